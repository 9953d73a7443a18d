"""The same results from a fill in one kernel and in two.  Each case makes its path, by the rows of the cache or the size of the
batch, and sees by the timed kernels that it was that one."""
import dataclasses

import numpy as np
import pytest

import wg_synth as ws
from oracle import oracle as O
from tests import helpers as H
from wg_synth.vocab import from_tokens

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2507_16768_amd as wg
    wg.load_library()
    return torch


_RUN = bytes(c for c in range(0x61, 0x7B)) * 6                      # 156 bytes
_TEXTS = ['Sequence(Write("%s"), Wait(denies={}, wait={<}, max=130), Write("c>"))' % _RUN.decode(),
          'Sequence(Wait(denies={}, wait={<}, max=64), Write("%s"))' % _RUN[:70].decode(),
          'DoWhile(body=Sequence(Wait(denies={9}, wait={<}), Write("%s")), condition=Wait(allow={\\x20}, true_waits={\\x2C}, '
          'false_waits={\\x5D}))' % _RUN[:63].decode()]


def _tokens():
    out = [b""] + [bytes([c]) for c in b"abcxyz<>9 ,]"]
    for n in (1, 7, 8, 9, 24, 25, 62, 63, 64, 65, 66, 127, 128, 129, 130, 131, 193):
        text, run = b"a" * n, (_RUN + b"x" * 60)[:n]
        out += [text, run, text[:-1] + b"<", text[:-1] + b"9", run[:-1] + b"!", b"x" + run[:-1],
                (b"xy<" + _RUN)[:n], (text + b"<" + _RUN)[:n + 5], (b"b" * 61 + b"<" + _RUN)[:n + 2], (b"<" + _RUN[:63] + b"  ,aa<")[:n + 6]]
    return list(dict.fromkeys(out))


@pytest.mark.parametrize("restart", [False, True])
def test_tokens_as_long_as_a_wavefront_and_longer(torch_cuda, restart):
    """Every state and budget with every token: through wg_advance (a request and four requests to a workgroup) and through
    the fill that advances in its one kernel, above a request per compute unit too, and in a lookup kernel, with a row for every key and without."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    toks = _tokens()
    vocab = from_tokens(toks, eos_id=0)
    o = O.Oracle(_TEXTS, None, O.OracleVocab(vocab.bytes, vocab.offsets, vocab.eos_id), restart=restart)
    h = wg.Handle(_TEXTS, None, wg.Vocab(vocab.bytes, vocab.offsets, vocab.eos_id), flags=wg.EOS_RESTART if restart else wg.EOS_STOP)
    h.reserve_batch(1024)
    st = [[O.SID_ERROR, 0]]
    for sid in range(o.num_states):
        d = o.describe(sid)
        st += [[sid, a] for a in (sorted({0, 1, d["max"] // 2, d["max"] - 1, d["max"], d["max"] + 1}) if d["kind"] == "WAIT" and d["max"] >= 0 else (0,))]
    st = np.array(st, dtype=np.uint32)
    rep, tk = np.repeat(st, vocab.V, axis=0), np.tile(np.arange(vocab.V, dtype=np.int32), len(st))
    want = o.advance(rep, tk)
    assert np.sum(want[:, 0] != O.SID_ERROR) >= 900
    got = H.dev_states(rep)
    h.advance(got, torch.from_numpy(tk).cuda())
    assert (H.host_states(got) == want).all()
    pick = np.random.default_rng(5).permutation(len(rep))
    pick = np.concatenate([pick[want[pick, 0] != O.SID_ERROR][:900], pick[:150]])
    keys = h.cache_stats()["keys"]
    for B, rows, kernels in ((256, keys, 1), (500, keys, 1), (300, keys, 1), (1000, keys, 2), (256, keys // 2, 2), (300, keys // 2, 2)):
        h.cache_resize(rows)
        for k in range(0, len(pick) - B + 1, B):
            p = pick[k:k + B]
            a, b = H.dev_states(rep[p]), H.dev_states(rep[p])
            mask = torch.empty((B, h.W), dtype=torch.int32, device="cuda")
            t = torch.from_numpy(tk[p]).cuda()
            h.advance(a, t)
            assert H.fill_kernels(h, lambda: h.advance_fill_masks(b, t, mask)) == kernels, (B, rows)
            assert (H.host_states(a) == want[p]).all() and torch.equal(a, b), (B, k)
            assert (H.host_mask(mask) == o.fill_masks(want[p])).all(), (B, k)


@pytest.mark.parametrize("n", [1, 6, 7, 8, 9, 56, 57, 63, 64, 65])
def test_walks_past_what_lies_ahead_of_their_state(torch_cuda, n):
    """A walk has eight states and 64 literal bytes from its state on at hand: runs that end on either side of both, in front of
    checkpoints, of conditions that lead back, over a body and past one, and of another run; in instances compiled first, added to the
    tables, and added with more than the tables had room for; through wg_advance and through the fill that advances, in its one kernel and in a
    lookup kernel."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    run = _RUN[:n].decode()
    text = ('DoWhile(body=Sequence(Write($r), Wait(denies={9}, wait={<}, max=40), IfElse(condition=Wait(allow={\\x20}, true_waits={\\x5B}, '
            'false_waits={\\x22}), if_body=Write($r), else_body=Sequence(Wait(allow={x}, wait={y}), Write("b"), Write("<c"))), Write($r)), '
            'condition=Wait(allow={\\x20}, true_waits={\\x2C}, false_waits={\\x5D}))')
    path = [b"%s<[%s%s" % ((run.encode(),) * 3), b'%s<"xyb<c%s' % ((run.encode(),) * 2), b"%s,%s]" % ((run.encode(),) * 2), b"ab<  [" + run.encode(), b"9", b"<9"]
    toks = [b""] + [bytes([c]) for c in b"abcxy<>9 ,[]\"!"] + [p[i:i + m] for p in path for i in (0, 1, n - 1, n, n + 1, n + 2, n + 5) for m in (2, 3, 7, 8, 9, 10, n, n + 1, n + 3, 2 * n + 4) if p[i:i + m]]
    vocab = from_tokens(list(dict.fromkeys(toks)), eos_id=0)
    args = [{"r": run.encode()}, {"r": run.encode()[::-1]}, {"r": b"<" * n}] + [{"r": (b"%d" % k).rjust(n, b"a")[-n:]} for k in range(40)]
    texts = [text] * len(args)
    o = O.Oracle(texts, args, O.OracleVocab(vocab.bytes, vocab.offsets, vocab.eos_id), restart=True)
    h = wg.Handle(texts[:1], args[:1], wg.Vocab(vocab.bytes, vocab.offsets, vocab.eos_id), flags=wg.EOS_RESTART)
    h.add_instances(texts[1:3], args[1:3])
    h.add_instances(texts[3:], args[3:])
    ends = o.num_states if len(args) * n < 200 else [k for k in range(o.num_states) if k < 3 * (o.num_states // len(args)) or k >= o.num_states - o.num_states // len(args)]
    st = []
    for sid in (range(ends) if isinstance(ends, int) else ends):
        d = o.describe(sid)
        st += [[sid, a] for a in ((0, 1, 39, 40) if d["kind"] == "WAIT" and d["max"] >= 0 else (0,))]
    st = np.array(st, dtype=np.uint32)
    rep, tk = np.repeat(st, vocab.V, axis=0), np.tile(np.arange(vocab.V, dtype=np.int32), len(st))
    want = o.advance(rep, tk)
    assert np.sum(want[:, 0] != O.SID_ERROR) >= 100
    got = H.dev_states(rep)
    h.advance(got, torch.from_numpy(tk).cuda())
    assert (H.host_states(got) == want).all()
    pick = np.random.default_rng(n).permutation(len(rep))
    pick = np.concatenate([pick[want[pick, 0] != O.SID_ERROR][:200], pick[:100]])
    keys = h.cache_stats()["keys"]
    for rows, kernels in ((keys, 1), (keys - 1, 2)):                   # in one kernel, and in a lookup kernel
        h.cache_resize(rows)
        for p in (pick[:200], pick):
            b, t = H.dev_states(rep[p]), torch.from_numpy(tk[p]).cuda()
            mask = torch.empty((len(p), h.W), dtype=torch.int32, device="cuda")
            assert H.fill_kernels(h, lambda: h.advance_fill_masks(b, t, mask)) == kernels
            assert (H.host_states(b) == want[p]).all() and (H.host_mask(mask) == o.fill_masks(want[p])).all()


def _unpack(torch, mask, V):
    shifts = torch.arange(32, dtype=torch.int32, device="cuda")
    return ((mask[:, :, None] >> shifts) & 1).bool().reshape(mask.shape[0], -1)[:, :V]


def _mask_by_itself_and_from_a_fill(torch, dtype, V, B, kernels):
    """Rows at lines and inside them, by wg_apply_mask and from the rows' kernel, the lookup in it or before it."""
    import paper_2507_16768_amd as wg
    dt, bits = (torch.float32, torch.int32) if dtype == "f32" else (torch.bfloat16, torch.int16)
    w = ws.make_workload(4, V=V, B=B, steps=2)
    o = H.make_oracle(w)
    v, h = H.make_gpu(w)
    cur = H.start_states(o, w)
    st = H.dev_states(cur)
    mask = torch.empty((B, h.W), dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(V + B)
    noise = torch.randint(-2 ** 31, 2 ** 31, (B, h.W), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    if V % 32:
        noise[:, -1] &= (1 << (V % 32)) - 1
    for off, pad in ((0, 0), (5, 0), (64, 61)):
        buf = torch.randn((B * (V + pad) + 128,), generator=g, device="cuda").to(dt)
        for m in (None, noise):
            x = buf[off:off + B * (V + pad)].view(B, V + pad)[:, :V]
            want = buf.clone()
            if m is None:
                assert H.fill_kernels(h, lambda: h.decode_step(st, None, mask, x)) == kernels
                assert (H.host_mask(mask[:3]) == o.fill_masks(cur[:3])).all()
            else:
                wg.apply_mask(x, m)
            want[off:off + B * (V + pad)].view(B, V + pad)[:, :V].masked_fill_(~_unpack(torch, mask if m is None else m, V), float("-inf"))
            assert torch.equal(buf.view(bits), want.view(bits)), (off, pad, m is None)


@pytest.mark.parametrize("dtype,V,B,through", [("f32", 1020, 257, False), ("f32", 1021, 257, True), ("bf16", 2040, 257, False), ("bf16", 2041, 257, True),
                                               ("f32", 340, 769, False), ("f32", 341, 769, True), ("bf16", 681, 769, False), ("bf16", 682, 769, True)])
def test_masking_either_side_of_the_least_that_goes_through_the_l2(torch_cuda, dtype, V, B, through):
    """1 MiB of logits, in one kernel and, above three requests per compute unit of so short rows, in two."""
    assert (B * V * (4 if dtype == "f32" else 2) > 1 << 20) == through
    _mask_by_itself_and_from_a_fill(torch_cuda, dtype, V, B, 1 if B <= 768 else 2)


@pytest.mark.parametrize("V,B", [(12001, 1), (20011, 31), (30000, 129), (98304, 96), (151936, 64), (20011, 255), (20011, 256), (20011, 257), (40000, 256)])
def test_keys_of_many_requests_of_one_call(torch_cuda, V, B):
    """Every workgroup of a row looks it up by itself up to a request per compute unit, and several make
    the same row and class rows: masks, counters and rows in use are as if one had, the rows are there for
    later calls in one kernel and in two, and they stay when the arena stops being addressed by key.  A class table
    counts once, in the call that takes it up, whatever the keys that share it."""
    torch = torch_cuda
    base = ws.make_workload(3, V=V, B=1, steps=1)
    args = list(base.args[:1]) + [{"x": bytes(np.random.default_rng(1).integers(1, 256, 5000, dtype=np.uint8))}]
    texts = list(base.texts[:1]) + ["Sequence(Write($x))"]
    w = dataclasses.replace(base, texts=texts, args=args, B=2, request_template=np.arange(2, dtype=np.int64))
    o = H.make_oracle(w)
    import paper_2507_16768_amd as wg
    h = wg.Handle(texts[:1], args[:1], wg.Vocab(w.vocab.bytes, w.vocab.offsets, w.vocab.eos_id), flags=wg.EOS_RESTART)
    own = h.num_states
    many = 300 if V > 16384 else 800                                # requests of a call that is two kernels
    mask = torch.empty((many, h.W), dtype=torch.int32, device="cuda")

    table = wg.Table(texts[:1], args[:1], flags=wg.EOS_RESTART, lmax=int(np.diff(w.vocab.offsets).max()))
    sets = {s: tuple(table.symbol_class(s, x) for x in range(256)) for s in range(own) if table.state(s)["kind"] in (2, 3)}

    def tables(sids):
        return {sets[s] for s in sids.tolist() if s in sets}

    def fill(sids, used_up=0):
        st = np.stack([sids, np.full_like(sids, used_up)], 1).astype(np.uint32)
        before = h.cache_stats()
        mask.fill_(0x35353535)
        direct = before["keys"] <= before["cache_rows"]
        assert H.fill_kernels(h, lambda: h.fill_masks(H.dev_states(st), mask[:len(st)])) == (1 if direct and len(st) <= 256 else 2)
        assert (H.host_mask(mask[:len(st)]) == o.fill_masks(st)).all()
        after = h.cache_stats()
        assert after["lookups"] - before["lookups"] == len(st)
        return {k: after[k] - before[k] for k in ("builds", "hits", "class_scans")}, after["rows_in_use"]

    sids = 1 + np.arange(B, dtype=np.uint32) % (own - 1)
    n = len(np.unique(sids))
    for _ in range(2):
        d, used = fill(sids)
        assert d["builds"] == n == used and d["hits"] == 0 and d["class_scans"] == len(tables(sids))
        d, used = fill(sids)
        assert d["builds"] == 0 and d["class_scans"] == 0 and d["hits"] == B and used == n
        h.cache_clear()
    fill(sids)
    rest = 1 + np.arange(many, dtype=np.uint32) % (own - 1)         # two kernels find them, and make the others
    d, used = fill(rest)
    assert d["builds"] == own - 1 - n and used == own - 1 and d["class_scans"] == len(tables(rest) - tables(sids))
    # new keys whose class table is there: a bounded Wait with a byte left, in as many requests as before and in more
    bounded = np.array([s for s in sets if table.state(s)["n_keys"] > 1], dtype=np.uint32)
    for i, size in enumerate((B, many)):
        d, now = fill(np.resize(bounded, size), 255 - i)
        used += min(size, len(bounded))
        assert d["builds"] == min(size, len(bounded)) and d["class_scans"] == 0 and now == used, size
    h.add_instances(texts[1:], args[1:])                            # more keys than rows
    s = h.cache_stats()
    assert s["keys"] > s["cache_rows"] and s["rows_in_use"] == used
    d, _ = fill(sids)
    assert d["builds"] == 0 and d["hits"] == B
    d, now = fill(np.arange(own, own + 40, dtype=np.uint32))
    assert d["builds"] == 40 and now == used + 40
    d, _ = fill(np.concatenate([sids[:200], np.arange(own, own + 40, dtype=np.uint32)]))
    assert d["builds"] == 0


@pytest.mark.parametrize("V,B,dtype,step,fill", [(9001, 257, "f32", 1, 1), (9001, 768, "bf16", 1, 1), (9001, 769, "bf16", 2, 2), (5003, 1024, "bf16", 2, 2), (16384, 448, "bf16", 1, 1),
                                                 (16384, 449, "f32", 2, 1), (16384, 512, "bf16", 2, 1), (16384, 513, "bf16", 2, 2), (16385, 300, "bf16", 2, 2), (99999, 384, "bf16", 2, 2),
                                                 (100000, 384, "bf16", 1, 2), (100000, 383, "f32", 2, 2), (100003, 1024, "bf16", 1, 2), (100003, 1025, "bf16", 2, 2)])
def test_batches_above_a_request_per_unit(torch_cuda, V, B, dtype, step, fill):
    """Either side of the lines up to which a batch of more than 256 requests is one kernel, with logits (step) and without (fill): masks, logits and
    states are those of batches of 100, and of a sample the oracle's, cold and cached, through each call; rows, hits and claims are counted as for any
    other batch."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    w = ws.make_workload(4, V=V, B=64, steps=1)
    o = H.make_oracle(w)
    _, h = H.make_gpu(w)
    _, ref = H.make_gpu(w)
    h.reserve_batch(B)
    rng = np.random.default_rng(V + B)
    at = np.stack([rng.integers(0, h.num_states, B), np.zeros(B)], 1).astype(np.uint32)
    at[:3] = at[B - 3:]                                                # requests of one key, at both ends of the batch
    tok = torch.empty(B, dtype=torch.int32, device="cuda")             # allowed ones, but for every ninth
    for b in range(0, B, 100):
        m = torch.empty((len(at[b:b + 100]), h.W), dtype=torch.int32, device="cuda")
        ref.fill_masks(H.dev_states(at[b:b + 100]), m)
        wg.select_tokens(m, V, torch.from_numpy(rng.integers(0, 1 << 62, len(m))).cuda(), tok[b:b + 100])
    tok[4::9] = 1
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    raw = torch.randn((B, V + 5), device="cuda").to(dt)
    want_states, want = H.dev_states(at), torch.empty((B, h.W), dtype=torch.int32, device="cuda")
    want_logits = raw.clone()
    for b in range(0, B, 100):
        s, m = want_states[b:b + 100], want[b:b + 100]
        ref.advance(s, tok[b:b + 100])
        ref.fill_masks(s, m)
        wg.apply_mask(want_logits[b:b + 100, :V], m)
    some = rng.permutation(B)[:40]
    sampled = o.advance(at[some], tok.cpu().numpy()[some])
    assert (H.host_states(want_states)[some] == sampled).all() and (H.host_mask(want)[some] == o.fill_masks(sampled)).all()
    keys = len(np.unique(H.host_mask(want), axis=0))
    live = int((H.host_states(want_states)[:, 0] != 0xFFFFFFFF).sum())
    assert B // 2 < live < B
    for cold in (True, False):
        for call in ("step", "advance_fill", "fill"):
            if cold:
                h.cache_clear()
            before = h.cache_stats()
            states = H.dev_states(at) if call != "fill" else want_states.clone()
            mask, logits = torch.full_like(want, -1), raw.clone()
            kernels = H.fill_kernels(h, {"step": lambda: h.decode_step(states, tok, mask, logits[:, :V]), "advance_fill": lambda: h.advance_fill_masks(states, tok, mask),
                                         "fill": lambda: h.fill_masks(states, mask)}[call])
            assert kernels == (step if call == "step" else fill), call
            assert torch.equal(states, want_states) and torch.equal(mask, want), (cold, call)
            assert call != "step" or torch.equal(logits.view(torch.int32 if dtype == "f32" else torch.int16), want_logits.view(torch.int32 if dtype == "f32" else torch.int16)), cold
            after = h.cache_stats()
            assert after["lookups"] - before["lookups"] == B
            assert after["hits"] - before["hits"] == (0 if cold else live)
            assert after["builds"] - before["builds"] == (after["rows_in_use"] if cold else 0), (cold, call)
            assert not cold or after["rows_in_use"] >= keys - 1
