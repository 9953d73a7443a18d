"""GPU parity of the walk of a token by a wavefront, a byte per lane: tokens as long as the wavefront, a byte less, a byte
more and of three of its windows, ended by every kind of state and budget; and of how a call of one kernel counts its
rows (groups of 16)."""
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
    the fill that advances in its one kernel and behind a lookup kernel."""
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
    for B in (256, 500, 300):
        for k in range(0, len(pick) - B + 1, B):
            p = pick[k:k + B]
            a, b = H.dev_states(rep[p]), H.dev_states(rep[p])
            mask = torch.empty((B, h.W), dtype=torch.int32, device="cuda")
            t = torch.from_numpy(tk[p]).cuda()
            h.advance(a, t)
            h.advance_fill_masks(b, t, mask)
            assert (H.host_states(a) == want[p]).all() and torch.equal(a, b), (B, k)
            assert (H.host_mask(mask) == o.fill_masks(want[p])).all(), (B, k)


@pytest.mark.parametrize("n", [1, 6, 7, 8, 9, 56, 57, 63, 64, 65])
def test_walks_past_what_lies_ahead_of_their_state(torch_cuda, n):
    """A walk has eight states and 64 literal bytes from its state on at hand: runs that end on either side of both, in front of
    checkpoints, of conditions that lead back, over a body and past one, and of another run; in instances compiled first, added to the
    tables, and added with more than the tables had room for."""
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
    for p in (pick[:200], pick):                                       # in one kernel, and behind a lookup kernel
        b = H.dev_states(rep[p])
        mask = torch.empty((len(p), h.W), dtype=torch.int32, device="cuda")
        h.advance_fill_masks(b, torch.from_numpy(tk[p]).cuda(), mask)
        assert (H.host_states(b) == want[p]).all() and (H.host_mask(mask) == o.fill_masks(want[p])).all()


@pytest.mark.parametrize("B", [1, 15, 16, 17, 31, 32, 33, 255, 256])
def test_calls_of_one_kernel_count_their_rows(torch_cuda, B):
    """Each call's states are written back, its lookups counted and its claims told from the next call's, whatever rows the
    last group holds."""
    torch = torch_cuda
    w = ws.make_workload(4, V=5003, B=B, steps=6)
    o = H.make_oracle(w)
    v, h = H.make_gpu(w)
    cur = H.start_states(o, w)
    st = H.dev_states(cur)
    mask = torch.empty((B, h.W), dtype=torch.int32, device="cuda")
    draws = w.token_draws()
    lookups = 0
    for k in range(6):
        h.fill_masks(st, mask)                             # (made, from the second call of a step on found)
        made = h.cache_stats()
        want = o.fill_masks(cur)
        assert (H.host_mask(mask) == want).all(), k
        t = np.array([O.select_bit(r, int(draws[k][b]) % int(np.unpackbits(r.view(np.uint8)).sum())) for b, r in enumerate(want)], dtype=np.int32)
        cur = o.advance(cur, t)
        h.fill_masks(st, mask)
        found = h.cache_stats()
        assert found["builds"] == made["builds"] and found["hits"] == made["hits"] + B, k
        h.advance_fill_masks(st, torch.from_numpy(t).cuda(), mask)
        assert (H.host_states(st) == cur).all() and (H.host_mask(mask) == o.fill_masks(cur)).all(), k
        lookups += 3 * B
        assert h.cache_stats()["lookups"] == lookups, k
        if k == 3:
            h.cache_clear()
    assert h.error_count() == 0


def test_advance_of_more_requests_than_the_grid_holds(torch_cuda):
    torch = torch_cuda
    w = ws.make_workload(2, V=2003, B=8, steps=1)
    o = H.make_oracle(w)
    v, h = H.make_gpu(w)
    st = H.start_states(o, w)
    few = np.arange(16, dtype=np.int32) + 60
    want = o.advance(np.repeat(st[:1], 16, axis=0), few)
    B = (4 << 20) + 21
    big = torch.from_numpy(st[:1].view(np.int32).copy()).cuda().repeat(B, 1)
    h.advance(big, (torch.arange(B, device="cuda", dtype=torch.int32) % 16 + 60))
    assert torch.equal(big, torch.from_numpy(want.view(np.int32)).cuda().repeat(B // 16 + 1, 1)[:B])


@pytest.mark.parametrize("B", [1, 63, 64, 65, 256, 257, 1000, 70000])
def test_rejected_tokens_are_counted(torch_cuda, B):
    """Each of them once, through wg_advance and through the fills that advance (in one kernel, whose workgroups all walk the token, and in
    two); requests that are in ERROR already count again."""
    torch = torch_cuda
    w = ws.make_workload(4, V=20011, B=8, steps=1)
    v, h = H.make_gpu(w)
    start = H.dev_states(np.array([[h.start_states[0][0], 0]], dtype=np.uint32)).repeat(B, 1)
    bad = (torch.arange(B, device="cuda") % 3 != 1).to(torch.int32)          # the template's first byte is no 0x00 token and no id above V
    tokens = torch.where(bad == 1, torch.where(torch.arange(B, device="cuda") % 2 == 0, 0, 1 << 30), -7).to(torch.int32)
    st = start.clone()
    h.advance(st, tokens)
    assert h.error_count() == B and bool((st[:, 0] == -1).all())
    h.advance(st, tokens)
    assert h.error_count() == 2 * B
    if B <= h.max_batch():
        mask = torch.empty((B, h.W), dtype=torch.int32, device="cuda")
        st = start.clone()
        h.advance_fill_masks(st, tokens, mask)
        assert h.error_count() == 3 * B and bool((st[:, 0] == -1).all()) and not bool(mask.any())


@pytest.mark.parametrize("B", [8191, 8192, 8193, 70001])
@pytest.mark.parametrize("cap", [1, 65, 300])
def test_forced_bytes_of_many_requests(torch_cuda, B, cap):
    """A wavefront per request and, above 32 requests to a unit, a thread."""
    test_forced_bytes_longer_than_a_wavefront(torch_cuda, B, cap)


@pytest.mark.parametrize("B", [1, 511, 512, 513, 1025])
@pytest.mark.parametrize("cap", [1, 63, 64, 65, 300])
def test_forced_bytes_longer_than_a_wavefront(torch_cuda, B, cap):
    """Forced runs of less and more bytes than lanes, of several Writes in a row, cut inside a Write and at its end, one
    request to a workgroup and four."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    text = 'Sequence(Write("%s"), Write("b"), Write("%s"), Wait(denies={}, wait={<}), Write("%s"))' % (_RUN.decode(), _RUN[:64].decode(), _RUN[:65].decode())
    vocab = from_tokens([b""] + [bytes([c]) for c in b"abcxyz<>"], 0)
    o = O.Oracle([text], [{}], O.OracleVocab(vocab.bytes, vocab.offsets, vocab.eos_id), restart=True)
    h = wg.Handle([text], [{}], wg.Vocab(vocab.bytes, vocab.offsets, vocab.eos_id), flags=wg.EOS_RESTART)
    sids = [(i * 7) % (o.num_states + 2) if i else 1 for i in range(B)]
    st = np.array([[s, 3] for s in sids], dtype=np.uint32)
    d_bytes = torch.full((B, cap), 0xEE, dtype=torch.uint8, device="cuda")
    d_lens = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    d_end = torch.full((B, 2), -1, dtype=torch.int32, device="cuda")
    h.forced_bytes(H.dev_states(st), d_bytes, d_lens, d_end)
    gb, gl, ge = d_bytes.cpu().numpy(), d_lens.cpu().numpy(), H.host_states(d_end)
    for i, s in enumerate(sids):
        want, end = o.forced_bytes(s, cap)
        assert gl[i] == len(want) and bytes(gb[i, :gl[i]]) == want and (gb[i, gl[i]:] == 0xEE).all(), (s, cap)
        assert ge[i, 0] == end and ge[i, 1] == (0 if want else 3), (s, cap)
