"""GPU parity of the row builder and of the masking at the sizes where they can go wrong: vocabularies
at the edges of token ranges and mask words, class tables at the edges of the two ways to take one,
logits at every alignment, and logits above the size from which whole lines are written."""
import dataclasses

import numpy as np
import pytest

import wg_synth as ws
from oracle import oracle as O
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2507_16768_amd as wg
    wg.load_library()
    return torch


def _set(chars):
    return "{" + ", ".join("\\x%02X" % c for c in chars) + "}"


# byte values that enter the table: 1, 2, 8 and 9 of them, a block of 16 that stays between blocks that
# do not, exits that share a block with rejected values, no value that stays, all of them
_TABLES = [((), b"a"), (b"b", b"a"), (b"bcdefgh", b"a"), (b"bcdefghi", b"a"), (bytes(range(0x60, 0x70)), b"pq"),
           (bytes(range(0x20, 0x30)) + b"abc", b"x/"), ((), bytes(range(0x30, 0x3A))), (bytes(range(256)), b"<"),
           (bytes(c for c in range(0x20, 0x7F) if c % 3), b"!$'"),
           # values rejected in blocks of 128, 64 and 32, at their edges
           (bytes(range(0x80, 0x100)), b"a"), (bytes(range(0x00, 0x80)), b"z"), (bytes(range(0x40, 0x80)), b" "),
           (bytes(range(0x20, 0x40)) + bytes(range(0xA0, 0xE0)), b"ab"), (bytes(range(0x00, 0x20)) + bytes([0x3F, 0x40, 0x7F, 0xC0]), b"c")]


def _texts():
    out = []
    for i, (allow, leave) in enumerate(_TABLES):
        stay = _set([c for c in allow if c not in leave])
        for bound in ("", ", max=3"):
            w = "Wait(allow=%s, wait=%s%s)" % (stay, _set(leave), bound)
            out.append('Sequence(%s, Write("ab"))' % w)
            out.append("Sequence(Write(\"z\"), %s, Wait(denies={}, wait={>}, max=2))" % w)      # a checkpoint behind it
        out.append('IfElse(condition=Wait(allow=%s, true_waits=%s, false_waits={\\x7E}), if_body=Write("a b c d e f g h i j k l m"), '
                   'else_body=Wait(allow={a, b}, wait={c}))' % (_set([c for c in allow if c not in leave and c != 0x7E]), _set(leave)))
    return out


@pytest.mark.parametrize("V,longest", [(257, 8), (2047, 24), (2049, 24), (4096, 9), (16384, 24), (16385, 33), (18432, 24)])
def test_rows_of_every_kind_of_table(torch_cuda, V, longest):
    torch = torch_cuda
    texts = _texts()
    base = ws.make_workload(2, V=V, B=1, steps=1)
    w = dataclasses.replace(base, vocab=ws.make_vocab(V, ("geometric", 4, longest), seed=V, utf8_tenths=1), texts=texts,
                            args=[{}] * len(texts), B=len(texts), request_template=np.arange(len(texts), dtype=np.int64))
    o = H.make_oracle(w)
    v, h = H.make_gpu(w)
    st = []
    for sid in range(1, o.num_states):
        d = o.describe(sid)
        st += [[sid, a] for a in range(d["max"] + 1)] if d["kind"] == "WAIT" and d["max"] >= 0 else [[sid, 0]]
    st = np.array(st + st[::7], dtype=np.uint32)                    # some states twice in a call
    want = o.fill_masks(st)
    d_mask = torch.empty((len(st), h.W), dtype=torch.int32, device="cuda")
    for rep in ("cold", "warm", "cleared"):
        if rep == "cleared":
            h.cache_clear()
        d_mask.fill_(0x35353535)
        h.fill_masks(H.dev_states(st), d_mask)
        assert (H.host_mask(d_mask) == want).all(), (rep, np.flatnonzero((H.host_mask(d_mask) != want).any(1))[:8])


def _unpack(torch, mask, V):
    shifts = torch.arange(32, dtype=torch.int32, device="cuda")
    return ((mask[:, :, None] >> shifts) & 1).bool().reshape(mask.shape[0], -1)[:, :V]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V", [1, 33, 65, 1000, 2047, 2049, 2113, 8191, 8193, 20001])
def test_masking_at_every_alignment(torch_cuda, V, dtype):
    """apply_mask on rows that start 0 .. 17 elements into a buffer, odd and even strides."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(V)
    B = 5
    mask = torch.randint(-2 ** 31, 2 ** 31, (B, (V + 31) // 32), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    mask[1], mask[2], mask[3, ::2] = 0, -1, 0
    if V % 32:
        mask[:, -1] &= (1 << (V % 32)) - 1
    for off in (0, 1, 3, 8, 17):
        for pad in (0, 1, 8, 63):
            buf = torch.randn((B * (V + pad) + 32,), generator=g, device="cuda").to(dt)
            x = buf[off:off + B * (V + pad)].view(B, V + pad)[:, :V]
            want = buf.clone()
            y = want[off:off + B * (V + pad)].view(B, V + pad)[:, :V]
            y.masked_fill_(~_unpack(torch, mask, V), float("-inf"))
            wg.apply_mask(x, mask)
            bits = torch.int32 if dtype == "f32" else torch.int16
            assert torch.equal(buf.view(bits), want.view(bits)), (off, pad)     # nothing outside the rows either


def _mask_by_itself_and_from_a_fill(torch, dtype, V, B):
    """Rows at lines and inside them, by wg_apply_mask and from the rows' kernel."""
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
                h.decode_step(st, None, mask, x)
                assert (H.host_mask(mask[:3]) == o.fill_masks(cur[:3])).all()
            else:
                wg.apply_mask(x, m)
            want[off:off + B * (V + pad)].view(B, V + pad)[:, :V].masked_fill_(~_unpack(torch, mask if m is None else m, V), float("-inf"))
            assert torch.equal(buf.view(bits), want.view(bits)), (off, pad, m is None)


@pytest.mark.parametrize("dtype,V,B,through", [("bf16", 100003, 209, True), ("bf16", 100003, 210, False), ("bf16", 99904, 209, True), ("bf16", 99904, 210, False), ("f32", 41003, 255, True),
                                               ("f32", 41003, 256, False), ("f32", 20011, 523, True), ("f32", 20011, 524, False), ("f32", 20011, 525, False)])
def test_masking_either_side_of_what_goes_through_the_l2(torch_cuda, dtype, V, B, through):
    """40 MiB of logits, in one kernel and, above a request per compute unit, in two."""
    assert (B * V * (4 if dtype == "f32" else 2) <= 40 << 20) == through
    _mask_by_itself_and_from_a_fill(torch_cuda, dtype, V, B)


@pytest.mark.parametrize("dtype,V,B,through", [("bf16", 32768, 16, False), ("bf16", 32769, 16, True), ("f32", 16384, 16, False), ("f32", 16385, 16, True), ("f32", 1020, 257, False),
                                               ("f32", 1021, 257, True), ("bf16", 2040, 257, False), ("bf16", 2041, 257, True)])
def test_masking_either_side_of_the_least_that_goes_through_the_l2(torch_cuda, dtype, V, B, through):
    """1 MiB of logits, as above."""
    assert (B * V * (4 if dtype == "f32" else 2) > 1 << 20) == through
    _mask_by_itself_and_from_a_fill(torch_cuda, dtype, V, B)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V", [257, 2049, 16385, 40003, 131073])
def test_masking_of_rows_with_one_token_disallowed(torch_cuda, V, dtype):
    """Wavefronts that have nothing to mask beside one that has a single token, at the edges of their shares."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    dt, bits = (torch.float32, torch.int32) if dtype == "f32" else (torch.bfloat16, torch.int16)
    at = [None] + [t for t in (0, 1, 255, 256, 511, 512, 2047, 2048, 16383, 16384, 32768) if t < V] + [V - 1]
    allowed = torch.ones((len(at), V), dtype=torch.bool, device="cuda")
    for b, t in enumerate(at):
        if t is not None:
            allowed[b, t] = False
    W = (V + 31) // 32
    packed = np.packbits(np.pad(allowed.cpu().numpy(), ((0, 0), (0, 32 * W - V))), axis=1, bitorder="little").view(np.int32)
    x = torch.randn((len(at), V), device="cuda").to(dt)
    want = x.masked_fill(~allowed, float("-inf"))
    wg.apply_mask(x, torch.from_numpy(packed.copy()).cuda())
    assert torch.equal(x.view(bits), want.view(bits))
    # the same from the rows' kernel: text without an end in which one byte, and so one token, is not allowed
    vocab = ws.make_vocab(V, ("uniform", 1, 8), seed=V, utf8_tenths=0)
    h = wg.Handle(["Sequence(Wait(denies={}, wait={<eos>}))", "Sequence(Wait(denies={\\x02}, wait={<eos>}))"], None,
                  wg.Vocab(vocab.bytes, vocab.offsets, vocab.eos_id), flags=wg.EOS_RESTART)
    st = H.dev_states(np.concatenate([h.start_states] * 3).view(np.uint32).reshape(-1, 2))
    mask = torch.empty((6, h.W), dtype=torch.int32, device="cuda")
    for cold in (True, False):
        x = torch.randn((6, V), device="cuda").to(dt)
        want = x.clone()
        h.decode_step(st, None, mask, x)
        ok = _unpack(torch, mask, V)
        assert (V - ok.sum(1)).tolist() == [0, 1] * 3
        want.masked_fill_(~ok, float("-inf"))
        assert torch.equal(x.view(bits), want.view(bits)), cold


@pytest.mark.parametrize("dtype,V,B", [(t, V, 24) for t in ("f32", "bf16") for V in (1536, 2048, 8191, 8193, 20001)] + [("bf16", 100003, 503), ("bf16", 100003, 504)])
def test_masking_of_few_scattered_tokens(torch_cuda, V, B, dtype):
    """Either side of 48 disallowed tokens in a wavefront's 2,048, or 36 in 1,536 (bf16 logits above 96 MiB), which it then
    lists and stores at once: at random places, side by side, at the ends of the share; rows at any address, nothing
    outside them touched."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    dt, bits = (torch.float32, torch.int32) if dtype == "f32" else (torch.bfloat16, torch.int16)
    share, edge = (1536, 36) if B == 504 else (2048, 48)
    rng = np.random.default_rng(V)
    rows = []
    for n in (1, 2, edge - 1, edge, edge + 1, 64, 65, 200):
        for places in (lambda m: rng.permutation(m)[:n], lambda m: np.arange(min(n, m)), lambda m: np.arange(max(0, m - n), m)):
            ok = np.ones(V, dtype=bool)
            for lo in range(0, V, share):
                ok[lo + places(min(share, V - lo))] = False
            rows.append(ok)
    allowed, W = np.stack(rows), (V + 31) // 32
    packed = np.packbits(np.pad(allowed, ((0, 0), (0, 32 * W - V))), axis=1, bitorder="little").view(np.int32)
    which = torch.arange(B, device="cuda") % len(rows)
    mask, allowed = torch.from_numpy(packed.copy()).cuda()[which], torch.from_numpy(allowed).cuda()[which]
    for off, pad in ((0, 0), (1, 3), (5, 64)):
        buf = torch.randn(B * (V + pad) + 24, device="cuda").to(dt)
        x = buf[off:off + B * (V + pad)].view(B, V + pad)[:, :V]
        want = buf.clone()
        want[off:off + B * (V + pad)].view(B, V + pad)[:, :V].masked_fill_(~allowed, float("-inf"))
        wg.apply_mask(x, mask)
        assert torch.equal(buf.view(bits), want.view(bits)), (off, pad)


@pytest.mark.parametrize("dtype,B,V,pad", [("bf16", 700, 151936, 0), ("bf16", 701, 151900, 3), ("bf16", 740, 151936, 0), ("bf16", 741, 151900, 3), ("f32", 400, 128256, 0), ("f32", 700, 128256, 0)])
def test_masking_of_logits_beyond_the_last_level_cache(torch_cuda, dtype, B, V, pad):
    """Either side of 208 MiB of bf16 and 320 MiB of fp32 logits; above them lines are read where they are
    mixed and written whole."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(B)
    buf = torch.randn((B, V + pad), generator=g, device="cuda").to(dt)
    mask = torch.randint(-2 ** 31, 2 ** 31, (B, (V + 31) // 32), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    mask[::3] = 0
    mask[1::3] |= torch.randint(-2 ** 31, 2 ** 31, mask[1::3].shape, generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    mask[1::6, : mask.shape[1] // 2] = -1
    if V % 32:
        mask[:, -1] &= (1 << (V % 32)) - 1
    want = buf.clone()
    for lo in range(0, B, 64):
        want[lo:lo + 64, :V].masked_fill_(~_unpack(torch, mask[lo:lo + 64], V), float("-inf"))
    wg.apply_mask(buf[:, :V], mask)
    bits = torch.int32 if dtype == "f32" else torch.int16
    assert torch.equal(buf.view(bits), want.view(bits))


@pytest.mark.parametrize("V,B", [(65535, 8), (65536, 8), (131072, 4), (131073, 5), (151936, 1), (98304, 33), (98304, 96), (98305, 97), (65536, 97), (131072, 48), (131073, 64), (147456, 64), (20481, 40), (24577, 300), (98304, 64), (98304, 112), (98304, 113), (32768, 224), (32768, 225), (32768, 256), (32769, 256), (32768, 257), (131072, 32), (131072, 33), (40000, 256), (40000, 257),
                                 (40000, 32), (40000, 33), (8200, 7), (3000, 512), (3000, 513)])
def test_decode_step_at_the_edges_of_the_split(torch_cuda, V, B):
    """Rows cut into 1 to 32 workgroups, looked up in the rows' kernel and before it; the advance by itself with
    one and with four requests to a wavefront."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    w = ws.make_workload(5, V=V, B=B, steps=4)
    o = H.make_oracle(w)
    v, h = H.make_gpu(w)
    st = H.dev_states(H.start_states(o, w))
    ref = st.clone()
    mask = torch.empty((B, h.W), dtype=torch.int32, device="cuda")
    draws = torch.from_numpy(w.token_draws(4).view(np.int64)).cuda()
    tok = torch.empty(B, dtype=torch.int32, device="cuda")
    for k in range(4):
        x = torch.randn((B, V), device="cuda").to(torch.bfloat16)
        y = x.clone()
        if k == 2:
            h.cache_clear()
        h.decode_step(st, tok if k else None, mask, x)
        if k:
            h.advance(ref, tok)
        assert torch.equal(st, ref), k
        assert (H.host_mask(mask) == o.fill_masks(H.host_states(st))).all(), k
        y.masked_fill_(~_unpack(torch, mask, V), float("-inf"))
        assert torch.equal(x.view(torch.int16), y.view(torch.int16)), k
        wg.select_tokens(mask, V, draws[k], tok)
    n = h.cache_stats()
    assert h.error_count() == 0 and n["lookups"] == 4 * B and n["hits"] + n["builds"] <= 4 * B


@pytest.mark.parametrize("V,B", [(16384, 16), (16385, 16), (16385, 17), (32768, 8), (32769, 9), (8192, 64), (8192, 65), (4096, 128), (98303, 257), (98304, 257), (49151, 512), (49151, 513), (49152, 513), (24575, 1024)])
def test_decode_step_at_the_edges_of_few_and_of_many_rows(torch_cuda, V, B):
    """Up to a workgroup per compute unit, and above a request per unit either side of eight workgroups to one."""
    test_decode_step_at_the_edges_of_the_split(torch_cuda, V, B)


@pytest.mark.parametrize("V,B", [(40959, 512), (40960, 512), (65599, 820), (65600, 820), (20479, 1024), (20480, 1024), (28800, 360), (28799, 360)])
def test_decode_step_where_shares_grow_with_the_batch(torch_cuda, V, B):
    """Above a request per compute unit either side of where a row is cut into fewer shares for the workgroups of the call."""
    test_decode_step_at_the_edges_of_the_split(torch_cuda, V, B)


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
    mask = torch.empty((300, h.W), dtype=torch.int32, device="cuda")

    table = wg.Table(texts[:1], args[:1], flags=wg.EOS_RESTART, lmax=int(np.diff(w.vocab.offsets).max()))
    sets = {s: tuple(table.symbol_class(s, x) for x in range(256)) for s in range(own) if table.state(s)["kind"] in (2, 3)}

    def tables(sids):
        return {sets[s] for s in sids.tolist() if s in sets}

    def fill(sids, used_up=0):
        st = np.stack([sids, np.full_like(sids, used_up)], 1).astype(np.uint32)
        before = h.cache_stats()
        mask.fill_(0x35353535)
        h.fill_masks(H.dev_states(st), mask[:len(st)])
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
    rest = 1 + np.arange(300, dtype=np.uint32) % (own - 1)          # two kernels find them, and make the others
    d, used = fill(rest)
    assert d["builds"] == own - 1 - n and used == own - 1 and d["class_scans"] == len(tables(rest) - tables(sids))
    # new keys whose class table is there: a bounded Wait with a byte left, in as many requests as before and in more
    bounded = np.array([s for s in sets if table.state(s)["n_keys"] > 1], dtype=np.uint32)
    for i, size in enumerate((B, 300)):
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


def test_additions_of_every_size(torch_cuda):
    """Slices of 1 to 40 states at every offset, with and without new class tables, and one above the
    handle's pinned memory: the states that arrive are those of a compilation at once."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    base = ws.make_workload(2, V=1031, B=1, steps=1)
    rng = np.random.default_rng(7)
    text = ["Sequence(Write($x))", 'Sequence(Write($x), Wait(allow=$x, wait={\\x00}))']
    sizes = list(range(1, 41)) + [60000, 3, 17]
    texts = [text[n % 2 if n < 100 else 0] for n in sizes]
    args = [{"x": bytes(rng.integers(1, 256, n, dtype=np.uint8))} for n in sizes]
    w = dataclasses.replace(base, texts=texts, args=args, B=len(texts), request_template=np.arange(len(texts), dtype=np.int64))
    o = H.make_oracle(w)
    h = wg.Handle(texts[:1], args[:1], wg.Vocab(w.vocab.bytes, w.vocab.offsets, w.vocab.eos_id), flags=wg.EOS_RESTART)
    for i in range(1, len(texts)):
        first = h.num_states
        new = h.add_instances(texts[i:i + 1], args[i:i + 1])
        assert int(new[0, 0]) == o.start_state(i)
        st = np.arange(first, h.num_states, dtype=np.uint32)[-900:]
        st = np.stack([st, np.zeros_like(st)], 1)
        mask = torch.empty((len(st), h.W), dtype=torch.int32, device="cuda")
        h.fill_masks(H.dev_states(st), mask)
        assert (H.host_mask(mask) == o.fill_masks(st)).all(), i
    assert h.num_states == o.num_states


@pytest.mark.parametrize("dtype,stride_pad", [("bf16", 0), ("f32", 5)])
def test_decode_step_of_a_large_batch(torch_cuda, dtype, stride_pad):
    """wg_decode_step with logits beyond the last-level cache against the separate calls (which the
    other tests compare with the oracle): masks, states and masked logits, cold and warm."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    w = ws.make_workload(5, V=151936 if dtype == "bf16" else 90001, B=720 if dtype == "bf16" else 1000, steps=3)
    o = H.make_oracle(w)
    v, h = H.make_gpu(w)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    st = H.dev_states(H.start_states(o, w))
    ref = st.clone()
    mask, ref_mask = (torch.empty((w.B, h.W), dtype=torch.int32, device="cuda") for _ in range(2))
    draws = torch.from_numpy(w.token_draws(3).view(np.int64)).cuda()
    tok = torch.empty(w.B, dtype=torch.int32, device="cuda")
    for k in range(3):
        x = torch.randn((w.B, w.vocab.V + stride_pad), device="cuda").to(dt)
        y = x.clone()
        if k != 1:
            h.cache_clear()
        h.decode_step(st, tok if k else None, mask, x[:, :w.vocab.V])
        if k:
            h.advance(ref, tok)
        h.cache_clear()
        h.fill_masks(ref, ref_mask)
        wg.apply_mask(y[:, :w.vocab.V], ref_mask)
        assert torch.equal(mask, ref_mask) and torch.equal(st, ref), k
        bits = torch.int32 if dtype == "f32" else torch.int16
        assert torch.equal(x.view(bits), y.view(bits)), k
        assert (H.host_mask(mask)[::90] == o.fill_masks(H.host_states(st)[::90])).all()
        wg.select_tokens(mask, w.vocab.V, draws[k], tok)
    assert h.error_count() == 0


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,V,off", [(1, 33, 0), (3, 8193, 1), (130, 5000, 3), (2, 90001, 0), (97, 90001, 5), (40, 151936, 0), (3, 300007, 1),
                                     (5, 90112, 3), (5, 90109, 3), (95, 90110, 2), (8, 49151, 0), (8, 49152, 1), (47, 50021, 0), (95, 50021, 0), (96, 50021, 0),
                                     (31, 114688, 1), (63, 114689, 0), (64, 114689, 0), (191, 90001, 1), (192, 90001, 1)])
def test_sampling_of_cut_and_whole_rows(torch_cuda, B, V, off, dtype):
    """masked_argmax and masked_topk where rows are cut and where they are not, at any alignment, with
    ties (as many as tie-breaking by token id decides), NaNs, both zeros, -inf and rows that allow
    little or nothing; each call twice, so that nothing is left behind in the merge arrays."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    rng = np.random.default_rng(V + B)
    x = rng.standard_normal((B, V)).astype(np.float32)
    x[:, rng.integers(0, V, V // 20)] = np.nan
    x[0] = np.round(x[0])                                           # thousands tie, zeros of both signs
    if B > 2:
        x[1], x[2] = -np.inf, np.nan
        x[2, V // 2] = -0.0
    host = x if dtype == "f32" else ws.to_bf16_bits(x)
    bits = rng.integers(0, 1 << 32, (B, (V + 31) // 32), dtype=np.uint32)
    if B > 3:
        bits[3], bits[4 % B] = 0, 0
        bits[4 % B, -1] = 1
    if V % 32:
        bits[:, -1] &= np.uint32((1 << (V % 32)) - 1)
    d = H.dev_logits(host)
    buf = torch.zeros((B * (V + off) + 64,), dtype=d.dtype, device="cuda")
    view = buf[off:off + B * (V + off)].view(B, V + off)[:, :V]
    view.copy_(d)
    mask = torch.from_numpy(bits.view(np.int32)).cuda()
    tok = torch.empty(B, dtype=torch.int32, device="cuda")
    want = O.masked_argmax(host, bits)
    for _ in range(2):
        tok.fill_(-7)
        wg.masked_argmax(view, mask, tok)
        assert (tok.cpu().numpy() == want).all()
    for k in (1, 7, 64):
        ids = torch.empty((B, k), dtype=torch.int32, device="cuda")
        vals = torch.empty((B, k), dtype=d.dtype, device="cuda")
        work = torch.empty(wg.masked_topk_workspace(B, V, k), dtype=torch.uint8, device="cuda")
        wg.masked_topk(view, mask, ids, vals, work)
        want_ids, want_vals = O.masked_topk(host, bits, k)
        assert (ids.cpu().numpy() == want_ids).all(), k
        assert (H.host_logit_bits(vals) == np.ascontiguousarray(want_vals).view(np.uint32 if dtype == "f32" else np.uint16)).all(), k


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,V,off", [(5, 8192, 0), (5, 8193, 1), (5, 12288, 0), (5, 12289, 0), (5, 12285, 3), (5, 16384, 0), (5, 24576, 0), (5, 24577, 0), (5, 24569, 7),
                                     (3, 98304, 0), (3, 98305, 0), (2, 196608, 0), (2, 196610, 1)])
def test_sampling_either_side_of_one_round(torch_cuda, B, V, off, dtype):
    """Rows, and shares of cut rows, of one, two and three pieces of a thread, of a piece more and where a row that begins
    inside a block has one more."""
    test_sampling_of_cut_and_whole_rows(torch_cuda, B, V, off, dtype)


@pytest.mark.parametrize("dtype,V", [("bf16", 262145), ("bf16", 286720), ("bf16", 286729), ("f32", 262149), ("f32", 274433)])
def test_sampling_of_whole_rows_of_two_segments(torch_cuda, V, dtype):
    """Rows whose mask comes to LDS in two turns, the second a single piece, one round and more than one."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    B, few = 130, 6
    g = torch.Generator(device="cuda").manual_seed(V)
    x = torch.randn((B, V), generator=g, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
    x[1, V - 1], x[2, 262143], x[3, 262144] = 50.0, 50.0, 50.0
    bits = torch.randint(-2 ** 31, 2 ** 31, (B, (V + 31) // 32), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    bits[1:4] = -1
    bits[4] = 0
    if V % 32:
        bits[:, -1] &= (1 << (V % 32)) - 1
    host, masks = H.host_logit_bits(x[:few]), H.host_mask(bits[:few])
    host = host.view(np.float32) if dtype == "f32" else host
    tok = torch.empty(B, dtype=torch.int32, device="cuda")
    ids, vals = torch.empty((B, 9), dtype=torch.int32, device="cuda"), torch.empty((B, 9), dtype=x.dtype, device="cuda")
    wg.masked_argmax(x, bits, tok)
    wg.masked_topk(x, bits, ids, vals, torch.empty(wg.masked_topk_workspace(B, V, 9), dtype=torch.uint8, device="cuda"))
    want_ids, want_vals = O.masked_topk(host, masks, 9)
    assert (ids[:few].cpu().numpy() == want_ids).all() and (tok[:few].cpu().numpy() == want_ids[:, 0]).all()
    assert (H.host_logit_bits(vals[:few]) == np.ascontiguousarray(want_vals).view(np.uint32 if dtype == "f32" else np.uint16)).all()
    assert torch.equal(tok, ids[:, 0])


@pytest.mark.parametrize("dtype,byte", [("bf16", 1), ("bf16", 3), ("f32", 1), ("f32", 2), ("f32", 3)])
@pytest.mark.parametrize("B,V,pad", [(3, 1, 0), (5, 3, 1), (5, 9, 0), (5, 4097, 2), (7, 8192, 1), (6, 8193, 0), (33, 20011, 1), (40, 57347, 3), (40, 114690, 1),
                                     (9, 100003, 0), (2, 262143, 1), (2, 262149, 0)])
def test_sampling_of_rows_at_odd_bytes(torch_cuda, B, V, pad, dtype, byte):
    """masked_argmax and masked_topk where logits do not lie at multiples of their size: rows of one piece, of pieces and a part, of
    several segments of the mask, whole and in slices, through the C ABI (no tensor has such an address)."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    L, code, e = wg.load_library(), wg.F32 if dtype == "f32" else wg.BF16, 4 if dtype == "f32" else 2
    rng = np.random.default_rng(V + B + byte)
    x = rng.standard_normal((B, V + pad)).astype(np.float32)
    x[:, rng.integers(0, V, V // 20)] = np.nan
    x[0] = np.round(x[0])                                           # ties, zeros of both signs
    x[1, V - 1] = 60.0                                              # the last token, in the part of a piece
    host = x if dtype == "f32" else ws.to_bf16_bits(x)
    bits = rng.integers(0, 1 << 32, (B, (V + 31) // 32), dtype=np.uint32)
    bits[1] = 0xFFFFFFFF
    if V % 32:
        bits[:, -1] &= np.uint32((1 << (V % 32)) - 1)
    if B > 3:
        bits[3] = 0
    raw = np.concatenate([np.full(byte, 0x7F, np.uint8), np.ascontiguousarray(host).view(np.uint8).ravel(), np.full(64, 0x7F, np.uint8)])
    buf = torch.from_numpy(raw).cuda()
    assert buf.data_ptr() % 16 == 0
    mask = torch.from_numpy(bits.view(np.int32)).cuda()
    rows, stream = np.ascontiguousarray(host[:, :V]), torch.cuda.current_stream().cuda_stream
    tok = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    assert L.wg_masked_argmax(buf.data_ptr() + byte, code, B, V, V + pad, mask.data_ptr(), tok.data_ptr(), stream) == 0
    assert (tok.cpu().numpy() == O.masked_argmax(rows, bits)).all()
    for k in (1, 20, 64):
        ids = torch.empty((B, k), dtype=torch.int32, device="cuda")
        vals = torch.empty((B, k), dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
        work = torch.empty(wg.masked_topk_workspace(B, V, k), dtype=torch.uint8, device="cuda")
        assert L.wg_masked_topk(buf.data_ptr() + byte, code, B, V, V + pad, mask.data_ptr(), k, ids.data_ptr(), vals.data_ptr(),
                                work.data_ptr(), work.numel(), stream) == 0
        want_ids, want_vals = O.masked_topk(rows, bits, k)
        assert (ids.cpu().numpy() == want_ids).all(), k
        assert (H.host_logit_bits(vals) == np.ascontiguousarray(want_vals).view(np.uint32 if dtype == "f32" else np.uint16)).all(), k


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,V,off", [(5, 32768, 0), (5, 32777, 1), (39, 114688, 1), (40, 114688, 0), (5, 163840, 3), (48, 57344, 0), (56, 65537, 2),
                                     (80, 81921, 0), (64, 131071, 1), (5, 262143, 3), (5, 262144, 1)])
def test_the_k_best_where_threads_hold_one_piece_or_more(torch_cuda, B, V, off, dtype):
    """Rows of a few pieces of a thread and of many, either side of the lines between slices and whole rows; the best
    tokens all in one thread's pieces, all in neighbouring pieces, fewer numbers than k among NaNs, thousands of ties, one
    value in every piece of a thread."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    rng = np.random.default_rng(V + B + off)
    x = rng.standard_normal((B, V)).astype(np.float32)
    per = 16384 // (4 if dtype == "f32" else 2)                     # tokens from a thread's piece to its next, 1,024 threads
    x[0, 5::per] = 40.0 + np.arange(len(x[0, 5::per]))
    x[1, 1000:1100] = 50.0 + rng.standard_normal(100)
    x[2] = np.nan
    x[2, rng.integers(0, V, 9)] = 1.0
    x[3] = np.where(rng.random(V) < 0.9, 2.0, 1.0)
    x[4, 8 * 77 % V::per] = 9.0
    host = x if dtype == "f32" else ws.to_bf16_bits(x)
    bits = rng.integers(0, 1 << 32, (B, (V + 31) // 32), dtype=np.uint32) | rng.integers(0, 1 << 32, (B, (V + 31) // 32), dtype=np.uint32)
    if V % 32:
        bits[:, -1] &= np.uint32((1 << (V % 32)) - 1)
    d = H.dev_logits(host)
    buf = torch.zeros((B * (V + off) + 64,), dtype=d.dtype, device="cuda")
    view = buf[off:off + B * (V + off)].view(B, V + off)[:, :V]
    view.copy_(d)
    mask = torch.from_numpy(bits.view(np.int32)).cuda()
    for k in (20, 33, 57):
        ids = torch.empty((B, k), dtype=torch.int32, device="cuda")
        vals = torch.empty((B, k), dtype=d.dtype, device="cuda")
        work = torch.empty(wg.masked_topk_workspace(B, V, k), dtype=torch.uint8, device="cuda")
        wg.masked_topk(view, mask, ids, vals, work)
        want_ids, want_vals = O.masked_topk(host, bits, k)
        assert (ids.cpu().numpy() == want_ids).all(), k
        assert (H.host_logit_bits(vals) == np.ascontiguousarray(want_vals).view(np.uint32 if dtype == "f32" else np.uint16)).all(), k


@pytest.mark.parametrize("B,V,off", [(32, 32769, 0), (33, 32768, 0), (33, 32769, 0), (33, 32769, 3), (40, 40957, 3), (40, 40958, 3), (40, 40961, 2),
                                     (65, 50021, 1), (129, 131072, 0), (1030, 33000, 0), (32, 57345, 0), (33, 57344, 0), (33, 57345, 3), (40, 65533, 3), (40, 65537, 2)])
def test_greedy_choice_of_fp32_rows_in_slices(torch_cuda, B, V, off):
    """Rows of five and more slices of 8,192 tokens and the sizes just below, rows that begin inside a
    16-byte block (so that the last tokens make a slice of their own), maxima on either side of a slice's edge,
    ties, NaNs, both zeros, rows that allow little or nothing; twice, so that no key is left behind."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    rng = np.random.default_rng(V + B + off)
    x = rng.standard_normal((B, V)).astype(np.float32)
    x[:, rng.integers(0, V, V // 50)] = np.nan
    bits = rng.integers(0, 1 << 32, (B, (V + 31) // 32), dtype=np.uint32)
    x[0] = np.round(x[0])                                           # thousands tie, zeros of both signs
    x[1], x[2] = -np.inf, np.nan
    x[2, V // 2] = -0.0
    x[3] = np.nan
    bits[4], bits[5], bits[5, -1] = 0, 0, 1
    for r in range(6, 26):                                          # the same maximum at both sides of an edge, one or both allowed
        t = 8192 * (1 + r % ((V - 1) // 8192)) - (r % 3)
        x[r, [t - 1, t]] = 50.0
        for i, u in enumerate((t - 1, t)):
            bits[r, u // 32] |= np.uint32(1 << (u % 32))
            if r % 5 == i:
                bits[r, u // 32] ^= np.uint32(1 << (u % 32))
    x[26:29, V - 1] = 60.0
    bits[26:28, -1] |= np.uint32(1 << ((V - 1) % 32))
    if V % 32:
        bits[:, -1] &= np.uint32((1 << (V % 32)) - 1)
    buf = torch.zeros((B * (V + off) + 64,), dtype=torch.float32, device="cuda")
    view = buf[off:off + B * (V + off)].view(B, V + off)[:, :V]
    view.copy_(torch.from_numpy(x))
    mask = torch.from_numpy(bits.view(np.int32)).cuda()
    tok = torch.empty(B, dtype=torch.int32, device="cuda")
    want = O.masked_argmax(x, bits)
    for _ in range(2):
        tok.fill_(-7)
        wg.masked_argmax(view, mask, tok)
        assert (tok.cpu().numpy() == want).all(), np.flatnonzero(tok.cpu().numpy() != want)[:8]


@pytest.mark.parametrize("V,B,dtype", [(9001, 257, "f32"), (9001, 768, "bf16"), (9001, 769, "bf16"), (5003, 1024, "bf16"), (16384, 448, "bf16"), (16384, 449, "f32"),
                                       (16385, 300, "bf16"), (99999, 384, "bf16"), (100000, 384, "bf16"), (100000, 383, "f32"), (100003, 1024, "bf16"), (100003, 1025, "bf16")])
def test_batches_above_a_request_per_unit(torch_cuda, V, B, dtype):
    """Either side of the lines up to which a batch of more than 256 requests is one kernel: masks, logits and states are those of batches of 100,
    cold and cached, through each call; rows, hits and claims are counted as for any other batch."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    w = ws.make_workload(4, V=V, B=64, steps=1)
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
            if call == "step":
                h.decode_step(states, tok, mask, logits[:, :V])
            elif call == "advance_fill":
                h.advance_fill_masks(states, tok, mask)
            else:
                h.fill_masks(states, mask)
            assert torch.equal(states, want_states) and torch.equal(mask, want), (cold, call)
            assert call != "step" or torch.equal(logits.view(torch.int32 if dtype == "f32" else torch.int16), want_logits.view(torch.int32 if dtype == "f32" else torch.int16)), cold
            after = h.cache_stats()
            assert after["lookups"] - before["lookups"] == B
            assert after["hits"] - before["hits"] == (0 if cold else live)
            assert after["builds"] - before["builds"] == (after["rows_in_use"] if cold else 0), (cold, call)
            assert not cold or after["rows_in_use"] >= keys - 1
