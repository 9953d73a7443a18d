"""GPU tests of what the per-step calls do beside their results: kernel timing and error reports."""
import numpy as np
import pytest

import wg_synth as ws
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2507_16768_amd as wg
    wg.load_library()
    return torch


def _batch(torch, B, V=20000):
    w = ws.make_workload(4, V=V, B=B, steps=2)
    o = H.make_oracle(w)
    v, h = H.make_gpu(w)
    st = H.dev_states(H.start_states(o, w))
    return w, o, h, st, torch.empty((B, h.W), dtype=torch.int32, device="cuda")


@pytest.mark.parametrize("call", ["fill", "advance_fill", "decode_step"])
def test_kernel_timing_of_batches_of_one_and_of_two_kernels(torch_cuda, call):
    """Each kernel that a fill launches is timed, and only those: a small batch (one kernel) after a large
    one (two), whose events it takes over, adds nothing to the lookup; the calls after a read succeed."""
    torch = torch_cuda
    _, _, h, st, mask = _batch(torch, 300)
    logits = torch.zeros((300, h.V), dtype=torch.bfloat16, device="cuda")
    tok = torch.full((300,), -1, dtype=torch.int32, device="cuda")
    h.profile_enable()
    for B, kernels in ((2, 1), (300, 2), (2, 1), (2, 1)):
        s, m, x, t = st[:B].clone(), mask[:B], logits[:B], tok[:B]
        for _ in range(3):
            if call == "fill":
                h.fill_masks(s, m)
            elif call == "advance_fill":
                h.advance_fill_masks(s, t, m)
            else:
                h.decode_step(s, None, m, x)
        h.advance(s, t)
        h.profile_apply_mask(x, m)
        p = h.profile_read()
        assert (p["fill_calls"], p["advance_calls"], p["apply_calls"]) == (3, 1, 1)
        assert p["build_ms"] > 0.0 and p["advance_ms"] > 0.0 and p["apply_ms"] > 0.0
        assert (p["lookup_ms"] > 0.0) == (kernels == 2), (B, p)
    h.profile_enable(False)
    h.fill_masks(st, mask)
    assert h.profile_read()["fill_calls"] == 0


@pytest.mark.parametrize("V,one", [(340001, True), (350000, False)])
def test_a_fill_without_logits_goes_by_its_own_workgroups(torch_cuda, V, one):
    """Logits that are masked by whole lines (above 208 MiB of bf16, 320 MiB of fp32) are masked behind a lookup of
    its own; a fill that masks no logits is one kernel while its workgroups are resident together."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    B = 256
    rng = np.random.default_rng(1)
    offsets = np.concatenate([[0], np.arange(257), 256 + np.cumsum(rng.integers(1, 5, V - 257))]).astype(np.uint64)
    data = np.concatenate([np.arange(256, dtype=np.uint8), rng.integers(0x20, 0x7F, int(offsets[-1]) - 256, dtype=np.uint8)])
    h = wg.Handle(['Sequence(Write("ab"), Wait(denies={}, wait={<}, max=256), Write("c"))'], None, wg.Vocab(data, offsets, 0), flags=wg.EOS_RESTART)
    st = H.dev_states(np.stack([1 + np.arange(B, dtype=np.uint32) % (h.num_states - 1), np.zeros(B, dtype=np.uint32)], 1))
    mask, want = (torch.empty((B, h.W), dtype=torch.int32, device="cuda") for _ in range(2))
    tok = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    h.profile_enable()
    for dt, kernels in ((torch.float32, 2), (torch.bfloat16, 1)):
        h.cache_clear()
        h.decode_step(st, None, want, torch.zeros((B, V), dtype=dt, device="cuda"))
        assert (h.profile_read()["lookup_ms"] > 0.0) == (kernels == 2), dt
        h.cache_clear()
        h.fill_masks(st, mask)
        assert torch.equal(mask, want)
        h.advance_fill_masks(st.clone(), tok, mask)
        p = h.profile_read()
        assert p["fill_calls"] == 2 and (p["lookup_ms"] == 0.0) == one, p


def test_errors_of_other_calls_are_not_reported_as_these(torch_cuda):
    """A call whose kernels were launched returns WG_OK, also when an earlier HIP call of the thread, made
    by somebody else, has failed: a caller who takes the step for failed would advance its states twice."""
    torch = torch_cuda
    import ctypes
    import paper_2507_16768_amd as wg
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip = ctypes.CDLL(path)                            # the runtime of this process
    w, o, h, st, mask = _batch(torch, 8)
    logits = torch.zeros((8, h.V), dtype=torch.float32, device="cuda")
    tok = torch.empty(8, dtype=torch.int32, device="cuda")
    ids, vals = torch.empty((8, 4), dtype=torch.int32, device="cuda"), torch.empty((8, 4), device="cuda")
    lens = torch.empty(8, dtype=torch.int32, device="cuda")
    out = torch.empty((8, 16), dtype=torch.uint8, device="cuda")
    draws = torch.zeros(8, dtype=torch.int64, device="cuda")
    calls = [lambda: h.fill_masks(st, mask), lambda: wg.apply_mask(logits, mask), lambda: wg.masked_argmax(logits, mask, tok),
             lambda: wg.masked_topk_static(logits, mask, ids, vals), lambda: h.forced_bytes(st, out, lens),
             lambda: wg.select_tokens(mask, h.V, draws, tok), lambda: h.advance(st, tok), lambda: h.advance_fill_masks(st, tok, mask),
             lambda: h.decode_step(st, None, mask, logits), lambda: h.add_instances(w.texts[:1], w.args[:1])]
    for i, call in enumerate(calls):
        torch.cuda.synchronize()
        ms = ctypes.c_float()
        assert hip.hipEventElapsedTime(ctypes.byref(ms), None, None) != 0        # no such events: refused by the runtime
        try:
            call()
        finally:
            hip.hipGetLastError()
    torch.cuda.synchronize()
    assert (H.host_mask(mask) == o.fill_masks(H.host_states(st))).all()


def test_start_states_of_additions(torch_cuda):
    """The start states of all instances, over additions of one and of many; what a caller took earlier stays as it was."""
    w, o, h, st, mask = _batch(torch_cuda, 8)
    want, taken = h.start_states.copy(), []
    for n in (1, 3, 8, 1, 8, 8):
        taken.append((h.start_states, want.copy()))
        want = np.concatenate([want, h.add_instances(w.texts[:n], w.args[:n])])
        assert (h.start_states == want).all() and len(h.start_states) == h.num_instances()
    assert all((a == b).all() for a, b in taken)


def test_start_states_given_out_are_the_callers(torch_cuda):
    """What a caller writes into an array that it was given before an addition is not in the handle's behind it; what it writes into
    the handle's present one is, and so is an array that it puts in its place.  Additions leave all of them as they are."""
    w, o, h, st, mask = _batch(torch_cuda, 8)
    add = lambda n: h.add_instances(w.texts[:n], w.args[:n])
    taken = []
    for n in (1, 8, 2, 40):                                            # also with additions in between that nobody looks behind
        mine, want = h.start_states, h.start_states.copy()
        for m in (n, 1, 3)[:1 + n % 3]:
            want = np.concatenate([want, add(m % 8 + 1)])
        mine[:] = 0xDEAD
        assert (h.start_states == want).all()
        taken.append((mine, np.full_like(mine, 0xDEAD)))
    h.start_states[0] = (7, 9)
    want = np.concatenate([h.start_states, add(2)])
    assert (h.start_states == want).all() and tuple(want[0]) == (7, 9)
    whole = h.start_states
    h.start_states = whole[:5]
    taken.append((whole, whole.copy()))
    want = np.concatenate([whole[:5], add(3)])
    want = np.concatenate([want, add(3)])
    assert (h.start_states == want).all()
    assert all((a == b).all() for a, b in taken)


@pytest.mark.parametrize("states", [1, 10790, 10820, 16385, 32768, 50007, 180007])
def test_additions_either_side_of_what_one_launch_uploads(torch_cuda, states):
    """1 MiB of tables, 97 bytes a state, goes to the device in one launch, more in halves of that: every state behind an addition of either kind takes tokens as the oracle's does, and so do those before it and those of an addition
    behind it, and all of them compiled at once."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    from oracle import oracle as O
    from wg_synth.vocab import from_tokens
    rng = np.random.default_rng(states)
    write = lambda n: 'Write("%s")' % bytes(rng.choice(np.frombuffer(b"ab", np.uint8), n)).decode()
    block = lambda i: "%s, Wait(denies={%s}, wait={<}, max=3)" % (write(8), "ab"[i % 2])       # nine states
    sizes = [min(9000, states - k) for k in range(0, states, 9000)]                            # an instance has an END behind its leaves
    texts = ["Sequence(%s)" % ", ".join([block(i) for i in range((n - 1) // 9)] + [write((n - 1) % 9)] * ((n - 1) % 9 > 0)) if n > 1 else 'Write("")'
             for n in sizes]
    base, last = ["Sequence(%s, %s)" % (block(0), write(3))], ["Sequence(%s, %s)" % (block(1), write(5))]
    vocab = from_tokens([b"", b"a", b"b", b"<", b"aa", b"ab", b"ba", b"bb", b"a<", b"b<a", b"abab", b"c"], eos_id=0)
    o = O.Oracle(base + texts + last, None, O.OracleVocab(vocab.bytes, vocab.offsets, vocab.eos_id), restart=True)
    v = wg.Vocab(vocab.bytes, vocab.offsets, vocab.eos_id)
    h = wg.Handle(base, None, v, flags=wg.EOS_RESTART)
    own = h.num_states
    h.add_instances(texts, None)
    assert h.num_states - own == states
    h.add_instances(last, None)
    at_once = wg.Handle(base + texts + last, None, v, flags=wg.EOS_RESTART)
    assert h.num_states == at_once.num_states == o.num_states
    st = np.zeros((h.num_states, 2), dtype=np.uint32)
    st[:, 0] = np.arange(h.num_states)
    for _ in range(4):
        tok = rng.integers(0, vocab.V, len(st)).astype(np.int32)
        want = o.advance(st, tok)
        for x in (h, at_once):
            got = H.dev_states(st)
            x.advance(got, torch.from_numpy(tok).cuda())
            assert (H.host_states(got) == want).all()
    some = rng.permutation(len(st))[:200]
    mask = torch.empty((len(some), h.W), dtype=torch.int32, device="cuda")
    for x in (h, at_once):
        x.fill_masks(H.dev_states(st[some]), mask)
        assert (H.host_mask(mask) == o.fill_masks(st[some])).all()
