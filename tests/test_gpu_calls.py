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
