"""The native module behind the binding, where it can be tested without a GPU: tensors that have no storage
to point to, and argument objects that are only held by what the caller passed."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

NO_STORAGE = r"""
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
import paper_2507_16768_amd as wg
from paper_2507_16768_amd import binding
binding.load_library()
n = binding._native
B, V, W, k = 4, 64, 2, 3
with FakeTensorMode(allow_non_fake_inputs=True):
    i32 = dict(dtype=torch.int32, device="cuda")
    # a batched tensor under vmap counts as a device tensor and has no storage of its own
    given = dict(states=torch.empty((5, B, 2), **i32), tokens=torch.empty((5, B), **i32), mask=torch.empty((5, B, W), **i32),
                 ids=torch.empty((5, B, k), **i32), logits=torch.empty((5, B, V), device="cuda"), values=torch.empty((5, B, k), device="cuda"),
                 work=torch.empty((5, 4096), dtype=torch.uint8, device="cuda"), out=torch.empty((5, B, 8), dtype=torch.uint8, device="cuda"),
                 draws=torch.empty((5, B), dtype=torch.int64, device="cuda"))
    CALLS = {
        "fill_masks": (("states", "mask"), lambda states, mask: n.fill_masks(0, W, states, mask, 0)),
        "advance": (("states", "tokens"), lambda states, tokens: n.advance(0, states, tokens, 0)),
        "advance_fill_masks": (("states", "tokens", "mask"), lambda states, tokens, mask: n.advance_fill_masks(0, W, states, tokens, mask, 0)),
        "decode_step": (("states", "tokens", "mask", "logits"),
                        lambda states, tokens, mask, logits: n.decode_step(0, W, V, states, tokens, mask, logits, 0)),
        "forced_bytes": (("states", "out", "tokens"), lambda states, out, tokens: n.forced_bytes(0, states, out, tokens, None, 0)),
        "apply_mask": (("logits", "mask"), lambda logits, mask: wg.apply_mask(logits, mask, 0)),
        "masked_argmax": (("logits", "mask", "tokens"), lambda logits, mask, tokens: wg.masked_argmax(logits, mask, tokens, 0)),
        "masked_topk": (("logits", "mask", "ids", "values", "work"),
                        lambda logits, mask, ids, values, work: wg.masked_topk(logits, mask, ids, values, work, 0)),
        "masked_topk_static": (("logits", "mask", "ids", "values"),
                               lambda logits, mask, ids, values: wg.masked_topk_static(logits, mask, ids, values, 0)),
        "select_tokens": (("mask", "draws", "tokens"), lambda mask, draws, tokens: wg.select_tokens(mask, V, draws, tokens, 0)),
    }
    for name, (names, call) in CALLS.items():
        for batched in names:                          # one argument at a time, then all
            for which in ((batched,), names):
                def body(*xs):
                    call(**{a: (xs[which.index(a)] if a in which else given[a][0]) for a in names})
                    return xs[0]
                try:
                    torch.func.vmap(body)(*[given[a] for a in which])
                    print(name, which, "returned")
                except RuntimeError as e:
                    assert not isinstance(e, wg.WgError), (name, which, e)
                    assert "storage" in str(e), (name, which, e)
    print("done")
"""


def test_tensors_without_storage_raise_instead_of_ending_the_process():
    """Asking such a tensor for its address throws in C++; the error has to arrive as an exception, with the
    interpreter's lock held, whichever argument it is."""
    r = subprocess.run([sys.executable, "-c", NO_STORAGE], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.split() == ["done"], (r.returncode, r.stdout, r.stderr[-2000:])


def test_arguments_of_add_instances_are_held_through_the_call():
    """The C call reads texts, names and values where they lie, so each is held whatever happens to the
    caller's list and dictionaries meanwhile: here a value's own conversion to bytes empties them."""
    import numpy as np
    import paper_2507_16768_amd as wg
    from paper_2507_16768_amd import binding
    binding.load_library()
    made = {k: "".join([k, "_of_this_test"]) for k in ("text", "name")}       # strings that nothing else refers to
    value = bytes(bytearray(b"a literal of its own"))
    texts, d = [made["text"], "Sequence(Write($x))"], {}
    args = [d, {"x": b"1"}]
    held = {}

    class Value:
        def __bytes__(self):
            d.clear(); args.clear(); texts.clear()
            held.update({k: sys.getrefcount(o) - 2 for k, o in made.items()}, value=sys.getrefcount(value) - 2)
            return b"2"

    d.update({made["name"]: value, "last": Value()})
    starts = np.zeros((2, 2), dtype=np.uint32)
    with pytest.raises(wg.WgError, match="null handle"):
        binding._native.add_instances(0, texts, args, starts.ctypes.data, 2, 0)
    # (beside the reference that this test itself has to each: `made`, the local `value`)
    assert held["text"] >= 2 and held["name"] >= 2 and held["value"] >= 1, held
    assert sys.getrefcount(value) == 2                                        # and let go of afterwards


def test_add_instances_takes_no_more_templates_than_it_has_room_for():
    import numpy as np
    from paper_2507_16768_amd import binding
    binding.load_library()
    starts = np.zeros((2, 2), dtype=np.uint32)
    with pytest.raises(ValueError, match="rows"):
        binding._native.add_instances(0, ["Sequence(Write(\"a\"))"] * 2, None, starts.ctypes.data, 1, 0)
