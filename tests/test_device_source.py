"""What the kernels rely on without the hardware's or the compiler's word, checked on the source and on the code that the compiler
makes of it: where arguments lie, what is waited for before a barrier, which words of LDS are exchanged between barriers.  CPU only."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2507_16768_amd import build

KERNELS = os.path.join(build.CSRC, "wg_kernels.hip")


def _compile(source, *more):
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC") and not f.startswith("-Wl,")]
    return subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + ["--cuda-device-only"] + list(more) + [source],
                          capture_output=True, text=True, timeout=300)


def _body(text, name):
    """The text of a function template, from its name to the closing brace in the first column."""
    at = text.index("\n%s(" % name)
    return text[at:text.index("\n}\n", at)]


@pytest.mark.parametrize("old,new", [("uint32_t n_states, uint32_t V, LateArgs", "uint32_t n_states, uint32_t V, uint32_t more, LateArgs"),
                                     ("const uint8_t *len8, uint32_t n_states", "uint32_t n_states"),
                                     ("struct LateArgs {", "struct alignas(16) LateArgs {")])
def test_arguments_that_would_lie_elsewhere_do_not_compile(tmp_path, old, new):
    """The late arguments are read at an offset behind the early ones, and the early ones are in registers: one more, one less and a
    wider alignment are refused."""
    shutil.copytree(build.CSRC, tmp_path / "library" / "csrc")
    shutil.copytree(os.path.join(build.HERE, "..", "include"), tmp_path / "include")
    path = tmp_path / "library" / "csrc" / "wg_kernels.hip"
    text = path.read_text()
    assert text.count(old) == 1
    path.write_text(text.replace(old, new))
    r = _compile(str(path), "-fsyntax-only")
    assert r.returncode != 0 and "early arguments" in r.stderr, r.stderr[-2000:]


def test_a_row_is_not_written_back_before_it_is_read(tmp_path):
    """The last workgroup of a row to take its ticket writes the row's state while others are still at work: what each reads of the state has to
    have arrived before its ticket counts, which is behind the first barrier."""
    head = _body(open(KERNELS).read(), "rows_kernel").split("__syncthreads();")[0]
    waits = [line for line in head.splitlines() if "asm volatile" in line]
    assert len(waits) == 1 and all('"s"(%s)' % x in waits[0] for x in ("launch", "sid", "aux")), waits
    out = str(tmp_path / "kernels.s")
    r = _compile(KERNELS, "-S", "-o", out)
    assert r.returncode == 0, r.stderr[-2000:]
    text = open(out).read()
    names = re.findall(r"^(_ZN2wg11rows_kernelI.*Lb1EE\S*):", text, re.M)
    assert len(names) == 5
    for name in names:
        at = text.index("\n%s:" % name)
        code = [line.split(";")[0].strip() for line in text[at:text.index("s_barrier", at)].splitlines()]
        code = [c for c in code if c]
        for load, count in ((("s_load", "ds_"), "lgkmcnt(0)"), (("global_load", "flat_load", "buffer_load"), "vmcnt(0)")):
            last = max([i for i, c in enumerate(code) if c.startswith(load)], default=-1)
            assert last < 0 or any(c.startswith("s_waitcnt") and count in c for c in code[last:]), (name, count)


def test_words_of_lds_are_not_rewritten_while_they_are_read():
    """Between two barriers of a row's lookup no word that one wavefront assigns is read by the others."""
    body = _body(open(KERNELS).read(), "rows_kernel")
    lookup = body[body.index("if (kWhole) {"):body.index("const RowTask in")]
    for part in lookup.split("__syncthreads();"):
        part = re.sub(r"//.*", "", part)
        written = set(re.findall(r"\bsh\.(\w+) = ", part))
        read = set(re.findall(r"\bsh\.(\w+)(?! = )\b", part))
        assert not written & read, (written & read, part)
