"""What the kernels rely on without the hardware's or the compiler's word, checked on the source.  CPU only."""
import os
import re

from paper_2507_16768_amd import build

KERNELS = os.path.join(build.CSRC, "wg_kernels.hip")


def _body(text, name):
    """The text of a function template, from its name to the closing brace in the first column."""
    at = text.index("\n%s(" % name)
    return text[at:text.index("\n}\n", at)]


def test_words_of_lds_are_not_rewritten_while_they_are_read():
    """Between two barriers of a row's lookup no word that one wavefront assigns is read by the others."""
    body = _body(open(KERNELS).read(), "rows_kernel")
    lookup = body[body.index("if (kWhole) {"):body.index("const RowTask in")]
    for part in lookup.split("__syncthreads();"):
        part = re.sub(r"//.*", "", part)
        written = set(re.findall(r"\bsh\.(\w+) = ", part))
        read = set(re.findall(r"\bsh\.(\w+)(?! = )\b", part))
        assert not written & read, (written & read, part)
