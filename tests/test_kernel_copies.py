"""gn_shared_kernel writes out gn_kernel's per-iteration arithmetic (register
allocation; gn_kernel's covers split columns and several groups too): the
statements must stay the same, in the same order."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KERNELS = os.path.join(ROOT, "paper_1910_01997_amd", "csrc", "sgn_kernels.hip")


def _statements(text):
    text = " ".join(re.sub(r"//.*|^\s*#.*", "", line).strip() for line in text.splitlines())
    return [re.sub(r"\s+", " ", s).strip() for s in re.split(r"(?<=[;{}])", text) if s.strip()]


def _between(src, start, first, last):
    a = src.index(first, src.index(start))
    return _statements(src[a:src.index(last, a)])


def _in_order(part, whole):
    """The statements of part that are not, in order, among whole's."""
    at, missing = 0, []
    for s in part:
        if s in whole[at:]:
            at = whole.index(s, at) + 1
        else:
            missing.append(s)
    return missing


def test_shared_kernel_linearises_as_gn_kernel_does():
    src = open(KERNELS).read()
    gn = _between(src, "void gn_kernel(", "const float4 sa = *(const float4*)(st + 0);", "// owner_step body begin")
    assert len(gn) > 100
    # the pixels' plane: sigma and its step down the column
    plane = _between(src, "void gn_shared_kernel(", "const float4 sa = *(const float4*)(st + 0);", "for (int j")
    assert len(plane) > 6 and _in_order(plane, gn) == []
    # the Jacobians and the normal equations of a lane's pixels
    sums = _between(src, "void gn_shared_kernel(", "const float4 sa2 = *(const float4*)(st + 0);", "pnv = (float)")
    sums = [s.replace("hdr->depth_only != 0 ?", "depth_only ?") for s in sums]
    assert len(sums) > 40 and _in_order(sums, gn) == []
    # the reduction over a surfel's lanes
    join = _between(src, "void gn_shared_kernel(", "const bool odd = (p & 1) != 0;", "if (last) {")
    join = [re.sub(r"^const float (s\d = pair_sum)<LANES>", r"\1<RL>", s) for s in join]
    join = [s.replace("lsm + r * SM_WORDS", "lsm + (k * SLOTS + r) * SM_WORDS").replace(
        "if (LANES == 4 || p < 2) {", "if (LANES == 4 || p < (RL == 4 ? 4 : 2)) {") for s in join]
    assert len(join) > 10 and _in_order(join, gn) == []
