"""Index and threshold arithmetic of the kernels, checked by the compiler on the
functions that they use: the kept prefixes that a tile's blocks load lie inside
the trace's own sample area, for every number of segments and first bit of a
segment mask, and the 32-bit threshold test agrees with the 64-bit one."""
import os
import subprocess

import pytest

from paper_2212_07597_amd import _build

SOURCE = """
#include "sampler_device.h"
using namespace smp;

// every block of every tile of a trace of nseg segments
constexpr bool inside(int nseg) {
    const uint64_t n = (uint64_t)(nseg - 1) * SEG + 1;                        // the shortest such trace
    const uint64_t kept = (n + 1) * sizeof(Sample) / (SEG * sizeof(int64_t));  // segments that its sample area can keep
    int built = 0;
    for (int k = 0; k * TILE < nseg; ++k) {
        const int nval = nseg - k * TILE < TILE ? nseg - k * TILE : TILE;
        for (int b = 0; b < TWAVES; ++b) {
            const int nb = block_segments(nval, b);
            if (nb < 0 || nb > 64) return false;
            built += nb;
            if (nb == 0) continue;
            for (int i = -1; i < nb; ++i) {  // none left, or the first left is i
                const uint64_t sims = i < 0 ? 0 : 1ull << i;
                const int64_t j = next_kept((int64_t)k * TILE + b * 64, sims);
                if (j < 0 || j >= nseg || (uint64_t)j >= kept) return false;
            }
        }
    }
    return built == nseg;
}
template <int LO, int HI>
constexpr bool all_inside() {
    for (int s = LO; s < HI; ++s)
        if (!inside(s)) return false;
    return true;
}
static_assert(all_inside<8, 80>() && all_inside<80, 151>() && all_inside<500, 530>() && all_inside<1020, 1030>(), "");
"""


BEYOND = """
#include "sampler_device.h"
using namespace smp;

// against the same comparison in 64 bits, at the ends of the range and around T (a signed overflow would not compile)
constexpr bool same(int32_t T) {
    const int32_t ends[] = {-(1 << 30) + 1, -(1 << 30) + 2, -T - 1, -T, -T + 1, -1, 0, 1, T - 1, T, (1 << 30) - 2, (1 << 30) - 1};
    for (int32_t v : ends)
        for (int32_t ref : ends) {
            const int64_t d = (int64_t)v - ref;
            if (beyond32(v, ref, T) != (d >= T || -d >= T)) return false;
        }
    return true;
}
static_assert(same(1) && same(2) && same(1 << 20) && same((1 << 30) / 3 * 2) && same((1 << 30) - 2) && same((1 << 30) - 1), "");
"""


@pytest.mark.skipif(not os.path.exists(_build.HIPCC), reason="no hipcc")
@pytest.mark.parametrize("text", [SOURCE, BEYOND], ids=["bounds", "threshold"])
def test_arithmetic(tmp_path, text):
    src = tmp_path / "check.hip"
    src.write_text(text)
    flags = [f for f in _build.HIP_FLAGS if f not in ("-shared", "-fPIC")]
    r = subprocess.run([_build.HIPCC, *flags, "-fconstexpr-steps=100000000", "-I", os.path.join(_build.PKG, "csrc"), "-I",
                        os.path.join(_build.ROOT, "include"), "--cuda-device-only", "-fsyntax-only", str(src)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_blocks_without_segments_load_nothing():
    """The block map's builder leaves before its first load."""
    with open(os.path.join(_build.PKG, "csrc", "sampler_kernels.hip")) as f:
        text = f.read()
    body = text[text.index(" build_block("):text.index(" block_source(")]
    assert 0 < body.find("if (nb == 0) return") < body.index("load_kept32(")
