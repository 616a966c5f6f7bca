"""CPU: the launches the host plans fit the hardware, over all sizes."""
from tests import host_check


def test_several_steps_launch_fits_the_kernels_that_serve_it(tmp_path):
    """Every plan of the sweep of short lists asks for at most a workgroup's
    160 KiB of LDS with the workgroup that is launched: 512 threads, and for
    lists of up to 128 packed entries also 256 or 1024.  Sizes that do not fit
    are refused (FP64, N = 995 and more, lists past 128 entries)."""
    rows = host_check.run(tmp_path, r"""
#include <cstdio>
#include "ahead.hpp"
using namespace rlpt;
int main() {
    for (int prec : {RLPT_FP32, RLPT_FP64})
        for (int layout : {kLayoutPacked, kLayoutChunked})
            for (int N = 4; N <= (layout == kLayoutChunked ? 256 : 1024); ++N)
                for (unsigned longest = 1; longest <= 600; longest += longest < 130 ? 1 : 7) {
                    AheadLaunch L{};
                    const bool ok = ahead_plan(prec, layout, longest, N, &L);
                    // the layout of the kernel's LDS: draws, decisions, list bounds, a copy of the amplitudes per wave
                    const size_t real = prec == RLPT_FP64 ? 8 : 4, w = L.block / 64;
                    const size_t fixed = (size_t)(N / 2) * (real == 8 ? 64 : 32) + w * 10 * real + w * 8 + (N + 1) * 4;
                    const size_t lds = (fixed + 15) / 16 * 16 + w * N * 2 * real;
                    const bool is_short = layout == kLayoutPacked && L.slots <= kShortSlots;
                    if (ok && (lds > 160 * 1024 || lds != ahead_lds_bytes(prec, L) || (!is_short && L.block != 512) ||
                               (L.block != 256 && L.block != 512 && L.block != 1024)))
                        printf("bad %d %d %d %u %d %zu\n", prec, layout, N, longest, L.block, lds);
                    if (layout == kLayoutPacked && prec == RLPT_FP64 && longest == 298 && N >= 993 && N <= 996)
                        printf("edge %d %d\n", N, (int)ok);
                    if (layout == kLayoutPacked && N == 1024 && longest == 100) printf("short %d %d %d\n", prec, (int)ok, L.block);
                }
}
""")
    assert [r for r in rows if r[0] == "bad"] == []
    assert [r[1:] for r in rows if r[0] == "edge"] == [["993", "1"], ["994", "1"], ["995", "0"], ["996", "0"]]
    assert [r[1:] for r in rows if r[0] == "short"] == [["0", "1", "1024"], ["1", "1", "256"]]
