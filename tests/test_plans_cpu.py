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


def test_energy_ranges_fit_a_workgroup(tmp_path):
    """The ranges of the banded energy recomputation fit a workgroup's LDS (the
    amplitudes of 16 copies, 4 B per pair of a range, 512 B of sums) at every N
    and number of copies, with partial energies that the entry point without
    allocations has room for (its limit of 32768 copies)."""
    rows = host_check.run(tmp_path, r"""
#include <cstdio>
#include "internal.hpp"
using namespace rlpt;
int main() {
    for (int N : {4, 5, 17, 64, 128, 200, 229, 230, 243, 255, 256}) {
        rlpt_graph_desc d{};
        d.n_modes = N;
        d.omega_kind = N == 4 ? RLPT_OMEGA_COMB : RLPT_OMEGA_RANDOM;
        d.seed = 2511135081;
        d.split_mask = RLPT_SPLIT_ALL;
        rlpt_graph* g = nullptr;
        if (rlpt_graph_build(&d, &g)) return 1;
        for (int prec : {RLPT_FP32, RLPT_FP64})
            for (int reps : {1, 50, 1000, 32768, 65536, 131072, 131073, 262144, 262145, 1 << 22}) {
                rlpt_config c;
                rlpt_config_default(&c);
                c.n_reps = reps;
                c.precision = prec;
                const int parts = energy_parts(c, &g, 1);
                const int tiles = (N * (N - 1) / 2 + 15) / 16;
                size_t lds = 0;  // as the kernel lays it out
                for (int p = 0; p < parts; ++p) {
                    const int t0 = (int)((long)tiles * p / parts), t1 = (int)((long)tiles * (p + 1) / parts);
                    if (t0 == t1) continue;
                    const size_t n = 16 * (t1 - t0) + 4 * (g->energy_tile[t1] - g->energy_tile[t1 - 1]);
                    const size_t b = (size_t)N * 16 * (prec == RLPT_FP64 ? 16 : 8) + 4 * n + 512;
                    if (b > lds) lds = b;
                }
                const bool scratch = reps > 32768 || (size_t)reps * parts * 8 <= kStaticScratchBytes;
                printf("%d %d %d %d %d %d\n", N, prec, reps, parts, (int)(lds <= 160 * 1024), (int)scratch);
            }
        rlpt_graph_free(g);
    }
}
""")
    assert len(rows) == 11 * 2 * 10
    assert [r for r in rows if int(r[3]) < 1 or int(r[3]) > 64 or r[4] == "0" or r[5] == "0"] == []
