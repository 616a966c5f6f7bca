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


def test_pair_space_is_left_to_cold_ladders(tmp_path):
    """The acceptance estimate rises with the temperature to 1, and the rule for
    pair space takes every size on a ladder of 0.25 to 1.5 and none on one of 5
    to 20, whatever the number of copies; once refused, a hotter ladder is
    refused too."""
    rows = host_check.run(tmp_path, r"""
#include <cstdio>
#include "route.hpp"
using namespace rlpt;
int main() {
    for (int rho : {4, 2}) {
        double last = 0;
        for (double T = 0.05; T < 300; T *= 1.01) {
            const double a = update_acceptance(T, rho);
            if (!(a >= last && a > 0 && a < 1)) printf("bad acceptance %g %g\n", T, a);
            last = a;
        }
    }
    std::vector<double> t(40);
    auto ladder = [&](double lo, double hi) {
        for (int i = 0; i < 40; ++i) t[i] = lo * pow(hi / lo, i / 39.0);
        return ladder_acceptance(t, 4);
    };
    const Ladder cold = ladder(0.25, 1.5), warm = ladder(1, 3), hot = ladder(5, 20);
    printf("ladders %.3f %.3f %.3f %.3f\n", cold.mean, cold.hottest, warm.mean, warm.hottest);
    for (int N = 88; N <= 256; ++N)
        for (long copies = 1; copies < 100000; copies += 1 + copies / 7)
            for (bool shared : {false, true}) {
                bool last = true;
                for (double f = 1; f < 8; f *= 1.1) {
                    const Ladder l = ladder(0.25 * f, 1.5 * f);
                    const bool now = pair_space_pays(N, copies, shared, 256, l.mean, l.hottest);
                    if (now && !last) printf("bad order %d %ld\n", N, copies);
                    last = now;
                }
                if (!pair_space_pays(N, copies, shared, 256, cold.mean, cold.hottest) ||
                    pair_space_pays(N, copies, shared, 256, hot.mean, hot.hottest))
                    printf("bad rule %d %ld %d\n", N, copies, (int)shared);
            }
}
""")
    assert [r for r in rows if r[0] == "bad"] == []
    # measured on those ladders over N and copies: 0.076-0.085, 0.25-0.28; 0.335-0.345, 0.57-0.59
    cold, hot_c, warm, hot_w = (float(x) for x in rows[0][1:])
    assert abs(cold - 0.08) < 0.02 and abs(hot_c - 0.27) < 0.03 and abs(warm - 0.34) < 0.03 and abs(hot_w - 0.58) < 0.03


def test_several_steps_are_left_to_cold_ladders(tmp_path):
    """Short lists on ladders of T = 0.25 to 1.5 take several steps at a time
    with a copy per compute unit, at any size; samples of 128 modes and more
    with short lists on ladders of 50 to 100 do not (but lists past 128 entries
    do, where a round costs less than the other sweep's step)."""
    rows = host_check.run(tmp_path, r"""
#include <cstdio>
#include "route.hpp"
using namespace rlpt;
int main() {
    std::vector<double> t(8);
    for (int prec : {RLPT_FP32, RLPT_FP64})
        for (int N = 8; N <= 1024; N += 8)
            for (unsigned longest : {100u, 250u})
                for (double f : {1.0, 100.0}) {
                    for (int i = 0; i < 8; ++i) t[i] = 0.25 * f * pow(6.0, i / 7.0);
                    AheadLaunch L{};
                    if (!ahead_plan(prec, kLayoutPacked, longest, N, &L)) continue;
                    const size_t lds = ahead_lds_bytes(prec, L);
                    for (int copies : {8, 256})
                        printf("%d %d %u %g %d %d\n", prec, N, longest, f, copies,
                               (int)ahead_pays(prec, L, lds, copies, 256, false, t, 4));
                }
}
""")
    assert all(r[5] == "1" for r in rows if r[3] == "1")
    hot = [r for r in rows if r[3] == "100" and int(r[1]) >= 128]
    assert all(r[5] == ("1" if r[2] == "250" else "0") for r in hot) and len(hot) > 800
