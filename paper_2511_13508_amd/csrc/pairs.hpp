// Pair-space sweep: tables and launchers.  A term conj(a_p) conj(a_s) a_m a_n
// couples the pair products a_p a_s and a_m a_n, and the frequency-matching
// filter keeps it when the pairs' frequency sums differ by less than gamma.
// With the N (N - 1) / 2 pairs sorted by that sum the couplings form a narrow
// band, and every local field (eq. local field, sec. III.A of Benedetti &
// Leuzzi, arXiv 2511.13508) follows from one banded product:
//   G_{lx} = sum over the band of J a_y a_z,   F_l = sum_x conj(a_x) G_{lx}.
// Each coupling is used twice per evaluation of all N fields instead of four
// times, with no index to read, and the products a_y a_z are formed once.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.hpp"

namespace rlpt {

constexpr int kPairTile = 32;   // rows of the band that share their columns (two matrix-core tiles)
constexpr int kCopyTile = 16;   // copies of one sample per matrix-core tile
constexpr int kListUnit = 16;      // entries padded and read together
constexpr int kStartBits = 13;     // of a list's start in its descriptor; the rest holds its role-0 units / 2
constexpr int kGatherModes = 136;  // up to here a copy's banded product fits the decisions' LDS

// one sample's pair tables
struct PairSample {
    int32_t N;
    int32_t n_pairs;
    int32_t n_tiles;       // ceil(n_pairs / 32)
    int32_t pad;
    int64_t pm_base;       // pairs by rank: p | s << 8
    int64_t pos_base;      // [N][N] rank of pair {l, x}
    int64_t tile_base;     // [n_tiles] offset in the band, first column | columns / 4 << 16
    int64_t band_base;     // band values
    int64_t prod_base;     // the banded product of the sample's copies
    int64_t desc_base;     // [N][N + 1] lists of source j by target l: their start in j's units | role-0 units / 2 << 13
    int64_t list_base;     // byte offset of the lists, source by source; the first unit is zero
};

// One term holding source j and target l: the other two members p1 | p2 << 8
// and the coupling J.  Role 0 (j is l's partner): F_l changes by J conj(d_j)
// a_p1 a_p2; role 1: by J conj(a_p1) d_j a_p2.  A list holds its role-0
// entries, padded with J = 0 to 32, then its role-1 entries, padded to 16.  The
// entries of a unit of 16 are stored as 16 p, then 16 J: 6 bytes each (8: 748 us, not 674, for
// the decisions of N = 256, 640 copies).
constexpr int kUnitBytes = kListUnit * 6, kUnitJ = kListUnit * 2;  // of a unit; where its J begin

// one step's draws: StepDraw<float>, opaque to the host
constexpr size_t kPairDrawBytes = 32;

struct PairDev {
    const PairSample* samples;
    const ItemDev* items;  // one copy each, hottest temperature slot first
    const uint16_t* pm;
    const uint16_t* pos;
    const uint2* tile;
    const uint32_t* first;  // first unit of each source, at the sample's list bounds
    float* band;
    uint16_t* desc;
    unsigned char* list;
    // per sweep: the banded product, the fields it gives, the draws, the
    // targets by latest need and their number per step
    float2* prod;     // [copy][pair] (N <= kGatherModes) or [copy / 16][pair][16]
    float2* fields;   // [copy][N], laid out as the amplitudes (N > kGatherModes)
    void* draws;      // [copy][max steps] StepDraw<float>
    uint16_t* order;  // [copy][max N]
    uint16_t* after;  // [copy][max steps + 1], the last: how many modes the sweep uses
    int32_t max_N;
    int32_t max_steps;
};

// what one launch covers: items [first, first + n), copies of samples of any N
// up to the launch's N on the same side of kGatherModes; N sizes the grid and
// the LDS, each block reads its own sample's
struct PairLaunch {
    int N, first, n;
    int threads;  // per workgroup of the decisions
    int samples;  // the launch's samples: every `samples`-th item is of one of them
    int columns;  // most columns (and 4) that the row tiles of one product workgroup span
};

int pairs_product_waves(int N);   // waves per workgroup of the banded product
int pairs_tiles_per_wave(int N);  // row tiles per wave of the banded product
int pairs_decide_threads(int N, int copies, int cus);

// fills band, desc and list of every sample (on the stream) from the context's
// lists and by-term arrays; band and list must hold zeros
hipError_t launch_pairs_tables(const DevPtrs<float>& P, const PairDev& Q, const ShapeInfo& sh, int n_samples, int max_N,
                               int64_t max_quads, hipStream_t st);
// one sweep of the launch's copies, `ahead` sweeps after the counters'
hipError_t launch_pair_fields(const DevPtrs<float>& P, const PairDev& Q, const ShapeInfo& sh, const PairLaunch& L,
                              int ahead, hipStream_t st);
hipError_t launch_pair_decide(const DevPtrs<float>& P, const PairDev& Q, const ShapeInfo& sh, const PairLaunch& L,
                              hipStream_t st);

}  // namespace rlpt
