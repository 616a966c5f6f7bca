// Pair-space sweep for CDNA4 (gfx950): all local fields of a copy from one
// banded product per sweep, then the sweep's two-mode updates decided in
// batches, the fields corrected where an accepted update changes them.
// Method: Benedetti & Leuzzi, arXiv 2511.13508, sec. III.A (the same chain
// and draws as the list-streaming sweep of kernels.hip).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"
#include "pairs.hpp"

namespace rlpt {
namespace {

// ---------------------------------------------------------------- tables
static_assert(sizeof(StepDraw<float>) == kPairDrawBytes, "draws as the host sizes them");

// place of (row, column) in the band, the matrix-core operand of 4 columns:
// lane (column % 4) * 16 + row % 16 holds its value in the first and in the
// second 16 rows of the tile
__device__ inline size_t band_at(const PairDev& Q, const PairSample& ps, uint32_t row, uint32_t col) {
    const uint2 b = Q.tile[ps.tile_base + (row >> 5)];
    const uint32_t c = col - (b.y & 0xffffu);
    return (size_t)b.x + 2 * ((size_t)(c >> 2) * 64 + (c & 3u) * 16 + (row & 15u)) + ((row >> 4) & 1u);
}

// the two off-diagonal places of every term in the band
__global__ __launch_bounds__(256) void k_band_fill(DevPtrs<float> P, PairDev Q) {
    const PairSample ps = Q.samples[blockIdx.y];
    if (ps.N == 0) return;  // a sample swept from its lists
    const SampleDev sd = P.samples[blockIdx.y];
    const ushort4* quads = P.quads + sd.quad_base;
    const double* Jq = P.Jq + sd.quad_base;
    const uint16_t* pos = Q.pos + ps.pos_base;
    float* band = Q.band + ps.band_base;
    for (int64_t q = blockIdx.x * (int64_t)256 + threadIdx.x; q < sd.n_quads; q += (int64_t)gridDim.x * 256) {
        const ushort4 t = quads[q];
        const float J = (float)Jq[q];
        const uint32_t u = pos[t.x * ps.N + t.y], v = pos[t.z * ps.N + t.w];
        band[band_at(Q, ps, u, v)] = J;
        band[band_at(Q, ps, v, u)] = J;
    }
}

constexpr int kListTile = 1024;

// entries of source l (one block each) by target j, in the order of l's list
template <int LAYOUT>
__global__ __launch_bounds__(256) void k_list_fill(DevPtrs<float> P, PairDev Q) {
    __shared__ uint32_t cnt[2][256];
    __shared__ uint32_t tv[kListTile];
    __shared__ float tj[kListTile];
    const PairSample ps = Q.samples[blockIdx.y];
    const SampleDev sd = P.samples[blockIdx.y];
    const int N = ps.N, l = blockIdx.x, j = threadIdx.x;
    if (l >= N) return;
    uint32_t beg, end;  // packed: entries; chunked: 4 entries per chunk
    if constexpr (LAYOUT == kLayoutChunked) {
        beg = 4 * P.chunk_start[sd.mode_base + l];
        end = 4 * P.chunk_start[sd.mode_base + l + 1];
    } else {
        beg = P.mode_start[sd.mode_base + l];
        end = P.mode_start[sd.mode_base + l + 1];
    }
    auto stage = [&](uint32_t t0) {  // entries [t0, t0 + tile) as x | y << 8 | z << 16 (padding: J = 0)
        for (uint32_t i = threadIdx.x; i < kListTile; i += 256) {
            const uint32_t e = t0 + i;
            uint32_t v = 0;
            float J = 0;
            if (e < end) {
                if constexpr (LAYOUT == kLayoutChunked) {
                    const uint2 yz = P.cyz[e >> 2];
                    const uint32_t w = (e & 2u) ? yz.y : yz.x;
                    v = (uint32_t)P.cx[e >> 2] | ((e & 1u) ? w >> 16 : w & 0xffffu) << 8;
                    J = P.cJ[e];
                } else {
                    const uint32_t p = P.idx[e];
                    v = (p & 255u) | ((p >> 10) & 255u) << 8 | ((p >> 20) & 255u) << 16;
                    J = P.J[e];
                }
            }
            tv[i] = v;
            tj[i] = J;
        }
    };
    cnt[0][j] = 0;
    cnt[1][j] = 0;
    for (uint32_t t0 = beg; t0 < end; t0 += kListTile) {
        __syncthreads();
        stage(t0);
        __syncthreads();
        for (int i = threadIdx.x; i < kListTile; i += 256)
            if (tj[i] != 0.0f) {
                atomicAdd(&cnt[0][tv[i] & 255u], 1u);
                atomicAdd(&cnt[1][(tv[i] >> 8) & 255u], 1u);
                atomicAdd(&cnt[1][tv[i] >> 16], 1u);
            }
    }
    __syncthreads();
    uint32_t at = 0;  // start of target j's list in l's units
    for (int i = 0; i < j; ++i) at += (cnt[0][i] + 31) / 32 * 2 + (cnt[1][i] + 15) / 16;
    const uint32_t n0 = (cnt[0][j] + 31) / 32, n1 = (cnt[1][j] + 15) / 16;
    if (j < N) {
        uint16_t* d = Q.desc + ps.desc_base + (int64_t)l * (N + 1);
        d[j] = (uint16_t)(at | n0 << kStartBits);
        if (j == N - 1) d[N] = (uint16_t)(at + 2 * n0 + n1);
    }
    unsigned char* list = Q.list + ps.list_base + (size_t)kUnitBytes * (Q.first[sd.mode_base + l] + at);
    uint32_t next0 = 0, next1 = 32 * n0;  // the padding of both roles holds zeros already
    const auto put = [&](uint32_t e, uint32_t p, float J) {
        unsigned char* unit = list + (size_t)kUnitBytes * (e / kListUnit);
        reinterpret_cast<uint16_t*>(unit)[e % kListUnit] = (uint16_t)p;
        reinterpret_cast<float*>(unit + kUnitJ)[e % kListUnit] = J;
    };
    for (uint32_t t0 = beg; t0 < end; t0 += kListTile) {
        __syncthreads();
        stage(t0);
        __syncthreads();
        if (j < N)
            for (int i = 0; i < kListTile; ++i) {
                const uint32_t v = tv[i];
                const float J = tj[i];
                if (J == 0.0f) continue;
                const uint32_t x = v & 255u, y = (v >> 8) & 255u, z = v >> 16;
                if (x == (uint32_t)j)  // l is the target's partner
                    put(next0++, y | z << 8, J);
                else if (y == (uint32_t)j || z == (uint32_t)j)  // the target's partner is the other of y and z
                    put(next1++, (y == (uint32_t)j ? z : y) | x << 8, J);
            }
    }
}

// ---------------------------------------------------------------- draws
// The state-independent part of one copy's sweep: every step's draws (four
// waves: the pair, the two phases, the magnitudes and the uniform), and the
// modes whose fields later steps read: order holds the sweep's modes by the
// last step that uses them, latest first, and after[s] says how many of them
// are used after step s.  need: N + N / 2 ints of LDS.
template <int BLOCK>
__device__ inline void draw_sweep(const PairDev& Q, const ShapeInfo& sh, int sample, int c, int64_t sweep, int N,
                                  int* need) {
    const int steps = N / 2, tid = threadIdx.x, lane = tid & 63;
    const int64_t pair_stream = sh.shared_pairs ? (int64_t)sample : (int64_t)c;
    StepDraw<float>* tab = static_cast<StepDraw<float>*>(Q.draws) + (size_t)c * Q.max_steps;
    uint16_t* order = Q.order + (size_t)c * Q.max_N;
    uint16_t* after = Q.after + (size_t)c * (Q.max_steps + 1);
    int* pair = need + N;
    for (int i = tid; i < N; i += BLOCK) need[i] = -1;
    __syncthreads();
    for (int i = tid; i < 4 * ((steps + 63) & ~63); i += BLOCK) {
        const int s = (i & 63) | (i >> 8) << 6, part = (i >> 6) & 3;
        if (s >= steps) continue;
        if (part == 0) {
            const int jk = draw_pair(sh.run_seed, pair_stream, sweep, s, N);
            tab[s].jk = jk;
            pair[s] = jk;
            atomicMax(&need[jk & 0xffff], s);
            atomicMax(&need[jk >> 16], s);
        } else {
            draw_part<float>(sh.run_seed, c, sweep, s, sh.rho, part, tab[s]);
        }
    }
    __syncthreads();
    if (tid >= 64) return;
    int run = 0;
    for (int top = steps - 1; top >= 0; top -= 64) {
        const int s = top - lane;
        int j = 0, k = 0;
        bool lj = false, lk = false;
        if (s >= 0) {
            j = pair[s] & 0xffff;
            k = pair[s] >> 16;
            lj = need[j] == s;
            lk = need[k] == s;
        }
        const unsigned long long below = (1ull << lane) - 1, mj = __ballot(lj), mk = __ballot(lk);
        const int at = run + __popcll(mj & below) + __popcll(mk & below);
        if (s >= 0) after[s] = (uint16_t)at;
        if (lj) order[at] = (uint16_t)j;
        if (lk) order[at + (lj ? 1 : 0)] = (uint16_t)k;
        run += __popcll(mj) + __popcll(mk);
    }
    if (lane == 0) after[steps] = (uint16_t)run;
}

// ---------------------------------------------------------------- fields
// The banded product of kCopyTile copies of one sample on the matrix cores:
// G = J b, J real (rows: pairs), b the pair products (columns: copies, their
// real and imaginary parts in two tiles).  A wave takes 32 rows at a time, so
// each product, formed from the amplitudes in LDS, feeds two row tiles.
// v_mfma_f32_16x16x4_f32: FP32 operands and accumulation.
// Blocks past the product's draw the copies' sweeps.
// It takes twice the time of its matrix-core products (4 of 32 cycles per 4
// columns of a wave's 32 rows); what a wave issues between them, 3 LDS reads and the
// operands they form, is the rest, so that is kept off the vector ALU where it can be
// (scalar tile, immediate offsets) and the loads in flight.  Eight waves share the amplitudes of large
// N: six waves per SIMD instead of four.  N = 256, 640 copies of 8 samples (the
// draws included): 166 us as first written, 149 with
// scalar addresses, 137 with eight waves (68 at the matrix cores' rate).
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_pair_product(DevPtrs<float> P, PairDev Q, ShapeInfo sh, int first_item,
                                                      int samples, int groups, int n_product, int per_wave, int ahead) {
    extern __shared__ __align__(16) unsigned char smem[];
    if ((int)blockIdx.x >= n_product) {
        const ItemDev it = Q.items[first_item + blockIdx.x - n_product];
        draw_sweep<BLOCK>(Q, sh, it.sample, it.first_copy, P.counters->sweeps_done + ahead, Q.samples[it.sample].N,
                               reinterpret_cast<int*>(smem));
        return;
    }
    // the launch's samples in turn (so that an XCD, which takes every eighth
    // block, reads few samples' bands), their copy tiles, then the rows
    const int sample = Q.items[first_item + blockIdx.x % samples].sample;
    const int group = (blockIdx.x / samples) % groups, chunk = blockIdx.x / (samples * groups);
    const PairSample ps = Q.samples[sample];
    const int N = ps.N, np = ps.n_pairs, R = sh.copies_per_sample;
    if (chunk * (BLOCK / 64) * per_wave >= ps.n_tiles) return;  // a sample smaller than the launch's largest
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, col = lane & 15, quad = lane >> 4;
    float2* a = reinterpret_cast<float2*>(smem);  // [mode][16 copies]
    {
        const int c = group * kCopyTile + col;
        const float2* amp = reinterpret_cast<const float2*>(P.amp) + P.samples[sample].amp_base + (int64_t)min(c, R - 1) * N;
        for (int m = tid >> 4; m < N; m += BLOCK / 16) a[m * kCopyTile + col] = c < R ? amp[m] : make_float2(0.0f, 0.0f);
    }
    // the pairs of the block's columns
    const int t0 = chunk * (BLOCK / 64) * per_wave, t1 = min(t0 + BLOCK / 64 * per_wave, ps.n_tiles) - 1;
    const uint2 b0 = Q.tile[ps.tile_base + t0], b1 = Q.tile[ps.tile_base + t1];
    const int first = (int)(b0.y & 0xffffu), end = (int)(b1.y & 0xffffu) + 4 * (int)(b1.y >> 16);
    uint32_t* pm = reinterpret_cast<uint32_t*>(a + N * kCopyTile);  // LDS offsets of the two modes' rows
    for (int i = tid; i < end - first + 4; i += BLOCK) {  // a tile's columns are whole 4s
        const uint32_t v = Q.pm[ps.pm_base + min(first + i, np - 1)];
        pm[i] = (v & 255u) * (kCopyTile * 8) | (v >> 8) * (kCopyTile * 8) << 16;
    }
    __syncthreads();
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);  // scalar: a tile's bounds and its operand's address
    for (int i = 0; i < per_wave; ++i) {
        const int t = (chunk * (BLOCK / 64) + wave_u) * per_wave + i;
        if (t >= ps.n_tiles) break;
        const uint2 blk = Q.tile[ps.tile_base + t];
        const int k0 = (int)(blk.y & 0xffffu), n4 = (int)(blk.y >> 16);
        // (reads up to kBandSlack values past the tile's, unused)
        const float2* A = reinterpret_cast<const float2*>(Q.band + ps.band_base + blk.x);
        f32x4 r0 = {0, 0, 0, 0}, i0 = r0, r1 = r0, i1 = r0;
        // eight operands ahead of their use
        float2 ra[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) ra[u] = (A + u * 64)[lane];
        const uint32_t* pq = pm + (k0 - first) + quad;
        const auto step = [&](int q, float2 j) {
            const uint32_t v = pq[4 * q];
            const float2 x = *reinterpret_cast<const float2*>(smem + (v & 0xffffu) + 8 * col);
            const float2 y = *reinterpret_cast<const float2*>(smem + (v >> 16) + 8 * col);
            const float br = x.x * y.x - x.y * y.y, bi = x.x * y.y + x.y * y.x;
            r0 = __builtin_amdgcn_mfma_f32_16x16x4f32(j.x, br, r0, 0, 0, 0);
            i0 = __builtin_amdgcn_mfma_f32_16x16x4f32(j.x, bi, i0, 0, 0, 0);
            r1 = __builtin_amdgcn_mfma_f32_16x16x4f32(j.y, br, r1, 0, 0, 0);
            i1 = __builtin_amdgcn_mfma_f32_16x16x4f32(j.y, bi, i1, 0, 0, 0);
        };
        int q0 = 0;
        for (; q0 + 8 <= n4; q0 += 8) {  // no branch inside: the next loads stay in flight
            A += 8 * 64;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float2 j = ra[u];
                ra[u] = (A + u * 64)[lane];
                step(q0 + u, j);
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (q0 + u < n4) step(q0 + u, ra[u]);
        // lane (quad, col) holds rows 4 quad .. 4 quad + 3 of copy col
        const int c = group * kCopyTile + col;
        float2* G = Q.prod + ps.prod_base;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = t * kPairTile + 16 * h + 4 * quad + r;
                const float2 g = h ? make_float2(r1[r], i1[r]) : make_float2(r0[r], i0[r]);
                if (row >= np) continue;
                if (N > kGatherModes) G[((size_t)group * np + row) * kCopyTile + col] = g;
                else if (c < R) G[(size_t)c * np + row] = g;
            }
    }
}

// Large N: the fields of kCopyTile copies from their banded product, a wave
// per mode, four pairs of the mode at a time (one row of 16 copies each).  The
// product is read twice (each pair belongs to two modes), 334 MB at N = 256 and
// 640 copies in 54 us: bound by that stream, 6.2 TB/s past the L2s.
__global__ __launch_bounds__(256) void k_pair_reduce(DevPtrs<float> P, PairDev Q, ShapeInfo sh, int first_item,
                                                     int samples, int groups, int per_wave) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int sample = Q.items[first_item + blockIdx.x % samples].sample;
    const int group = (blockIdx.x / samples) % groups, chunk = blockIdx.x / (samples * groups);
    const PairSample ps = Q.samples[sample];
    const int N = ps.N, np = ps.n_pairs, R = sh.copies_per_sample;
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, quad = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float2* a = reinterpret_cast<float2*>(smem);
    const int c = group * kCopyTile + col;
    const int64_t at = P.samples[sample].amp_base + (int64_t)min(c, R - 1) * N;
    {
        const float2* amp = reinterpret_cast<const float2*>(P.amp) + at;
        for (int m = tid >> 4; m < N; m += 16) a[m * kCopyTile + col] = c < R ? amp[m] : make_float2(0.0f, 0.0f);
    }
    __syncthreads();
    const float2* G = Q.prod + ps.prod_base + (size_t)group * np * kCopyTile + col;
    const uint16_t* pos = Q.pos + ps.pos_base;
    float2* F = reinterpret_cast<float2*>(Q.fields) + at;
    for (int i = 0; i < per_wave; ++i) {
        const int l = (chunk * 4 + wave) * per_wave + i;
        if (l >= N) break;
        float fr = 0, fi = 0;
        for (int x0 = quad; x0 < N; x0 += 32) {
            float2 g[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) g[u] = G[(size_t)pos[l * N + min(x0 + 4 * u, N - 1)] * kCopyTile];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int x = x0 + 4 * u;
                const float2 v = x < N && x != l ? a[x * kCopyTile + col] : make_float2(0.0f, 0.0f);
                fr += v.x * g[u].x + v.y * g[u].y;
                fi += v.x * g[u].y - v.y * g[u].x;
            }
        }
        fr += __shfl_xor(fr, 16);
        fi += __shfl_xor(fi, 16);
        fr += __shfl_xor(fr, 32);
        fi += __shfl_xor(fi, 32);
        if (quad == 0 && c < R) F[l] = make_float2(fr, fi);
    }
}

// ---------------------------------------------------------------- decisions
constexpr int kWindow = 14;  // steps decided together

// LDS of one copy; the amplitudes come first (a list entry holds their offsets)
struct DecideLds {
    size_t F, tab, order, after, first, flag, ev, desc, total;
};

__host__ __device__ inline DecideLds decide_lds(int N, int groups, bool gather) {
    DecideLds o{};
    const size_t steps = N / 2;
    size_t off = ((size_t)N * 2 * sizeof(float) + 15) & ~(size_t)15;
    auto take = [&](size_t b) {
        const size_t at = off;
        off += (b + 15) & ~(size_t)15;
        return at;
    };
    o.F = take((size_t)N * 2 * sizeof(float));
    o.tab = take(steps * sizeof(StepDraw<float>));
    o.order = take((size_t)N * 2);
    o.after = take((steps + 1) * 2);
    o.first = take((size_t)N * 4);
    o.flag = take(2 * (size_t)groups * 4);
    o.ev = take(2 * (size_t)groups * 9 * sizeof(float));
    const size_t prod = gather ? (size_t)N * (N - 1) / 2 * 2 * sizeof(float) : 0, desc = (size_t)N * (N + 1) * 2;
    o.desc = take(prod > desc ? prod : desc);
    o.total = off;
    return o;
}

// a list: byte offset of its entries, and how many of role 0 and of role 1 (padding included)
struct PairList {
    uint32_t at, n0, n1;
};

__device__ inline uint32_t units_of(uint32_t n) { return n / kListUnit * kUnitBytes; }

struct PairEntry {
    uint32_t p;  // p1 | p2 << 8
    float J;
};

// this lane's share, entries t, t + G, ... of the n at byte offset `at`, K of
// them, issued together (0 past the end).  ALL: lanes past the end read the
// zero unit, so that no branch separates the loads (us per sweep, N = 256, 640
// copies 894 -> 872, 160 692 -> 664; N = 128, 1920 copies 399 -> 377); otherwise
// they are left out, which is faster where most lists end early (N = 96, 640
// copies 114, not 117)
template <int K, int G, bool ALL>
__device__ inline void list_load(const unsigned char* __restrict__ list, uint32_t at, uint32_t n, uint32_t t,
                                 PairEntry* e) {
    static_assert(G % kListUnit == 0, "a lane keeps its place in the unit");
    const uint32_t unit = at + units_of(t), in = t % kListUnit;
    const uint32_t at_p = unit + 2 * in, at_J = unit + kUnitJ + 4 * in;
#pragma unroll
    for (int u = 0; u < K; ++u) {
        const bool in_list = t + (uint32_t)(u * G) < n;
        constexpr uint32_t kStep = G / kListUnit * kUnitBytes;
        e[u].p = 0;
        e[u].J = 0;
        if (ALL || in_list) {
            e[u].p = *reinterpret_cast<const uint16_t*>(list + (in_list ? at_p + u * kStep : 0u));
            e[u].J = *reinterpret_cast<const float*>(list + (in_list ? at_J + u * kStep : 0u));
        }
    }
}

// sums J a_p1 a_p2 (ROLE 0) or J conj(a_p1) a_p2 (ROLE 1) over the entries
// loaded; n: entries of the list (a wave stops where no lane has one left)
template <int K, int G, int ROLE>
__device__ inline void list_use(const PairEntry* e, uint32_t n, const unsigned char* a, float& sr, float& si) {
    const float2* amp = reinterpret_cast<const float2*>(a);
#pragma unroll
    for (int u = 0; u < K; ++u) {
        if (u >= K / 2 && !__any((uint32_t)(u * G) < n)) break;
        const float2 x = amp[e[u].p & 0xffu];
        const float2 y = amp[e[u].p >> 8];
        const float vr = e[u].J * x.x, vi = ROLE == 0 ? e[u].J * x.y : -e[u].J * x.y;
        sr += vr * y.x - vi * y.y;
        si += vr * y.y + vi * y.x;
        if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // a few LDS reads ahead, not all of them (registers)
    }
}

// the entries past the first K0 and K1 per lane (none at the sizes they are chosen for)
template <int K0, int K1, int G>
__device__ inline void list_rest(const unsigned char* list, const PairList& p, uint32_t t, const unsigned char* a, float& pr,
                                 float& pi, float& mr, float& mi) {
    PairEntry e[4];
    for (uint32_t i = K0 * G; i < p.n0; i += 4 * G) {
        list_load<4, G, false>(list, p.at, p.n0, i + t, e);
        list_use<4, G, 0>(e, p.n0 - i, a, pr, pi);
    }
    for (uint32_t i = K1 * G; i < p.n1; i += 4 * G) {
        list_load<4, G, false>(list, p.at + units_of(p.n0), p.n1, i + t, e);
        list_use<4, G, 1>(e, p.n1 - i, a, mr, mi);
    }
}

// the field change of a source's move by d: conj(d) times the role-0 sum, d times the role-1 sum
__device__ inline void list_change(float2 d, float pr, float pi, float mr, float mi, float& fr, float& fi) {
    fr = d.x * (pr + mr) + d.y * (pi - mi);
    fi = d.x * (pi + mi) - d.y * (pr - mr);
}

// sum over each half-wave, in every lane of it
__device__ inline float half_sum(float v) {
    v = row_sum(v);
    return v + __shfl_xor(v, 16);
}

// One workgroup per copy: the sweep's steps, decided kWindow at a time, 32
// lanes per step, each on the configuration before them all.  As most updates
// are rejected, the first accepted step of a window (if any) is the only one
// whose result the chain sees, and the steps after it are taken again from
// the changed configuration.  An accepted step corrects the fields that later
// steps still read, from the terms holding both the moved mode and the
// target, 32 lanes per target (16 for each of the two moved modes).  A step's
// own list, from its j to its k, is held from the moment the step's turn comes
// near.  K0, K1: entries of role 0 and 1 per lane of a target's list that are
// loaded at once.  GATHER: the fields are summed here from the copy's banded
// product (which the lists' descriptors then replace in LDS).
// Bound by the chains of accepted updates of the hottest copies, which accept a
// third of their steps: at N = 256 some 43 in a row, 13 us each, for two
// sources' lists to half of the targets (200 KB), two passes of 12 targets in
// flight.  The chip as a whole reads 1.8 GB past the L2s per sweep of 640
// equilibrated copies in 663 us (2.7 TB/s), 5.9 GB before they relax (7.9 TB/s,
// with 8 B per entry: then the bandwidth bound it, 748 us).  The list-streaming
// sweep read every list of every step instead: 2625 us per sweep there.
// 32 lanes per step because a wave per step repeats the scalar work 64 times;
// all of a target's entries are asked for before any is used, as one more
// access at a time exposes its whole latency (957 us).  N > 136: 768 threads,
// for the registers that hold two targets' entries (1024 spilled).
template <int BLOCK, int LANES, int K0, int K1, bool GATHER>
__global__ __launch_bounds__(BLOCK) void k_pair_decide(DevPtrs<float> P, PairDev Q, ShapeInfo sh, int first_item) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int kGroups = BLOCK / 16, kSlots = BLOCK / 32;
    constexpr bool kAll = BLOCK != 1024;
    const ItemDev it = Q.items[first_item + blockIdx.x];
    const PairSample ps = Q.samples[it.sample];
    const int N = ps.N, steps = N / 2;
    const int tid = threadIdx.x, lane = tid & 63, grp = tid >> 4, gl = tid & 15, hl = tid & 31;
    const DecideLds o = decide_lds(N, kSlots, GATHER);
    float2* a = reinterpret_cast<float2*>(smem);
    float2* F = reinterpret_cast<float2*>(smem + o.F);
    StepDraw<float>* tab = reinterpret_cast<StepDraw<float>*>(smem + o.tab);
    uint16_t* order = reinterpret_cast<uint16_t*>(smem + o.order);
    uint16_t* after = reinterpret_cast<uint16_t*>(smem + o.after);
    uint32_t* first = reinterpret_cast<uint32_t*>(smem + o.first);
    int* flag = reinterpret_cast<int*>(smem + o.flag);
    float* ev = reinterpret_cast<float*>(smem + o.ev);
    uint16_t* desc = reinterpret_cast<uint16_t*>(smem + o.desc);

    // the copy at this item's temperature slot (descending temperature, then
    // ladder: the hottest copies accept the most updates and start first)
    int c;
    {
        const int i = it.first_copy - it.sample * sh.copies_per_sample;
        c = P.copy_at[((size_t)it.sample * sh.n_reps + i % sh.n_reps) * sh.n_temps + (sh.n_temps - 1 - i / sh.n_reps)];
    }
    const SampleDev* sd = P.samples + it.sample;
    const int64_t at = sd->amp_base + (int64_t)(c - it.sample * sh.copies_per_sample) * N;
    float2* amp_g = reinterpret_cast<float2*>(P.amp) + at;
    const unsigned char* list = Q.list + ps.list_base;
    {
        const float2* F_g = reinterpret_cast<const float2*>(Q.fields) + at;
        const uint32_t* first_g = Q.first + sd->mode_base;
        const uint16_t* ord_g = Q.order + (size_t)c * Q.max_N;
        const uint16_t* aft_g = Q.after + (size_t)c * (Q.max_steps + 1);
        const float* tab_g = reinterpret_cast<const float*>(static_cast<const StepDraw<float>*>(Q.draws) + (size_t)c * Q.max_steps);
        for (int i = tid; i < N; i += BLOCK) {
            a[i] = amp_g[i];
            if constexpr (!GATHER) F[i] = F_g[i];
            first[i] = first_g[i];
            order[i] = ord_g[i];
        }
        for (int i = tid; i <= steps; i += BLOCK) after[i] = aft_g[i];
        constexpr int kWords = (int)(sizeof(StepDraw<float>) / sizeof(float));
        for (int i = tid; i < steps * kWords; i += BLOCK) reinterpret_cast<float*>(tab)[i] = tab_g[i];
    }
    if constexpr (GATHER) {
        float2* G = reinterpret_cast<float2*>(desc);
        const float2* G_g = Q.prod + ps.prod_base + (size_t)(c - it.sample * sh.copies_per_sample) * ps.n_pairs;
        for (int i0 = tid; i0 < ps.n_pairs; i0 += 8 * BLOCK) {
            float2 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = G_g[min(i0 + u * BLOCK, ps.n_pairs - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i0 + u * BLOCK < ps.n_pairs) G[i0 + u * BLOCK] = v[u];
        }
        __syncthreads();
        const uint16_t* pos = Q.pos + ps.pos_base;
        for (int i = grp; i < after[steps]; i += kGroups) {
            const int l = order[i];
            float fr = 0, fi = 0;
            for (int x0 = gl; x0 < N; x0 += 64) {
                int r[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) r[u] = pos[l * N + min(x0 + 16 * u, N - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int x = x0 + 16 * u;
                    const float2 g = G[r[u]];
                    const float2 v = x < N && x != l ? a[x] : make_float2(0, 0);
                    fr += v.x * g.x + v.y * g.y;
                    fi += v.x * g.y - v.y * g.x;
                }
            }
            fr = row_sum(fr);
            fi = row_sum(fi);
            if (gl == 0) F[l] = make_float2(fr, fi);
        }
        __syncthreads();
    }
    {   // N (N + 1) is even and the rows start at an even element: two descriptors at a time
        const uint32_t* g = reinterpret_cast<const uint32_t*>(Q.desc + ps.desc_base);
        uint32_t* d = reinterpret_cast<uint32_t*>(desc);
        const int n = N * (N + 1) / 2;
        for (int i0 = tid; i0 < n; i0 += 8 * BLOCK) {
            uint32_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = g[min(i0 + u * BLOCK, n - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i0 + u * BLOCK < n) d[i0 + u * BLOCK] = v[u];
        }
    }
    const int t_idx = P.temp_of[c];
    const float beta = P.beta[t_idx];
    float E = P.E[c];
    unsigned int n_acc = 0;

    auto find = [&](int j, int l) {  // the list from source j to target l
        const uint32_t v = desc[j * (N + 1) + l], w = desc[j * (N + 1) + l + 1], start = v & ((1u << kStartBits) - 1);
        PairList p;
        p.n0 = (v >> kStartBits) * 2 * kListUnit;
        p.n1 = ((w & ((1u << kStartBits) - 1)) - start) * kListUnit - p.n0;
        p.at = (first[j] + start) * (uint32_t)kUnitBytes;
        return p;
    };
    // step s belongs to half-wave s mod kSlots; its list entries come ahead,
    // for both steps of a wave at once (a wave waits for all its loads)
    constexpr int kOwn0 = (K0 * LANES + 31) / 32, kOwn1 = (K1 * LANES + 31) / 32;
    PairEntry own0[kOwn0], own1[kOwn1];
    PairList op{0, 0, 0};
    auto take_step = [&](int s) {
        op = PairList{0, 0, 0};
        if (s < steps) op = find(tab[s].jk & 0xffff, tab[s].jk >> 16);
        list_load<kOwn0, 32, kAll>(list, op.at, op.n0, hl, own0);
        list_load<kOwn1, 32, kAll>(list, op.at + units_of(op.n0), op.n1, hl, own1);
    };
    __syncthreads();
    int my = tid >> 5, base = 0, par = 0;
    take_step(my);
    while (base < steps) {
        if (my >= base && my < steps && my < base + kWindow) {
            const StepDraw<float> d = tab[my];
            const int j = d.jk & 0xffff, k = d.jk >> 16;
            const float2 ajo = a[j], ako = a[k];
            const float uj = ajo.x * ajo.x + ajo.y * ajo.y, uk = ako.x * ako.x + ako.y * ako.y;
            const float K = pair_radius<float, false>(uj, uk, sh.rho);
            const float2 ajn = make_float2(K * d.cj * d.ejr, K * d.cj * d.eji);
            const float2 akn = make_float2(K * d.sk * d.ekr, K * d.sk * d.eki);
            const float2 dj = make_float2(ajn.x - ajo.x, ajn.y - ajo.y);
            // F_k's change from the new a_j, terms holding both
            float pr = 0, pi = 0, mr = 0, mi = 0, cr, ci;
            list_use<kOwn0, 32, 0>(own0, op.n0, smem, pr, pi);
            list_use<kOwn1, 32, 1>(own1, op.n1, smem, mr, mi);
            list_rest<kOwn0, kOwn1, 32>(list, op, hl, smem, pr, pi, mr, mi);
            list_change(dj, pr, pi, mr, mi, cr, ci);
            cr = half_sum(cr);
            ci = half_sum(ci);
            const float2 Fj = F[j];
            float2 Fk = F[k];
            Fk.x += cr;
            Fk.y += ci;
            const float dE = pair_delta<float>(ajo, ajn, ako, akn, Fj, Fk);
            const bool acc = (dE <= 0.0f) || (d.u < exp(-beta * dE));
            if (hl == 0) {
                flag[par * kSlots + my % kSlots] = acc ? 1 : 0;
                if (acc) {
                    float* e = ev + (par * kSlots + my % kSlots) * 9;
                    e[0] = dE;
                    e[1] = ajn.x;
                    e[2] = ajn.y;
                    e[3] = akn.x;
                    e[4] = akn.y;
                    e[5] = dj.x;
                    e[6] = dj.y;
                    e[7] = akn.x - ako.x;
                    e[8] = akn.y - ako.y;
                }
            }
        }
        block_sync_lds();
        // first accepted step of the window
        const int s_l = base + lane;
        const unsigned long long hit =
            __ballot(lane < kWindow && s_l < steps && flag[par * kSlots + s_l % kSlots] != 0);
        int advance = base + kWindow;  // steps below this are decided
        if (hit) {
            const int s = base + (int)__ffsll((long long)hit) - 1;
            const float* e = ev + (par * kSlots + s % kSlots) * 9;
            const int j = tab[s].jk & 0xffff, k = tab[s].jk >> 16;
            const float2 dj = make_float2(e[5], e[6]), dk = make_float2(e[7], e[8]);
            advance = s + 1;
            // fields that later steps read, a_j new and a_k old: a target's
            // entries are on their way before the others see a_j
            constexpr int kTargets = BLOCK / (2 * LANES);  // corrected together
            const int nt = after[s], mine = tid / (2 * LANES), src = (tid / LANES) & 1 ? k : j, ll = tid & (LANES - 1);
            struct Fetch {
                PairList p;
                PairEntry ea[K0], eb[K1];
            };
            auto fetch = [&](int i, Fetch& f) {
                f.p = find(src, order[i]);
                list_load<K0, LANES, kAll>(list, f.p.at, f.p.n0, ll, f.ea);
                list_load<K1, LANES, kAll>(list, f.p.at + units_of(f.p.n0), f.p.n1, ll, f.eb);
            };
            auto correct = [&](int i, const Fetch& f) {
                float pr = 0, pi = 0, mr = 0, mi = 0, fr, fi;
                list_use<K0, LANES, 0>(f.ea, f.p.n0, smem, pr, pi);
                list_use<K1, LANES, 1>(f.eb, f.p.n1, smem, mr, mi);
                list_rest<K0, K1, LANES>(list, f.p, ll, smem, pr, pi, mr, mi);
                list_change((tid / LANES) & 1 ? dk : dj, pr, pi, mr, mi, fr, fi);
                fr = row_sum(fr);
                fi = row_sum(fi);
                // the last row of the target's lanes gathers the totals of the others
                fr += dpp_bcast<0x142, 0xA>(fr);
                fi += dpp_bcast<0x142, 0xA>(fi);
                if constexpr (LANES == 32) {
                    fr += dpp_bcast<0x143, 0xC>(fr);
                    fi += dpp_bcast<0x143, 0xC>(fi);
                }
                const int l = order[i];
                if ((tid & (2 * LANES - 1)) == 2 * LANES - 1) F[l] = make_float2(F[l].x + fr, F[l].y + fi);
            };
            Fetch f0, f1;
            if (mine < nt) fetch(mine, f0);
            if (tid == 0) {
                E += e[0];
                ++n_acc;
                a[j] = make_float2(e[1], e[2]);
            }
            block_sync_lds();
            if constexpr (LANES == 32) {  // the next target's entries come while this one's are used
                for (int i = mine; i < nt; i += 2 * kTargets) {
                    if (i + kTargets < nt) fetch(i + kTargets, f1);
                    correct(i, f0);
                    if (i + kTargets >= nt) break;
                    if (i + 2 * kTargets < nt) fetch(i + 2 * kTargets, f0);
                    correct(i + kTargets, f1);
                }
            } else {
                for (int i = mine; i < nt; i += kTargets) {
                    if (i != mine) fetch(i, f0);
                    correct(i, f0);
                }
            }
            block_sync_lds();
            if (tid == 0) a[k] = make_float2(e[3], e[4]);
            block_sync_lds();
        }
        if ((my | 1) < advance) {  // both steps of the wave are decided
            my += kSlots;
            take_step(my);
        }
        base = advance;
        par ^= 1;
    }
    __syncthreads();
    for (int i = tid; i < N; i += BLOCK) amp_g[i] = a[i];
    if (tid == 0) {
        P.E[c] = E;
        atomicAdd(&P.acc[(size_t)it.sample * sh.n_temps + t_idx], (unsigned long long)n_acc);
    }
}

// more than the default 64 KiB of dynamic LDS has to be asked for
template <typename K>
hipError_t allow_lds(K kernel, size_t bytes) {
    if (bytes <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)bytes);
}

template <int BLOCK, int LANES, int K0, int K1, bool GATHER>
hipError_t decide_b(const DevPtrs<float>& P, const PairDev& Q, const ShapeInfo& sh, const PairLaunch& L,
                    hipStream_t st) {
    static_assert(BLOCK / 32 > kWindow, "a window's steps, and the rest of their waves, in different slots");
    const size_t lds = decide_lds(L.N, BLOCK / 32, GATHER).total;
    auto kernel = &k_pair_decide<BLOCK, LANES, K0, K1, GATHER>;
    hipError_t e = allow_lds(kernel, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_pair_decide<BLOCK, LANES, K0, K1, GATHER>), dim3(L.n), dim3(BLOCK), lds, st, P, Q, sh,
                       L.first);
    return hipGetLastError();
}

}  // namespace

// a block's prologue (16 copies into LDS) is worth several row tiles per wave once there are many
int pairs_product_waves(int N) { return N * (N - 1) / 2 >= 512 * kPairTile ? 8 : 4; }
int pairs_tiles_per_wave(int N) { return N * (N - 1) / 2 >= 512 * kPairTile ? 2 : 1; }

hipError_t launch_pair_fields(const DevPtrs<float>& P, const PairDev& Q, const ShapeInfo& sh, const PairLaunch& L,
                              int ahead, hipStream_t st) {
    const int groups = (sh.copies_per_sample + kCopyTile - 1) / kCopyTile;
    const int tiles = (L.N * (L.N - 1) / 2 + kPairTile - 1) / kPairTile;
    const int per_wave = pairs_tiles_per_wave(L.N);
    const int chunks = (tiles + pairs_product_waves(L.N) * per_wave - 1) / (pairs_product_waves(L.N) * per_wave);
    const int n_product = chunks * groups * L.samples;
    const size_t lds = (size_t)L.N * kCopyTile * sizeof(float2) + (size_t)L.columns * 4;
    if (pairs_product_waves(L.N) == 8)
        hipLaunchKernelGGL(k_pair_product<512>, dim3(n_product + L.n), dim3(512), lds, st, P, Q, sh, L.first, L.samples,
                           groups, n_product, per_wave, ahead);
    else
        hipLaunchKernelGGL(k_pair_product<256>, dim3(n_product + L.n), dim3(256), lds, st, P, Q, sh, L.first, L.samples,
                           groups, n_product, per_wave, ahead);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (L.N > kGatherModes) {
        const int modes = 4;  // per wave
        const int blocks = (L.N + 4 * modes - 1) / (4 * modes) * groups * L.samples;
        hipLaunchKernelGGL(k_pair_reduce, dim3(blocks), dim3(256), (size_t)L.N * kCopyTile * sizeof(float2), st, P, Q, sh,
                           L.first, L.samples, groups, modes);
        e = hipGetLastError();
    }
    return e;
}

hipError_t launch_pair_decide(const DevPtrs<float>& P, const PairDev& Q, const ShapeInfo& sh, const PairLaunch& L,
                              hipStream_t st) {
    switch (L.threads) {
        case 512: return decide_b<512, 16, 6, 10, true>(P, Q, sh, L, st);
        case 768: return decide_b<768, 32, 4, 9, false>(P, Q, sh, L, st);
        case 1024: return decide_b<1024, 16, 6, 10, true>(P, Q, sh, L, st);
        default: return hipErrorInvalidValue;
    }
}

int pairs_decide_threads(int N, int copies, int cus) {
    if (N > kGatherModes) return 768;
    // A copy's chain of accepted updates is latency; 1024 threads shorten it,
    // 512 let a compute unit interleave two copies' chains.  Us per sweep on 256
    // units, 1024 -> 512: N = 96, 640 copies 121 -> 143, 960 146 -> 156, 1280
    // 180 -> 167, 3200 461 -> 366; N = 128 198 -> 237, 255 -> 280, 331 -> 314,
    // 809 -> 675; 1024 copies beside a list sweep 381 -> 354.
    return copies >= 4 * cus ? 512 : 1024;
}

hipError_t launch_pairs_tables(const DevPtrs<float>& P, const PairDev& Q, const ShapeInfo& sh, int n_samples, int max_N,
                               int64_t max_quads, hipStream_t st) {
    const int blocks = (int)std::min<int64_t>((max_quads + 1023) / 1024, 1024);
    hipLaunchKernelGGL(k_band_fill, dim3(blocks < 1 ? 1 : blocks, n_samples), dim3(256), 0, st, P, Q);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (sh.layout == kLayoutChunked)
        hipLaunchKernelGGL((k_list_fill<kLayoutChunked>), dim3(max_N, n_samples), dim3(256), 0, st, P, Q);
    else
        hipLaunchKernelGGL((k_list_fill<kLayoutPacked>), dim3(max_N, n_samples), dim3(256), 0, st, P, Q);
    return hipGetLastError();
}

}  // namespace rlpt
