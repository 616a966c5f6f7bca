// Sweep of few copies with short lists for CDNA4 (gfx950): a copy's two-mode
// updates decided several at a time.  Method: Benedetti & Leuzzi, arXiv 2511.13508, sec. III.A
// (the same chain and draws as the list-streaming sweep of kernels.hip).
#include <hip/hip_runtime.h>

#include "ahead.hpp"
#include "device.hpp"
#include "lists.hpp"

namespace rlpt {
namespace {

// LDS before the private amplitudes: draws, decisions, list bounds
template <typename R>
__host__ __device__ inline size_t ahead_fixed_bytes(int max_N, int waves) {
    const size_t b = (size_t)(max_N / 2) * sizeof(StepDraw<R>) + (size_t)waves * 10 * sizeof(R) + (size_t)waves * 8 +
                     (size_t)(max_N + 1) * 4;
    return (b + 15) & ~(size_t)15;
}

// One workgroup per copy, one wave per step.  A step's update depends on the
// steps before it only where one of them is accepted, and most are rejected:
// the kWaves / 2 next steps are evaluated at once, each on the configuration
// before them all (in a private copy of the amplitudes that holds its own
// a_j'), and the first accepted one of them, if any, ends the round: the steps
// before it are rejected, those after it are evaluated again from the changed
// configuration.  Step s belongs to wave s mod kWaves, so a step's lists are
// in registers a round before it can be evaluated.
// A step at a time, the chain of list load, reduction, barrier and decision
// bounds a small copy; here a round pays it for several steps.  Us per sweep:
// N = 1024 of mean degree 32, 160 copies 410 -> 190; N = 24, 384 copies 31 -> 18;
// N = 32, 8 copies 28 -> 18; past a few waves per SIMD the LDS reads of the
// evaluations bound it instead, and the host takes the other kernels.
// SHORT: packed lists of at most 32 * PF entries, half a wave each; otherwise
// chunked lists of at most PF chunks per lane.
template <typename R, int BLOCK, bool SHORT, int PF>
__global__ __launch_bounds__(BLOCK) void k_sweep_ahead(DevPtrs<R> P, ShapeInfo sh, const ItemDev* items, int max_N,
                                                       int n_sweeps) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int kWaves = BLOCK / 64, kWindow = kWaves / 2;
    const ItemDev it = items[blockIdx.x];
    const SampleDev sd = P.samples[it.sample];
    const int N = sd.N, steps = sd.n_steps;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    StepDraw<R>* tab = reinterpret_cast<StepDraw<R>*>(smem);
    R* ev = reinterpret_cast<R*>(tab + max_N / 2);             // [2][kWaves][5] dE, a_j', a_k'
    int* flag = reinterpret_cast<int*>(ev + 2 * kWaves * 5);   // [2][kWaves]
    uint32_t* lb = reinterpret_cast<uint32_t*>(flag + 2 * kWaves);  // [max_N + 1]
    R2<R>* a = reinterpret_cast<R2<R>*>(smem + ahead_fixed_bytes<R>(max_N, kWaves)) + (size_t)wave * max_N;

    // the copy at this item's temperature slot (descending temperature, then
    // ladder: the hottest copies accept the most updates and start first)
    int c;
    {
        const int i = it.first_copy - it.sample * sh.copies_per_sample;
        c = P.copy_at[((size_t)it.sample * sh.n_reps + i % sh.n_reps) * sh.n_temps + (sh.n_temps - 1 - i / sh.n_reps)];
    }
    R2<R>* amp_g = reinterpret_cast<R2<R>*>(P.amp) + sd.amp_base + (int64_t)(c - it.sample * sh.copies_per_sample) * N;
    for (int i = lane; i < N; i += 64) a[i] = amp_g[i];
    {
        const uint32_t* gb = (SHORT ? P.mode_start : P.chunk_start) + sd.mode_base;
        for (int i = tid; i <= N; i += BLOCK) lb[i] = gb[i];
    }
    const int t_idx = P.temp_of[c];
    const R beta = P.beta[t_idx];
    R E = P.E[c];
    unsigned int n_acc = 0;
    const int64_t pair_stream = sh.shared_pairs ? (int64_t)it.sample : (int64_t)c;
    const int64_t sweep0 = P.counters->sweeps_done;

    // this wave's lists
    uint32_t sv[PF];
    R sj[PF];
    ChunkRegs<R, PF> rj, rk;
    auto take_step = [&](int s) {
        if (s >= steps) return;
        const int j = tab[s].jk & 0xffff, k = tab[s].jk >> 16;
        if constexpr (SHORT) {  // lanes 0-31: list of j, 32-63: of k; past the end the sample's first entry, weighted 0
            const int l = lane < 32 ? j : k;
            const uint32_t b = lb[l], e = lb[l + 1];
#pragma unroll
            for (int i = 0; i < PF; ++i) {
                const uint32_t x = b + (uint32_t)((lane & 31) + 32 * i);
                sv[i] = P.idx[x < e ? x : lb[0]];
                const R J = P.J[x < e ? x : lb[0]];
                sj[i] = x < e ? J : (R)0;
            }
        } else {
            chunk_prefetch<R, PF>(P, lb, j, lane, 64, rj);
            chunk_prefetch<R, PF>(P, lb, k, lane, 64, rk);
        }
    };
    for (int sw = 0; sw < n_sweeps; ++sw) {
        __syncthreads();
        // a step's draws over four waves: the pair, the two phases, the magnitudes and the uniform
        for (int i = tid; i < 4 * ((steps + 63) & ~63); i += BLOCK) {
            const int s = (i & 63) | (i >> 8) << 6, part = (i >> 6) & 3;
            if (s >= steps) continue;
            if (part == 0) tab[s].jk = draw_pair(sh.run_seed, pair_stream, sweep0 + sw, s, N);
            else draw_part<R>(sh.run_seed, c, sweep0 + sw, s, sh.rho, part, tab[s]);
        }
        __syncthreads();
        int my = wave, base = 0, par = 0;
        take_step(my);
        while (base < steps) {
            if (my >= base && my < steps && my < base + kWindow) {
                const StepDraw<R> d = tab[my];
                const int j = d.jk & 0xffff, k = d.jk >> 16;
                const R2<R> ajo = a[j], ako = a[k];
                const R uj = ajo.x * ajo.x + ajo.y * ajo.y, uk = ako.x * ako.x + ako.y * ako.y;
                const R K = pair_radius<R, SHORT && PF == kShortSlots>(uj, uk, sh.rho);
                const R2<R> ajn = mk2<R>(K * d.cj * d.ejr, K * d.cj * d.eji);
                const R2<R> akn = mk2<R>(K * d.sk * d.ekr, K * d.sk * d.eki);
                wave_sync();
                if (lane == 0) a[j] = ajn;  // the step's snapshot: a_j new, a_k old
                wave_sync();
                R2<R> Fj, Fk;
                if constexpr (SHORT) {
                    R fr = 0, fi = 0;
#pragma unroll
                    for (int i = 0; i < PF; ++i) field_term<R>(sv[i], sj[i], a, fr, fi);
                    fr = row_sum(fr);
                    fi = row_sum(fi);
                    Fj = mk2<R>(read_lane(fr, 0) + read_lane(fr, 16), read_lane(fi, 0) + read_lane(fi, 16));
                    Fk = mk2<R>(read_lane(fr, 32) + read_lane(fr, 48), read_lane(fi, 32) + read_lane(fi, 48));
                } else {
                    R jr = 0, ji = 0, kr = 0, ki = 0;
                    chunk_consume<R, PF>(rj, a, jr, ji);
                    chunk_consume<R, PF>(rk, a, kr, ki);
                    Fj = mk2<R>(wave_sum(jr), wave_sum(ji));
                    Fk = mk2<R>(wave_sum(kr), wave_sum(ki));
                }
                wave_sync();
                const R dE = pair_delta<R>(ajo, ajn, ako, akn, Fj, Fk);
                const bool acc = (dE <= (R)0) || (d.u < exp(-beta * dE));
                if (lane == 0) {
                    a[j] = ajo;
                    flag[par * kWaves + wave] = acc ? 1 : 0;
                    R* e = ev + (par * kWaves + wave) * 5;
                    e[0] = dE;
                    e[1] = ajn.x;
                    e[2] = ajn.y;
                    e[3] = akn.x;
                    e[4] = akn.y;
                }
            }
            block_sync_lds();
            const int s_l = base + lane;
            const unsigned long long hit =
                __ballot(lane < kWindow && s_l < steps && flag[par * kWaves + s_l % kWaves] != 0);
            base += kWindow;  // steps below it are decided
            if (hit) {
                base += (int)__ffsll((long long)hit) - kWindow;
                const int s = base - 1;
                const R* e = ev + (par * kWaves + s % kWaves) * 5;
                if (lane == 0) {
                    a[tab[s].jk & 0xffff] = mk2<R>(e[1], e[2]);
                    a[tab[s].jk >> 16] = mk2<R>(e[3], e[4]);
                }
                if (tid == 0) {
                    E += e[0];
                    ++n_acc;
                }
                wave_sync();
            }
            if (my < base) {
                my += kWaves;
                take_step(my);
            }
            par ^= 1;
        }
    }
    if (wave == 0)
        for (int i = lane; i < N; i += 64) amp_g[i] = a[i];
    if (tid == 0) {
        P.E[c] = E;
        atomicAdd(&P.acc[(size_t)it.sample * sh.n_temps + t_idx], (unsigned long long)n_acc);
    }
}

template <typename R, int BLOCK, bool SHORT, int PF>
hipError_t ahead_b(const DevPtrs<R>& P, const ShapeInfo& sh, const AheadLaunch& L, int n_sweeps, hipStream_t st) {
    const size_t lds = ahead_fixed_bytes<R>(L.max_N, BLOCK / 64) + (size_t)(BLOCK / 64) * L.max_N * 2 * sizeof(R);
    auto kernel = &k_sweep_ahead<R, BLOCK, SHORT, PF>;
    if (lds > 64 * 1024) {  // more than the default dynamic LDS has to be asked for
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_sweep_ahead<R, BLOCK, SHORT, PF>), dim3(L.n_items), dim3(BLOCK), lds, st, P, sh, L.items,
                       L.max_N, n_sweeps);
    return hipGetLastError();
}

template <typename R>
hipError_t ahead_t(const DevPtrs<R>& P, const ShapeInfo& sh, const AheadLaunch& L, int n_sweeps, hipStream_t st) {
    // lists past the short ones have instances of 512 threads only
    if (L.block != 512 && (sh.layout == kLayoutChunked || L.slots > kShortSlots)) return hipErrorInvalidValue;
    if (sh.layout != kLayoutChunked) {
        if (L.slots > 12) return ahead_b<R, 512, true, 16>(P, sh, L, n_sweeps, st);
        if (L.slots > 8) return ahead_b<R, 512, true, 12>(P, sh, L, n_sweeps, st);
        if (L.slots > kShortSlots) return ahead_b<R, 512, true, 8>(P, sh, L, n_sweeps, st);
        if (L.block == 1024) return ahead_b<R, 1024, true, kShortSlots>(P, sh, L, n_sweeps, st);
        if (L.block == 512) return ahead_b<R, 512, true, kShortSlots>(P, sh, L, n_sweeps, st);
        return ahead_b<R, 256, true, kShortSlots>(P, sh, L, n_sweeps, st);
    }
    if (L.chunks <= 2) return ahead_b<R, 512, false, 2>(P, sh, L, n_sweeps, st);
    if (L.chunks <= 4) return ahead_b<R, 512, false, 4>(P, sh, L, n_sweeps, st);
    return ahead_b<R, 512, false, 6>(P, sh, L, n_sweeps, st);
}

}  // namespace

size_t ahead_lds_bytes(int precision, const AheadLaunch& L) {
    const int w = L.block / 64;
    return precision == RLPT_FP64 ? ahead_fixed_bytes<double>(L.max_N, w) + (size_t)w * L.max_N * 16
                                  : ahead_fixed_bytes<float>(L.max_N, w) + (size_t)w * L.max_N * 8;
}

bool ahead_plan(int precision, int layout, uint32_t longest, int max_N, AheadLaunch* L) {
    L->max_N = max_N;
    L->chunks = L->slots = 0;
    L->block = 512;
    if (layout == kLayoutChunked) {
        L->chunks = (int)(longest + 63) / 64;
        if (L->chunks > 6) return false;
    } else {
        L->slots = (int)(longest + 31) / 32;
        if (L->slots > 16) return false;
        const bool is_short = L->slots <= kShortSlots;
        if (is_short) L->block = 1024;
        // no wave without a step: the window is half the waves
        while (L->block > 256 && L->block / 128 > max_N / 2) L->block /= 2;
        if (!is_short && L->block < 512) return false;
        while (is_short && L->block > 256 && ahead_lds_bytes(precision, *L) > kMaxLds) L->block /= 2;
    }
    return ahead_lds_bytes(precision, *L) <= kMaxLds;
}

hipError_t launch_sweep_ahead(int precision, const void* ptrs, const ShapeInfo& sh, const AheadLaunch& L, int n_sweeps,
                              hipStream_t st) {
    return precision == RLPT_FP64 ? ahead_t<double>(*static_cast<const DevPtrs<double>*>(ptrs), sh, L, n_sweeps, st)
                                  : ahead_t<float>(*static_cast<const DevPtrs<float>*>(ptrs), sh, L, n_sweeps, st);
}

}  // namespace rlpt
