// Device helpers shared by the sweep kernels (kernels.hip, pairs.hip): complex
// values in the context's precision, cross-lane sums, the LDS-only workgroup
// barrier, and the draws and energy change of one two-mode update (sec. III.A
// of Benedetti & Leuzzi, arXiv 2511.13508).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "philox.hpp"

namespace rlpt {
namespace {

template <typename R>
struct V2;
template <>
struct V2<float> {
    using T = float2;
};
template <>
struct V2<double> {
    using T = double2;
};
template <typename R>
using R2 = typename V2<R>::T;

template <typename R>
struct J4;
template <>
struct J4<float> {
    using T = float4;
};
template <>
struct J4<double> {
    using T = double4;
};

template <typename R>
__device__ inline R2<R> mk2(R x, R y) {
    R2<R> v;
    v.x = x;
    v.y = y;
    return v;
}

template <typename R>
__device__ inline R pi_v() {
    return (R)3.14159265358979323846;
}

__device__ inline void sincos_r(float x, float* s, float* c) { sincosf(x, s, c); }
__device__ inline void sincos_r(double x, double* s, double* c) { sincos(x, s, c); }

// cross-lane moves within rows of 16 lanes (DPP: quad_perm [1,0,3,2] = 0xB1,
// [2,3,0,1] = 0x4E, row_half_mirror = 0x141, row_mirror = 0x140) and reads of
// one lane's value into every lane (v_readlane, the lane index wave-uniform)
template <int CTRL>
__device__ inline float dpp_move(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ inline double dpp_move(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ inline float read_lane(float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); }
__device__ inline double read_lane(double v, int l) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ inline int read_lane(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ inline uint32_t read_lane(uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); }

// sum over each row of 16 lanes, in every lane of the row
template <typename R>
__device__ inline R row_sum(R v) {
    v += dpp_move<0xB1>(v);
    v += dpp_move<0x4E>(v);
    v += dpp_move<0x141>(v);
    v += dpp_move<0x140>(v);
    return v;
}

// row broadcasts (DPP row_bcast:15 = 0x142 into rows 1 and 3, row_bcast:31 =
// 0x143 into rows 2 and 3); lanes of the other rows receive 0
template <int CTRL, int ROWS>
__device__ inline float dpp_bcast(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xF, false));
}
template <int CTRL, int ROWS>
__device__ inline double dpp_bcast(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xF, false);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// sum over the wave, the same value in every lane (all lanes active)
template <typename R>
__device__ inline R wave_sum(R v) {
    v = row_sum(v);
    return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

// the same sum, valid in lane 63 only, without lane reads: rows 1 and 3 add
// the totals of rows 0 and 2, then row 3 adds row 1's; (r3 + r2) + (r1 + r0)
// rounds exactly as wave_sum's (r0 + r1) + (r2 + r3)
template <typename R>
__device__ inline R wave_sum_last(R v) {
    v = row_sum(v);
    v += dpp_bcast<0x142, 0xA>(v);
    v += dpp_bcast<0x143, 0xC>(v);
    return v;
}

// workgroup barrier that waits for LDS operations only (s_waitcnt lgkmcnt(0)
// with vmcnt and expcnt at their maxima, 0xC07F): global loads issued before
// it stay in flight.  Only for loops whose global memory traffic is loads.
__device__ inline void block_sync_lds() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// energy change of the two-mode update from the two fields of one snapshot:
// dE = -2 Re(conj(aj_new - aj_old) F_j) - 2 Re(conj(ak_new - ak_old) F_k)
template <typename R>
__device__ inline R pair_delta(R2<R> ajo, R2<R> ajn, R2<R> ako, R2<R> akn, R2<R> Fj, R2<R> Fk) {
    const R djr = ajn.x - ajo.x, dji = ajn.y - ajo.y;
    const R dkr = akn.x - ako.x, dki = akn.y - ako.y;
    return (R)-2 * (djr * Fj.x + dji * Fj.y) - (R)2 * (dkr * Fk.x + dki * Fk.y);
}

// K of the pair's circle from |a_j|^2 and |a_k|^2.  The compiler may contract
// the sum of squares either way round; the order is written out, so that the
// same proposal has the same bits whichever kernel forms it: FIRST_J squares
// |a_j|^2 first (the sweep from short packed lists), otherwise |a_k|^2 (the
// other sweeps)
template <typename R, bool FIRST_J>
__device__ inline R pair_radius(R uj, R uk, int rho) {
    if (rho == 2) return sqrt(uj + uk);
    const R u = FIRST_J ? uj : uk, v = FIRST_J ? uk : uj;
    return sqrt(sqrt(fma(v, v, u * u)));
}

// state-independent part of step s of sweep w for one copy (sec. III.A):
// distinct j, k; unit phasors of the new phases; sqrt(cos theta), sqrt(sin theta);
// acceptance uniform
template <typename R>
struct StepDraw {
    int32_t jk;  // j | k << 16
    R ejr, eji, ekr, eki, cj, sk, u;
};

// the step's two distinct modes j | k << 16
__device__ __forceinline__ int pair_of(const Philox4& wp, int N) {
    const int j = index_below(wp.v[0], N);
    int k = index_below(wp.v[1], N - 1);
    k += (k >= j) ? 1 : 0;
    return j | (k << 16);
}

__device__ inline int draw_pair(uint64_t seed, int64_t pair_stream, int64_t sweep, int step, int N) {
    return pair_of(philox4x64((uint64_t)step, (uint64_t)sweep, (uint64_t)pair_stream, 0, seed, kTagPair), N);
}

// part of the move's draws: 1 the phase of a_j, 2 the phase of a_k, 3 the
// magnitudes and the acceptance uniform
template <typename R>
__device__ __forceinline__ void move_part(const Philox4& wm, int rho, int part, StepDraw<R>& d) {
    const R two_pi = (R)2 * pi_v<R>();
    R s, c;
    if (part == 1) {
        sincos_r(two_pi * uniform01<R>(wm.v[0]), &s, &c);
        d.ejr = c;
        d.eji = s;
    } else if (part == 2) {
        sincos_r(two_pi * uniform01<R>(wm.v[1]), &s, &c);
        d.ekr = c;
        d.eki = s;
    } else {
        if (rho == 2) {  // sin^2 theta uniform: A_j' = K sqrt(1 - u), A_k' = K sqrt(u)
            const R u = uniform01<R>(wm.v[2]);
            d.cj = sqrt((R)1 - u);
            d.sk = sqrt(u);
        } else {  // theta uniform: A_j' = K sqrt(cos theta), A_k' = K sqrt(sin theta)
            sincos_r((R)0.5 * pi_v<R>() * uniform01<R>(wm.v[2]), &s, &c);
            d.cj = sqrt(c > (R)0 ? c : (R)0);
            d.sk = sqrt(s > (R)0 ? s : (R)0);
        }
        d.u = uniform01<R>(wm.v[3]);
    }
}

__device__ inline Philox4 draw_move(uint64_t seed, int64_t copy_id, int64_t sweep, int step) {
    return philox4x64((uint64_t)step, (uint64_t)sweep, (uint64_t)copy_id, 0, seed, kTagMove);
}

// one part of step's draws into its table entry (the parts of a step may run in different threads)
template <typename R>
__device__ inline void draw_part(uint64_t seed, int64_t copy_id, int64_t sweep, int step, int rho, int part,
                                 StepDraw<R>& d) {
    move_part<R>(draw_move(seed, copy_id, sweep, step), rho, part, d);
}

template <typename R>
__device__ inline StepDraw<R> draw_step(uint64_t seed, int64_t pair_stream, int64_t copy_id, int64_t sweep,
                                        int step, int N, int rho) {
    const Philox4 wp = philox4x64((uint64_t)step, (uint64_t)sweep, (uint64_t)pair_stream, 0, seed, kTagPair);
    const Philox4 wm = draw_move(seed, copy_id, sweep, step);
    StepDraw<R> d;
    d.jk = pair_of(wp, N);
    move_part<R>(wm, rho, 1, d);
    move_part<R>(wm, rho, 2, d);
    move_part<R>(wm, rho, 3, d);
    return d;
}

}  // namespace
}  // namespace rlpt
