// Per-mode lists as the sweep kernels read them: the field contributions of
// packed entries and of chunks, and chunks held in registers ahead of their
// step.  F_l = sum over l's list of J conj(a_x) a_y a_z (eq. local field,
// sec. III.A of Benedetti & Leuzzi, arXiv 2511.13508).
#pragma once
#include "device.hpp"
#include "internal.hpp"

namespace rlpt {
namespace {

// contribution J conj(a_x) a_y a_z of one packed entry
template <typename R>
__device__ inline void field_term(uint32_t e, R j, const R2<R>* __restrict__ a, R& fr, R& fi) {
    const R2<R> ax = a[e & 1023u];
    const R2<R> ay = a[(e >> 10) & 1023u];
    const R2<R> az = a[e >> 20];
    const R pr = ax.x * ay.x + ax.y * ay.y;
    const R pi = ax.x * ay.y - ax.y * ay.x;
    const R qr = pr * az.x - pi * az.y;
    const R qi = pr * az.y + pi * az.x;
    fr += j * qr;
    fi += j * qi;
}

// chunked layout: a chunk holds 4 entries sharing the partner x; the field
// contribution is conj(a_x) * sum_i J_i a_{y_i} a_{z_i}
template <typename R>
__device__ inline void chunk_pair(uint32_t v, R j, const R2<R>* __restrict__ a, R& gr, R& gi) {
    const R2<R> ay = a[v & 0xffu];
    const R2<R> az = a[(v >> 8) & 0xffu];
    gr += j * (ay.x * az.x - ay.y * az.y);
    gi += j * (ay.x * az.y + ay.y * az.x);
}

template <typename R>
__device__ inline void chunk_term(uint32_t x, uint2 yz, typename J4<R>::T j, const R2<R>* __restrict__ a, R& fr,
                                  R& fi) {
    R gr = 0, gi = 0;
    chunk_pair<R>(yz.x & 0xffffu, j.x, a, gr, gi);
    chunk_pair<R>(yz.x >> 16, j.y, a, gr, gi);
    chunk_pair<R>(yz.y & 0xffffu, j.z, a, gr, gi);
    chunk_pair<R>(yz.y >> 16, j.w, a, gr, gi);
    const R2<R> ax = a[x];
    fr += ax.x * gr + ax.y * gi;
    fi += ax.x * gi - ax.y * gr;
}

// list chunks of one mode held in registers ahead of their step: thread t of a
// group of nt owns chunks beg + t + m * nt, m < PF (the host picks PF so that
// every list of the launch fits); consumed in the order the streaming loop
// of field_partial_chunk would take them
template <typename R, int PF>
struct ChunkRegs {
    uint32_t x[PF];
    uint2 yz[PF];
    typename J4<R>::T J[PF];
    uint32_t n;  // chunks of this thread
};

template <typename R, int PF>
__device__ inline void chunk_prefetch(const DevPtrs<R>& P, const uint32_t* lb, int l, int t, int nt,
                                      ChunkRegs<R, PF>& rg) {
    using JT = typename J4<R>::T;
    const uint32_t beg = lb[l], end = lb[l + 1];
    const JT* __restrict__ Jv = reinterpret_cast<const JT*>(P.cJ);
    // a lane past the list's end reads chunk 0: a load behind a branch would
    // keep the registers' old values alive and wait for the loads before it
    rg.n = 0;
#pragma unroll
    for (int m = 0; m < PF; ++m) {
        const uint32_t c = beg + t + (uint32_t)m * nt;
        const uint32_t at = c < end ? c : 0;
        rg.x[m] = P.cx[at];
        rg.yz[m] = P.cyz[at];
        rg.J[m] = Jv[at];
        rg.n += c < end ? 1 : 0;
    }
}

template <typename R, int PF>
__device__ inline void chunk_consume(const ChunkRegs<R, PF>& rg, const R2<R>* __restrict__ a, R& fr, R& fi) {
#pragma unroll
    for (int m = 0; m < PF; ++m)
        if ((uint32_t)m < rg.n) chunk_term<R>(rg.x[m], rg.yz[m], rg.J[m], a, fr, fi);
}

// keep the compiler from moving LDS accesses across a write by one lane that
// all lanes then read (the hardware runs one wave's LDS accesses in order);
// emits no wait, so global loads in flight stay in flight
__device__ inline void wave_sync() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_wave_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

}  // namespace
}  // namespace rlpt
