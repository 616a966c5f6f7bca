// FP64 energies of dense graphs for CDNA4 (gfx950): the first stage of an
// energy recomputation as a banded product on the FP64 matrix cores.
// H = -2 sum_q J_q Re(conj(a_p a_s) a_m a_n), eq. 4-body Hamiltonian of
// Benedetti & Leuzzi, arXiv 2511.13508, in pair space: with the pairs sorted
// by frequency sum, H = -2 sum_x Re(conj(b_x) G_x), G_x = sum_{y > x} J_xy b_y,
// b_x the product of pair x, J a narrow band.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"
#include "internal.hpp"

namespace rlpt {
namespace {

constexpr int kRows = 16, kCols = 16;  // of a matrix-core tile: pairs, copies
constexpr size_t kRedBytes = 4 * kCols * sizeof(double);  // the waves' sums, static LDS
typedef double f64x4 __attribute__((ext_vector_type(4)));

// every term's place above the diagonal: the operand of 4 columns holds, at
// lane (column % 4) * 16 + row % 16, the value of that row and column
template <typename R>
__global__ __launch_bounds__(256) void k_energy_fill(DevPtrs<R> P) {
    const SampleDev sd = P.samples[blockIdx.y];
    const EnergySample es = P.en_samples[blockIdx.y];
    const uint16_t* pos = P.en_rank + es.rank_base;
    const uint32_t* tile = P.en_tile + es.tile_base;
    double* band = P.en_band + es.band_base;
    for (int64_t q = blockIdx.x * (int64_t)256 + threadIdx.x; q < sd.n_quads; q += (int64_t)gridDim.x * 256) {
        const ushort4 t = P.quads[sd.quad_base + q];
        const uint32_t u = pos[t.x * sd.N + t.y], v = pos[t.z * sd.N + t.w];
        const uint32_t row = min(u, v), c = max(u, v) - row / kRows * kRows;
        band[(size_t)tile[row / kRows] * 64 + (size_t)(c >> 2) * 64 + (c & 3u) * 16 + row % kRows] = P.Jq[sd.quad_base + q];
    }
}

// Partial energies of kCols copies of one sample over one of `parts` ranges of
// row tiles, a tile at a time per wave; the pair products, formed in FP64 from
// the amplitudes in LDS, are the second operand and, for the tile's own rows,
// what its product is contracted with.  groups: copy tiles of a sample.
// Summed term by term (k_resync_part) a term costs every copy four FP64
// amplitudes from LDS, which bounds it; here a pair's two amplitudes serve the
// 16 rows of a tile, and the FP64 matrix cores bound it: 16 rows rather than
// 32 because a tile also multiplies the half of its diagonal block that is
// empty.  Us for the energies, terms -> band, on an MI355X: N = 256, 640 copies
// of 8 samples 585 -> 133; 4 copies 264 -> 39; N = 128, 640 copies 103 -> 36;
// N = 64, 384 copies 17 -> 11; N = 16, 16 copies 8.8 -> 8.1.
template <typename R>
__global__ __launch_bounds__(256) void k_energy_band(DevPtrs<R> P, ShapeInfo sh, int groups) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[4][kCols];
    // the samples in turn (an XCD takes every eighth block and so reads few
    // samples' bands), their copy tiles, then the row tiles
    const int S = sh.n_samples, parts = sh.en_parts;
    const int mu = blockIdx.x % S, group = (blockIdx.x / S) % groups, part = blockIdx.x / (S * groups);
    const SampleDev sd = P.samples[mu];
    const EnergySample es = P.en_samples[mu];
    const int N = sd.N, np = N * (N - 1) / 2, n_tiles = (np + kRows - 1) / kRows, Rc = sh.copies_per_sample;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, col = lane & 15, quad = lane >> 4;
    const int t0 = (int)((int64_t)n_tiles * part / parts), t1 = (int)((int64_t)n_tiles * (part + 1) / parts);
    const int c = group * kCols + col;
    R2<R>* a = reinterpret_cast<R2<R>*>(smem);  // [mode][16 copies]
    const uint32_t* tile = P.en_tile + es.tile_base;
    double H = 0;
    if (t0 < t1) {
        const R2<R>* amp = reinterpret_cast<const R2<R>*>(P.amp) + sd.amp_base + (int64_t)min(c, Rc - 1) * N;
        for (int m = tid >> 4; m < N; m += 16) a[m * kCols + col] = c < Rc ? amp[m] : mk2<R>(0, 0);
        // LDS offsets of the two modes of the block's pairs (band values past the last pair are zero)
        uint32_t* pm = reinterpret_cast<uint32_t*>(a + N * kCols);
        const int first = t0 * kRows, n = (t1 - 1) * kRows + 4 * (int)(tile[t1] - tile[t1 - 1]) + kRows - first;
        constexpr uint32_t kRowBytes = kCols * sizeof(R2<R>);
        for (int i = tid; i < n; i += 256) {
            const uint32_t v = P.en_pairs[es.pair_base + min(first + i, np - 1)];
            pm[i] = (v & 255u) * kRowBytes | (v >> 8) * kRowBytes << 16;
        }
        __syncthreads();
        const auto product = [&](uint32_t v, double& br, double& bi) {
            const R2<R> x = *reinterpret_cast<const R2<R>*>(smem + (v & 0xffffu) + sizeof(R2<R>) * col);
            const R2<R> y = *reinterpret_cast<const R2<R>*>(smem + (v >> 16) + sizeof(R2<R>) * col);
            const double xr = x.x, xi = x.y, yr = y.x, yi = y.y;
            br = xr * yr - xi * yi;
            bi = xr * yi + xi * yr;
        };
        for (int t = t0 + wave; t < t1; t += 4) {
            const int n4 = (int)(tile[t + 1] - tile[t]);
            // (reads up to kBandSlack words past the tile's values, unused)
            const double* A = P.en_band + es.band_base + (size_t)tile[t] * 64;
            const uint32_t* pq = pm + (t * kRows - first);
            f64x4 gr = {0, 0, 0, 0}, gi = gr;
            double ra[8];  // eight operands ahead of their use
#pragma unroll
            for (int u = 0; u < 8; ++u) ra[u] = (A + u * 64)[lane];
            const auto step = [&](int q, double j) {
                double br, bi;
                product(pq[4 * q + quad], br, bi);
                gr = __builtin_amdgcn_mfma_f64_16x16x4f64(j, br, gr, 0, 0, 0);
                gi = __builtin_amdgcn_mfma_f64_16x16x4f64(j, bi, gi, 0, 0, 0);
            };
            int q0 = 0;
            for (; q0 + 8 <= n4; q0 += 8) {  // no branch inside: the next loads stay in flight
                A += 8 * 64;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const double j = ra[u];
                    ra[u] = (A + u * 64)[lane];
                    step(q0 + u, j);
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (q0 + u < n4) step(q0 + u, ra[u]);
            // lane (quad, col) holds rows quad, 4 + quad, 8 + quad, 12 + quad of copy col
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double br, bi;
                product(pq[4 * r + quad], br, bi);
                H += br * gr[r] + bi * gi[r];
            }
        }
    }
    H += __shfl_xor(H, 16);
    H += __shfl_xor(H, 32);
    if (quad == 0) red[wave][col] = H;
    __syncthreads();
    if (tid < kCols && c < Rc)
        P.rs_part[((int64_t)mu * Rc + c) * parts + part] =
            -2.0 * ((red[0][col] + red[1][col]) + (red[2][col] + red[3][col]));
}

template <typename R>
hipError_t fill_t(const void* ptrs, const ShapeInfo& sh, int64_t max_quads, hipStream_t st) {
    const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((max_quads + 1023) / 1024, 1024));
    hipLaunchKernelGGL(k_energy_fill<R>, dim3(blocks, sh.n_samples), dim3(256), 0, st,
                       *static_cast<const DevPtrs<R>*>(ptrs));
    return hipGetLastError();
}

template <typename R>
hipError_t band_t(const void* ptrs, const ShapeInfo& sh, hipStream_t st) {
    const int groups = (sh.copies_per_sample + kCols - 1) / kCols;
    const size_t lds = energy_lds_bytes(sizeof(R) == 8 ? RLPT_FP64 : RLPT_FP32, sh.spec_stride, sh.en_columns) - kRedBytes;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_energy_band<R>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_energy_band<R>, dim3(sh.n_samples * groups * sh.en_parts), dim3(256), lds, st,
                       *static_cast<const DevPtrs<R>*>(ptrs), sh, groups);
    return hipGetLastError();
}

}  // namespace

// of a workgroup: the amplitudes of a copy tile, its pairs' offsets, the waves' sums
size_t energy_lds_bytes(int precision, int max_N, int columns) {
    return (size_t)max_N * kCols * 2 * (precision == RLPT_FP64 ? 8 : 4) + (size_t)columns * 4 + kRedBytes;
}

hipError_t launch_energy_fill(int precision, const void* ptrs, const ShapeInfo& sh, int64_t max_quads, hipStream_t st) {
    return precision == RLPT_FP64 ? fill_t<double>(ptrs, sh, max_quads, st) : fill_t<float>(ptrs, sh, max_quads, st);
}

hipError_t launch_energy_band(int precision, const void* ptrs, const ShapeInfo& sh, hipStream_t st) {
    return precision == RLPT_FP64 ? band_t<double>(ptrs, sh, st) : band_t<float>(ptrs, sh, st);
}

}  // namespace rlpt
