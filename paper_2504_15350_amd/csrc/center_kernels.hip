// Fluctuation snapshots (Sec. 4.1) without forming them.
//
// The snapshot matrix holds M = n / N blocks of N consecutive columns (one
// block per parameter, its N time instants); the fluctuation matrix is
// S' = S - Msum E^T / N, with Msum (m x M) the block sums of S's columns and
// E (n x M) the block indicator. The library never writes S' out:
//   - the first pass over S multiplies S by [Omega, E] (the indicator columns
//     written by k_center_prep after the sketch), so Msum comes out of that
//     pass as M extra output columns;
//   - S' X = S X - Msum (E^T X / N): k_center_prep forms C = E^T X / N from
//     the operand the pass used, k_center_y subtracts Msum C from the pass's
//     output (FP64 arithmetic, one rounding to the storage type);
//   - S'^T Q = S^T Q - E (Msum^T Q) / N: k_center_cross forms Msum^T Q in
//     FP64 (partial sums over row chunks, added up by k_center_sum), k_center_z
//     subtracts it block by block from the reduced S^T Q.
// Every reduction has a fixed order, so results are deterministic.
#include "device_common.hpp"
#include "internal.hpp"

namespace rpod {

template <typename A>
static Group<A> mkgc(const GroupLaunch<A>& L) {
    Group<A> g;
    g.args = L.args;
    g.tstart = L.tstart;
    g.calls = L.calls;
    g.count = L.count;
    g.skip = L.skip;
    g.skip_mask = L.skip_mask;
    return g;
}

template <typename T>
__device__ __forceinline__ double to_d(T x) {
    if constexpr (sizeof(T) == 2) return (double)(float)x;
    else return (double)x;
}

// tile t = (block k, quad cq): wave w sums column 4 cq + w of block k over its
// N rows (lanes over rows, a fixed butterfly); tiles with cq = 0 also write
// column lp + k of X = the indicator of block k over all ld rows (ind)
template <typename T>
__global__ __launch_bounds__(256) void k_center_prep(Group<CprepArgs> g) {
    if (group_skipped(g)) return;
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const CprepArgs& a = g.args[it];
    const int t = blockIdx.x - g.tstart[it];
    const int k = t % a.K, cq = t / a.K;
    GLOBAL T* X = gbl((T*)a.X);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t j0 = (int64_t)k * a.N;
    const int c = 4 * cq + wave;
    if (c < a.lp) {
        const GLOBAL T* col = X + (int64_t)c * a.ld + j0;
        double s = 0.0;
        for (int64_t j = lane; j < a.N; j += 64) s += to_d(col[j]);
        for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
        if (lane == 0) a.C[k + (int64_t)c * a.K] = s / (double)a.N;
    }
    if (a.ind && cq == 0) {
        GLOBAL T* ind = X + (int64_t)(a.lp + k) * a.ld;
        for (int64_t j = threadIdx.x; j < a.ld; j += 256) ind[j] = (T)((j >= j0 && j < j0 + a.N) ? 1.0f : 0.0f);
    }
}

// 256 rows per tile: Y[i, c] -= sum_k Msum[i, k] C[k + c K] on the FP64 matrix cores, whose chain of fused
// multiply-adds takes the blocks in order, 16 at a time with one rounding to the storage type after each.
// Wave w has rows 64 w ..; lane (n, g) holds rows 4 n .. 4 n + 3 of columns g + 4 v (the C operand; 16 lanes
// read 256 consecutive bytes of a column) and of block sums k0 + 4 s + g (the B operand).
// Bound by reading and writing Y. 100003 x 64 FP32, five blocks: 17.3 us against 20.7 us with a row per
// thread on the vector units (the same bits).
template <typename T>
__global__ __launch_bounds__(256) void k_center_y(Group<CenterYArgs> g) {
    if (group_skipped(g)) return;
    typedef typename vec4_of<T>::type Vec;
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const CenterYArgs& a = g.args[it];
    __shared__ double cs[4096];  // K lp <= 4096
    for (int e = threadIdx.x; e < a.K * a.lp; e += 256) cs[e] = a.C[e];
    __syncthreads();
    const int lane = threadIdx.x & 63, n = lane & 15, kg = lane >> 4;
    const int64_t iw = (int64_t)(blockIdx.x - g.tstart[it]) * 256 + (threadIdx.x >> 6) * 64, i = iw + 4 * n;
    if (iw >= a.m) return;
    GLOBAL T* Y = gbl((T*)a.Y);
    const GLOBAL T* Ms = Y + (int64_t)a.lp * a.ld;
    for (int k0 = 0; k0 < a.K; k0 += 16) {
        Vec mk[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = k0 + 4 * s + kg;
            mk[s] = *reinterpret_cast<const GLOBAL Vec*>(Ms + (int64_t)(k < a.K ? k : 0) * a.ld + i);
            if (k >= a.K) mk[s] = Vec{0, 0, 0, 0};
        }
        for (int c0 = 0; c0 < a.lp; c0 += 16) {
            Vec y[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) y[v] = *reinterpret_cast<const GLOBAL Vec*>(Y + (int64_t)(c0 + kg + 4 * v) * a.ld + i);
            f64x4 acc[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] = f64x4{to_d(y[0][t]), to_d(y[1][t]), to_d(y[2][t]), to_d(y[3][t])};
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int k = k0 + 4 * s + kg;
                const double c = k < a.K ? -cs[k + (c0 + n) * a.K] : 0.0;
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[t] = mfma_16x16x4(c, to_d(mk[s][t]), acc[t]);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                GLOBAL T* py = Y + (int64_t)(c0 + kg + 4 * v) * a.ld + i;
                if (iw + 64 <= a.m) {
                    *reinterpret_cast<GLOBAL Vec*>(py) = Vec{(T)acc[0][v], (T)acc[1][v], (T)acc[2][v], (T)acc[3][v]};
                } else {
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        if (i + t < a.m) py[t] = (T)acc[t][v];
                }
            }
        }
    }
}

// one tile per chunk of rows: the chunk's slab of Msum^T Q (K x lp, FP64 products and sums) on the FP64
// matrix cores. Wave w takes the 16-row blocks w, w + 4, .. (lane (r, g): rows 4 g .. + 3 of its column of
// either operand; rows past m are zero), 16 block sums at a time; the waves' sums are added in order.
// Bound by the latency of its few loads per wave and the ordered sum of the waves. 100003 rows, 64 columns, five blocks: 25.7 us against 28.2 us with 1 x 4
// register blocks on the vector units.
constexpr int CX_NT = 7;  // lp <= 112 (with the indicator columns at most 128)
template <typename T, int NT>
__device__ __forceinline__ void center_cross(const CrossArgs& a, int ch, double* red) {
    typedef typename vec4_of<T>::type Vec;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15, kg = lane >> 4;
    const int64_t i0 = (int64_t)ch * a.chunk, i1 = (i0 + a.chunk < a.m) ? i0 + a.chunk : a.m;
    const GLOBAL T* M = gbl((const T*)a.M);
    const GLOBAL T* Q = gbl((const T*)a.Q);
    for (int k0 = 0; k0 < a.K; k0 += 16) {
        f64x4 acc[NT];
#pragma unroll
        for (int c = 0; c < NT; ++c) acc[c] = f64x4{0, 0, 0, 0};
        const int k = k0 + r16;
        for (int64_t i = i0 + 16 * wave; i < i1; i += 64) {
            Vec x = *reinterpret_cast<const GLOBAL Vec*>(M + (int64_t)(k < a.K ? k : 0) * a.ld + i + 4 * kg), q[NT];
#pragma unroll
            for (int c = 0; c < NT; ++c)
                q[c] = *reinterpret_cast<const GLOBAL Vec*>(Q + (int64_t)(16 * c + r16) * a.ld + i + 4 * kg);
            if (k >= a.K) x = Vec{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int c = 0; c < NT; ++c) acc[c] = mfma_16x16x4(to_d(x[s]), to_d(q[c][s]), acc[c]);
        }
        for (int w = 0; w < 4; ++w) {
            if (wave == w) {
#pragma unroll
                for (int c = 0; c < NT; ++c)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int e = c * 256 + r16 * 16 + mfma_row<double>(kg, v);
                        red[e] = (w == 0 ? 0.0 : red[e]) + acc[c][v];
                    }
            }
            __syncthreads();
        }
        for (int e = threadIdx.x; e < NT * 256; e += 256)  // e: column e / 16, block sum k0 + e mod 16
            if (k0 + e % 16 < a.K) a.Pp[(k0 + e % 16 + (int64_t)(e / 16) * a.K) * a.nchunk + ch] = red[e];
        __syncthreads();
    }
}
template <typename T>
__global__ __launch_bounds__(256) void k_center_cross(Group<CrossArgs> g) {
    if (group_skipped(g)) return;
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const CrossArgs& a = g.args[it];
    const int ch = blockIdx.x - g.tstart[it];
    __shared__ double red[CX_NT * 256];
    switch (a.lp / 16) {  // uniform
        case 1: center_cross<T, 1>(a, ch, red); break;
        case 2: center_cross<T, 2>(a, ch, red); break;
        case 3: center_cross<T, 3>(a, ch, red); break;
        case 4: center_cross<T, 4>(a, ch, red); break;
        case 5: center_cross<T, 5>(a, ch, red); break;
        case 6: center_cross<T, 6>(a, ch, red); break;
        case 7: center_cross<T, 7>(a, ch, red); break;
    }
}

// one tile per entry o: P[o] = the sum of its nchunk partial sums (contiguous);
// thread t adds chunks t, t + 256, .. in order, then a fixed tree in LDS
__global__ __launch_bounds__(256) void k_center_sum(Group<CrossSumArgs> g) {
    if (group_skipped(g)) return;
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const CrossSumArgs& a = g.args[it];
    const int o = blockIdx.x - g.tstart[it];
    const double* src = a.Pp + (int64_t)o * a.nchunk;
    double s = 0.0;
    for (int c = threadIdx.x; c < a.nchunk; c += 256) s += src[c];
    __shared__ double red[256];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) a.P[o] = red[0];
}

// 256 entries per tile over the ld x lp array Z
__global__ __launch_bounds__(256) void k_center_z(Group<CenterZArgs> g) {
    if (group_skipped(g)) return;
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const CenterZArgs& a = g.args[it];
    const int64_t e = (int64_t)(blockIdx.x - g.tstart[it]) * 256 + threadIdx.x;
    const int64_t j = e % a.ld;
    const int64_t c = e / a.ld;
    if (c >= a.lp || j >= a.n) return;
    a.Z[c * a.ld + j] -= a.P[j / a.N + c * a.K] / (double)a.N;
}

hipError_t launch_center_prep(int tx, const GroupLaunch<CprepArgs>& L, hipStream_t st) {
    switch (tx) {
        case DT_F64: hipLaunchKernelGGL(k_center_prep<double>, dim3(L.tiles), dim3(256), 0, st, mkgc(L)); break;
        case DT_F32: hipLaunchKernelGGL(k_center_prep<float>, dim3(L.tiles), dim3(256), 0, st, mkgc(L)); break;
        case DT_BF16: hipLaunchKernelGGL(k_center_prep<__bf16>, dim3(L.tiles), dim3(256), 0, st, mkgc(L)); break;
        case DT_F16: hipLaunchKernelGGL(k_center_prep<_Float16>, dim3(L.tiles), dim3(256), 0, st, mkgc(L)); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_center_y(int tacc, const GroupLaunch<CenterYArgs>& L, hipStream_t st) {
    if (tacc == DT_F64)
        hipLaunchKernelGGL(k_center_y<double>, dim3(L.tiles), dim3(256), 0, st, mkgc(L));
    else
        hipLaunchKernelGGL(k_center_y<float>, dim3(L.tiles), dim3(256), 0, st, mkgc(L));
    return hipGetLastError();
}

hipError_t launch_center_cross(int tacc, const GroupLaunch<CrossArgs>& L, hipStream_t st) {
    if (tacc == DT_F64)
        hipLaunchKernelGGL(k_center_cross<double>, dim3(L.tiles), dim3(256), 0, st, mkgc(L));
    else
        hipLaunchKernelGGL(k_center_cross<float>, dim3(L.tiles), dim3(256), 0, st, mkgc(L));
    return hipGetLastError();
}

hipError_t launch_center_sum(const GroupLaunch<CrossSumArgs>& L, hipStream_t st) {
    hipLaunchKernelGGL(k_center_sum, dim3(L.tiles), dim3(256), 0, st, mkgc(L));
    return hipGetLastError();
}

hipError_t launch_center_z(const GroupLaunch<CenterZArgs>& L, hipStream_t st) {
    hipLaunchKernelGGL(k_center_z, dim3(L.tiles), dim3(256), 0, st, mkgc(L));
    return hipGetLastError();
}

}  // namespace rpod
