// Reduced-order reconstruction (Sec. 4: a field is its zeroth-order time
// average plus the modes weighted by their time-dependent coefficients) and
// the relative L2 error of time-averaged fields against full-order ones
// (Sec. 5). Plain launches (no grouping): the caller's pointers are kernel
// arguments.
//   k_recon_abar  abar_k = (1/T) sum_t alpha[k, t], one wave per mode
//   k_recon_fields32, k_recon_fields64
//                 out[i, t] = mean[i] + sum_k Phi[i, k] alpha[k, t] on the matrix
//                 cores: FP32 with operands split exactly into three BF16 parts,
//                 FP64 on the FP64 matrix cores
//   k_recon_err   per tile of 256 rows: sums of (f - g)^2 and f^2 with
//                 f = avg_t ref[i, t], g = mean[i] + sum_k Phi[i, k] abar_k,
//                 in a fixed order; the tile that ends last adds the tiles'
//                 sums, in order
#include <mutex>

#include "device_common.hpp"
#include "internal.hpp"
#include "split_ops.hpp"

namespace rpod {

// Scratch of the entry point that allocates nothing (rpod_reconstruct_noalloc):
// abar (doubles 0..127), the two sums (128, 129) and the error's partial sums
// (from 256: two per 256-row tile, for m up to RECON_NOALLOC_MAX_M). Each GPU
// holds its own copy until the process ends; every call on a GPU shares it.
static __device__ __align__(256) double scratch[RECON_NOALLOC_DOUBLES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[MAX_DEVICES] = {};
}  // namespace

hipError_t recon_scratch(double** ptr) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[dev] == nullptr) {
        // the device address of this GPU's copy (the array's name in host code
        // is only a stand-in for the symbol)
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = static_cast<double*>(p);
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

template <typename T>
__global__ __launch_bounds__(64) void k_recon_abar(const T* __restrict__ alpha, int r, int64_t T_, double* abar,
                                                   int* arrived) {
    const int k = blockIdx.x;
    if (k == 0 && threadIdx.x == 0) *arrived = 0;
    double s = 0.0;
    for (int64_t t = threadIdx.x; t < T_; t += 64) s += (double)alpha[t * r + k];
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if (threadIdx.x == 0) abar[k] = s / (double)T_;
}

// One pass over ref. Each lane takes 16 bytes of a column (V rows) and a wave RW = 64 V rows of it; the
// waves of a workgroup share its 256 rows and take every TW-th column each, eight columns in flight.
// Bound by the reads of ref. Measured at 262144 x 500 FP32 (524 MB): 102 us against 142 us with
// one row per lane and 4-byte loads, eight in flight.
template <typename T>
__global__ __launch_bounds__(256) void k_recon_err(const T* __restrict__ Phi, const T* __restrict__ mean,
                                                   const double* __restrict__ abar, const T* __restrict__ ref,
                                                   int64_t ld_ref, int64_t m, int r, int64_t T_, double* part,
                                                   double* out2, int* arrived) {
    constexpr int V = 16 / sizeof(T), RW = 64 * V, TW = 4 * RW / 256;
    typedef T Vec __attribute__((ext_vector_type(V)));
    __shared__ double sf[TW][256], sg[TW][256];
    __shared__ bool s_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tw = wave % TW, lr = wave / TW * RW + V * lane;  // first column, first row within the tile
    // a run past row m is moved inside the column; lanes then sum the same rows, and write the same sums
    const int64_t i0 = (int64_t)blockIdx.x * 256, i = i0 + lr < m - V ? i0 + lr : m < V ? 0 : m - V;
    double f[V], g[V];
#pragma unroll
    for (int v = 0; v < V; ++v) f[v] = g[v] = 0.0;
    // columns j = tw, tw + TW, .. < count of p, eight loads at a time (past the end the last column again,
    // not added)
    auto columns = [&](const GLOBAL T* p, int64_t stride, int64_t count, auto add) {
        for (int64_t j = tw; j < count; j += 8 * TW) {
            Vec x[8];
            auto col = [&](int u) { return p + (j + u * TW < count ? j + u * TW : count - 1) * stride; };
            if (m >= V) {  // outside the loop over the loads: behind a branch each they wait for one another
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    x[u] = __builtin_nontemporal_load(reinterpret_cast<const GLOBAL run_vec_u<T, V>*>(col(u) + i));
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = run_load<T, V>(col(u), 0, m, 1, i, 0);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (j + u * TW < count) add(x[u], j + u * TW);
        }
    };
    columns(gbl(ref), ld_ref, T_, [&](const Vec& x, int64_t) {
#pragma unroll
        for (int v = 0; v < V; ++v) f[v] += (double)x[v];
    });
    columns(gbl(Phi), m, r, [&](const Vec& x, int64_t k) {
        const double ab = abar[k];
#pragma unroll
        for (int v = 0; v < V; ++v) g[v] += (double)x[v] * ab;
    });
#pragma unroll
    for (int v = 0; v < V; ++v) {
        if (i + v >= i0 && i + v < m) {
            sf[tw][i + v - i0] = f[v];
            sg[tw][i + v - i0] = g[v];
        }
    }
    __syncthreads();
    double d2 = 0.0, f2 = 0.0;
    if (i0 + tid < m) {
        double fs = 0.0, gs = mean != nullptr ? (double)mean[i0 + tid] : 0.0;
#pragma unroll
        for (int w = 0; w < TW; ++w) {
            fs += sf[w][tid];
            gs += sg[w][tid];
        }
        fs /= (double)T_;
        d2 = (fs - gs) * (fs - gs);
        f2 = fs * fs;
    }
    auto tree = [&](double d, double q) {  // sums over the workgroup in sf[0][0], sg[0][0]
        __syncthreads();
        sf[0][tid] = d;
        sg[0][tid] = q;
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if (tid < h) {
                sf[0][tid] += sf[0][tid + h];
                sg[0][tid] += sg[0][tid + h];
            }
            __syncthreads();
        }
    };
    tree(d2, f2);
    if (tid == 0) {
        GLOBAL double* pp = gbl(part);
        __hip_atomic_store(pp + 2 * blockIdx.x, sf[0][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(pp + 2 * blockIdx.x + 1, sg[0][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the sums are out before the tile is counted
        s_last = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
    }
    __syncthreads();
    if (!s_last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // the other tiles' sums, not older copies
    d2 = f2 = 0.0;
    for (int64_t w = tid; w < gridDim.x; w += 256) {
        d2 += part[2 * w];
        f2 += part[2 * w + 1];
    }
    tree(d2, f2);
    if (tid == 0) {
        out2[0] = sf[0][0];
        out2[1] = sg[0][0];
    }
}

// FP32 fields on the BF16 matrix cores: out = [Phi, mean] [alpha; 1], K = r + 1 in
// steps of 32, operands split exactly into three BF16 parts (FP32-accurate products,
// FP32 sums). Wave w of a workgroup keeps the split operands of its 16 U rows in
// registers for all times (lane (n, g): rows U n .. U n + U - 1) and goes through the
// times 32 at a step, whose coefficients are split as they are staged in LDS for the
// four waves (double-buffered; operand of 16 times: lane (n, g): time n, modes 32 s +
// 8 g .. + 7). With the times as the rows of the matrix-core tile, a lane ends with U
// consecutive rows of a time: stores are runs of 16 lanes x 4 U bytes, at any alignment.
// U = 4 while the rows' operands leave room for two workgroups per CU (NK <= 2 steps),
// else 2. Workgroups short of four per CU split the times too.
// Bound by the writes of the fields. Measured at 262144 x 500, r = 50 (524 MB):
// 118 us, against 392 us for launches of 128 times with [Phi, mean] copied, read and
// split for each and 16-byte stores (the same bits); 131073 x 300, r = 50: 82 us a call
// against 199 us by fused multiply-adds on the vector units, the path of odd sizes until then.
// A value that is not the sum of its parts has parts that are not finite (an infinity, a NaN, a value past
// BF16's largest) or, where it has bits below BF16's smallest, is staged as NaN; every field that comes out of
// the matrix cores not finite is formed again by fused multiply-adds in FP32, in the order of the modes: what
// FP32 arithmetic gives. The test costs 0.1 us of 123 at 262144 x 500, r = 50, and 9 us of 255 at 400000 x
// 300, r = 128.
constexpr int RF_TIMES = 32;  // per step: two operand tiles
constexpr int RF_WG = 1024;   // workgroups to aim at

// the split operands of eight values; NaN with one under 2^-110, which may have bits below 2^-133
__device__ __forceinline__ void split8_or_nan(f32x4 x0, f32x4 x1, e6_u16x8& h, e6_u16x8& m, e6_u16x8& l) {
    split8(x0, x1, h, m, l);
    unsigned least = ~0u;  // of 2 |x| - 1 as bits: a zero is the largest
#pragma unroll
    for (int i = 0; i < 8; ++i) least = min(least, (__builtin_bit_cast(unsigned, i < 4 ? x0[i & 3] : x1[i & 3]) << 1) - 1u);
    if (least < (((127u - 110u) << 23) << 1) - 1u) h[0] = 0x7fc0;
}

// The split coefficients of all times, as the operands lie in LDS: [time tile][K step][part][lane]; one
// thread per (tile, step, lane). Splitting them in every workgroup instead costs 8 us of 125 at 262144 x
// 500, r = 50, and 75 us of 365 at 400000 x 300, r = 128.
__global__ __launch_bounds__(256) void k_recon_prep(const float* __restrict__ alpha, int r, int64_t T_, int nk,
                                                    int64_t count, e6_u16x8* __restrict__ op) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= count) return;
    const int lane = (int)(e & 63), n = lane & 15, g = lane >> 4;
    const int64_t ts = e >> 6, t = ts / nk * 16 + n;  // ts: tile * nk + step
    f32x4 x[2];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int k = 32 * (int)(ts % nk) + 8 * g + i;
        x[i / 4][i % 4] = t < T_ ? (k < r ? alpha[t * r + k] : k == r ? 1.0f : 0.0f) : 0.0f;
    }
    e6_u16x8* d = op + 192 * ts + lane;
    e6_u16x8 h, m, l;
    split8_or_nan(x[0], x[1], h, m, l);
    d[0] = h;
    d[64] = m;
    d[128] = l;
}

// PREP: op holds the split coefficients; else they are split here as they are staged
template <int NK, int U, bool PREP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_recon_fields32(
    const float* __restrict__ Phi, const float* __restrict__ mean, const float* __restrict__ alpha,
    const e6_u16x8* __restrict__ op, float* __restrict__ out, int64_t m, int r, int64_t T_) {
    typedef float Vec __attribute__((ext_vector_type(U)));
    typedef float VecU __attribute__((ext_vector_type(U), aligned(4)));
    constexpr int OPS = 2 * NK * 3 * 64;        // operands (16 bytes) of a step
    constexpr int OPT = (OPS + 255) / 256;      // ... per thread
    constexpr int PPT = (2 * NK + 3) / 4;       // pairs of time tile and K step per wave (w, w + 4, ..)
    __shared__ e6_u16x8 xs[2][OPS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    const int64_t row = (int64_t)blockIdx.x * (64 * U) + wave * (16 * U) + U * n;
    e6_u16x8 ph[NK][U], pm[NK][U], pl[NK][U];
    const GLOBAL float* P = gbl(Phi);
#pragma unroll
    for (int s = 0; s < NK; ++s) {
        Vec v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = 32 * s + 8 * g + i;
            const bool live = k < r || (k == r && mean != nullptr);
            const GLOBAL float* src = k < r ? P + (int64_t)k * m : live ? gbl(mean) : P;
            v[i] = run_load<float, U>(src, 0, m, 1, row, 0);
            v[i] = run_fix<float, U>(v[i], m, 1, row, live ? 0 : 1);
        }
#pragma unroll
        for (int t = 0; t < U; ++t)
            split8_or_nan(f32x4{v[0][t], v[1][t], v[2][t], v[3][t]}, f32x4{v[4][t], v[5][t], v[6][t], v[7][t]}, ph[s][t],
                          pm[s][t], pl[s][t]);
    }
    const int64_t ng = (T_ + RF_TIMES - 1) / RF_TIMES;
    const GLOBAL float* A = gbl(alpha);
    const GLOBAL e6_u16x8* O = gbl(op);
    e6_u16x8 xo[PREP ? OPT : 1];
    f32x4 xr[PREP ? 1 : PPT][2];
    // pair ts = tile * NK + step; modes past r and times past T read as zero
    auto fetch = [&](int64_t q) {
        if constexpr (PREP) {
#pragma unroll
            for (int c = 0; c < OPT; ++c)
                if (OPS % 256 == 0 || tid + 256 * c < OPS) xo[c] = O[q * OPS + tid + 256 * c];
            return;
        }
#pragma unroll
        for (int c = 0; c < (PREP ? 0 : PPT); ++c) {
            const int ts = wave + 4 * c, k0 = 32 * (ts % NK) + 8 * g;
            const int64_t t = q * RF_TIMES + 16 * (ts / NK) + n;
            if (ts >= 2 * NK) continue;
            if (32 * (ts % NK) + 32 <= r && (q + 1) * RF_TIMES <= T_) {
                const GLOBAL run_vec_u<float, 4>* p = reinterpret_cast<const GLOBAL run_vec_u<float, 4>*>(A + t * r + k0);
                xr[c][0] = p[0];
                xr[c][1] = p[1];
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h) xr[c][h] = run_load<float, 4>(A, r, r, T_, k0 + 4 * h, t);
            }
        }
    };
    auto stage = [&](int64_t q, int buf) {
        if constexpr (PREP) {
#pragma unroll
            for (int c = 0; c < OPT; ++c)
                if (OPS % 256 == 0 || tid + 256 * c < OPS) xs[buf][tid + 256 * c] = xo[c];
            return;
        }
#pragma unroll
        for (int c = 0; c < (PREP ? 0 : PPT); ++c) {
            const int ts = wave + 4 * c, k0 = 32 * (ts % NK) + 8 * g;
            const int64_t t = q * RF_TIMES + 16 * (ts / NK) + n;
            if (ts >= 2 * NK) continue;
            if (!(32 * (ts % NK) + 32 <= r && (q + 1) * RF_TIMES <= T_)) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    xr[c][h] = run_fix<float, 4>(xr[c][h], r, T_, k0 + 4 * h, t);
#pragma unroll
                    for (int i = 0; i < 4; ++i) xr[c][h][i] = k0 + 4 * h + i == r ? 1.0f : xr[c][h][i];
                }
            }
            e6_u16x8* x = xs[buf] + 192 * ts + lane;
            e6_u16x8 h, m, l;
            split8_or_nan(xr[c][0], xr[c][1], h, m, l);
            x[0] = h;
            x[64] = m;
            x[128] = l;
        }
    };
    int64_t q = blockIdx.y;
    if (q < ng) fetch(q);
    for (int buf = 0; q < ng; q += gridDim.y, buf ^= 1) {  // uniform
        stage(q, buf);
        if (q + gridDim.y < ng) fetch(q + gridDim.y);
        __syncthreads();  // step staged; the other buffer was read before the last step's barrier
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            f32x4 acc[U];
#pragma unroll
            for (int u = 0; u < U; ++u) acc[u] = f32x4{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < NK; ++s) {
                const e6_u16x8* x = xs[buf] + (tt * NK + s) * 192 + lane;
                const e6_u16x8 ah = x[0], am = x[64], al = x[128];
#pragma unroll
                for (int u = 0; u < U; ++u) {  // the terms of mma6, in its order, with the operands' places changed
                    acc[u] = mma_bf16(ah, pl[s][u], acc[u]);
                    acc[u] = mma_bf16(am, pm[s][u], acc[u]);
                    acc[u] = mma_bf16(al, ph[s][u], acc[u]);
                    acc[u] = mma_bf16(ah, pm[s][u], acc[u]);
                    acc[u] = mma_bf16(am, ph[s][u], acc[u]);
                    acc[u] = mma_bf16(ah, ph[s][u], acc[u]);
                }
            }
            // D[4 g + v][n] of tile u: time 4 g + v, row U n + u
            const int64_t t0 = q * RF_TIMES + 16 * tt + 4 * g;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (t0 + v >= T_) continue;
                GLOBAL float* o = gbl(out) + (t0 + v) * m + row;
                Vec y;
#pragma unroll
                for (int u = 0; u < U; ++u) y[u] = acc[u][v];
                if (row + U <= m) {
                    *reinterpret_cast<GLOBAL VecU*>(o) = y;
                } else {
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (row + u < m) o[u] = y[u];
                }
            }
            f32x4 fin = {0, 0, 0, 0};  // NaN if some field is not finite
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) fin[v] = fmaf(acc[u][v], 0.0f, fin[v]);
            if (__ballot((fin[0] + fin[1]) + (fin[2] + fin[3]) != 0.0f) != 0) {  // uniform; rare
                unsigned again = 0;
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        again |= !(fabsf(acc[u][v]) < INFINITY) && t0 + v < T_ && row + u < m ? 1u << (4 * u + v) : 0u;
                while (again != 0) {
                    const int e = __builtin_ctz(again);
                    const int64_t t = t0 + (e & 3), i = row + (e >> 2);
                    float y = mean != nullptr ? gbl(mean)[i] : 0.0f;
                    for (int k = 0; k < r; ++k) y = fmaf(P[k * m + i], A[t * r + k], y);
                    gbl(out)[t * m + i] = y;
                    again &= again - 1;
                }
            }
        }
    }
}

template <int NK, int U>
static hipError_t recon_fields_nk(int64_t m, int r, int64_t T_, const float* Phi, const float* mean,
                                  const float* alpha, e6_u16x8* op, int64_t op_bytes, float* out, hipStream_t st) {
    const int64_t ng = (T_ + RF_TIMES - 1) / RF_TIMES, gx = (m + 64 * U - 1) / (64 * U), count = ng * 2 * NK * 64;
    int64_t gy = (RF_WG + gx - 1) / gx;
    if (gy > ng) gy = ng;
    const dim3 grid((unsigned)gx, (unsigned)gy);
    // one launch more, where the coefficients are split often enough to pay for it
    if (gx * gy >= RF_WG / 2 && count * 48 <= op_bytes) {
        hipLaunchKernelGGL(k_recon_prep, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, alpha, r, T_, NK,
                           count, op);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_recon_fields32<NK, U, true>), grid, dim3(256), 0, st, Phi, mean, alpha,
                           (const e6_u16x8*)op, out, m, r, T_);
    } else {
        hipLaunchKernelGGL((k_recon_fields32<NK, U, false>), grid, dim3(256), 0, st, Phi, mean, alpha,
                           (const e6_u16x8*)nullptr, out, m, r, T_);
    }
    return hipGetLastError();
}

// op: scratch of op_bytes bytes for the split coefficients (may be null with 0)
static hipError_t recon_fields(int64_t m, int r, int64_t T_, const float* Phi, const float* mean, const float* alpha,
                               float* out, hipStream_t st, void* scratch_op = nullptr, int64_t op_bytes = 0) {
    e6_u16x8* op = static_cast<e6_u16x8*>(scratch_op);
    switch ((r + 32) / 32) {  // K = r + 1
        case 1: return recon_fields_nk<1, 4>(m, r, T_, Phi, mean, alpha, op, op_bytes, out, st);
        case 2: return recon_fields_nk<2, 4>(m, r, T_, Phi, mean, alpha, op, op_bytes, out, st);
        case 3: return recon_fields_nk<3, 2>(m, r, T_, Phi, mean, alpha, op, op_bytes, out, st);
        case 4: return recon_fields_nk<4, 2>(m, r, T_, Phi, mean, alpha, op, op_bytes, out, st);
        case 5: return recon_fields_nk<5, 2>(m, r, T_, Phi, mean, alpha, op, op_bytes, out, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_reconstruct_mfma(int64_t m, int r, int64_t T_, const float* Phi, const float* mean,
                                   const float* alpha, float* out, float* op, int64_t op_bytes, float*, int, SxArgs*,
                                   int*, hipStream_t st) {
    return recon_fields(m, r, T_, Phi, mean, alpha, out, st, op, op_bytes);
}

// FP64 fields on the FP64 matrix cores: mean[i] + sum_k Phi[i, k] alpha[k, t], a chain of fused
// multiply-adds in the order of k (the same bits as on the vector units). Each wave keeps Phi for its 32 rows
// in registers (lane (n, kg): rows 2 n, 2 n + 1, modes 4 s + kg) and goes through the times 16 at a step,
// alpha staged in LDS (double-buffered); a lane ends with two consecutive rows of a time. Bound by the FP64
// matrix cores at r = 50 and more, by the writes of the fields below that. Measured at 131072 x 300, r = 50: a call of 166 us
// against 292 us on the vector units.
template <int NS>  // steps of four modes
__global__ __launch_bounds__(256) void k_recon_fields64(const double* __restrict__ Phi, const double* __restrict__ mean,
                                                        const double* __restrict__ alpha, double* __restrict__ out,
                                                        int64_t m, int r, int64_t T_) {
    typedef double d2 __attribute__((ext_vector_type(2)));
    typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
    constexpr int LDA = 4 * NS + 1;  // odd: the 16 times of an operand read meet different banks
    constexpr int APT = NS / 4;      // alpha values per thread and step
    __shared__ double as[2][16 * LDA];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, kg = lane >> 4;
    const int64_t row = (int64_t)blockIdx.x * 128 + wave * 32 + 2 * n;
    const GLOBAL double *P = gbl(Phi), *al = gbl(alpha);
    double b[NS][2];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int k = 4 * s + kg;
        const d2 x = run_load<double, 2>(P, m, m, r, row, k);
        const d2 y = run_fix<double, 2>(x, m, r, row, k);
        b[s][0] = y[0];
        b[s][1] = y[1];
    }
    d2 base = {0.0, 0.0};
    if (mean != nullptr) base = run_fix<double, 2>(run_load<double, 2>(gbl(mean), 0, m, 1, row, 0), m, 1, row, 0);
    for (int e = tid; e < 16 * LDA; e += 256) as[0][e] = as[1][e] = 0.0;
    const int64_t nt = (T_ + 15) / 16;
    double ar[APT];
    auto fetch = [&](int64_t q) {
#pragma unroll
        for (int c = 0; c < APT; ++c) {
            const int e = tid + 256 * c;
            if (e < 16 * r) ar[c] = q * 16 + e / r < T_ ? al[q * 16 * r + e] : 0.0;
        }
    };
    int64_t q = blockIdx.y;
    if (q < nt) fetch(q);
    __syncthreads();
    for (int buf = 0; q < nt; q += gridDim.y, buf ^= 1) {  // uniform
#pragma unroll
        for (int c = 0; c < APT; ++c) {
            const int e = tid + 256 * c;
            if (e < 16 * r) as[buf][e / r * LDA + e % r] = ar[c];
        }
        if (q + gridDim.y < nt) fetch(q + gridDim.y);
        __syncthreads();  // step staged; the other buffer was read before the last step's barrier
        f64x4 acc[2] = {{base[0], base[0], base[0], base[0]}, {base[1], base[1], base[1], base[1]}};
        const double* a = as[buf] + n * LDA + kg;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const double x = a[4 * s];
            acc[0] = mfma_16x16x4(x, b[s][0], acc[0]);
            acc[1] = mfma_16x16x4(x, b[s][1], acc[1]);
        }
        // D[kg + 4 v][n] of tile u: time kg + 4 v, row 2 n + u
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t t = q * 16 + kg + 4 * v;
            if (t >= T_) continue;
            GLOBAL double* o = gbl(out) + t * m + row;
            if (row + 2 <= m)
                *reinterpret_cast<GLOBAL d2u*>(o) = d2{acc[0][v], acc[1][v]};
            else if (row < m)
                o[0] = acc[0][v];
        }
    }
}

static hipError_t recon_fields(int64_t m, int r, int64_t T_, const double* Phi, const double* mean,
                                 const double* alpha, double* out, hipStream_t st) {
    const int64_t gx = (m + 127) / 128, nt = (T_ + 15) / 16;
    int64_t gy = (RF_WG + gx - 1) / gx;
    if (gy > nt) gy = nt;
    const dim3 grid((unsigned)gx, (unsigned)gy);
    if (r <= 16) hipLaunchKernelGGL(k_recon_fields64<4>, grid, dim3(256), 0, st, Phi, mean, alpha, out, m, r, T_);
    else if (r <= 32) hipLaunchKernelGGL(k_recon_fields64<8>, grid, dim3(256), 0, st, Phi, mean, alpha, out, m, r, T_);
    else if (r <= 64) hipLaunchKernelGGL(k_recon_fields64<16>, grid, dim3(256), 0, st, Phi, mean, alpha, out, m, r, T_);
    else hipLaunchKernelGGL(k_recon_fields64<32>, grid, dim3(256), 0, st, Phi, mean, alpha, out, m, r, T_);
    return hipGetLastError();
}

template <typename T>
static hipError_t recon_t(int64_t m, int r, int64_t T_, const void* Phi, const void* mean, const void* alpha,
                          void* out, const void* ref, int64_t ld_ref, double* abar, double* part, double* out2,
                          hipStream_t st) {
    const unsigned rows = (unsigned)((m + 255) / 256);
    if (out != nullptr) {
        hipError_t e = recon_fields(m, r, T_, (const T*)Phi, (const T*)mean, (const T*)alpha, (T*)out, st);
        if (e != hipSuccess) return e;
    }
    if (ref != nullptr) {
        int* arrived = reinterpret_cast<int*>(out2 + 2);  // tiles that are done
        hipLaunchKernelGGL(k_recon_abar<T>, dim3(r), dim3(64), 0, st, (const T*)alpha, r, T_, abar, arrived);
        hipLaunchKernelGGL(k_recon_err<T>, dim3(rows), dim3(256), 0, st, (const T*)Phi, (const T*)mean,
                           (const double*)abar, (const T*)ref, ld_ref, m, r, T_, part, out2, arrived);
    }
    return hipGetLastError();
}

hipError_t launch_reconstruct(int dt, int64_t m, int r, int64_t T_, const void* Phi, const void* mean,
                              const void* alpha, void* out, const void* ref, int64_t ld_ref, double* abar,
                              double* part, double* out2, hipStream_t st) {
    if (dt == DT_F64) return recon_t<double>(m, r, T_, Phi, mean, alpha, out, ref, ld_ref, abar, part, out2, st);
    if (dt == DT_F32) return recon_t<float>(m, r, T_, Phi, mean, alpha, out, ref, ld_ref, abar, part, out2, st);
    return hipErrorInvalidValue;
}

}  // namespace rpod
