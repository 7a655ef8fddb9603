// Small FP64 linear algebra of the rPOD path and the Gaussian sketch.
//
//   k_omega        Gaussian sketch (Alg. 1 step 1) from Philox4x32-10
//   k_gram         FP64 Gram matrix Y^T Y of a tall matrix on FP64 MFMA
//   k_gram_reduce  its partial sums, then Cholesky + triangular inverse for CholeskyQR (step 4)
//   k_jacobi       SVD of the small T of step 6 via the eigenvectors of T T^T
//                  (pivoted Cholesky, then preconditioned one-sided Jacobi)
//   k_lift_coef    the small factors of the lift (step 7) and the coefficients
//   k_colmax/...   deterministic sign convention and output packing
#include <type_traits>

#include "device_common.hpp"
#include "internal.hpp"

namespace rpod {

template <typename T>
using V4 = typename vec4_of<T>::type;

template <typename A>
static Group<A> mkg(const GroupLaunch<A>& L) {
    Group<A> g;
    g.args = L.args;
    g.tstart = L.tstart;
    g.calls = L.calls;
    g.count = L.count;
    g.skip = L.skip;
    g.skip_mask = L.skip_mask;
    return g;
}

__global__ void k_zero_ints(Group<ZeroArgs> g) {
    if (group_skipped(g)) return;
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const ZeroArgs& a = g.args[it];
    const int i = (blockIdx.x - g.tstart[it]) * blockDim.x + threadIdx.x;
    if (i < a.count) a.p[i] = 0;
}

hipError_t launch_zero_ints(const GroupLaunch<ZeroArgs>& L, hipStream_t st) {
    hipLaunchKernelGGL(k_zero_ints, dim3(L.tiles), dim3(256), 0, st, mkg(L));
    return hipGetLastError();
}

// Per-call table: one entry per matrix, written from kernel arguments so
// that it needs no host staging buffer (and may precede a graph launch).
constexpr int CALLS_PER_LAUNCH = 16;
struct CallBatch {
    CallDesc d[CALLS_PER_LAUNCH];
    int first, count;
};

__global__ void k_set_calls(CallDesc* table, CallBatch b) {
    const int i = threadIdx.x;
    if (i < b.count) table[b.first + i] = b.d[i];
}

hipError_t launch_set_calls(CallDesc* table, const CallDesc* host, int count, hipStream_t st) {
    for (int first = 0; first < count; first += CALLS_PER_LAUNCH) {
        CallBatch b;
        b.first = first;
        b.count = count - first < CALLS_PER_LAUNCH ? count - first : CALLS_PER_LAUNCH;
        for (int i = 0; i < b.count; ++i) b.d[i] = host[first + i];
        hipLaunchKernelGGL(k_set_calls, dim3(1), dim3(CALLS_PER_LAUNCH), 0, st, table, b);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Gaussian sketch. Thread per (row j, column pair t).
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void omega_body(uint64_t seed, int64_t n, int l, int lpad, int64_t rows_pad, GLOBAL T* out,
                                           int64_t ldo, int64_t bx, int t /* column pair */, uint32_t stream) {
    const int64_t j = bx * blockDim.x + threadIdx.x;
    if (j >= rows_pad) return;
    const int c0 = 2 * t, c1 = 2 * t + 1;
    double g0 = 0.0, g1 = 0.0;
    if (j < n && c0 < l) {
        const philox_out o = philox4x32_10((uint32_t)j, (uint32_t)((uint64_t)j >> 32), (uint32_t)t, stream,
                                           (uint32_t)seed, (uint32_t)(seed >> 32));
        const uint64_t a = ((uint64_t)(o.x[0] >> 5) << 26) + (o.x[1] >> 6);
        const uint64_t b = ((uint64_t)(o.x[2] >> 5) << 26) + (o.x[3] >> 6);
        const double u1 = ((double)a + 0.5) * 0x1.0p-53;
        const double u2 = (double)b * 0x1.0p-53;
        const double rho = sqrt(-2.0 * log(u1));
        const double th = 6.283185307179586 * u2;
        g0 = rho * cos(th);
        g1 = rho * sin(th);
    }
    if (c0 < lpad) out[(int64_t)c0 * ldo + j] = narrow<T>(g0);
    if (c1 < lpad) out[(int64_t)c1 * ldo + j] = narrow<T>(c1 < l ? g1 : 0.0);
}

// grouped: local tile t covers rows 256 (t % nb) .. and column pair t / nb
template <typename T>
__global__ void k_omega(Group<OmegaArgs> g) {
    if (group_skipped(g)) return;
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const OmegaArgs& a = g.args[it];
    const int t = blockIdx.x - g.tstart[it];
    const int nb = (int)((a.rows_pad + 255) / 256);
    const uint64_t seed = a.call >= 0 ? g.calls[a.call].seed : a.seed;
    omega_body<T>(seed, a.n, a.l, a.lpad, a.rows_pad, gbl((T*)a.out), a.ldo, t % nb, t / nb, a.stream);
}

template <typename T>
__global__ void k_omega_direct(uint64_t seed, int64_t n, int l, int64_t ldo, T* out) {
    omega_body<T>(seed, n, l, l, n, gbl(out), ldo, blockIdx.x, blockIdx.y, 0u);
}

hipError_t launch_omega(int tout, const GroupLaunch<OmegaArgs>& L, hipStream_t st) {
    if (tout == DT_F64)
        hipLaunchKernelGGL(k_omega<double>, dim3(L.tiles), dim3(256), 0, st, mkg(L));
    else if (tout == DT_F32)
        hipLaunchKernelGGL(k_omega<float>, dim3(L.tiles), dim3(256), 0, st, mkg(L));
    else if (tout == DT_BF16)
        hipLaunchKernelGGL(k_omega<__bf16>, dim3(L.tiles), dim3(256), 0, st, mkg(L));
    else if (tout == DT_F16)
        hipLaunchKernelGGL(k_omega<_Float16>, dim3(L.tiles), dim3(256), 0, st, mkg(L));
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_omega_direct(int tout, uint64_t seed, int64_t n, int l, void* out, int64_t ldo, hipStream_t st) {
    dim3 grid((unsigned)((n + 255) / 256), (unsigned)((l + 1) / 2));
    if (tout == DT_F64)
        hipLaunchKernelGGL(k_omega_direct<double>, grid, dim3(256), 0, st, seed, n, l, ldo, (double*)out);
    else if (tout == DT_F32)
        hipLaunchKernelGGL(k_omega_direct<float>, grid, dim3(256), 0, st, seed, n, l, ldo, (float*)out);
    else if (tout == DT_BF16)
        hipLaunchKernelGGL(k_omega_direct<__bf16>, grid, dim3(256), 0, st, seed, n, l, ldo, (__bf16*)out);
    else if (tout == DT_F16)
        hipLaunchKernelGGL(k_omega_direct<_Float16>, grid, dim3(256), 0, st, seed, n, l, ldo, (_Float16*)out);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

__global__ void k_sketch_bits(uint64_t seed, int64_t n, int npairs, uint32_t* out) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int t = blockIdx.y;
    if (j >= n) return;
    const philox_out o = philox4x32_10((uint32_t)j, (uint32_t)((uint64_t)j >> 32), (uint32_t)t, 0u,
                                       (uint32_t)seed, (uint32_t)(seed >> 32));
    uint32_t* p = out + (j * npairs + t) * 4;
    p[0] = o.x[0]; p[1] = o.x[1]; p[2] = o.x[2]; p[3] = o.x[3];
}

hipError_t launch_sketch_bits(uint64_t seed, int64_t n, int l, uint32_t* out, hipStream_t st) {
    const int npairs = (l + 1) / 2;
    hipLaunchKernelGGL(k_sketch_bits, dim3((unsigned)((n + 255) / 256), (unsigned)npairs), dim3(256), 0, st, seed,
                       n, npairs, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Gram matrix in FP64 on MFMA: G[16a + mm][16b + nn] = sum_i Y[i][16a+mm] Y[i][16b+nn]
// for tile pairs a <= b. Each wave walks row blocks of 16 (grid-stride); a
// lane loads rows 4*(l/16)..+3 of column 16a + l%16 for every tile a, and
// MFMA (pair, s) uses row slot s of that vector as the K index.
// Pairs [PLO, PHI) of the NT(NT+1)/2 upper-triangle tile pairs belong to one
// pair group of the launch; partials are reduced over the 4 waves in LDS in a
// fixed order and written per workgroup.
// ---------------------------------------------------------------------------
constexpr int GRAM_WGS = 512;

__host__ __device__ constexpr int npairs_of(int nt) { return nt * (nt + 1) / 2; }
__host__ __device__ constexpr int gram_groups(int nt) { return nt <= 4 ? 1 : 3; }
__host__ __device__ constexpr int gram_pg(int nt) {
    return (npairs_of(nt) + gram_groups(nt) - 1) / gram_groups(nt);
}

int64_t gram_partial_count(int nt) { return (int64_t)GRAM_WGS * npairs_of(nt) * 256; }

template <typename Tin, int NT, int PLO, int PHI>
__device__ __forceinline__ void gram_body(const GLOBAL Tin* __restrict__ Y, int64_t ld, int64_t M,
                                          GLOBAL double* __restrict__ Gpart, double* red, int bx, int nwg) {
    constexpr int PG = PHI - PLO;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, kg = lane >> 4;
    f64x4 acc[PG];
#pragma unroll
    for (int p = 0; p < PG; ++p) acc[p] = f64x4{0, 0, 0, 0};

    const int64_t nrb = (M + 15) / 16, rstride = (int64_t)nwg * 4;
    // the next row block is loaded while the matrix cores work on this one
    V4<Tin> vn[NT];
    auto load = [&](int64_t rb) {
#pragma unroll
        for (int a = 0; a < NT; ++a)
            vn[a] = *reinterpret_cast<const GLOBAL V4<Tin>*>(Y + (int64_t)(16 * a + r16) * ld + rb * 16 + 4 * kg);
    };
    int64_t rb = (int64_t)bx * 4 + wave;
    if (rb < nrb) load(rb);
    for (; rb < nrb; rb += rstride) {
        double x[NT][4];
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
            for (int s = 0; s < 4; ++s) x[a][s] = (double)vn[a][s];
        if (rb + rstride < nrb) load(rb + rstride);
        // row slot outermost: consecutive matrix-core instructions are independent
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            int p = 0;
#pragma unroll
            for (int a = 0; a < NT; ++a)
#pragma unroll
                for (int b = a; b < NT; ++b) {
                    if (p >= PLO && p < PHI) acc[p - PLO] = mfma_16x16x4(x[a][s], x[b][s], acc[p - PLO]);
                    ++p;
                }
        }
    }
    // fixed-order reduction over the 4 waves
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int p = 0; p < PG; ++p)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int idx = p * 256 + mfma_row<double>(kg, v) * 16 + r16;
                    red[idx] = (w == 0 ? 0.0 : red[idx]) + acc[p][v];
                }
        }
        __syncthreads();
    }
    constexpr int NP = npairs_of(NT);
    for (int e = threadIdx.x; e < PG * 256; e += 256) {
        const int p = PLO + e / 256;
        Gpart[((int64_t)bx * NP + p) * 256 + (e % 256)] = red[e];
    }
}

// grouped: local tile t is partial workgroup bx of pair group grp. With
// several pair groups, the groups of one row block sit 8 tiles apart (the
// same XCD when the item starts at a multiple of 8, at about the same time),
// so the second and third reads of the rows come from that XCD's L2.
template <typename Tin, int NT>
__global__ __launch_bounds__(256) void k_gram(Group<GramArgs> g) {
    if (group_skipped(g)) return;
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const GramArgs& a = g.args[it];
    if (a.cond != nullptr && !(*a.cond & a.cond_mask)) return;
    const int t = blockIdx.x - g.tstart[it];
    constexpr int NG = gram_groups(NT);
    int bx = t % a.nwg, grp = t / a.nwg;
    if (NG > 1 && (a.nwg & 7) == 0 && (g.tstart[it] & 7) == 0) {
        grp = (t >> 3) % NG;
        bx = (t / (8 * NG)) * 8 + (t & 7);
    }
    constexpr int NP = npairs_of(NT), PG = gram_pg(NT);
    __shared__ double red[PG * 256];
    const GLOBAL Tin* Y = gbl((const Tin*)a.Y);
    GLOBAL double* Gp = gbl(a.Gpart);
    if (grp == 0) gram_body<Tin, NT, 0, (PG < NP ? PG : NP)>(Y, a.ld, a.M, Gp, red, bx, a.nwg);
    if constexpr (gram_groups(NT) > 1) {
        if (grp == 1) gram_body<Tin, NT, PG, (2 * PG < NP ? 2 * PG : NP)>(Y, a.ld, a.M, Gp, red, bx, a.nwg);
        if (grp == 2) gram_body<Tin, NT, 2 * PG, NP>(Y, a.ld, a.M, Gp, red, bx, a.nwg);
    }
}

// 1 / sqrt(x) and 1 / x for x > 0 (finite): the hardware estimates refined by
// two Newton steps each (the error of the estimate squares at every step).
__device__ __forceinline__ double rsqrt_nr(double x) {
    double y = __builtin_amdgcn_rsq(x);
    const double hx = 0.5 * x;
    y = y * fma(-hx * y, y, 1.5);
    y = y * fma(-hx * y, y, 1.5);
    return y;
}
__device__ __forceinline__ double rcp_nr(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    y = fma(y, fma(-x, y, 1.0), y);
    return y;
}

// v of lane `lane` (wave-uniform lane index), as a uniform value.
__device__ __forceinline__ double read_lane(double v, int lane) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// ---------------------------------------------------------------------------
// Cholesky G = R^T R and X = R^-1 for lp = 16 NB <= 128, by the workgroup that
// finishes the reduction of G. Wave w keeps the blocks (i, w), i <= w, of the
// 16 x 16 blocks of A as FP64 MFMA accumulators (right-looking; lane (n, kg)
// holds rows kg + 4 v of column n). A 16 x 16 block stored row-major is then
// both operands of the next update as it stands: A_iw -= R_pi^T R_pw takes row
// 4 s + kg of either block in MFMA step s. gfx950's FP64 MFMA is a chain of
// fused multiply-adds in the order of k, so every entry sees the updates of a
// step-by-step elimination, in its order.
//   Panel row p is factorised by one wave per 64 columns: lane j holds the 16
// entries of column j, and next to them a copy of the diagonal block's column
// j mod 16, so that the multipliers R[k][16 p + r] are broadcast over each row
// of 16 lanes by the multiply-add itself. The other waves meanwhile apply the
// previous panel to their blocks below the next panel row.
//   X: the diagonal blocks by forward substitution on rows (lane t: x[c] =
// (delta_tc - sum_{k<c} x[k] R[k][c]) / R[c][c]), then wave j goes up its block
// column, X_ij = -X_ii sum_{k=i+1..j} R_ik X_kj, the X_kj in registers as they
// come out of the matrix cores. Rows are padded to 17 entries, so that the
// transposed operand reads of that product meet no bank twice.
//   Bound by the serial chain of one workgroup (instruction issue of one wave
// per SIMD in the panels). Measured at lp = 32 / 64 / 96 / 128, a whole launch
// with the reduction of one partial: 10.4 / 18.9 / 30.8 / 44 us, against 15.4 /
// 28.2 / 55.5 / 76 us for the factorisation alone in a kernel of its own (rows
// of 16 in the registers of a wave, multipliers by readlane and LDS broadcast);
// the same bits.
// Padding rows and columns of R become identity, so X has identity padding.
// ---------------------------------------------------------------------------
constexpr int CHOL_LD = 17, CHOL_BLK = 16 * CHOL_LD;
__device__ __forceinline__ int blk(int ib, int jb) { return (jb * (jb + 1) / 2 + ib) * CHOL_BLK; }  // ib <= jb

// v of lane K of each row of 16 lanes
template <int K> __device__ __forceinline__ double row_bcast(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)b, 0x150 + K, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), 0x150 + K, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// a[r] -= x(lane r of the row) m, b[r] -= x(lane r of the row) n for R <= r < R + N (a DPP operand needs two
// wait states after a VALU write: inside)
template <int R, int N> __device__ __forceinline__ void fms_bcast(double* a, double* b, double x, double m, double n) {
#define RPOD_FMS(A, M, K) "v_fmac_f64_dpp " A ", -%[x], " M " row_newbcast:" K " row_mask:0xf bank_mask:0xf\n"
    if constexpr (N >= 4) {
        asm volatile("s_nop 1\n" RPOD_FMS("%0", "%[m]", "%[k0]") RPOD_FMS("%4", "%[n]", "%[k0]")
                     RPOD_FMS("%1", "%[m]", "%[k1]") RPOD_FMS("%5", "%[n]", "%[k1]")
                     RPOD_FMS("%2", "%[m]", "%[k2]") RPOD_FMS("%6", "%[n]", "%[k2]")
                     RPOD_FMS("%3", "%[m]", "%[k3]") RPOD_FMS("%7", "%[n]", "%[k3]")
                     : "+v"(a[R]), "+v"(a[R + 1]), "+v"(a[R + 2]), "+v"(a[R + 3]), "+v"(b[R]), "+v"(b[R + 1]),
                       "+v"(b[R + 2]), "+v"(b[R + 3])
                     : [x] "v"(x), [m] "v"(m), [n] "v"(n), [k0] "n"(R), [k1] "n"(R + 1), [k2] "n"(R + 2),
                       [k3] "n"(R + 3));
        fms_bcast<R + 4, N - 4>(a, b, x, m, n);
    } else if constexpr (N > 0) {
        asm volatile("s_nop 1\n" RPOD_FMS("%0", "%[m]", "%[k0]") RPOD_FMS("%1", "%[n]", "%[k0]")
                     : "+v"(a[R]), "+v"(b[R])
                     : [x] "v"(x), [m] "v"(m), [n] "v"(n), [k0] "n"(R));
        fms_bcast<R + 1, N - 1>(a, b, x, m, n);
    }
#undef RPOD_FMS
}
// s[c] -= r[c](lane K of the row) x for C <= c < C + N
template <int K, int C, int N> __device__ __forceinline__ void fms_from(double* s, const double* r, double x) {
#define RPOD_FMS(A, B) "v_fmac_f64_dpp " A ", -" B ", %[x] row_newbcast:%[k] row_mask:0xf bank_mask:0xf\n"
    if constexpr (N >= 4) {
        asm volatile("s_nop 1\n" RPOD_FMS("%0", "%[r0]") RPOD_FMS("%1", "%[r1]") RPOD_FMS("%2", "%[r2]")
                     RPOD_FMS("%3", "%[r3]")
                     : "+v"(s[C]), "+v"(s[C + 1]), "+v"(s[C + 2]), "+v"(s[C + 3])
                     : [x] "v"(x), [r0] "v"(r[C]), [r1] "v"(r[C + 1]), [r2] "v"(r[C + 2]), [r3] "v"(r[C + 3]), [k] "n"(K));
        fms_from<K, C + 4, N - 4>(s, r, x);
    } else if constexpr (N > 0) {
        asm volatile("s_nop 1\n" RPOD_FMS("%0", "%[r0]") : "+v"(s[C]) : [x] "v"(x), [r0] "v"(r[C]), [k] "n"(K));
        fms_from<K, C + 1, N - 1>(s, r, x);
    }
#undef RPOD_FMS
}
template <int I, int N, typename F> __device__ __forceinline__ void unroll(F f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unroll<I + 1, N>(f);
    }
}

struct CholShared {
    double* R;   // upper blocks of R, then R^-1's diagonal blocks in X
    double* X;
    double* gd;  // diagonal of G
    int* fail;
};

template <int NB>
__device__ __forceinline__ void chol_body(const GramArgs& a, const CholShared& sh) {
    constexpr int LP = 16 * NB, PW = (NB + 3) / 4;  // PW: panel waves
    double *Rs = sh.R, *Xs = sh.X, *gd = sh.gd;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // branches on it are scalar: no masks to keep
    const int n = lane & 15, kg = lane >> 4;  // MFMA lane; kg is also the lane's row of 16 lanes
    const CholArgs& c = a.chol;
    const int l = c.l, mode = c.mode;
    int* local = c.flags + 1;
    const GLOBAL double* G = gbl(a.G);
    if (mode == 2 && !(*local & DEV_FLAG_SHIFTED)) return;  // uniform
    if (mode == 0 && tid == 0) *local = 0;

    f64x4 w[NB];  // A[16 i + kg + 4 v][16 wave + n], then X
    bool fin = true;
    auto load = [&](bool first, double shift) {
        // formed anew by the second call: kept from the first, its masks and addresses spill
        int ln = n, ll = l;
        asm volatile("" : "+v"(ln), "+s"(ll));
#pragma unroll
        for (int i = 0; i < NB; ++i)
            if (wave < NB && i <= wave) {
#pragma unroll
                for (int v = 0; v < 4; ++v) w[i][v] = G[(16 * i + kg + 4 * v) * LP + 16 * wave + ln];
            }
#pragma unroll
        for (int i = 0; i < NB; ++i)
            if (wave < NB && i <= wave) {
#pragma unroll
                for (int v = 0; v < 4; ++v) fin = fin && isfinite(w[i][v]);
                if (i == wave) {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (kg + 4 * v == ln) {
                            if (first) gd[16 * wave + ln] = w[i][v];
                            w[i][v] += shift;
                        }
                }
                if (16 * wave + 16 > ll) {  // padding (i <= wave: its rows are in the same block column)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int row = 16 * i + kg + 4 * v, col = 16 * wave + ln;
                        if (row >= ll || col >= ll) w[i][v] = row == col ? 1.0 : 0.0;
                    }
                }
            }
    };
    load(true, 0.0);
    bool ok = __syncthreads_and(fin) != 0;
    if (!ok && tid == 0) atomicOr(c.flags, DEV_FLAG_NONFINITE);
    if (ok) {
#pragma unroll 1
        for (int attempt = 0; attempt < 2; ++attempt) {
            if (attempt == 1) {
                double tr = 0.0;
                for (int k = 0; k < l; ++k) tr += gd[k];
                load(false, 11.0 * ((double)a.M * l + (double)l * (l + 1)) * 0x1.0p-53 * tr);
            }
            if (tid == 0) *sh.fail = 0;
            // a panel row to be factorised: its diagonal block apart (both panel waves read it), the
            // others where R goes
            auto put = [&](int i, const f64x4& x) {
                double* d = (i == wave ? Xs + i * CHOL_BLK : Rs + blk(i, wave)) + kg * CHOL_LD + n;
#pragma unroll
                for (int v = 0; v < 4; ++v) d[4 * v * CHOL_LD] = x[v];
            };
            // w[i] -= R_pi^T R_p,wave
            auto update = [&](int i, int p, const double (&rb)[4], f64x4& x) {
                const double* ra = Rs + blk(p, i) + kg * CHOL_LD + n;
#pragma unroll
                for (int s = 0; s < 4; ++s) x = mfma_16x16x4(-ra[4 * s * CHOL_LD], rb[s], x);
            };
            auto row_of = [&](int p, double (&rb)[4]) {
                const double* r = Rs + blk(p, wave) + kg * CHOL_LD + n;
#pragma unroll
                for (int s = 0; s < 4; ++s) rb[s] = r[4 * s * CHOL_LD];
            };
            if (wave < NB) put(0, w[0]);
            __syncthreads();
#pragma unroll 1
            for (int p = 0; p < NB; ++p) {
                if (wave < PW && 4 * wave + 3 >= p) {
                    const int cb = 4 * wave + kg;  // this row of lanes' block column
                    const bool live = cb >= p && cb < NB;
                    const double* dsrc = Xs + p * CHOL_BLK + n;
                    double* xdst = Rs + blk(p, live ? cb : p) + n;
                    const double* xsrc = cb > p && live ? xdst : dsrc;
                    double d[16], x[16];
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        d[r] = dsrc[r * CHOL_LD];
                        x[r] = xsrc[r * CHOL_LD];
                    }
                    double piv = 0.0;  // lane n of a row: pivot 16 p + n
                    unroll<0, 16>([&](auto KK) {
                        constexpr int kk = KK;
                        piv = n == kk ? d[kk] : piv;
                        const double rinv = rsqrt_nr(row_bcast<kk>(d[kk]));
                        d[kk] *= rinv;  // R[k][:] (left of column k: of no use, never read)
                        x[kk] *= rinv;
                        fms_bcast<kk + 1, 15 - kk>(d, x, d[kk], d[kk], x[kk]);
                    });
                    // a non-positive, tiny or NaN pivot (the rows after it are thrown away)
                    const bool bad = !(piv > (double)l * 0x1.0p-52 * gd[16 * p + n]) || !(piv > 0.0);
                    if (bad) *sh.fail = 1;
                    if (live) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) xdst[r * CHOL_LD] = x[r];
                    }
                }
                double rb[4];
                if (p > 0 && wave > p && wave < NB) {  // panel p - 1 on the blocks below panel row p
                    row_of(p - 1, rb);
#pragma unroll
                    for (int i = 2; i < NB; ++i)
                        if (i > p && i <= wave) update(i, p - 1, rb, w[i]);
                }
                __syncthreads();  // panel row p final
                if (wave > p && wave < NB) {
                    row_of(p, rb);
#pragma unroll
                    for (int i = 1; i < NB; ++i)
                        if (i == p + 1) {
                            update(i, p, rb, w[i]);
                            put(i, w[i]);
                        }
                }
                __syncthreads();  // panel row p + 1 staged
            }
            const bool fail = *sh.fail != 0;
            __syncthreads();  // every thread has read it
            if (!fail) break;
            if (attempt == 0) {
                if (tid == 0) {
                    atomicOr(c.flags, DEV_FLAG_SHIFTED);
                    *local |= DEV_FLAG_SHIFTED;
                }
            } else {
                if (tid == 0) atomicOr(c.flags, DEV_FLAG_BREAKDOWN);
                ok = false;
            }
        }
    }
    GLOBAL double* R64 = gbl(c.R64);
    GLOBAL float* R32 = gbl(c.R32);
    if (ok) {
        if (wave < PW) {  // diagonal blocks 4 wave + kg, lane n = row n
            const int b = min(4 * wave + kg, NB - 1);
            const double* Rd = Rs + blk(b, b) + n * CHOL_LD;
            double rd[16], s0[16], s1[16];  // rd[c]: R[n][c]; even and odd k of x[c]'s sum, then x[c] in s0
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                rd[c] = Rd[c];
                s0[c] = c == n ? 1.0 : 0.0;
                s1[c] = 0.0;
            }
            const double rc = rcp_nr(Rd[n]);
            unroll<0, 16>([&](auto KK) {
                constexpr int k = KK;
                s0[k] = (s0[k] + s1[k]) * row_bcast<k>(rc);
                fms_from<k, k + 1, 15 - k>(k & 1 ? s1 : s0, rd, s0[k]);
            });
            double* Xd = Xs + b * CHOL_BLK + n * CHOL_LD;
#pragma unroll
            for (int c = 0; c < 16; ++c) Xd[c] = s0[c];  // zero below the diagonal
        }
        __syncthreads();
        if (wave < NB) {
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (i == wave) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) w[i][v] = Xs[i * CHOL_BLK + (kg + 4 * v) * CHOL_LD + n];
                }
#pragma unroll
            for (int ib = NB - 2; ib >= 0; --ib)
                if (ib < wave) {
                    f64x4 t = {0.0, 0.0, 0.0, 0.0}, x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int kb = ib + 1; kb < NB; ++kb)
                        if (kb <= wave) {
                            const double* ra = Rs + blk(ib, kb) + n * CHOL_LD + kg;
#pragma unroll
                            for (int s = 0; s < 4; ++s) t = mfma_16x16x4(ra[4 * s], w[kb][s], t);
                        }
                    const double* xa = Xs + ib * CHOL_BLK + n * CHOL_LD + kg;
#pragma unroll
                    for (int s = 0; s < 4; ++s) x = mfma_16x16x4(-xa[4 * s], t[s], x);
                    w[ib] = x;
                }
            // column-major
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const double x = i <= wave ? w[i][v] : 0.0;
                    const int e = (16 * wave + n) * LP + 16 * i + kg + 4 * v;
                    R64[e] = x;
                    R32[e] = (float)x;
                }
        }
    } else {
        for (int e = tid; e < LP * LP; e += blockDim.x) {
            const double v = (e % LP == e / LP) ? 1.0 : 0.0;
            R64[e] = v;
            R32[e] = (float)v;
        }
    }
}

// Reduction of the partial Gram matrices; with chol.R64 set, the workgroup that ends last goes on to the
// Cholesky factor and its inverse (a launch and its gap less than a kernel of its own).
// TPB / 8 entries per workgroup, eight threads per entry: thread t sums the partials w = t, t + 8, ..
// (independent loads in flight), and the eight sums are combined in a fixed order.
constexpr int reduce_threads(int nt) { return nt <= 4 ? 256 : 512; }  // a wave per block column at least

template <int NT>
__global__ __launch_bounds__(reduce_threads(NT)) void k_gram_reduce(Group<GramArgs> g) {
    if (group_skipped(g)) return;
    constexpr int TPB = reduce_threads(NT), EPB = TPB / 8, NP = npairs_of(NT), LP = 16 * NT;
    static_assert(NP * 256 % EPB == 0, "whole tiles");
    __shared__ double part[8][EPB];
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const GramArgs& ga = g.args[it];
    if (ga.cond != nullptr && !(*ga.cond & ga.cond_mask)) return;
    const int el = threadIdx.x % EPB, t = threadIdx.x / EPB;
    const int e = (blockIdx.x - g.tstart[it]) * EPB + el;
    const GLOBAL double* src = gbl(ga.Gpart) + e;  // entry e = pair e / 256, element e mod 256
    constexpr int64_t wstride = (int64_t)NP * 256;
    const int nwg = ga.nwg;
    double a4[4] = {0, 0, 0, 0};
    int w = t;
    for (; w + 24 < nwg; w += 32)
#pragma unroll
        for (int u = 0; u < 4; ++u) a4[u] += src[(int64_t)(w + 8 * u) * wstride];
    for (; w < nwg; w += 8) a4[0] += src[(int64_t)w * wstride];
    part[t][el] = (a4[0] + a4[1]) + (a4[2] + a4[3]);
    __syncthreads();
    if (t == 0) {
        const double s = ((part[0][el] + part[1][el]) + (part[2][el] + part[3][el])) +
                         ((part[4][el] + part[5][el]) + (part[6][el] + part[7][el]));
        const int p = e / 256, mm = (e % 256) / 16, nn = e % 16;
        int a = 0, q = p;
        while (q >= NT - a) { q -= NT - a; ++a; }
        const int b = a + q;
        // agent scope: written through this XCD's L2 (a fence that writes the whole L2 back from every
        // workgroup cost 25 us of 30 at lp = 128)
        GLOBAL double* G = gbl(ga.G);
        __hip_atomic_store(G + (16 * a + mm) * LP + 16 * b + nn, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(G + (16 * b + nn) * LP + 16 * a + mm, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the entries are out ...
    }
    if (ga.chol.R64 == nullptr) return;  // uniform
    __shared__ __attribute__((aligned(16))) double Rs[NP * CHOL_BLK];
    __shared__ __attribute__((aligned(16))) double Xs[NT * CHOL_BLK];
    __shared__ double gd[LP];
    __shared__ int s_fail, s_last;
    __syncthreads();
    if (threadIdx.x == 0) {
        int* arrived = ga.chol.flags + FLAG_ARRIVED;
        const int tiles = g.tstart[it + 1] - g.tstart[it];
        // ... before the workgroup is counted
        s_last = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == tiles - 1;
        if (s_last) *arrived = 0;
    }
    __syncthreads();
    if (!s_last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // the other workgroups' entries, not older copies
    chol_body<NT>(ga, CholShared{Rs, Xs, gd, &s_fail});
}

// Partial workgroups per pair group: one per 4 row blocks, at most `cap`;
// by default (cap 0) 256 for a single pair group (measured: more partials
// cost more in the reduction than they save) and about 512 workgroups over
// several pair groups (two waves per SIMD), rounded down to a multiple of 8.
int gram_nwg(int64_t M, int cap, int nt) {
    const int64_t nrb = (M + 15) / 16;
    int64_t nwg = (nrb + 3) / 4;
    if (cap < 1 || cap > GRAM_WGS) cap = gram_groups(nt) == 1 ? 256 : (GRAM_WGS / gram_groups(nt)) & ~7;
    if (nwg > cap) nwg = cap;
    if (nwg < 1) nwg = 1;
    return (int)nwg;
}

int gram_tiles(int nt, int nwg) { return nwg * gram_groups(nt); }
int gram_reduce_tiles(int nt) { return npairs_of(nt) * 256 / (reduce_threads(nt) / 8); }

template <typename Tin, int NT>
static hipError_t gram_nt(const GroupLaunch<GramArgs>& L, const GroupLaunch<GramArgs>& R, hipStream_t st) {
    hipLaunchKernelGGL((k_gram<Tin, NT>), dim3(L.tiles), dim3(256), 0, st, mkg(L));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gram_reduce<NT>, dim3(R.tiles), dim3(reduce_threads(NT)), 0, st, mkg(R));
    return hipGetLastError();
}

template <typename Tin>
static hipError_t gram_dispatch(int nt, const GroupLaunch<GramArgs>& L, const GroupLaunch<GramArgs>& R,
                                hipStream_t st) {
    switch (nt) {
#define RPOD_GRAM_CASE(K) case K: return gram_nt<Tin, K>(L, R, st);
        RPOD_GRAM_CASE(1) RPOD_GRAM_CASE(2) RPOD_GRAM_CASE(3) RPOD_GRAM_CASE(4)
        RPOD_GRAM_CASE(5) RPOD_GRAM_CASE(6) RPOD_GRAM_CASE(7) RPOD_GRAM_CASE(8)
#undef RPOD_GRAM_CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gram(int tin, int nt, const GroupLaunch<GramArgs>& L, const GroupLaunch<GramArgs>& R,
                       hipStream_t st) {
    if (tin == DT_F64) return gram_dispatch<double>(nt, L, R, st);
    if (tin == DT_F32) return gram_dispatch<float>(nt, L, R, st);
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Small SVD of step 6 (eigenvectors of G_B = T T^T), one workgroup per matrix.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double shfl_xor_d(double v, int mask) {
    return __shfl_xor(v, mask, 64);
}

// Value of another lane of the row of 16 by a DPP move (both halves); every lane has a source, so
// nothing is kept of the destination (bound_ctrl).
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
constexpr int DPP_XOR1 = 0xB1 /* quad_perm 1,0,3,2 */, DPP_XOR2 = 0x4E /* quad_perm 2,3,0,1 */,
              DPP_XOR7 = 0x141 /* row_half_mirror */, DPP_XOR15 = 0x140 /* row_mirror */,
              DPP_XOR8 = 0x128 /* row_ror:8 */;

// x of lanes l and l ^ 16 (permlane16_swap) or l ^ 32 (permlane32_swap), in the same order in both:
// a swap of a register with its copy leaves the even rows' (lower half's) values in both places of
// the first result and the odd rows' (upper half's) in both places of the second.
template <int BIT>
__device__ __forceinline__ void both_of(unsigned v, unsigned& even, unsigned& odd) {
    const auto r = BIT == 16 ? __builtin_amdgcn_permlane16_swap(v, v, false, false)
                             : __builtin_amdgcn_permlane32_swap(v, v, false, false);
    even = r[0];
    odd = r[1];
}
template <int BIT>
__device__ __forceinline__ double pair_sum(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    unsigned l0, l1, h0, h1;
    both_of<BIT>((unsigned)b, l0, l1);
    both_of<BIT>((unsigned)(b >> 32), h0, h1);
    return __builtin_bit_cast(double, ((unsigned long long)h0 << 32) | l0) +
           __builtin_bit_cast(double, ((unsigned long long)h1 << 32) | l1);
}
// Sum over the eight lanes that share l mod 8, the same bits in all of them (commuting operands).
__device__ __forceinline__ double sum_sub(double x) {
    x += dpp_d<DPP_XOR8>(x);
    return pair_sum<32>(pair_sum<16>(x));
}
// Maximum over the wave of non-NaN values, in every lane.
__device__ __forceinline__ double wave_max(double x) {
    x = fmax(x, dpp_d<DPP_XOR1>(x));
    x = fmax(x, dpp_d<DPP_XOR2>(x));
    x = fmax(x, dpp_d<DPP_XOR7>(x));
    x = fmax(x, dpp_d<DPP_XOR15>(x));
    return fmax(fmax(read_lane(x, 0), read_lane(x, 16)), fmax(read_lane(x, 32), read_lane(x, 48)));
}
__device__ __forceinline__ int wave_max(int x) {
    x = max(x, dpp_i<DPP_XOR1>(x));
    x = max(x, dpp_i<DPP_XOR2>(x));
    x = max(x, dpp_i<DPP_XOR7>(x));
    x = max(x, dpp_i<DPP_XOR15>(x));
    unsigned a, b;
    both_of<16>((unsigned)x, a, b);
    x = max((int)a, (int)b);
    both_of<32>((unsigned)x, a, b);
    return max((int)a, (int)b);
}

// a[k] += x(lane 16 (l / 16) + k) m for k < 16: the multipliers of a row of 16 lanes, each broadcast
// over its row by the multiply-add itself (no LDS broadcast reads, no register moves). The wait
// states a DPP operand needs after a VALU write are inside.
__device__ __forceinline__ void fma16_bcast(double (&a)[16], double x, double m) {
    asm volatile(
        "s_nop 1\n"
        "v_fmac_f64_dpp %0, %8, %9 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %1, %8, %9 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %2, %8, %9 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %3, %8, %9 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %4, %8, %9 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %5, %8, %9 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %6, %8, %9 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %7, %8, %9 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7])
        : "v"(x), "v"(m));
    asm volatile(
        "s_nop 1\n"
        "v_fmac_f64_dpp %0, %8, %9 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %1, %8, %9 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %2, %8, %9 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %3, %8, %9 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %4, %8, %9 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %5, %8, %9 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %6, %8, %9 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %7, %8, %9 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
        : "+v"(a[8]), "+v"(a[9]), "+v"(a[10]), "+v"(a[11]), "+v"(a[12]), "+v"(a[13]), "+v"(a[14]), "+v"(a[15])
        : "v"(x), "v"(m));
}

// sqrt(x) for x > 0 and 1 / x: the hardware estimates with one step that cubes their error
__device__ __forceinline__ double sqrt_3(double x) {
    const double y = __builtin_amdgcn_rsq(x), z = x * y, e = fma(-z, y, 1.0);
    return fma(z * e, fma(e, 0.375, 0.5), z);
}
__device__ __forceinline__ double rcp_3(double x) {
    const double y = __builtin_amdgcn_rcp(x), e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// One rotation per group of eight lanes that makes the columns own and part (RPL rows per lane)
// orthogonal: own' = c own - s part, part' = s own + c part; no, np are their squared norms. The
// rotation is orthogonal to rounding whatever the half-angle tangent u: s = 2 u / (1 + u^2) and
// c = 1 - u s follow from it to FP64 (through a rounded c sigma's error is twice as large). FINE: u and the tangent t of the norms' update to FP64; else from the hardware's estimates,
// which leaves 2^-23 of the inner product over. That is 1e-15 where pairs count as orthogonal from
// 1e-8 on, and the modes' errors are the same to four digits (lp = 16 .. 128, 0.5 to 4e-8 rms) for
// sweeps 4 to 6 % shorter; at a threshold of FP64 rounding it shows (modes of a 16 x 16 factor 1.27e-15
// rms from the exact ones instead of 1.00e-15).
// SYM: the two groups of a pair within a block compute the same rotation, each as "own"; every
// expression is then symmetric (or antisymmetric) in the exchange bit for bit, `low` deciding where
// the norms are equal. Otherwise the update is three shears in place, (1 -u; 0 1) (1 0; s 1) (1 -u; 0 1).
template <int RPL, bool SYM, bool FINE>
__device__ __forceinline__ bool jacobi_rotate(double (&own)[RPL], double (&part)[RPL], double& no, double& np,
                                              double tol2, bool low) {
    double g0 = 0.0, g1 = 0.0;
#pragma unroll
    for (int k = 0; k < RPL; k += 2) {
        g0 = fma(own[k], part[k], g0);
        g1 = fma(own[k + 1], part[k + 1], g1);
    }
    const double ga = sum_sub(g0 + g1);
    const bool rot = ga * ga > tol2 * (no * np);  // |ga| > tol sqrt(no np); false when a column is zero
    if (__ballot(rot) == 0) return false;
    // tan(theta) = y / p, tan(theta / 2) = y / (p + sqrt(2 r p)), with y = |2 ga|, r = sqrt(d^2 + y^2),
    // p = r + |d|, d = np - no; theta has the sign of d ga
    double d = np - no;
    const double e2 = ga + ga;
    if (SYM && d == 0.0) d = low ? 0.0 : -0.0;
    const double h2 = fma(d, d, e2 * e2);
    const double r = FINE ? sqrt_3(h2) : h2 * __builtin_amdgcn_rsq(h2);
    const double p = r + fabs(d);
    const double w = (0.5 * r) * p;  // <= h2: no overflow of its own
    const double q = fma(2.0, FINE ? sqrt_3(w) : w * __builtin_amdgcn_rsq(w), p);
    double u = fabs(e2) * (FINE ? rcp_3(q) : __builtin_amdgcn_rcp(q));
    double t = fabs(e2) * (FINE ? rcp_3(p) : __builtin_amdgcn_rcp(p));
    const double sgn = __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, d) ^
                                                      __builtin_bit_cast(unsigned long long, e2));
    u = rot ? __builtin_copysign(u, sgn) : 0.0;
    t = rot ? __builtin_copysign(t, sgn) : 0.0;
    const double y = rcp_3(fma(u, u, 1.0)), s = (u + u) * y;
    if constexpr (SYM) {
#pragma unroll
        for (int k = 0; k < RPL; ++k) {  // own - s (part + u own), part + s (own - u part): one rounding at full size
            const double a = own[k], b = part[k];
            own[k] = fma(-s, fma(u, a, b), a);
            part[k] = fma(s, fma(-u, b, a), b);
        }
    } else {
#pragma unroll
        for (int k = 0; k < RPL; ++k) own[k] = fma(-u, part[k], own[k]);
#pragma unroll
        for (int k = 0; k < RPL; ++k) part[k] = fma(s, own[k], part[k]);
#pragma unroll
        for (int k = 0; k < RPL; ++k) own[k] = fma(-u, part[k], own[k]);
    }
    no = fma(-t, ga, no);
    np = fma(t, ga, np);
    return rot;
}

// Preconditioned one-sided Jacobi (Drmac and Veselic, SIMAX 2008): with the
// diagonally pivoted Cholesky factorisation G = P L L^T P^T, the left
// singular vectors of P L are the eigenvectors of G and its singular values
// the square roots of G's eigenvalues. One-sided Jacobi on the columns of
// P L (a row permutation does not change the column inner products) then
// needs few sweeps. Results: UB[:, k] = (P L V)[:, k] / sigma_k by
// descending sigma_k = ||(P L V)[:, k]||; factorisation stops at the first
// pivot below lp u times the largest diagonal entry of G (the remaining
// columns are zero, as are their sigma and UB columns).
// Factorisation: lane i of wave w keeps rows i, i + 64 and columns 16 w .. 16 w + 15 of the
// Schur complement (original order) in registers. Every wave carries the diagonal and finds the
// pivot by itself (the largest remaining entry, lowest index on ties, compared by the halves of its
// bits; the next pivot is found while the update runs), the lane holding the pivot row publishes
// its part, and one barrier later every wave reads the row as the multipliers (the matrix is
// symmetric): one barrier per step, no data moved, and the reciprocal root is taken before it.
// Sweeps: the columns form blocks of eight. A wave holds two blocks in registers, one column of
// each per group of eight lanes (group = lane mod 8, rows 16 kc + 2 (lane / 8), + 1), so the 8 x 8
// pairs between them, and the pairs within each once per sweep, need no LDS and no barrier: from
// one round to the next the second block's columns move between the groups by one DPP lane
// exchange. Blocks meet by the circle method: lp / 8 - 1 exchanges through LDS, one barrier each,
// per sweep of lp - 1 rounds. A round is bound by the issue of one wave's instructions (about 8
// cycles each with one wave per SIMD, 6 with two): 760 cycles at lp = 64, 1650 at lp = 128, where
// a round through LDS with its own barrier took 1500 and 3300. Per launch, spectra decaying by
// e^-6 over l, Gram route: lp = 32, 64, 96, 128 64, 179, 462, 791 us, against 104, 341, 886, 1577 us
// for rounds through LDS; the factorisation is 28 us of it at lp = 64 and 95 us at lp = 128. The
// errors of a factor's modes against the exact ones are no larger than there (lp = 16, 32, 64, 128:
// 1.00, 3.2, 11, 40e-15 rms, there 1.08, 3.5, 13, 45e-15). Sixteen lanes per pair, and so two
// waves per SIMD at lp = 64, would issue 1.6 x the instructions for 1.3 x the issue rate.
// LDS holds the blocks as register images: chunk kc of block b at ((b KC + kc) 64 + lane) 16 bytes,
// so every access is 1 KB contiguous.
// Squared norms are recomputed at every load and updated over the eight rounds after it; a sweep
// without rotations therefore tests every pair with norms just computed.
// Factor route (C non-NULL): the columns of C (C C^T = T T^T, from an
// orthonormal basis of T^T rather than from the Gram matrix) are loaded as
// they are, with no permutation, and the sweeps start at once.
template <int LP>
__device__ __forceinline__ void jacobi_chol_body(const double* __restrict__ G, int l, double* __restrict__ UB,
                                                 double* __restrict__ sig, int* flags, double tol,
                                                 const double* __restrict__ C, int64_t ldc) {
    constexpr int NW = LP / 16, NTHR = 64 * NW, NB = 2 * NW, KC = LP / 16, RPL = 2 * KC, CPL = (LP + 63) / 64;
    typedef double d2 __attribute__((ext_vector_type(2)));
    __shared__ __attribute__((aligned(16))) double W[LP * LP];         // register images of the blocks
    __shared__ __attribute__((aligned(16))) double buf[2][64 * CPL];   // pivot rows, alternating
    __shared__ double nrm[LP];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // place of row `row` of column `col` in W
    auto at = [](int row, int col) {
        return (((col >> 3) * KC + (row >> 4)) * 64 + ((row & 15) >> 1) * 8 + (col & 7)) * 2 + (row & 1);
    };
    if (C != nullptr) {
        const GLOBAL double* Cg = gbl(C);
        for (int e = tid; e < LP * LP; e += NTHR) {
            const int c = e / LP, row = e % LP;
            W[at(row, c)] = (c < l && row < l) ? Cg[(int64_t)c * ldc + row] : 0.0;
        }
    } else {
        const GLOBAL double* Gg = gbl(G);
        for (int e = tid; e < LP * LP; e += NTHR) W[e] = 0.0;
        double a[CPL][16], dg[CPL];
        bool done[CPL];
#pragma unroll
        for (int cc = 0; cc < CPL; ++cc) {
            const int row = lane + 64 * cc;
            const bool live = row < l;
            const int rc = row < LP ? row : 0;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                a[cc][k] = Gg[(16 * wave + k) * LP + rc];
            }
            dg[cc] = Gg[rc * LP + rc];
            done[cc] = !live;
        }
        // rows and columns past l (read all the same, so that the loads are in flight together) count as zero
#pragma unroll
        for (int cc = 0; cc < CPL; ++cc) {
            const bool live = lane + 64 * cc < l;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                asm volatile("" : "+v"(a[cc][k]));
                a[cc][k] = (live && 16 * wave + k < l) ? a[cc][k] : 0.0;
            }
            asm volatile("" : "+v"(dg[cc]));
            dg[cc] = live ? dg[cc] : 0.0;
        }
        // the largest diagonal entry scales the threshold
        double dm = dg[0];
        if constexpr (CPL > 1) dm = fmax(dm, dg[CPL - 1]);
        const double thr = (double)LP * 0x1.0p-53 * wave_max(dm);
        // the next pivot: row and value, and whether one is left that is not negligible (or not finite).
        // Positive doubles are in the order of their bits: the upper halves decide, the lower ones
        // between equals (a negative or NaN remainder and a finished row lose against any).
        auto find = [&](int& pv, double& app) {
            int v[CPL], vm = -1;
#pragma unroll
            for (int cc = 0; cc < CPL; ++cc) {
                v[cc] = !done[cc] && dg[cc] > 0.0 ? (int)(__builtin_bit_cast(unsigned long long, dg[cc]) >> 32) : -1;
                vm = max(vm, v[cc]);
            }
            const int vmax = wave_max(vm);
            unsigned long long m[CPL];
            int count = 0;
#pragma unroll
            for (int cc = 0; cc < CPL; ++cc) {
                m[cc] = __ballot(v[cc] == vmax);
                count += __popcll(m[cc]);
            }
            if (count > 1) {  // uniform
                int w[CPL], wm = INT32_MIN;
#pragma unroll
                for (int cc = 0; cc < CPL; ++cc) {
                    const int lo = (int)((unsigned)__builtin_bit_cast(unsigned long long, dg[cc]) ^ 0x80000000u);
                    w[cc] = v[cc] == vmax ? lo : INT32_MIN;
                    wm = max(wm, w[cc]);
                }
                const int wmax = wave_max(wm);
#pragma unroll
                for (int cc = 0; cc < CPL; ++cc) m[cc] &= __ballot(w[cc] == wmax);
            }
            pv = 0;
#pragma unroll
            for (int cc = CPL - 1; cc >= 0; --cc)
                if (m[cc] != 0) pv = 64 * cc + __ffsll(m[cc]) - 1;
            app = CPL > 1 && pv >= 64 ? read_lane(dg[CPL - 1], pv & 63) : read_lane(dg[0], pv & 63);
            return __builtin_amdgcn_readfirstlane(vmax) >= 0 && app > thr;
        };
        int rank = l, pv;
        double app;
        bool more = find(pv, app);
        __syncthreads();
        for (int j = 0; j < l; ++j) {
            if (!more) {  // the same in every wave
                rank = j;
                break;
            }
            double* pr = buf[j & 1];
#pragma unroll
            for (int cc = 0; cc < CPL; ++cc)
                if (lane + 64 * cc == pv) {
#pragma unroll
                    for (int k = 0; k < 16; k += 2)
                        *reinterpret_cast<d2*>(pr + 16 * wave + k) = d2{a[cc][k], a[cc][k + 1]};
                }
            const double inv = rsqrt_nr(app), ljj = app * inv;
            __syncthreads();
            double lij[CPL], m[CPL];
#pragma unroll
            for (int cc = 0; cc < CPL; ++cc) lij[cc] = pr[lane + 64 * cc];  // rows >= LP: never used
            const double rk = pr[16 * wave + (lane & 15)];
#pragma unroll
            for (int cc = 0; cc < CPL; ++cc) {
                const int row = lane + 64 * cc;
                lij[cc] = done[cc] ? 0.0 : lij[cc] * inv;
                if (row == pv) {
                    done[cc] = true;
                    lij[cc] = ljj;
                }
                if (row < LP && wave == j % NW) W[at(row, j)] = lij[cc];
                dg[cc] = fma(-lij[cc], lij[cc], dg[cc]);
                m[cc] = -lij[cc] * inv;
            }
            more = find(pv, app);
#pragma unroll
            for (int cc = 0; cc < CPL; ++cc) fma16_bcast(a[cc], rk, m[cc]);
        }
        if (tid == 0 && rank < l) atomicOr(flags, DEV_FLAG_RANK_CUT);
    }
    // ---- one-sided Jacobi on the columns ----
    const int grp = lane & 7, sub = lane >> 3;
    const double tol2 = tol * tol;
    double A[RPL], B[RPL];
    auto load = [&](double (&x)[RPL], int b) {
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
            const d2 v = *reinterpret_cast<const d2*>(W + ((b * KC + kc) * 64 + lane) * 2);
            x[2 * kc] = v[0];
            x[2 * kc + 1] = v[1];
        }
    };
    auto store = [&](const double (&x)[RPL], int b, int ln) {
#pragma unroll
        for (int kc = 0; kc < KC; ++kc)
            *reinterpret_cast<d2*>(W + ((b * KC + kc) * 64 + ln) * 2) = d2{x[2 * kc], x[2 * kc + 1]};
    };
    auto norm2 = [&](const double (&x)[RPL]) {
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int k = 0; k < RPL; k += 2) {
            s0 = fma(x[k], x[k], s0);
            s1 = fma(x[k + 1], x[k + 1], s1);
        }
        return sum_sub(s0 + s1);
    };
    auto move = [&](auto ctrl, double (&x)[RPL], double& nx) {
        constexpr int CTRL = decltype(ctrl)::value;
#pragma unroll
        for (int k = 0; k < RPL; ++k) x[k] = dpp_d<CTRL>(x[k]);
        nx = dpp_d<CTRL>(nx);
    };
    // group offsets of the eight rounds: 0, then 1, 3, 2, 5, 4, 6, 7
    std::integral_constant<int, DPP_XOR1> x1;
    std::integral_constant<int, DPP_XOR2> x2;
    std::integral_constant<int, DPP_XOR7> x7;
    // the 28 pairs within a block: each pair computed by both of its groups
    auto within = [&](auto fine, double (&x)[RPL], double& nx) {
        double P[RPL], np = nx;
        bool rot = false;
#pragma unroll
        for (int k = 0; k < RPL; ++k) P[k] = x[k];
        auto step = [&](auto ctrl, int k) {
            move(ctrl, P, np);
            rot |= jacobi_rotate<RPL, true, decltype(fine)::value>(x, P, nx, np, tol2, grp < (grp ^ k));
        };
        step(x1, 1); step(x2, 3); step(x1, 2); step(x7, 5); step(x1, 4); step(x2, 6); step(x1, 7);
        return rot;
    };
    int sweep = 0;
    constexpr int max_sweeps = 40;
    auto sweeps = [&](auto fine) {
        for (; sweep < max_sweeps; ++sweep) {
            bool rot = false;  // this lane's pairs rotated during the sweep
            int any = 0;
            for (int t = 0; t < NB - 1; ++t) {
                int ba = t + wave, bb = t - wave;  // circle method: block NB - 1 stays, the others turn
                if (ba >= NB - 1) ba -= NB - 1;
                if (bb < 0) bb += NB - 1;
                if (wave == 0) ba = NB - 1;
                load(A, ba);
                load(B, bb);
                double na = norm2(A), nb = norm2(B);
                if (t == 0) {
                    rot |= within(fine, A, na);
                    rot |= within(fine, B, nb);
                }
                rot |= jacobi_rotate<RPL, false, decltype(fine)::value>(A, B, na, nb, tol2, true);
                auto step = [&](auto ctrl) {
                    move(ctrl, B, nb);
                    rot |= jacobi_rotate<RPL, false, decltype(fine)::value>(A, B, na, nb, tol2, true);
                };
                step(x1); step(x2); step(x1); step(x7); step(x1); step(x2); step(x1);
                store(A, ba, lane);
                store(B, bb, lane ^ 7);  // the last partner was the column of group grp ^ 7
                // a slot is written by its holder and, after the barrier, read and later written by the next
                // holder only
                if (t < NB - 2) __syncthreads();
                else any = __syncthreads_or(rot);
            }
            if (!any) break;
        }
    };
    __syncthreads();
    if (C != nullptr) sweeps(std::true_type{});
    else sweeps(std::false_type{});
    if (sweep == max_sweeps && tid == 0) atomicOr(flags, DEV_FLAG_JACOBI_SLOW);
    load(A, 2 * wave);
    load(B, 2 * wave + 1);
    const double va = sqrt(norm2(A)), vb = sqrt(norm2(B));
    const int ca = 16 * wave + grp, cb = ca + 8;
    if (sub == 0) {
        nrm[ca] = va;
        nrm[cb] = vb;
    }
    __syncthreads();
    int ra = 0, rb = 0;  // ranks by descending norm, lowest column first on ties
    for (int k = sub; k < LP; k += 8) {
        const double v = nrm[k];
        ra += (v > va) || (v == va && k < ca);
        rb += (v > vb) || (v == vb && k < cb);
    }
#pragma unroll
    for (int off = 8; off < 64; off <<= 1) {
        ra += __shfl_xor(ra, off, 64);
        rb += __shfl_xor(rb, off, 64);
    }
    if (sub == 0) {
        sig[ra] = va;
        sig[rb] = vb;
    }
    const double ia = va > 0.0 ? 1.0 / va : 0.0, ib = vb > 0.0 ? 1.0 / vb : 0.0;
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
        *reinterpret_cast<d2*>(UB + ra * LP + 16 * kc + 2 * sub) = d2{A[2 * kc] * ia, A[2 * kc + 1] * ia};
        *reinterpret_cast<d2*>(UB + rb * LP + 16 * kc + 2 * sub) = d2{B[2 * kc] * ib, B[2 * kc + 1] * ib};
    }
}

// lp / 16 waves per workgroup, two blocks of eight columns each
template <int LP>
__global__ __launch_bounds__(4 * LP) void k_jacobi(Group<JacobiArgs> g) {
    if (group_skipped(g)) return;
    const JacobiArgs& a = g.args[blockIdx.x];  // one workgroup per matrix
    jacobi_chol_body<LP>(a.G, a.l, a.UB, a.sig, a.flags, a.tol, a.C, a.ldc);
}

int jacobi_threads(int lp) { return 4 * lp; }

hipError_t launch_jacobi(int lp, const GroupLaunch<JacobiArgs>& L, hipStream_t st) {
    switch (lp) {
#define RPOD_JAC_CASE(K) \
    case K: hipLaunchKernelGGL(k_jacobi<K>, dim3(L.count), dim3(4 * K), 0, st, mkg(L)); break;
        RPOD_JAC_CASE(16) RPOD_JAC_CASE(32) RPOD_JAC_CASE(48) RPOD_JAC_CASE(64)
        RPOD_JAC_CASE(80) RPOD_JAC_CASE(96) RPOD_JAC_CASE(112) RPOD_JAC_CASE(128)
#undef RPOD_JAC_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// M = Rinv * UB[:, :r] and Ur = UB[:, :r], both lp x rp column-major (zero pad). Bound by load latency:
// sixteen terms' loads in flight (16.2 -> 6.8 us at lp = 64, 25.4 -> 10.1 at 128).
__global__ void k_lift_coef(Group<LiftArgs> g) {
    if (group_skipped(g)) return;
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const LiftArgs& la = g.args[it];
    const double* __restrict__ Rinv = la.Rinv;
    const double* __restrict__ UB = la.UB;
    double* __restrict__ M64 = la.M64;
    float* __restrict__ M32 = la.M32;
    double* __restrict__ Ur = la.Ur;
    const int lp = la.lp, r = la.r, rp = la.rp;
    const int e = (blockIdx.x - g.tstart[it]) * blockDim.x + threadIdx.x;
    if (e >= lp * rp) return;
    const int k = e % lp, c = e / lp;
    double s = 0.0, u = 0.0;
    if (c < r) {
#pragma unroll 16
        for (int j = 0; j < lp; ++j) s += Rinv[(int64_t)j * lp + k] * UB[(int64_t)c * lp + j];
        u = UB[(int64_t)c * lp + k];
    }
    M64[e] = s;
    M32[e] = (float)s;
    Ur[e] = u;
}

hipError_t launch_lift_coef(const GroupLaunch<LiftArgs>& L, hipStream_t st) {
    hipLaunchKernelGGL(k_lift_coef, dim3(L.tiles), dim3(256), 0, st, mkg(L));
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Sign convention: per column, the entry of largest magnitude (lowest row on
// ties) is made positive. Partial argmax per (column, row chunk), then one
// thread per column combines chunks in order.
// ---------------------------------------------------------------------------
// grouped: local tile t covers row chunk t % nchunk of column t / nchunk
template <typename T>
__global__ __launch_bounds__(256) void k_colmax(Group<ColmaxArgs> g) {
    if (group_skipped(g)) return;
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const ColmaxArgs& a = g.args[it];
    const int t = blockIdx.x - g.tstart[it];
    const int c = t / a.nchunk, ch = t % a.nchunk;
    const GLOBAL T* __restrict__ Phi = gbl((const T*)a.Phi);
    const int64_t i0 = (int64_t)ch * a.chunk;
    const int64_t i1 = (i0 + a.chunk < a.m) ? i0 + a.chunk : a.m;
    double best = -1.0, bval = 0.0;
    int64_t bidx = INT64_MAX;
    const GLOBAL T* col = Phi + (int64_t)c * a.ld;
    auto visit = [&](double v, int64_t i) {  // increasing i per thread: strict > keeps the first
        const double av = fabs(v);
        if (av > best) { best = av; bidx = i; bval = v; }
    };
    constexpr int V = 16 / sizeof(T);  // 16-byte loads when the chunk starts on one
    if ((a.ld % V) == 0 && (i0 % V) == 0) {
        typedef T TV __attribute__((ext_vector_type(V)));
        for (int64_t i = i0 + (int64_t)threadIdx.x * V; i < i1; i += 256 * V) {
            if (i + V <= i1) {
                const TV v = *reinterpret_cast<const GLOBAL TV*>(col + i);
#pragma unroll
                for (int k = 0; k < V; ++k) visit((double)v[k], i + k);
            } else {
                for (int64_t k = i; k < i1; ++k) visit((double)col[k], k);
            }
        }
    } else {
        for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) visit((double)col[i], i);
    }
    __shared__ double sb[256], sv[256];
    __shared__ int64_t si[256];
    sb[threadIdx.x] = best; sv[threadIdx.x] = bval; si[threadIdx.x] = bidx;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) {
            const int o = threadIdx.x + off;
            if (sb[o] > sb[threadIdx.x] || (sb[o] == sb[threadIdx.x] && si[o] < si[threadIdx.x])) {
                sb[threadIdx.x] = sb[o]; sv[threadIdx.x] = sv[o]; si[threadIdx.x] = si[o];
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const int64_t slot = (int64_t)c * a.nchunk + ch;
        a.pval[slot] = (sb[0] < 0.0) ? 0.0 : sv[0];
        a.pidx[slot] = si[0];
    }
}

// One wave per column: lane k takes chunks k, k + 64, .., then a butterfly
// keeps the largest magnitude, lowest row on ties (the same entry whatever
// the order of the comparisons).
__global__ __launch_bounds__(64) void k_signs(Group<SignArgs> g) {
    if (group_skipped(g)) return;
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const SignArgs& a = g.args[it];
    const int c = blockIdx.x - g.tstart[it];
    if (c >= a.r) return;  // uniform
    const int lane = threadIdx.x;
    double best = -1.0, bval = 0.0;
    int64_t bidx = INT64_MAX;
    for (int k = lane; k < a.nchunk; k += 64) {
        const double v = a.pval[(int64_t)c * a.nchunk + k];
        const int64_t ix = a.pidx[(int64_t)c * a.nchunk + k];
        const double av = fabs(v);
        if (av > best || (av == best && ix < bidx)) { best = av; bval = v; bidx = ix; }
    }
    for (int off = 32; off >= 1; off >>= 1) {
        const double ob = shfl_xor_d(best, off), ov = shfl_xor_d(bval, off);
        const unsigned long long ub = (unsigned long long)bidx;
        const unsigned lo = (unsigned)__shfl_xor((int)(unsigned)ub, off, 64);
        const unsigned hi = (unsigned)__shfl_xor((int)(unsigned)(ub >> 32), off, 64);
        const int64_t oi = (int64_t)(((unsigned long long)hi << 32) | lo);
        if (ob > best || (ob == best && oi < bidx)) { best = ob; bval = ov; bidx = oi; }
    }
    if (lane == 0) a.signs[c] = (bval < 0.0) ? -1.0 : 1.0;
}

hipError_t launch_signs(int tphi, const GroupLaunch<ColmaxArgs>& C, const GroupLaunch<SignArgs>& S, hipStream_t st) {
    if (tphi == DT_F64)
        hipLaunchKernelGGL(k_colmax<double>, dim3(C.tiles), dim3(256), 0, st, mkg(C));
    else
        hipLaunchKernelGGL(k_colmax<float>, dim3(C.tiles), dim3(256), 0, st, mkg(C));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_signs, dim3(S.tiles), dim3(64), 0, st, mkg(S));
    return hipGetLastError();
}

// grouped: Phi tiles (rows 256 V (t % nb).., column t / nb, V elements of 16 bytes per
// thread); outputs from the call table
template <typename T>
__global__ void k_fin_phi(Group<FinArgs> g) {
    if (group_skipped(g)) return;
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const FinArgs& a = g.args[it];
    const int t = blockIdx.x - g.tstart[it];
    constexpr int V = 16 / sizeof(T);  // elements per thread
    const int nb = (int)((a.m + 256 * V - 1) / (256 * V));
    const int c = t / nb;
    const int64_t i = ((int64_t)(t % nb) * 256 + threadIdx.x) * V;
    if (i >= a.m) return;
    GLOBAL T* Pout = gbl((T*)g.calls[a.call].Phi) + (int64_t)c * a.m;
    const GLOBAL T* Pin = gbl((const T*)a.Phi_int) + (int64_t)c * a.ldP;
    const double sg = a.signs[c];  // +1 or -1: the products are exact
    if (i + V <= a.m && (a.m % V) == 0 && (a.ldP % V) == 0 && ((uintptr_t)Pout % 16) == 0) {
        typedef T TV __attribute__((ext_vector_type(V)));
        const TV v = *reinterpret_cast<const GLOBAL TV*>(Pin + i);
        TV o;
#pragma unroll
        for (int k = 0; k < V; ++k) o[k] = (T)(sg * (double)v[k]);
        *reinterpret_cast<GLOBAL TV*>(Pout + i) = o;
    } else {
        for (int64_t k = i; k < i + V && k < a.m; ++k) Pout[k] = (T)(sg * (double)Pin[k]);
    }
}

template <typename T>
__global__ void k_fin_a(Group<FinArgs> g) {
    if (group_skipped(g)) return;
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const FinArgs& a = g.args[it];
    const int64_t e = (int64_t)(blockIdx.x - g.tstart[it]) * blockDim.x + threadIdx.x;
    const CallDesc& cd = g.calls[a.call];
    if (e < (int64_t)a.r) cd.sigma[e] = a.sig[e];
    if (e >= a.n * a.r) return;
    const int64_t j = e / a.r;
    const int k = (int)(e % a.r);
    gbl((T*)cd.A)[e] = (T)(a.signs[k] * gbl(a.At)[(int64_t)k * a.ldA + j]);
}

int fin_phi_tiles(int64_t m, int r, int tphi) {
    const int64_t span = 256 * (tphi == DT_F64 ? 2 : 4);
    return (int)((m + span - 1) / span) * r;
}
int fin_a_tiles(int64_t n, int r) { return (int)(((n * r > r ? n * r : r) + 255) / 256); }

hipError_t launch_finalize(int tphi, const GroupLaunch<FinArgs>& P, const GroupLaunch<FinArgs>& A, hipStream_t st) {
    if (tphi == DT_F64) {
        hipLaunchKernelGGL(k_fin_phi<double>, dim3(P.tiles), dim3(256), 0, st, mkg(P));
        hipLaunchKernelGGL(k_fin_a<double>, dim3(A.tiles), dim3(256), 0, st, mkg(A));
    } else {
        hipLaunchKernelGGL(k_fin_phi<float>, dim3(P.tiles), dim3(256), 0, st, mkg(P));
        hipLaunchKernelGGL(k_fin_a<float>, dim3(A.tiles), dim3(256), 0, st, mkg(A));
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Adaptive rank: identity factor, stopping decision, energy rank
// ---------------------------------------------------------------------------
__global__ void k_eye(Group<EyeArgs> g) {
    if (group_skipped(g)) return;
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const EyeArgs& a = g.args[it];
    const int e = (blockIdx.x - g.tstart[it]) * 256 + threadIdx.x;
    if (e < a.lp * a.lp) a.R[e] = (e / a.lp == e % a.lp) ? 1.0 : 0.0;
}

hipError_t launch_eye(const GroupLaunch<EyeArgs>& L, hipStream_t st) {
    hipLaunchKernelGGL(k_eye, dim3(L.tiles), dim3(256), 0, st, mkg(L));
    return hipGetLastError();
}

__global__ void k_adapt_decide(Group<AdaptDecideArgs> g) {
    if (group_skipped(g)) return;
    const AdaptDecideArgs& a = g.args[blockIdx.x];
    if (threadIdx.x != 0) return;
    const double f = *a.fro2;
    double E = f;
    for (int j = 0; j <= a.i; ++j) E -= a.cap[j];
    a.E[a.i] = E;
    const bool stop = E <= (1.0 - a.delta) * f || !(E == E) || a.i + 1 >= a.kmax;
    if (stop) {
        a.flags[ADAPT_STOP] |= 1 << (a.i + 1);
        a.flags[ADAPT_LUSED] = (a.i + 1) * a.b;
    } else {
        a.flags[ADAPT_ACTIVE] |= 1 << (a.i + 1);
    }
}

hipError_t launch_adapt_decide(const GroupLaunch<AdaptDecideArgs>& L, hipStream_t st) {
    hipLaunchKernelGGL(k_adapt_decide, dim3(L.count), dim3(64), 0, st, mkg(L));
    return hipGetLastError();
}

__global__ void k_adapt_rank(Group<AdaptRankArgs> g) {
    if (group_skipped(g)) return;
    const AdaptRankArgs& a = g.args[blockIdx.x];
    if (threadIdx.x != 0) return;
    const double f = *a.fro2;
    double cum = 0.0;
    int r = -1;
    for (int k = 0; k < a.l; ++k) {
        cum += __dmul_rn(a.sig[k], a.sig[k]);  // no fused multiply-add: the host's rounding
        if (cum / f >= a.delta) {
            r = k + 1;
            break;
        }
    }
    a.flags[ADAPT_RANK] = r;
}

hipError_t launch_adapt_rank(const GroupLaunch<AdaptRankArgs>& L, hipStream_t st) {
    hipLaunchKernelGGL(k_adapt_rank, dim3(L.count), dim3(64), 0, st, mkg(L));
    return hipGetLastError();
}

}  // namespace rpod
