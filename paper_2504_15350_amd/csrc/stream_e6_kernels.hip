// Passes over an FP32 snapshot matrix on the BF16 matrix cores.
//
// Every FP32 value x is split exactly into three bfloat16 parts
//   x = h + m + l,  h = bf16(x), m = bf16(x - h), l = bf16(x - h - m)
// (each difference is exact in FP32). A product of two split operands keeps
// the six terms hh, hm, mh, hl, mm, lh, each an exact BF16 x BF16 product
// accumulated in FP32 by the 16x16x32 MFMA. With |m| <= 2^-8 |x| and
// |l| <= 2^-16 |x| the dropped terms ml, lm, ll weigh together about
// 2^-23 |x| |y|, the size of one FP32 rounding of the product, so a dot
// product is as accurate as one with FP32 products and FP32 accumulation.
// The BF16 matrix cores run 16 times the FP32 rate: with six products per
// term both passes stay bound by HBM, not by the FP32 matrix-core rate.
//
//   k_sx_e6   Y = S X   (X in FP32, split as it is staged)
//   k_stq_e6  slabs of Z = S^T Q (Q split as it is staged), interleaved row splits
//
// MFMA operand layout (16x16x32 bf16, gfx950): lane l supplies
// A[l%16][8(l/16) + i] and B[8(l/16) + i][l%16], i = 0..7; the result holds
// D[4(l/16) + v][l%16].
#include "device_common.hpp"
#include "internal.hpp"
#include "offsets.hpp"
#include "split_ops.hpp"

namespace rpod {

// A 16-byte load at any 4-byte alignment: gfx950 global loads need no more, so odd leading
// dimensions of S take the same path as padded ones (100003 x 2000, ld 100003, 60 columns: S X 184 us,
// against 283 with four scalar loads). Times of passes in this file are those inside a call.
typedef float e6_f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// ---------------------------------------------------------------------------
// Y = S X. Workgroup = W waves = 256 rows, U = 16 / W row tiles per wave. Per
// 32-column step lane (r, g) of a wave holds rows U r .. U r + U - 1 of columns
// j0 + 8 g + i, i = 0..7 (a wave instruction covers 4 columns x 64 U bytes);
// element t of these is the A operand of row tile t (MFMA row r of tile t is row
// U r + t of the wave), K index 8 g + i. The step's block of X (32 rows x 16 NT
// columns, read in FP32 and split into its three BF16 parts as it is staged) is
// kept in LDS, double-buffered, and shared by the waves. All tiles are split before
// the matrix-core work.
// Bound by the reads of S up to 64 columns of X, by the matrix cores beyond (and
// there by the loads and splits that a SIMD's one or two waves leave exposed).
// Waves: four of four tiles, whose operand reads from LDS serve four products
// each; at 128 columns these take more than half of the register file and leave
// one wave per SIMD, and eight of two tiles are the faster (262144 x 1000: 376
// against 484 us, 65536 x 3000: 270 against 358; 1048576 x 128 times 128 x 128:
// 338 against 387; at 112 columns, where two waves still fit, 625 against 466 at
// 131072 x 3500). Every entry has the same order of sums in either.
// ---------------------------------------------------------------------------
constexpr int E6_XLD = 40;  // halfwords per staged X column (32 rows + pad)
// (EN sums S's squares in an order that belongs to four waves)
constexpr int sx_waves(int nt, bool en) { return nt == 8 && !en ? 8 : 4; }
// EARLY: the next step's S columns are loaded as soon as the current ones are split, before the
// matrix-core work; else after it. Early in products with few columns of S (the tall R^-1 applications,
// the lift: with four steps per workgroup every exposed load latency counts), with one workgroup per CU
// or less, which has no other to hide the loads (20000 x 1000, 60 columns: 66 against 75 us; 5003 x 701:
// 45 against 51), at 16 columns (131072 x 2000: 165 against 173) and at 128 (65536 x 3000: 270 against 303
// us; 262144 x 1000: 374 against 418); else late (262144 x 5000, 60 columns: 958 against 968 us; 100003 x
// 2000: 184 against 195; 131072 x 3500, 110 columns: 470 against 509).
constexpr int64_t SX_FEW_TILES = 256;
constexpr bool sx_early_always(int nt) { return nt == 1 || nt == 8; }

template <int NT, bool EN, bool EARLY, int W>
__device__ __forceinline__ void sx_e6_body(const GLOBAL float* S, int64_t ldS, int64_t m, int64_t n,
                                           const GLOBAL float* __restrict__ X, int64_t ldX,
                                           GLOBAL float* Y, int64_t ldY, int64_t mstore, int cmax, int64_t bx,
                                           unsigned short* xs, double* ssq = nullptr) {
    constexpr int XPART = 16 * NT * E6_XLD;     // one staged part
    constexpr int XB = 3 * XPART;               // one staged X block (three parts)
    constexpr int XCH = 16 * NT * 8;            // 16-byte FP32 chunks of a block (4 rows each)
    constexpr int U = 16 / W;                   // row tiles per wave
    constexpr int NTHR = 64 * W, XPT = (XCH + NTHR - 1) / NTHR;
    typedef float Vec __attribute__((ext_vector_type(U)));
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int64_t iw = bx * (16 * U * W) + wave * (16 * U);
    const int64_t irow = iw + U * r16;
    // Unguarded vector loads, a uniform base per column plus a 32-bit lane offset. A wave with rows past
    // m takes whole runs too (rows of the column's padding or of the next column, which meet only
    // output rows past m, written as zero), except where the last column of S is in the step, whose
    // runs could leave S, or a column is shorter than a tile. Where ldS is too large for 32-bit offsets,
    // 64-bit addresses at 16 columns, and the guarded loads of the edges at more, whose matrix-core work
    // hides their selects (34000000 x 80: 16 columns 2780 -> 2660 us, 60 columns 5060 with either).
    const bool narrow = row_offset_fits(ldS), inside = iw + 16 * U <= m;
    const bool fast = (inside || ldS >= 256) && (narrow || NT == 1);
    auto plain = [&](int64_t j0) { return fast && j0 + 32 <= (inside ? n : n - 1); };
    const uint32_t so = row_offset(g, ldS, irow);
    f32x4 acc[U][NT];
#pragma unroll
    for (int t = 0; t < U; ++t)
#pragma unroll
        for (int c = 0; c < NT; ++c) acc[t][c] = f32x4{0, 0, 0, 0};
    Vec sv[8];
    auto load_s = [&](int64_t j0) {
        if (plain(j0) && (NT > 1 || narrow)) {
            const GLOBAL char* p = reinterpret_cast<const GLOBAL char*>(S + j0 * ldS);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                sv[i] = __builtin_nontemporal_load(reinterpret_cast<const GLOBAL run_vec_u<float, U>*>(p + 4 * i * ldS + so));
        } else if (NT == 1 && plain(j0)) {
            const GLOBAL float* p = S + (j0 + 8 * g) * ldS + irow;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                sv[i] = __builtin_nontemporal_load(reinterpret_cast<const GLOBAL run_vec_u<float, U>*>(p + i * ldS));
        } else if (m >= U) {
#pragma unroll
            for (int i = 0; i < 8; ++i) sv[i] = run_load<float, U, true>(S, ldS, m, n, irow, j0 + 8 * g + i);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) sv[i] = run_load<float, U>(S, ldS, m, n, irow, j0 + 8 * g + i);
        }
    };
    f32x4 xr[XPT];
    auto load_x = [&](int64_t j0) {
#pragma unroll
        for (int q = 0; q < XPT; ++q) {
            const int ch = tid + NTHR * q;
            if (ch < XCH) xr[q] = *reinterpret_cast<const GLOBAL f32x4*>(X + (int64_t)(ch >> 3) * ldX + j0 + 4 * (ch & 7));
        }
    };
    // chunk (rows 4 k .. 4 k + 3 of a column) -> 8 bytes of each part
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    auto put_x = [&](int buf) {
#pragma unroll
        for (int q = 0; q < XPT; ++q) {
            const int ch = tid + NTHR * q;
            if (ch < XCH) {
                unsigned h0, m0, l0, h1, m1, l1;
                split_pair(xr[q][0], xr[q][1], h0, m0, l0);
                split_pair(xr[q][2], xr[q][3], h1, m1, l1);
                unsigned short* d = xs + buf * XB + (ch >> 3) * E6_XLD + 4 * (ch & 7);
                *reinterpret_cast<u32x2*>(d) = u32x2{h0, h1};
                *reinterpret_cast<u32x2*>(d + XPART) = u32x2{m0, m1};
                *reinterpret_cast<u32x2*>(d + 2 * XPART) = u32x2{l0, l1};
            }
        }
    };
    load_s(0);
    load_x(0);
    put_x(0);
    int buf = 0;
    double sq = 0.0;  // EN: sum of the squares of this lane's S entries (FP32 per step, FP64 across steps)
    for (int64_t j0 = 0; j0 < n; j0 += 32) {  // uniform trip count: the barriers below are reached by all waves
        const bool more = j0 + 32 < n;
        if (!plain(j0)) {
#pragma unroll
            for (int i = 0; i < 8; ++i) sv[i] = run_fix<float, U>(sv[i], m, n, irow, j0 + 8 * g + i);
        }
        if constexpr (EN) {
            float p = 0.0f;
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    const float x = inside || irow + t < m ? sv[i][t] : 0.0f;
                    p = fmaf(x, x, p);
                }
            sq += (double)p;
        }
        e6_u16x8 ah[U], am[U], al[U];
#pragma unroll
        for (int t = 0; t < U; ++t)
            split8(f32x4{sv[0][t], sv[1][t], sv[2][t], sv[3][t]}, f32x4{sv[4][t], sv[5][t], sv[6][t], sv[7][t]}, ah[t],
                   am[t], al[t]);
        if (more) {
            load_x(j0 + 32);
            if (EARLY) load_s(j0 + 32);  // sv is free once split
        }
        __syncthreads();  // block buf staged
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            const unsigned short* xb = xs + buf * XB + (16 * c + r16) * E6_XLD + 8 * g;
            const e6_u16x8 bh = *reinterpret_cast<const e6_u16x8*>(xb);
            const e6_u16x8 bm = *reinterpret_cast<const e6_u16x8*>(xb + XPART);
            const e6_u16x8 bl = *reinterpret_cast<const e6_u16x8*>(xb + 2 * XPART);
#pragma unroll
            for (int t = 0; t < U; ++t) mma6(ah[t], am[t], al[t], bh, bm, bl, acc[t][c]);
        }
        if (more) {
            if (!EARLY) load_s(j0 + 32);
            put_x(buf ^ 1);  // block buf ^ 1 was last read before this step's barrier
            buf ^= 1;
        }
    }
    if constexpr (EN) *ssq = sq;
    // D[4 g + v][r] of tile t: row iw + U (4 g + v) + t, output column 16 c + r
#pragma unroll
    for (int c = 0; c < NT; ++c) {
        if (16 * c + r16 >= cmax) continue;
        GLOBAL float* py = Y + (int64_t)(16 * c + r16) * ldY;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t row = iw + U * (4 * g + v);
            Vec o;
#pragma unroll
            for (int t = 0; t < U; ++t) o[t] = acc[t][c][v];
            if (!inside) {
#pragma unroll
                for (int t = 0; t < U; ++t) o[t] = row + t < m ? o[t] : 0.0f;
            }
            if (row + U <= mstore) {
                *reinterpret_cast<GLOBAL Vec*>(py + row) = o;
            } else {
#pragma unroll
                for (int t = 0; t < U; ++t)
                    if (row + t < mstore) py[row + t] = o[t];
            }
        }
    }
}

// EN: the energy report's variant (also each tile's sum of squares of S, in
// a fixed order: per lane, then a tree over the workgroup)
template <int NT, bool EN, bool EARLY>
__global__ __launch_bounds__(64 * sx_waves(NT, EN))
__attribute__((amdgpu_waves_per_eu(EN && NT == 8 ? 1 : 2, sx_waves(NT, EN) == 8 ? 4 : 2))) void k_sx_e6(
    Group<SxArgs> g) {
    if (group_skipped(g)) return;
    constexpr int W = sx_waves(NT, EN);
    __shared__ __attribute__((aligned(16))) unsigned short xs[2 * 3 * 16 * NT * E6_XLD];
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const SxArgs& a = g.args[it];
    if (a.cond != nullptr && !(*a.cond & a.cond_mask)) return;
    const void* S = static_cast<const char*>(a.call >= 0 ? g.calls[a.call].S : a.S) + a.col0 * a.ldS * 4;
    if constexpr (EN) {
        __shared__ double red[256];
        double sq = 0.0;
        sx_e6_body<NT, true, EARLY, W>(gbl((const float*)S), a.ldS, a.m, a.n, gbl((const float*)a.X), a.ldX,
                                  gbl((float*)a.Y), a.ldY, a.mstore, a.cmax > 0 ? a.cmax : 16 * NT,
                                  blockIdx.x - g.tstart[it], xs, &sq);
        red[threadIdx.x] = sq;
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
            __syncthreads();
        }
        if (threadIdx.x == 0 && a.fpart != nullptr) a.fpart[blockIdx.x - g.tstart[it]] = red[0];
    } else {
        sx_e6_body<NT, false, EARLY, W>(gbl((const float*)S), a.ldS, a.m, a.n, gbl((const float*)a.X), a.ldX,
                                         gbl((float*)a.Y), a.ldY, a.mstore, a.cmax > 0 ? a.cmax : 16 * NT,
                                         blockIdx.x - g.tstart[it], xs);
    }
}

// ---------------------------------------------------------------------------
// Z_s = S^T Q. Workgroup: 256 columns of S (16 / W column tiles of 16
// for each of the W waves), 32 rows per step; the step's S block (32 x 256, FP32) and the three
// BF16 parts of the Q block (32 x 16 NT, read as FP32 and split when staged)
// are staged in LDS column-major and the next step's blocks are loaded into
// registers during the matrix-core work. Lane (r, g) reads rows 8 g .. 8 g + 7
// of its S column (the A operand, split in registers) and of each Q column
// part (the B operand).
// Columns are stored unpadded with their 16-byte chunks XOR-swizzled (S
// column c: chunk k at k ^ ((c / 2) mod 8); Q column c: chunk k at
// k ^ ((c / 4) mod 4)), which keeps both the staging writes and the operand
// reads free of bank conflicts for every 16 lanes.
// Splits interleaved in units of 64 rows (256 bytes of an FP32 Q column):
// unit k of split s covers rows 64 (k nsplit + s) .. + 63, two steps. Each
// workgroup writes its FP32 accumulators as its split's slab (summed in FP64
// afterwards).
// Tiles go to the XCDs (workgroup b runs on XCD b mod 8) so that each XCD
// holds every column block of its splits: the Q rows of a split are then
// fetched into one L2 only.
// ---------------------------------------------------------------------------
constexpr int E6_R = 32, E6_LDS = E6_R, E6_LDQ = E6_R, E6_HB = 256;

// Waves per workgroup: four of four column tiles while two of them fit a SIMD's registers (two workgroups
// per CU); at 112 and 128 columns of Q they do not, and eight of two tiles hide more of the loads and
// splits than one such wave (65536 x 3000, 128 columns: 332 -> 303 us; 131072 x 3500, 110 columns: 688 ->
// 604; but at 80 columns 40000 x 4000 194 against 174 us, at 60 262144 x 5000 1372 against 1071). Two LDS
// buffers and one barrier per step measured no better on the whole (back to back: 349 against 363 us at
// 262144 x 1000 with 128 columns, but 612 against 590 with 110 and 1242 against 1108 at 262144 x 5000
// with 60).
constexpr int stq_waves(int nt, bool lines) { return lines && nt >= 7 ? 8 : 4; }

template <int NT, int W>
__device__ __forceinline__ void stq_e6_body(const GLOBAL float* __restrict__ S, int64_t ldS, int64_t m, int64_t n,
                                            const GLOBAL float* __restrict__ Q, int64_t ldQ,
                                            GLOBAL float* __restrict__ Zp, int64_t nP, int nsplit, int ncb,
                                            int tile, float* ss, unsigned short* qs) {
    constexpr int R = E6_R, LD = E6_LDS, LDQ = E6_LDQ, HB = E6_HB, U = HB / (16 * W), NTHR = 64 * W;
    constexpr int CPC = R / 4;                  // 16-byte S chunks per column
    constexpr int SPT = HB * CPC / NTHR;       // S chunks per thread
    constexpr int QCPC = R / 4;                 // 16-byte FP32 Q chunks per column
    constexpr int QCH = 16 * NT * QCPC;         // Q chunks per step
    constexpr int QPT = (QCH + NTHR - 1) / NTHR;
    constexpr int QPART = 16 * NT * LDQ;        // halfwords per staged part
    const int cb = tile % ncb, sp = tile / ncb;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int64_t j0 = (int64_t)cb * HB;
    const int64_t ib = (int64_t)sp * (2 * R), jump = (int64_t)nsplit * (2 * R) - R;
    // next step: the second half of the unit, or the first half of the next unit
    auto next = [&](int64_t i) { return ((i / R) & 1) ? i + jump : i + R; };

    f32x4 acc[U][NT];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < NT; ++c) acc[u][c] = f32x4{0, 0, 0, 0};

    f32x4 sr[SPT];
    f32x4 qr[QPT];
    // chunk q of a thread: column j0 + tid / CPC + q (NTHR / CPC), rows 4 (tid mod CPC) .. +3 of the step
    constexpr int CSTEP = NTHR / CPC;
    const GLOBAL float* sbase = S + (j0 + tid / CPC) * ldS + 4 * (tid % CPC);
    auto fetch = [&](int64_t i0) {
        if (j0 + HB <= n) {  // whole step in range: one unguarded vector load per chunk
            const GLOBAL float* p = sbase + i0;
#pragma unroll
            for (int q = 0; q < SPT; ++q)
                sr[q] = __builtin_nontemporal_load(reinterpret_cast<const GLOBAL e6_f32x4u*>(p + CSTEP * q * ldS));
        } else {  // columns past n read column n - 1 and are written as zero at the end
#pragma unroll
            for (int q = 0; q < SPT; ++q) {
                const int jl = min(tid / CPC + CSTEP * q, (int)(n - 1 - j0));
                sr[q] = __builtin_nontemporal_load(
                    reinterpret_cast<const GLOBAL e6_f32x4u*>(S + (j0 + jl) * ldS + i0 + 4 * (tid % CPC)));
            }
        }
    };
    auto fetch_q = [&](int64_t i0) {
#pragma unroll
        for (int q = 0; q < QPT; ++q) {
            const int ch = tid + NTHR * q;
            if (QCH % NTHR == 0 || ch < QCH)
                qr[q] = *reinterpret_cast<const GLOBAL f32x4*>(Q + (int64_t)(ch / QCPC) * ldQ + i0 + 4 * (ch % QCPC));
        }
    };
    static_assert(CPC == 8 && QCPC == 8, "swizzle patterns assume 32-row steps");
    auto put_s = [&]() {
#pragma unroll
        for (int q = 0; q < SPT; ++q) {
            const int ch = tid + NTHR * q, col = ch / CPC;
            *reinterpret_cast<f32x4*>(ss + col * LD + 4 * ((ch % CPC) ^ ((col >> 1) & 7))) = sr[q];
        }
    };
    // a last step past row m (rows past m must count as zero against any padding of S)
    auto put_edge = [&](int64_t i0) {
        const int64_t i = i0 + 4 * (tid % CPC), j = j0 + tid / CPC;
        if (m >= 4) {
#pragma unroll
            for (int q = 0; q < SPT; ++q) sr[q] = run_load<float, 4, true>(S, ldS, m, n, i, j + CSTEP * q);
        } else {
#pragma unroll
            for (int q = 0; q < SPT; ++q) sr[q] = run_load<float, 4>(S, ldS, m, n, i, j + CSTEP * q);
        }
#pragma unroll
        for (int q = 0; q < SPT; ++q)
            sr[q] = run_fix<float, 4>(sr[q], m, n, i, j + CSTEP * q);
        put_s();
    };
    auto put_q = [&]() {
        // Q chunk (rows 4 k .. 4 k + 3 of a column) -> 8 bytes of each part, in
        // half k mod 2 of the part's 16-byte chunk k / 2
        typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int q = 0; q < QPT; ++q) {
            const int ch = tid + NTHR * q, col = ch / QCPC, k = ch % QCPC;
            if (QCH % NTHR == 0 || ch < QCH) {
                unsigned h0, m0, l0, h1, m1, l1;
                split_pair(qr[q][0], qr[q][1], h0, m0, l0);
                split_pair(qr[q][2], qr[q][3], h1, m1, l1);
                const int o = col * LDQ + 8 * ((k >> 1) ^ ((col >> 2) & 3)) + 4 * (k & 1);
                *reinterpret_cast<u32x2*>(qs + o) = u32x2{h0, h1};
                *reinterpret_cast<u32x2*>(qs + QPART + o) = u32x2{m0, m1};
                *reinterpret_cast<u32x2*>(qs + 2 * QPART + o) = u32x2{l0, l1};
            }
        }
    };

    auto work = [&]() {
        e6_u16x8 ah[U], am[U], al[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int col = 16 * U * wave + 16 * u + r16, sw = (col >> 1) & 7;
            const float* src = ss + col * LD;
            split8(*reinterpret_cast<const f32x4*>(src + 4 * ((2 * g) ^ sw)),
                   *reinterpret_cast<const f32x4*>(src + 4 * ((2 * g + 1) ^ sw)), ah[u], am[u], al[u]);
        }
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            const int col = 16 * c + r16;
            const int o = col * LDQ + 8 * (g ^ ((col >> 2) & 3));
            const e6_u16x8 bh = *reinterpret_cast<const e6_u16x8*>(qs + o);
            const e6_u16x8 bm = *reinterpret_cast<const e6_u16x8*>(qs + QPART + o);
            const e6_u16x8 bl = *reinterpret_cast<const e6_u16x8*>(qs + 2 * QPART + o);
#pragma unroll
            for (int u = 0; u < U; ++u) mma6(ah[u], am[u], al[u], bh, bm, bl, acc[u][c]);
        }
    };
    int64_t i0 = ib;
    if (i0 < m) fetch_q(i0);
    if (i0 + R <= m) fetch(i0);
    while (i0 + R <= m) {
        const int64_t nx = next(i0);
        __syncthreads();  // previous step consumed
        put_s();
        put_q();
        __syncthreads();
        if (nx < m) fetch_q(nx);  // in flight during the matrix-core work
        if (nx + R <= m) fetch(nx);
        work();
        i0 = nx;
    }
    if (i0 < m) {
        __syncthreads();
        put_edge(i0);
        put_q();
        __syncthreads();
        work();
    }
    // D[4 g + v][r]: S column j0 + 16 U w + 16 u + 4 g + v, Q column 16 c + r; the
    // slab keeps the FP32 accumulators as they are (summed in FP64 afterwards)
    GLOBAL float* zp = Zp + (int64_t)sp * nP * (16 * NT);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            const int64_t j = j0 + 16 * U * wave + 16 * u + 4 * g;
            if (j0 + HB > n) {
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[u][c][v] = j + v < n ? acc[u][c][v] : 0.0f;
            }
            *reinterpret_cast<GLOBAL f32x4*>(zp + (int64_t)(16 * c + r16) * nP + j) = acc[u][c];
        }
}

// ---------------------------------------------------------------------------
// The same product where S's columns do not start on 128-byte lines (odd or
// padded leading dimensions): a 32-row run of a column then straddles two lines,
// so the workgroup takes its units of 64 rows in two steps of 128 columns x 64
// rows (runs of 256 bytes, three lines instead of four). The accumulation
// order of every entry is the one above. 100003 x 2000, 60 columns, ld 100003 /
// 100008: 293 / 268 -> 234 / 223 us; with columns on lines the steps above are
// the faster (131072 x 2000: by 9 %), because here a staged Q operand serves two
// column tiles instead of four. S or Q of 2^26 rows and more
// stays with the steps above: a thread's columns here lie within a 32-bit offset
// of a uniform base, which in 64 bits takes registers that 96 columns do not have.
// A last, short unit is loaded ahead like any other, its runs moved inside the
// column, and shifted back when it is staged (loaded when it is staged: 1000 x
// 20000, ld 1001, 12 columns 39 -> 30 us; 5003 x 701 16.6 -> 11.6).
// The S block (128 x 64, FP32) of a step and once per unit the parts of the Q
// block (64 x 16 NT) are staged in LDS column-major. Wave w owns columns 32 w ..
// 32 w + 31 of each half (two column tiles). S column c holds its 16-byte
// chunk k at k ^ sw_s(c), Q column c at k ^ sw_q(c): the 32 lanes one LDS cycle
// serves (16 columns, two g) touch every 16-byte slot of its 512-byte window once.
// ---------------------------------------------------------------------------
constexpr int E6U_R = 64, E6U_HC = 128;

__device__ __forceinline__ int sw_s(int c) { return ((c >> 1) & 1) | (((c >> 1) & 6) << 1); }  // of 16 chunks
__device__ __forceinline__ int sw_q(int c) { return ((c >> 2) & 3) << 1; }                     // of 8 chunks

template <int NT>
__device__ __forceinline__ void stq_e6u_body(const GLOBAL float* __restrict__ S, int64_t ldS, int64_t m, int64_t n,
                                           const GLOBAL float* __restrict__ Q, int64_t ldQ,
                                           GLOBAL float* __restrict__ Zp, int64_t nP, int nsplit, int ncb,
                                           int tile, float* ss, unsigned short* qs) {
    constexpr int R = E6U_R, U = 2;             // column tiles per wave and half
    constexpr int CPC = R / 4;                  // 16-byte FP32 chunks per column
    constexpr int SPT = E6U_HC * CPC / 256;      // S chunks per thread and step
    constexpr int QCH = 16 * NT * CPC;          // Q chunks per unit
    constexpr int QPT = QCH / 256;
    constexpr int QPART = 16 * NT * R;          // halfwords per staged part
    const int cb = tile % ncb, sp = tile / ncb;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int64_t j0 = (int64_t)cb * E6_HB;

    f32x4 acc[2][U][NT];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < NT; ++c) acc[h][u][c] = f32x4{0, 0, 0, 0};

    f32x4 sr[SPT];
    f32x4 qr[QPT];
    // chunk q of a thread: column (of the half) tid / CPC + q (256 / CPC), rows 4 (tid mod CPC) .. + 3.
    // Addresses are a uniform base per chunk plus one 32-bit offset per thread (the launch goes to the
    // other steps where it does not fit).
    constexpr int CSTEP = 256 / CPC;
    const int tc = tid / CPC, tk = tid % CPC;
    const uint32_t so = chunk_offset(tc, ldS, tk), qo = chunk_offset(tc, ldQ, tk);
    const int sws = sw_s(tc), swq = sw_q(tc);  // of every column tc + 16 q
    // a last unit past row m: runs moved inside the column (m >= 4), shifted back when they are staged
    auto fetch_s = [&](int64_t i0, int h) {
        const int64_t jh = j0 + E6U_HC * h;
        const bool edge = i0 + R > m;
        if (edge && m < 4) return;  // loaded when it is staged
        if (jh + E6U_HC <= n) {  // every column in range: a uniform base
            const GLOBAL char* p = reinterpret_cast<const GLOBAL char*>(S + jh * ldS + (edge ? 0 : i0));
            const uint32_t o = edge ? chunk_offset(tc, ldS, 0) + 4 * (uint32_t)min(i0 + 4 * tk, m - 4) : so;
#pragma unroll
            for (int q = 0; q < SPT; ++q)
                sr[q] = __builtin_nontemporal_load(
                    reinterpret_cast<const GLOBAL e6_f32x4u*>(p + 4 * CSTEP * q * ldS + o));
        } else {  // columns past n read column n - 1 and are written as zero at the end
            const GLOBAL float* p = S + (edge ? min(i0 + 4 * tk, m - 4) : i0 + 4 * tk);
#pragma unroll
            for (int q = 0; q < SPT; ++q) {
                const int64_t j = jh + tc + CSTEP * q;
                sr[q] = __builtin_nontemporal_load(reinterpret_cast<const GLOBAL e6_f32x4u*>(p + (j < n ? j : n - 1) * ldS));
            }
        }
    };
    auto fetch_q = [&](int64_t i0) {
        const GLOBAL char* p = reinterpret_cast<const GLOBAL char*>(Q + i0);
#pragma unroll
        for (int q = 0; q < QPT; ++q)
            qr[q] = *reinterpret_cast<const GLOBAL f32x4*>(p + 4 * CSTEP * q * ldQ + qo);
    };
    auto put_s = [&](int64_t i0, int h) {
        float* d = ss + tc * R + 4 * (tk ^ sws);
        if (i0 + R > m) {
            const int64_t i = i0 + 4 * tk, j = j0 + E6U_HC * h + tc;
            if (m >= 4) {
#pragma unroll
                for (int q = 0; q < SPT; ++q)
                    *reinterpret_cast<f32x4*>(d + CSTEP * q * R) = run_fix<float, 4>(sr[q], m, 1, i, 0);
            } else {
#pragma unroll 1
                for (int q = 0; q < SPT; ++q)
                    *reinterpret_cast<f32x4*>(d + CSTEP * q * R) =
                        run_fix<float, 4>(run_load<float, 4>(S, ldS, m, n, i, j + CSTEP * q), m, n, i, j + CSTEP * q);
            }
        } else {
#pragma unroll
            for (int q = 0; q < SPT; ++q) *reinterpret_cast<f32x4*>(d + CSTEP * q * R) = sr[q];
        }
    };
    // Q chunk (rows 4 k .. 4 k + 3 of a column) -> 8 bytes of each part, in half k mod 2 of the
    // part's 16-byte chunk k / 2
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    auto put_q = [&]() {
        unsigned short* d = qs + tc * R + 8 * ((tk >> 1) ^ swq) + 4 * (tk & 1);
#pragma unroll
        for (int q = 0; q < QPT; ++q) {
            const int o = CSTEP * q * R;
            unsigned h0, m0, l0, h1, m1, l1;
            split_pair(qr[q][0], qr[q][1], h0, m0, l0);
            split_pair(qr[q][2], qr[q][3], h1, m1, l1);
            *reinterpret_cast<u32x2*>(d + 2 * QPART + o) = u32x2{l0, l1};
            *reinterpret_cast<u32x2*>(d + o) = u32x2{h0, h1};
            *reinterpret_cast<u32x2*>(d + QPART + o) = u32x2{m0, m1};
        }
    };
    // the staged half times the staged unit of Q, 32 rows at a time
    auto half = [&](f32x4 (&ac)[U][NT]) {
#pragma unroll 1
        for (int kh = 0; kh < 2; ++kh) {
            const float* src = ss + (32 * wave + r16) * R;
            const int c0 = (8 * kh + 2 * g) ^ sw_s(r16), cq = (4 * kh + g) ^ sw_q(r16);
            f32x4 x0[U], x1[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                x0[u] = *reinterpret_cast<const f32x4*>(src + 16 * u * R + 4 * c0);
                x1[u] = *reinterpret_cast<const f32x4*>(src + 16 * u * R + 4 * (c0 ^ 1));
            }
            const unsigned short* qp0 = qs + r16 * R + 8 * cq;
            e6_u16x8 ah[U], am[U], al[U];
#pragma unroll
            for (int u = 0; u < U; ++u) split8(x0[u], x1[u], ah[u], am[u], al[u]);
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                const unsigned short* qp = qp0 + 16 * c * R;
                const e6_u16x8 bh = *reinterpret_cast<const e6_u16x8*>(qp);
                const e6_u16x8 bm = *reinterpret_cast<const e6_u16x8*>(qp + QPART);
                const e6_u16x8 bl = *reinterpret_cast<const e6_u16x8*>(qp + 2 * QPART);
#pragma unroll
                for (int u = 0; u < U; ++u) mma6(ah[u], am[u], al[u], bh, bm, bl, ac[u][c]);
            }
        }
    };

    const int64_t ib = (int64_t)sp * R, jump = (int64_t)nsplit * R;
    if (ib < m) {
        fetch_s(ib, 0);
        fetch_q(ib);
    }
    for (int64_t i0 = ib; i0 < m; i0 += jump) {
        __syncthreads();  // the previous unit is consumed
        put_s(i0, 0);
        put_q();
        fetch_s(i0, 1);  // in flight during the matrix-core work
        __syncthreads();
        half(acc[0]);
        __syncthreads();
        put_s(i0, 1);
        if (i0 + jump < m) {
            fetch_s(i0 + jump, 0);
            fetch_q(i0 + jump);
        }
        __syncthreads();
        half(acc[1]);
    }
    // D[4 g + v][r]: S column j0 + 128 h + 32 w + 16 u + 4 g + v, Q column 16 c + r; the slab keeps the
    // FP32 accumulators as they are (summed in FP64 afterwards)
    GLOBAL float* zp = Zp + (int64_t)sp * nP * (16 * NT);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                const int64_t j = j0 + E6U_HC * h + 32 * wave + 16 * u + 4 * g;
                if (j0 + E6_HB > n) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[h][u][c][v] = j + v < n ? acc[h][u][c][v] : 0.0f;
                }
                *reinterpret_cast<GLOBAL f32x4*>(zp + (int64_t)(16 * c + r16) * nP + j) = acc[h][u][c];
            }
}

// LINES: S's columns start on 128-byte lines
template <int NT, bool LINES>
__global__ __launch_bounds__(64 * stq_waves(NT, LINES)) __attribute__((amdgpu_waves_per_eu(
    NT <= 6 || stq_waves(NT, LINES) == 8 ? 2 : 1, 2))) void k_stq_e6(
    Group<StqArgs> g) {
    if (group_skipped(g)) return;
    __shared__ __attribute__((aligned(16))) float ss[E6_HB * E6_LDS];  // = 128 x 64
    __shared__ __attribute__((aligned(16))) unsigned short qs[3 * 16 * NT * (LINES ? E6_LDQ : E6U_R)];
    const int it = group_item(g.tstart, g.count, blockIdx.x);
    const StqArgs& a = g.args[it];
    const void* S = a.call >= 0 ? g.calls[a.call].S : a.S;
    // XCD-aware order: local tile b (XCD b mod 8 when the item starts at a
    // multiple of 8) takes tile (b mod 8) T / 8 + b / 8 of the item's T
    const int local = blockIdx.x - g.tstart[it], ntl = a.ncb * a.nsplit;
    const int tile = ((ntl & 7) == 0 && (g.tstart[it] & 7) == 0) ? (local & 7) * (ntl >> 3) + (local >> 3) : local;
    if constexpr (LINES)
        stq_e6_body<NT, stq_waves(NT, true)>(gbl((const float*)S), a.ldS, a.m, a.n, gbl((const float*)a.Q), a.ldQ, gbl((float*)a.Zp),
                        a.nP, a.nsplit, a.ncb, tile, ss, qs);
    else
        stq_e6u_body<NT>(gbl((const float*)S), a.ldS, a.m, a.n, gbl((const float*)a.Q), a.ldQ, gbl((float*)a.Zp),
                         a.nP, a.nsplit, a.ncb, tile, ss, qs);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <typename A>
static Group<A> mke6(const GroupLaunch<A>& L) {
    Group<A> g;
    g.args = L.args;
    g.tstart = L.tstart;
    g.calls = L.calls;
    g.count = L.count;
    g.skip = L.skip;
    g.skip_mask = L.skip_mask;
    return g;
}

template <int NT>
static hipError_t sxe6_nt(const GroupLaunch<SxArgs>& L, bool en, bool tall, hipStream_t st) {
    constexpr int NTHR = 64 * sx_waves(NT, false);
    if (en)
        hipLaunchKernelGGL((k_sx_e6<NT, true, false>), dim3(L.tiles), dim3(256), 0, st, mke6(L));
    else if (tall || sx_early_always(NT) || L.tiles <= SX_FEW_TILES)
        hipLaunchKernelGGL((k_sx_e6<NT, false, true>), dim3(L.tiles), dim3(NTHR), 0, st, mke6(L));
    else
        hipLaunchKernelGGL((k_sx_e6<NT, false, sx_early_always(NT)>), dim3(L.tiles), dim3(NTHR), 0, st, mke6(L));
    return hipGetLastError();
}

hipError_t launch_sx_e6(int nt, bool /*vec*/, bool en, bool tall, const GroupLaunch<SxArgs>& L, hipStream_t st) {
    switch (nt) {
#define RPOD_E6_CASE(K) case K: return sxe6_nt<K>(L, en, tall, st);
        RPOD_E6_CASE(1) RPOD_E6_CASE(2) RPOD_E6_CASE(3) RPOD_E6_CASE(4)
        RPOD_E6_CASE(5) RPOD_E6_CASE(6) RPOD_E6_CASE(7) RPOD_E6_CASE(8)
#undef RPOD_E6_CASE
        default: return hipErrorInvalidValue;
    }
}

template <int NT>
static hipError_t stqe6_nt(const GroupLaunch<StqArgs>& L, bool lines, hipStream_t st) {
    if (lines)
        hipLaunchKernelGGL((k_stq_e6<NT, true>), dim3(L.tiles), dim3(64 * stq_waves(NT, true)), 0, st, mke6(L));
    else
        hipLaunchKernelGGL((k_stq_e6<NT, false>), dim3(L.tiles), dim3(256), 0, st, mke6(L));
    return hipGetLastError();
}

hipError_t launch_stq_e6(int nt, bool vec, const GroupLaunch<StqArgs>& L, hipStream_t st) {
    switch (nt) {
#define RPOD_E6_CASE(K) case K: return stqe6_nt<K>(L, vec, st);
        RPOD_E6_CASE(1) RPOD_E6_CASE(2) RPOD_E6_CASE(3) RPOD_E6_CASE(4)
        RPOD_E6_CASE(5) RPOD_E6_CASE(6) RPOD_E6_CASE(7) RPOD_E6_CASE(8)
#undef RPOD_E6_CASE
        default: return hipErrorInvalidValue;
    }
}

int stq_e6_block_cols() { return E6_HB; }

}  // namespace rpod
