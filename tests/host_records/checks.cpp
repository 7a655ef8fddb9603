// Host-only stand-ins as in ../host_sanitizer/stubs.cpp, with the launchers below in place of the ones there:
// they check what a launch record promises its kernel (the tiles of a Gram reduction that its Cholesky
// factorisation counts, the factorisation's record, operands within the 32-bit offsets of the FP32 S^T Q) and
// play the stopping test of an adaptive plan, so that every part of its program is walked.
#include <sys/mman.h>

#include "../../include/rpod.h"
#include "../../paper_2504_15350_amd/csrc/internal.hpp"
#include "../../paper_2504_15350_amd/csrc/offsets.hpp"

#define hipMemsetAsync stand_in_hipMemsetAsync
#define gram_reduce_tiles stand_in_gram_reduce_tiles
#define launch_gram stand_in_launch_gram
#define launch_zero_ints stand_in_launch_zero_ints
#define launch_stq_e6 stand_in_launch_stq_e6
#define launch_adapt_decide stand_in_launch_adapt_decide
#define launch_adapt_rank stand_in_launch_adapt_rank
#include "../host_sanitizer/stubs.cpp"
#undef hipMemsetAsync
#undef gram_reduce_tiles
#undef launch_gram
#undef launch_zero_ints
#undef launch_stq_e6
#undef launch_adapt_decide
#undef launch_adapt_rank

static int g_stop = 1;                        // blocks that an adaptive call takes
static int g_decided, g_finishes, g_fin_l;    // blocks decided, finishes run, width of the last one
static int g_grams, g_chols, g_stq, g_stq_wide;

#define EXPECT(c)                                                  \
    do {                                                           \
        if (!(c)) {                                                \
            printf("%s:%d: %s\n", __FILE__, __LINE__, #c);         \
            ++g_bad;                                               \
        }                                                          \
    } while (0)

// plans clear their workspace when they are made: fresh pages are zero
extern "C" hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }

namespace rpod {
int gram_reduce_tiles(int nt) { return npairs_of(nt) * 256 / ((nt <= 4 ? 256 : 512) / 8); }

hipError_t launch_gram(int, int nt, const GroupLaunch<GramArgs>& L, const GroupLaunch<GramArgs>& R, hipStream_t) {
    EXPECT(chk(L) == hipSuccess && chk(R) == hipSuccess && L.count == R.count);
    for (int i = 0; i < R.count; ++i) {
        const GramArgs& a = R.args[i];
        const CholArgs& c = a.chol;
        EXPECT(L.tstart[i + 1] - L.tstart[i] == gram_tiles(nt, a.nwg));
        EXPECT(R.tstart[i + 1] - R.tstart[i] == gram_reduce_tiles(nt));
        ++g_grams;
        if (c.R64 == nullptr) continue;
        ++g_chols;
        EXPECT(c.R32 != nullptr && c.flags != nullptr && c.l >= 1 && c.l <= 16 * nt && c.mode >= 0 && c.mode <= 2);
        EXPECT(c.flags[FLAG_ARRIVED] == 0);
        EXPECT(c.mode == 2 ? a.cond == c.flags + 1 && a.cond_mask == 1 /* shifted */ : a.cond == nullptr);
    }
    return hipSuccess;
}
hipError_t launch_zero_ints(const GroupLaunch<ZeroArgs>& L, hipStream_t) {
    for (int i = 0; i < L.count; ++i) memset(L.args[i].p, 0, sizeof(int) * L.args[i].count);
    return chk(L);
}
hipError_t launch_stq_e6(int, bool vec, const GroupLaunch<StqArgs>& L, hipStream_t) {
    for (int i = 0; i < L.count; ++i) {
        const StqArgs& a = L.args[i];
        EXPECT(L.tstart[i + 1] - L.tstart[i] == a.ncb * a.nsplit && a.ncb * stq_e6_block_cols() == a.nP);
        const bool fits = chunk_offset_fits(a.ldS) && chunk_offset_fits(a.ldQ);
        EXPECT(vec || fits);
        if (!vec) EXPECT(a.ldS % 32 != 0 || L.count > 1);
        ++g_stq;
        g_stq_wide += !fits;
    }
    return chk(L);
}
hipError_t launch_adapt_decide(const GroupLaunch<AdaptDecideArgs>& L, hipStream_t) {
    const AdaptDecideArgs& a = L.args[0];
    ++g_decided;
    if (a.i + 1 == g_stop || a.i + 1 >= a.kmax) {
        a.flags[ADAPT_STOP] |= 1 << (a.i + 1);
        a.flags[ADAPT_LUSED] = (a.i + 1) * a.b;
    } else {
        a.flags[ADAPT_ACTIVE] |= 1 << (a.i + 1);
    }
    return chk(L);
}
hipError_t launch_adapt_rank(const GroupLaunch<AdaptRankArgs>& L, hipStream_t) {
    ++g_finishes;
    g_fin_l = L.args[0].l;
    L.args[0].flags[ADAPT_RANK] = g_fin_l;
    return chk(L);
}
}  // namespace rpod

struct Map {  // zero pages, so that a workspace of many GB costs nothing until it is written
    size_t bytes;
    void* p;
    explicit Map(size_t n) : bytes(n) {
        p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
        if (p == MAP_FAILED) abort();
    }
    ~Map() { munmap(p, bytes); }
};

static rpod_desc desc(int64_t m, int64_t n, int64_t ld, int dt, int r, int p, int q) {
    rpod_desc d{};
    d.m = m; d.n = n; d.ld = ld; d.dtype = dt; d.r = r; d.p = p; d.q = q;
    return d;
}

static void run(const rpod_desc* d, int count) {
    size_t need = 0;
    EXPECT(rpod_workspace_size_batched(d, count, &need) == RPOD_OK);
    Map ws(need);
    rpod_plan p = nullptr;
    EXPECT(rpod_plan_create_batched(&p, d, count, ws.p, need, nullptr) == RPOD_OK);
    if (p) rpod_plan_destroy(p);  // recorded and launched once under (stand-in) capture
}

static void offsets() {
    for (int64_t ld : {(int64_t)1, (int64_t)100003, (int64_t)33554431, (int64_t)33554432, (int64_t)67108863,
                       (int64_t)67108864, (int64_t)71582720, (int64_t)71582976, (int64_t)400000000}) {
        for (int c = 0; c < 16 && rpod::chunk_offset_fits(ld); ++c) {
            for (int k = 0; k < 16; ++k) EXPECT((int64_t)rpod::chunk_offset(c, ld, k) == 4 * ld * c + 16 * k);
            EXPECT((int64_t)(rpod::chunk_offset(c, ld, 0) + 4 * (uint32_t)(ld - 1)) == 4 * ld * c + 4 * (ld - 1));
        }
        for (int g = 0; g < 4 && rpod::row_offset_fits(ld); ++g)
            for (int64_t i : {(int64_t)0, ld / 2, ld + 255})
                EXPECT((int64_t)rpod::row_offset(g, ld, i) == 32 * ld * g + 4 * i);
    }
}

static void adaptive(int dt) {
    const int kmax = 4, b = 16;
    const rpod_desc a = desc(20001, 700, 20001, dt, kmax * b, b, 1);
    size_t need = 0;
    EXPECT(rpod_workspace_size_adaptive(&a, 0.99, &need) == RPOD_OK);
    Map ws(need), buf(256);
    rpod_plan p = nullptr;
    EXPECT(rpod_plan_create_adaptive(&p, &a, 0.99, ws.p, need, nullptr) == RPOD_OK);
    for (int rep = 0; p != nullptr && rep < 2; ++rep)
        for (g_stop = 1; g_stop <= kmax + 1; ++g_stop) {  // kmax + 1: the widths run out
            g_decided = g_finishes = g_fin_l = 0;
            int32_t lu = -1, rk = -1;
            double res = 0;
            EXPECT(rpod_compute_adaptive(p, buf.p, 3, buf.p, static_cast<double*>(buf.p), buf.p, &lu, &rk, &res) ==
                   RPOD_OK);
            const int k = g_stop < kmax ? g_stop : kmax;
            EXPECT(lu == k * b && rk == k * b && g_decided == k && g_finishes == 1 && g_fin_l == k * b);
        }
    if (p) rpod_plan_destroy(p);
}

int main() {
    offsets();
    for (int dt : {RPOD_F64, RPOD_F32, RPOD_BF16, RPOD_F16}) {
        for (int l : {16, 17, 64, 65, 96, 128}) {
            const rpod_desc d = desc(9001, 300, 9001, dt, l - 3, 3, 2);
            run(&d, 1);
        }
        rpod_desc d[3] = {desc(20000, 700, 20000, dt, 25, 10, 1), desc(9000, 1200, 9008, dt, 90, 10, 1),
                          desc(30001, 500, 30001, dt, 10, 10, 1)};
        run(d, 3);
        d[1].block_cols = 100;
        run(d + 1, 1);
        adaptive(dt);
    }
    // S^T Q of very tall FP32 matrices, columns on and off the 128-byte lines, alone and beside another
    const int before = g_stq_wide;
    for (int64_t m : {(int64_t)67108600, (int64_t)67108865, (int64_t)71582721, (int64_t)72000000}) {
        rpod_desc d[2] = {desc(m, 20, m | 1, RPOD_F32, 12, 4, 1), desc(1000, 40, 1001, RPOD_F32, 12, 4, 1)};
        run(d, 1);
        run(d, 2);
        d[0].ld = (m + 31) / 32 * 32;
        run(d, 1);
    }
    EXPECT(g_stq_wide > before && g_grams > g_chols && g_chols > 0);
    const int bad = stub_report();
    printf("%d Gram reductions, %d with a factorisation, %d S^T Q: %s\n", g_grams, g_chols, g_stq, bad ? "FAILED" : "PASSED");
    return bad != 0;
}
