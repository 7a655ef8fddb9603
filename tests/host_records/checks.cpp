// Host-only stand-ins as in ../host_sanitizer/stubs.cpp, with the launchers below in place of the ones there:
// they check what a launch record promises its kernel (operands within the 32-bit offsets of the FP32 S^T Q).
#include <sys/mman.h>

#include "../../include/rpod.h"
#include "../../paper_2504_15350_amd/csrc/internal.hpp"
#include "../../paper_2504_15350_amd/csrc/offsets.hpp"

#define hipMemsetAsync stand_in_hipMemsetAsync
#define launch_stq_e6 stand_in_launch_stq_e6
#include "../host_sanitizer/stubs.cpp"
#undef hipMemsetAsync
#undef launch_stq_e6

static int g_stq, g_stq_wide;

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
        for (int c = 0; c < 16 && rpod::chunk_offset_fits(ld); ++c)
            for (int k = 0; k < 16; ++k) EXPECT((int64_t)rpod::chunk_offset(c, ld, k) == 4 * ld * c + 16 * k);
        for (int g = 0; g < 4 && rpod::row_offset_fits(ld); ++g)
            for (int64_t i : {(int64_t)0, ld / 2, ld + 255})
                EXPECT((int64_t)rpod::row_offset(g, ld, i) == 32 * ld * g + 4 * i);
    }
}

int main() {
    offsets();
    // S^T Q of very tall FP32 matrices, columns on and off the 128-byte lines, alone and beside another
    for (int64_t m : {(int64_t)67108600, (int64_t)67108865, (int64_t)71582721, (int64_t)72000000}) {
        rpod_desc d[2] = {desc(m, 20, m | 1, RPOD_F32, 12, 4, 1), desc(1000, 40, 1001, RPOD_F32, 12, 4, 1)};
        run(d, 1);
        run(d, 2);
        d[0].ld = (m + 31) / 32 * 32;
        run(d, 1);
    }
    EXPECT(g_stq > g_stq_wide && g_stq_wide > 0);
    const int bad = stub_report();
    printf("%d S^T Q, %d of them wide: %s\n", g_stq, g_stq_wide, bad ? "FAILED" : "PASSED");
    return bad != 0;
}
