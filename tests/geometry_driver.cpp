// CPU check of the LDS sizes that go with a plan: for every workgroup size, a
// sweep of chunk lengths and delays around the LDS limit, both plans a bank can
// take (pieces of max_block samples, short segments) carry LDS sizes that hold
// the batches of their own length, with the window in LDS and in global memory.
// Built by tests/test_geometry.py; exits non-zero on the first violation.
#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "layout.h"

using namespace spiir;
using namespace spiir::layout;

namespace {

// What the forward kernel lays out: the window, a tile of lane sums per wave, two
// buffers of row sums (odd row stride) and key slots of one batch.
size_t kernel_lds(int wpg, const Geometry &g, int dmax, bool window, int sumb) {
    const size_t steps = (size_t)sumb, rows = 4 * (size_t)wpg + 1;
    const size_t win = window ? (size_t)((dmax + g.nb + kFwdTile + 3) / 4 * 4) * 4 : 0;
    return win + (size_t)wpg * kFwdTile * 64 * 8 + 2 * steps * rows * 8 + 2 * steps * 8;
}

int bad(const char *what, int wpg, int L, int dmax, const Geometry &g) {
    std::fprintf(stderr, "FAIL %s: wpg %d chunk_len %d delay %d: batch %d, lds %zu, lds_tile %zu\n", what, wpg, L, dmax,
                 g.sumb, g.lds_run, g.lds_tile);
    return 1;
}

int check(int wpg, int L, int dmax, int max_block, size_t cap, const Geometry &g) {
    if (L % g.tt || g.nb < std::min(L, max_block)) return bad("chunk", wpg, L, dmax, g);
    if (g.sumb < kFwdTile || g.sumb > kLongBatch || g.sumb % kFwdTile) return bad("batch", wpg, L, dmax, g);
    if (g.lds_tile < kernel_lds(wpg, g, dmax, false, kLongBatch)) return bad("comparator", wpg, L, dmax, g);
    if (g.lds_run < kernel_lds(wpg, g, dmax, g.xlds, g.sumb)) return bad("bank", wpg, L, dmax, g);
    if (g.lds > g.lds_run || g.lds_run > cap || g.lds_tile > cap) return bad("over the device's LDS", wpg, L, dmax, g);
    return 0;
}

}  // namespace

int main() {
    const size_t cap = 160 * 1024;
    long plans = 0, differ = 0;
    for (int wpg = 1; wpg <= kMaxWaves; ++wpg)
        for (int L = 8; L <= 4096; L += L < 512 ? 8 : 64)
            for (int dmax = 0; dmax <= 42000; dmax += dmax < 15000 ? 2500 : 61) {
                const int max_block = std::max(L, 16384 / L * L);
                const Geometry whole = plan_geometry(wpg, dmax, L, max_block, cap);
                const Geometry part = plan_short_geometry(wpg, dmax, L, max_block, cap);
                if (check(wpg, L, dmax, max_block, cap, whole)) return 1;
                if (check(wpg, L, dmax, max_block, cap, part)) return 1;
                ++plans;
                differ += whole.sumb != part.sumb;
            }
    if (!differ) {
        std::fprintf(stderr, "FAIL the two plans never differ in batch length: the sweep misses the limit\n");
        return 1;
    }
    std::printf("geometry ok: %ld plans, %ld with different batches\n", plans, differ);
    return 0;
}
