// Layers whose kernels trade places with the batch: planned for both on the same weight tiles,
// inside the packed bytes, and sent to each by some batch.  Returns the number of faults.
#include <cstdio>

#include "bsp_common.h"

using namespace bsp;

namespace {

int bad = 0;

void check(int cin, int h, int w, int cout, int k, int s, int reg, int bh, int bw, int rate, int n_main, int n_alt) {
    bsp_scheme q;
    memset(&q, 0, sizeof(q));
    q.rows = cout; q.cols = cin * std::max(1, k * k); q.regularity = reg; q.bh = bh; q.bw = bw; q.rate = rate;
    q.khw = reg == BSP_PUNCHED ? k * k : 1;
    const bsp_conv_shape c = {1, cin, h, w, k, k, s, s, k / 2, k / 2};
    Plan p, a;
    const bsp_status st = make_plan(&q, k ? &c : nullptr, BSP_BF16, 0, &p, &a);
    bool ok = st == BSP_OK && p.alt;
    if (ok) {
        ok = a.pl && a.S == p.S && a.L == p.L && a.n_groups == p.n_groups && a.mt_per_group == p.mt_per_group &&
             a.shared == p.shared && a.off_a == p.off_a && a.fingerprint == p.fingerprint &&
             a.n_mb * a.MBT <= p.n_mt_pad && p.off_a + (int64_t)p.n_mt_pad * p.S * 1024 <= p.tile_bytes;
        if (!p.shared)
            ok = ok && a.off_desc16 == p.off_alt && p.alt_g_pad >= a.n_mb * a.MBG && p.alt_g_pad >= p.n_groups &&
                 p.off_alt >= p.off_counts && p.off_alt % 4 == 0 &&
                 p.off_alt + (int64_t)2 * p.alt_g_pad * p.LP <= p.tile_bytes;
        ok = ok && !alt_takes(p, a, n_main, 1) && alt_takes(p, a, n_alt, 1);
    }
    if (ok) return;
    printf("%d x %d -> %d, %dx%d: status %d alt %d takes %d %d\n", cin, k, cout, h, w, st, p.alt,
           p.alt ? alt_takes(p, a, n_main, 1) : -1, p.alt ? alt_takes(p, a, n_alt, 1) : -1);
    ++bad;
}

}  // namespace

int main() {
    // measured (us): the planned kernel and the other one at the second batch
    check(512, 14, 14, 512, 3, 2, BSP_COL, 16, 32, 4, 64, 1);    // 25 and 15 at 1 image
    check(648, 16, 16, 214, 3, 2, BSP_COL, 64, 32, 2, 64, 1);    // 31 and 13
    check(512, 4, 4, 512, 3, 1, BSP_DENSE, 0, 0, 1, 1024, 4);    // 50 and 14 at 4
    check(516, 7, 10, 163, 3, 2, BSP_PUNCHED, 64, 16, 2, 256, 1);   // 26 and 12
    check(454, 25, 25, 24, 1, 1, BSP_COL, 64, 64, 4, 1, 64);     // 24 and 11 at 64
    check(214, 63, 63, 41, 1, 1, BSP_COL, 32, 32, 2, 1, 64);     // 68 and 32
    check(512, 62, 58, 287, 1, 1, BSP_COL, 16, 32, 4, 1, 16);    // 76 and 44 at 16
    check(3960, 0, 0, 424, 0, 1, BSP_COL, 64, 32, 4, 1, 554);    // 17 and 12 at 554 vectors
    printf("%d faults\n", bad);
    return bad;
}
