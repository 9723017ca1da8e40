// Enumerates what the kernel of 3-wide convs reads of its input, on the host: every unit of
// every tile of a grid of layers, at every place a chunk may start, with the planner and the
// address arithmetic that the kernel uses.  Prints the layers whose element-wise path does not
// cover a read outside x, and returns how many there are.
#include <cstdio>

#include "bsp_common.h"

using namespace bsp;

namespace {

int bad = 0, n_layers = 0, n_far = 0;   // far: layers with a column group before the image and three chunks

void check(int cin, int h, int w, int kh, int sh, int sw, int ph, int pw, const bsp_scheme &s) {
    const bsp_conv_shape c = {1, cin, h, w, kh, 3, sh, sw, ph, pw};
    Plan p;
    if (make_plan(&s, &c, BSP_BF16, 0, &p) != BSP_OK || !p.cv) return;
    ++n_layers;
    n_far += pw > 1 && p.cv_nch > 2;
    const int NE = 4 * sw;
    for (int n = 1; n <= 2; ++n) {
        CvArgs a;
        memset(&a, 0, sizeof(a));
        cv_geometry(p, n, &a);
        const int groups = n * p.Ho * p.GPR;
        for (int TG : {8, 16, 32, 64, 128, (4 * p.NT) << p.lg_wp})   // the tiles the launcher may choose
            for (int G0 = 0; G0 < groups; G0 += TG) {
                const int g0 = G0 / p.GPR, g1 = (std::min(G0 + TG, groups) - 1) / p.GPR;
                const int img0 = g0 / p.Ho, img1 = g1 / p.Ho;
                const int edge = cv_edge(a, img0, g0 - img0 * p.Ho, img1, g1 - img1 * p.Ho, NE);
                for (int g = g0; g <= g1; ++g)
                    for (int r = 0; r < kh; ++r) {
                        const int img = g / p.Ho, ih = (g - img * p.Ho) * sh - ph + r;
                        const bool live = ih >= 0 && ih < h;
                        const int row = img * cin * a.x_cs + ih * w;
                        for (int oc = 0; oc < p.GPR; ++oc)
                            for (int ch = 0; ch < p.CC; ch = ch + 1 < p.CC ? p.CC - 1 : p.CC) {
                                const uint32_t off =
                                    live ? cv_off(a, row, ch, cv_col0(a, oc, NE), NE) : (uint32_t)a.shift;
                                // a read moves with the chunk, so the ends of the range decide
                                for (int cf = 0; cf <= cin - p.CC; cf = cf + 9 < cin - p.CC && cf > 8 ? cin - p.CC - 8 : cf + 1) {
                                    if (cv_safe(a, edge, cf, NE)) continue;
                                    const int64_t at = 2 * cv_first(a, 0, cf) + (uint32_t)(off * 2u);   // bytes
                                    if (at >= 0 && at + 2 * NE <= 2 * a.x_total && at == 2 * cv_first(a, off, cf)) continue;
                                    if (bad++ < 10)
                                        printf("cin %d %dx%d kh %d s %d p %d,%d n %d: row %d group %d channel %d + %d: byte %lld\n",
                                               cin, h, w, kh, sw, ph, pw, n, g, oc, cf, ch, (long long)at);
                                }
                            }
                    }
            }
    }
}

}  // namespace

int main() {
    for (int cin : {1, 2, 17, 64, 256})
        for (int hw : {3, 7, 14, 30})
            for (int w : {1, hw, hw + 3})
                for (int kh : {1, 3})
                    for (int sw : {1, 2})
                        for (int pw : {1, 2, 3, 5, 12, 40})
                            for (int bw : {16, 0}) {
                                const int ph = pw > 12 ? 12 : pw / 2;
                                if (w + 2 * pw < 3 || hw + 2 * ph < kh) continue;
                                bsp_scheme s;
                                memset(&s, 0, sizeof(s));
                                s.rows = 64; s.cols = cin * kh * 3; s.bh = 16; s.bw = bw; s.rate = 4; s.khw = kh * 3;
                                for (int reg : {BSP_DENSE, BSP_COL, BSP_PUNCHED}) {
                                    s.regularity = reg;
                                    check(cin, hw, w, kh, sw, sw, ph, pw, s);
                                }
                            }
    printf("%d layers, %d with far columns, %d reads outside x\n", n_layers, n_far, bad);
    return bad ? 1 : n_layers < 1000 || n_far < 50 ? 2 : 0;
}
