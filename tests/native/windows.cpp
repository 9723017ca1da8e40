// Steps of drawn column lists against the channel windows of their plans, on the host: the
// kernels that stage a window per chunk (3-wide convs, pointwise layers) hold every step, for
// kept columns anywhere in their blocks and at either end of the input.  Prints the layers
// whose pack would be refused, and returns how many there are.
#include <cstdio>
#include <random>
#include <vector>

#include "bsp_common.h"

using namespace bsp;

namespace {

int bad = 0, n_windowed = 0, n_whole = 0;
std::mt19937 rng(5);

// Kept columns of one block-row: `k` of every block of `bw` columns (of every `khw` locations
// of a channel when punched, the same locations in a block of channels).  place 0: anywhere;
// 1: the first ones of the block; 2: the last ones; 3: both ends; 4: by turns 1 and 2.
std::vector<int> columns(const Plan &p, int place, int row) {
    std::vector<int> out;
    const bool punched = p.reg == BSP_PUNCHED;
    const int unit = punched ? p.khw : 1, width = p.C / unit;
    for (int b = 0; b < p.nbc; ++b) {
        const int c0 = b * p.bw_eff, cn = std::min(width, c0 + p.bw_eff) - c0;
        const int n = punched ? p.khw : cn, k = kept_count(n, p.rate);
        std::vector<char> keep(n, 0);
        const int how = place == 4 ? 1 + (b + row) % 2 : place;
        for (int i = 0; i < k; ++i) {
            if (how == 0) {
                int q;
                do q = (int)(rng() % (uint32_t)n); while (keep[q]);
                keep[q] = 1;
            } else {
                keep[how == 1 ? i : how == 2 ? n - 1 - i : i % 2 ? n - 1 - i / 2 : i / 2] = 1;
            }
        }
        if (punched) {
            for (int c = c0; c < c0 + cn; ++c)
                for (int q = 0; q < n; ++q)
                    if (keep[q]) out.push_back(c * p.khw + q);
        } else {
            for (int q = 0; q < n; ++q)
                if (keep[q]) out.push_back(c0 + q);
        }
    }
    return out;
}

void check(const bsp_scheme &s, const bsp_conv_shape *c) {
    Plan p;
    if (make_plan(&s, c, BSP_BF16, 0, &p) != BSP_OK || p.shared || p.im2col || !(p.cv || p.p1)) return;
    ++n_windowed;
    n_whole += p.CC == p.Cin;
    const int khw = p.KH * p.KW;
    for (int place = 0; place < 5; ++place) {
        std::vector<std::vector<int>> lists;
        for (int i = 0; i < p.nbr; ++i) lists.push_back(columns(p, place, i));
        for (int st = 0; st < p.S; ++st) {
            int lo = 1 << 30, hi = -1;
            for (const auto &l : lists) {
                if ((int)l.size() != p.L) { printf("list of %d, planned %d\n", (int)l.size(), p.L); ++bad; return; }
                lo = std::min(lo, l[32 * st] / khw);
                hi = std::max(hi, l[std::min(p.L, 32 * st + 32) - 1] / khw);
            }
            if (hi - std::min(lo, p.Cin - p.CC) + 1 <= p.CC) continue;
            if (bad++ < 10)
                printf("%d x %d, blocks %d x %d, regularity %d, 1/%d, %dx%d image, place %d: step %d spans %d channels of %d\n",
                       p.R, p.C, s.bh, s.bw, s.regularity, s.rate, p.H, p.W, place, st, hi - lo + 1, p.CC);
            break;
        }
    }
}

}  // namespace

int main() {
    for (int cin : {16, 60, 130, 512, 1024})
        for (int bw : {0, 16, 36, 300})
            for (int rate : {2, 4, 8})
                for (int reg : {BSP_COL, BSP_ROWCOL, BSP_PUNCHED})
                    for (int k : {0, 1, 3})
                        for (int hw : {4, 7, 14, 30})
                            for (int stride : {1, 2}) {
                                bsp_scheme s;
                                memset(&s, 0, sizeof(s));
                                s.rows = 96; s.cols = cin * (k ? k * k : 1); s.bh = 32; s.bw = bw; s.rate = rate;
                                s.regularity = reg; s.khw = reg == BSP_PUNCHED ? std::max(k * k, 1) : 1;
                                const bsp_conv_shape c = {1, cin, hw, hw, k, k, stride, stride, k / 2, k / 2};
                                check(s, k ? &c : nullptr);
                            }
    // a filter too tall for a staged tile: planned over its im2col input, not refused
    bsp_scheme s;
    memset(&s, 0, sizeof(s));
    s.rows = 16; s.cols = 299 * 3; s.rate = 1; s.regularity = BSP_DENSE;
    const bsp_conv_shape tall = {1, 1, 300, 8, 299, 3, 1, 1, 0, 1};
    Plan p;
    if (make_plan(&s, &tall, BSP_BF16, 0, &p) != BSP_OK || !p.im2col) { printf("299 x 3 refused\n"); ++bad; }
    printf("%d windowed plans (%d of the whole input), %d refused\n", n_windowed, n_whole, bad);
    return bad ? 1 : n_windowed < 500 ? 2 : 0;
}
