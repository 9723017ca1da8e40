// 3-wide lists of block-rows shorter than half an m-tile, on the host: k_cv runs them as
// lists or stored with zeros, each where it measured better (64 images and 4 images).
#include <cstdio>
#include <cstring>

#include "bsp_common.h"

using namespace bsp;

int main() {
    const struct {
        int cin, hw, stride, reg, bh, bw, rate, zeros;
    } layers[] = {
        // us at 64 and 4 images, lists against zeros
        {256, 56, 1, BSP_COL, 4, 4, 4, 1},        // 798, 375 at 64
        {64, 56, 1, BSP_COL, 4, 4, 4, 1},         // 84, 43; 12, 15
        {64, 56, 1, BSP_COL, 2, 32, 4, 1},        // 186, 43; 17, 15
        {64, 56, 1, BSP_PUNCHED, 4, 32, 4, 1},    // 89, 43; 12, 15
        {128, 28, 1, BSP_COL, 4, 4, 4, 1},        // 77, 35; 13, 16
        {256, 28, 2, BSP_COL, 2, 32, 4, 1},       // 118, 44; 18, 27
        {64, 56, 1, BSP_COL, 8, 32, 4, 0},        // 54, 43; 10, 15
        {128, 28, 1, BSP_COL, 8, 32, 4, 0},       // 40, 35; 11, 16
        {43, 46, 1, BSP_PUNCHED, 8, 32, 4, 0},    // to 663; one image 13, 23
        {256, 14, 1, BSP_COL, 4, 4, 4, 0},        // 56, 47; 13, 28
        {512, 7, 1, BSP_COL, 4, 4, 4, 0},         // 48, 84; 20, 56
        {256, 56, 1, BSP_COL, 16, 32, 2, 0},      // full tiles
    };
    int bad = 0;
    for (const auto &l : layers) {
        bsp_scheme s;
        std::memset(&s, 0, sizeof(s));
        s.rows = l.cin == 43 ? 663 : l.cin; s.cols = 9 * l.cin; s.bh = l.bh; s.bw = l.bw;
        s.regularity = (bsp_regularity)l.reg; s.rate = l.rate; s.khw = 9;
        const bsp_conv_shape c = {64, l.cin, l.hw, l.hw, 3, 3, l.stride, l.stride, 1, 1};
        Plan p;
        if (make_plan(&s, &c, BSP_BF16, 0, &p) == BSP_OK && p.cv && p.shared == l.zeros) continue;
        ++bad;
        printf("%d at %dx%d, stride %d, regularity %d, %dx%d blocks, 1/%d: %s\n", l.cin, l.hw, l.hw, l.stride, l.reg,
               l.bh, l.bw, l.rate, p.shared ? "zeros" : "lists");
    }
    return bad;
}
