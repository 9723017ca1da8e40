// Forward kernel of bf16 convolutions with 3-wide filters at stride 1 or 2 and padding
// (template; instantiated in bsp_cv_*.hip): implicit GEMM over the kept columns only
// (Sec. 4.2, Sec. 4.3), with output pixels as the MFMA rows and filters as its columns.
//
//  * A workgroup (8 waves) computes a tile of 16 NT x 2^lg_wp output pixels (in groups of
//    4 adjacent pixels of one output row) for TM x 8 / 2^lg_wp m-tiles of 16 filters.  A
//    wave owns NT pixel tiles of 16 and TM m-tiles.
//  * The K loop walks chunks: ranges of at most SMAX 32-wide steps whose kept columns
//    fall in CC consecutive input channels.  The patch of a chunk holds, per channel and
//    filter column s, the tile's input rows as output column ow needs them:
//    T_s[row][ow] = x[row][ow * SW + s - PW], zero outside the image.  So every read of
//    the multiply is aligned, at any image width, padding and stride.
//  * A unit stages 4 output columns of one channel and row: it loads its own 4 or 8 input
//    columns once and takes the columns beside them from the neighbouring lanes, so an
//    input element is loaded once for its three copies.  Which units a thread stages is
//    the same in every chunk (each chunk stages CC channels): offsets are computed once,
//    the chunk only moves the scalar base.  Rows outside the image are zeroed once.
//  * A step's 16-pixel operand (32 kept columns x 16 pixels) is read with two
//    transposing LDS reads: lane i of 16 names the row of kept column i / 4 and pixel
//    group i % 4, and gets four kept columns of its own pixel.  A lane decodes one gather
//    offset per read and nothing is re-packed.
//  * A chunk's weights and offsets go straight to registers, issued after the next chunk's
//    input so that waiting for the input leaves them in flight.  Two workgroups share a
//    CU: one stages while the other multiplies.
//  * Epilogue: a lane holds 4 adjacent pixels of one filter per pixel tile; where rows are
//    whole groups its tiles are 8 adjacent pixels (16-byte stores).  16 pixels a lane are
//    no better: 56-wide rows 5% faster, 14-wide rows 10% slower (bank conflicts).
//
// What bounds it: no unit is saturated (128 -> 128 at 28x28, 64 images, 23 us: VALU issue
// 8 us, LDS 6 us of which half bank conflicts, input loads 6 us, MFMA 1.5 us); a chunk's
// chain of load, staging, barrier and multiply is what is left, so many waves per CU beat
// large tiles per wave (4 waves of 2 x 8 tiles per workgroup: 30 us).  Measured against
// the general kernel that ran these layers before (batch 64, cold cache; 16x32 column
// blocks 4x unless said): 64 at 56x56 57 -> 40 us, 128 at 28x28 53 -> 24, 256 at 14x14
// 45 -> 25, 512 at 7x7 72 -> 32, 128 at 56x56 stride 2 75 -> 36, 256 at 28x28 stride 2
// 69 -> 29, 512 at 14x14 stride 2 80 -> 30, 32x32 punched 256 at 56x56 477 -> 218, dense
// 256 at 56x56 682 -> 375; the 8x16 column layers at 8x of 32 images from 16-25 to 8-13.
#pragma once

#include "bsp_fwd.h"

namespace bsp {
namespace cv {

using fwd::epi;
using fwd::f32_to_bf16_rne;
using fwd::lds_addr;
using fwd::pk_bf16;
using fwd::uni;

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kNone = -2147483647 - 1;   // slot of an input row outside the image

// A unit stages the input of 4 output columns of one channel and input row: it loads its
// own 4 SW input columns (ND dwords) and takes the columns beside them from the units of
// the neighbouring lanes.
template <int SW>
struct Own {
    static constexpr int ND = 2 * SW, NE = 4 * SW;
};

template <int ND>
struct __attribute__((packed, aligned(2))) Raw {
    uint32_t d[ND];
};

__device__ __forceinline__ void barrier_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The value of the lane below / above (0 past the ends of the wave).
__device__ __forceinline__ uint32_t lane_below(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, true);   // wave_shr:1
}
__device__ __forceinline__ uint32_t lane_above(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xf, 0xf, true);   // wave_shl:1
}
// Stores a run of SP 4-pixel groups of one filter, k_cv's and k_p1's: o rounded to bf16, or fp32
// from element `at` on.  ybase, nval: element offset of each group in filter 0 and its valid
// pixels; yrow: offset of the filter; whole: the groups are whole and contiguous in memory.
template <int SP>
__device__ __forceinline__ void store_run(void *yv, bool bf16, int64_t at, const float (&o)[SP][4], const int *ybase,
                                          const int *nval, int yrow, bool whole) {
    if (bf16) {
        uint32_t w[SP][2];
#pragma unroll
        for (int t = 0; t < SP; ++t) {
            w[t][0] = pk_bf16(o[t][0], o[t][1]);
            w[t][1] = pk_bf16(o[t][2], o[t][3]);
        }
        if (whole) {
            uint16_t *y = (uint16_t *)yv + (uint32_t)(ybase[0] + yrow);
#pragma unroll
            for (int t = 0; t < SP; t += 2) {
                const Raw<4> v = {{w[t][0], w[t][1], w[t + 1][0], w[t + 1][1]}};
                *(Raw<4> *)(y + 4 * t) = v;
            }
        } else {
#pragma unroll
            for (int t = 0; t < SP; ++t) {
                uint16_t *y = (uint16_t *)yv + (uint32_t)(ybase[t] + yrow);
                if (nval[t] == 4) {
                    const Raw<2> v = {{w[t][0], w[t][1]}};
                    *(Raw<2> *)y = v;
                } else {
                    if (nval[t] > 0) y[0] = (uint16_t)w[t][0];
                    if (nval[t] > 1) y[1] = (uint16_t)(w[t][0] >> 16);
                    if (nval[t] > 2) y[2] = (uint16_t)w[t][1];
                }
            }
        }
    } else {
#pragma unroll
        for (int t = 0; t < SP; ++t) {
            float *y = (float *)yv + at + (uint32_t)(ybase[t] + yrow);
            if (nval[t] == 4) {
                struct __attribute__((packed, aligned(4))) F4 { float f[4]; };
                const F4 v = {{o[t][0], o[t][1], o[t][2], o[t][3]}};
                *(F4 *)y = v;
            } else {
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    if (i < nval[t]) y[i] = o[t][i];
            }
        }
    }
}

// All ones when bit i of v is set, else 0.
__device__ __forceinline__ uint32_t bit_mask(uint32_t v, int i) { return (uint32_t)__builtin_amdgcn_sbfe((int)v, i, 1); }
__device__ __forceinline__ uint32_t half_mask(uint32_t v, int i) {   // halves by bits i and i + 1
    return (bit_mask(v, i) & 0xffffu) | (bit_mask(v, i + 1) & 0xffff0000u);
}

template <int SW, int TM, int TPG, int NT, bool MAP>
__global__ __launch_bounds__(kCvThreads, cv_wps(TM, NT)) void k_cv(CvArgs a) {
    constexpr int GW = TM / TPG;              // lists of a wave
    constexpr int SMAX = cv_smax(TM, NT);         // steps of a chunk
    constexpr int UPT = cv_upt(SW);           // units a thread holds
    constexpr int ND = Own<SW>::ND, NE = Own<SW>::NE;
    extern __shared__ __attribute__((aligned(256))) unsigned char lds[];
    __shared__ int s_rowbase[kMaxTileRows];
    __shared__ int s_slot[kMaxSlots];

    const int per = gridDim.x >> 3;
    const int lid = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (lid >= a.grid_valid) return;
    const int pt = (int)fdiv((uint32_t)lid, a.div_nmb);
    const int mb = lid - pt * a.n_mb;

    const TileHeader *hdr = (const TileHeader *)a.tiles;
    const bool ok = hdr->magic == kMagic && hdr->fp_lo == a.fp_lo && hdr->fp_hi == a.fp_hi;
    const int nch = ok ? uni(hdr->n_chunks) : 0;
    const const_int *table = (const const_int *)(a.tiles + a.off_chunks);
    const unsigned char *A_g = a.tiles + a.off_a;
    const uint32_t *desc = (const uint32_t *)(a.tiles + a.off_desc16);

    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int wp = wave & ((1 << a.lg_wp) - 1), wm = wave >> a.lg_wp;
    const int mt0 = mb * a.MBT + wm * TM;     // the wave's first m-tile
    int grp[GW];                              // its lists
#pragma unroll
    for (int g = 0; g < GW; ++g) grp[g] = a.n_groups == 1 ? 0 : (mt0 + g * TPG) / a.mt_per_group;

    // ---- weights and gather offsets of a chunk (always SMAX steps; steps past the end
    // repeat the last one and are not multiplied) ----
    uint4 wr[SMAX][TM];
    uint32_t of[SMAX][GW];
    auto load_w = [&](int4 cd) {
#pragma unroll
        for (int k = 0; k < SMAX; ++k) {
            const int s = min(cd.x + k, cd.y - 1);
#pragma unroll
            for (int g = 0; g < GW; ++g)
                of[k][g] = desc[(size_t)(grp[g] * a.S + s) * 16 + (lane >> 4) * 4 + ((lane >> 2) & 3)];
#pragma unroll
            for (int t = 0; t < TM; ++t)
                wr[k][t] = *(const uint4 *)(A_g + ((size_t)(mt0 + t) * a.S + s) * 1024 + lane * 16);
        }
    };

    // ---- the tile's output rows, staged input rows (slots) and unit table ----
    const int TG = (4 * NT) << a.lg_wp;
    const int G0 = pt * TG;
    const int G1 = min(G0 + TG, a.n_groups_total) - 1;
    const int g0 = (int)fdiv((uint32_t)G0, a.div_GPR), g1 = (int)fdiv((uint32_t)G1, a.div_GPR);
    const int nrows = g1 - g0 + 1;
    const int img0 = (int)fdiv((uint32_t)g0, a.div_Ho);
    const int kl = (int)fdiv((uint32_t)g1, a.div_Ho) - img0;   // image boundaries crossed
    const int rstep = min(a.SH, a.KH);
    const int used = (nrows - 1 - kl) * rstep + kl * a.KH + a.KH;   // slots of this tile
    if (tid < nrows) {
        const int g = g0 + tid;
        const int img = (int)fdiv((uint32_t)g, a.div_Ho), oh = g - img * a.Ho;
        const int k = img - img0;
        const int base = (tid - k) * rstep + k * a.KH;
        for (int r = 0; r < a.KH; ++r) {
            const int ih = oh * a.SH - a.PH + r;
            s_slot[base + r] = ih >= 0 && ih < a.H ? img * a.Cin * a.x_cs + ih * a.W : kNone;
        }
        s_rowbase[tid] = base;
    }
    barrier_lds();
    const int UC = used * a.GPR;       // units of a channel
    const int n_units = a.CC * UC;     // units of a chunk (every chunk stages CC channels)
    // unit -> channel by a float multiply: exact, since u + 1/2 is at least 1 / (2 UC) off
    // every multiple of UC and u < 2^20
    const float rUC = 1.f / (float)UC;
    unsigned char *patch = lds;
    // A wave handles 62 units per round in lanes 1 .. 62; lanes 0 and 63 load the units
    // beside them for their neighbours.  unit(i): offset of the unit's own input columns at
    // the chunk's first channel (cv_off), LDS offset of its copies (-1: not written), and
    // which of its own columns, and the ones below and above them, lie in the image.
    auto unit = [&](int i, uint32_t &off, int &dst, uint32_t &own, uint32_t &below, uint32_t &above) {
        const int uu = (i * kCvWaves + wave) * 62 + lane - 1;
        const int u = min(max(uu, 0), n_units - 1);
        const int c = (int)(((float)u + 0.5f) * rUC), r = u - c * UC;
        const int slot = (int)fdiv((uint32_t)r, a.div_GPR), oc = r - slot * a.GPR;
        const int so = s_slot[slot];
        const int col0 = cv_col0(a, oc, NE);
        const bool live = so != kNone;
        off = live ? cv_off(a, so, c, col0, NE) : (uint32_t)a.shift;
        dst = (c * a.CH_STRIDE + 4 * r) * 2;
        own = 0;
        if (a.mask_own) {   // columns max(0, -col0) .. min(NE, W - col0) - 1 of the unit
            const int lo = max(0, -col0), hi = min(NE, a.W - col0);
            own = hi > lo ? (1u << hi) - (1u << lo) : 0u;
        }
        below = oc > 0;
        above = oc + 1 < a.GPR;
        const bool mine = uu == u && lane != 0 && lane != 63;
        if (mine && !live) {   // a row outside the image: zeros, written once
#pragma unroll
            for (int k = 0; k < 3; ++k) *(uint2 *)(patch + dst + 2 * k * a.VS) = make_uint2(0u, 0u);
        }
        if (!mine || !live) dst = -1;
    };
    // the units held in registers: offset, LDS offset, flags (own: NE bits of NPW units per word)
    constexpr int NPW = 32 / NE;
    uint32_t u_off[UPT];
    int u_dst[UPT];
    uint32_t f_own[(UPT + NPW - 1) / NPW] = {}, f_below = 0, f_above = 0;
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
        uint32_t own, be, ab;
        unit(i, u_off[i], u_dst[i], own, be, ab);
        f_own[i / NPW] |= own << (i % NPW * NE);
        f_below |= be << i;
        f_above |= ab << i;
    }
    Raw<ND> st[UPT];
    // input of one unit (xc: `shift` elements before x at the chunk's first channel)
    auto load_fast = [&](const uint16_t *xc, uint32_t off) { return *(const Raw<ND> *)((const char *)xc + off * 2u); };
    auto load_safe = [&](int c_first, uint32_t off) {
        Raw<ND> v;
        const int64_t e = cv_first(a, off, c_first);
        if (e >= 0 && e + NE <= a.x_total) {
            const Raw<ND> w = *(const Raw<ND> *)(a.x + e);
#pragma unroll
            for (int d = 0; d < ND; ++d) v.d[d] = w.d[d];
        } else {
#pragma unroll
            for (int d = 0; d < ND; ++d) {
                const uint32_t lo = e + 2 * d >= 0 && e + 2 * d < a.x_total ? a.x[e + 2 * d] : 0;
                const uint32_t hi = e + 2 * d + 1 >= 0 && e + 2 * d + 1 < a.x_total ? a.x[e + 2 * d + 1] : 0;
                v.d[d] = lo | hi << 16;
            }
        }
        return v;
    };
    // the three copies of a unit: T_s[ow] = x[ow SW + s - PW]
    auto put = [&](const Raw<ND> &v, int dst, uint32_t own, uint32_t below, uint32_t above) {
        uint32_t d[ND];
#pragma unroll
        for (int j = 0; j < ND; ++j) d[j] = a.mask_own ? v.d[j] & half_mask(own, 2 * j) : v.d[j];
        const uint32_t lo = lane_below(d[ND - 1]) & below;
        uint2 t0, t1, t2;
        if constexpr (SW == 1) {
            const uint32_t hi = lane_above(d[0]) & above;
            const uint32_t mid = __builtin_amdgcn_alignbyte(d[1], d[0], 2);
            t0 = make_uint2(__builtin_amdgcn_alignbyte(d[0], lo, 2), mid);
            t1 = make_uint2(d[0], d[1]);
            t2 = make_uint2(mid, __builtin_amdgcn_alignbyte(hi, d[1], 2));
        } else {
            t0 = make_uint2(fwd::perm(d[0], lo, 0x07060302u), fwd::perm(d[2], d[1], 0x07060302u));
            t1 = make_uint2(fwd::perm(d[1], d[0], 0x05040100u), fwd::perm(d[3], d[2], 0x05040100u));
            t2 = make_uint2(fwd::perm(d[1], d[0], 0x07060302u), fwd::perm(d[3], d[2], 0x07060302u));
        }
        if (dst >= 0) {
            *(uint2 *)(patch + dst) = t0;
            *(uint2 *)(patch + dst + 2 * a.VS) = t1;
            *(uint2 *)(patch + dst + 4 * a.VS) = t2;
        }
    };
    auto write_x = [&](int c_first, bool safe) {
#pragma unroll
        for (int i = 0; i < UPT; ++i)
            put(st[i], u_dst[i], f_own[i / NPW] >> (i % NPW * NE), bit_mask(f_below, i), bit_mask(f_above, i));
        // units past the registers (lists whose steps span many channels)
        for (int i = UPT; i * kCvRound < n_units; ++i) {
            int dst;
            uint32_t off, own, be, ab;
            unit(i, off, dst, own, be, ab);
            const Raw<ND> v = safe ? load_safe(c_first, off) : load_fast(a.x + cv_first(a, 0, c_first), off);
            put(v, dst, own, (uint32_t)-(int)be, (uint32_t)-(int)ab);
        }
    };

    // ---- the lane's pixel groups.  Rows of whole groups: tile t's group q is group q SP + t
    // of a run of 4 SP, so that a lane of the output holds SP consecutive groups; other rows:
    // group 4 t + q, whose reads conflict less.  Byte offset of the group that the lane
    // names in tile t's reads (q = lane % 4) ----
    constexpr int SP = 2;
    const int Gw = G0 + wp * (4 * NT);
    const bool runs = (a.Wo & 3) == 0;
    auto group = [&](int t, int q) { return Gw + t / SP * (4 * SP) + (runs ? q * SP + t % SP : t % SP * 4 + q); };
    const uint32_t patch0 = lds_addr(patch);
    uint32_t pixb[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int G = min(group(t, lane & 3), G1);
        const int row = (int)fdiv((uint32_t)G, a.div_GPR);
        pixb[t] = patch0 + (uint32_t)((s_rowbase[row - g0] * a.GPR + (G - row * a.GPR)) * 8);
    }

    f32x4 acc[TM][NT];
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto compute = [&](int ns) {
#pragma unroll
        for (int k = 0; k < SMAX; ++k) {
            if (k >= ns) break;
#pragma unroll
            for (int g = 0; g < GW; ++g) {
                const uint32_t o0 = (of[k][g] & 0xffffu) << 1, o1 = (of[k][g] >> 16) << 1;
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(uintptr_t)(pixb[t] + o0));
                    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(uintptr_t)(pixb[t] + o1));
                    const s16x8 f = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                    for (int i = 0; i < TPG; ++i)
                        acc[g * TPG + i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            f, __builtin_bit_cast(s16x8, wr[k][g * TPG + i]), acc[g * TPG + i][t], 0, 0, 0);
                }
            }
        }
    };

    const int edge = uni(cv_edge(a, img0, g0 - img0 * a.Ho, img0 + kl, g1 - (img0 + kl) * a.Ho, NE));
    const uint16_t *x0 = a.x - a.shift;   // unit offsets count from here (cv_first)
    // Pipeline over the chunks: the input of chunk c is loaded while chunk c - 1
    // multiplies, then its weights (waiting for the input leaves them in flight).
    int4 cp = make_int4(0, 0, 0, 0);
    for (int c = 0; c <= nch; ++c) {
        // the units' values stay as they are held: derived ones, hoisted out of the loop,
        // would not fit the registers
#pragma unroll
        for (int i = 0; i < UPT; ++i) asm volatile("" : "+v"(u_off[i]), "+v"(u_dst[i]));
        asm volatile("" : "+v"(f_below), "+v"(f_above));
        int4 cd = cp;
        bool safe = false;
        if (c < nch) {
            cd = fwd::chunk_at(table, c);
            safe = edge != 0 && cv_safe(a, edge, cd.z, NE);
            if (safe) {
#pragma unroll
                for (int i = 0; i < UPT; ++i) st[i] = load_safe(cd.z, u_off[i]);
            } else {
                const uint16_t *xc = x0 + (int64_t)cd.z * a.x_cs;
#pragma unroll
                for (int i = 0; i < UPT; ++i) st[i] = load_fast(xc, u_off[i]);
            }
        }
        if (c > 0) compute(cp.y - cp.x);
        if (c == nch) break;
        load_w(cd);
        barrier_lds();   // everyone is done with the patch
        write_x(cd.z, safe);
        barrier_lds();
        cp = cd;
    }

    // ---- bias, ReLU, rounding, stores: lane = filter lane % 16, pixel group lane / 16 ----
    const float qnan = __builtin_nanf("");
    // element offset of the groups in filter 0 and their valid pixels (0: none); whole: the
    // SP groups of run r are consecutive whole groups of one image, contiguous in memory
    int ybase[NT], nval[NT];
    bool whole[NT / SP];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int G = group(t, lane >> 4);
        const int row = (int)fdiv((uint32_t)min(G, G1), a.div_GPR);
        const int ow = 4 * (min(G, G1) - row * a.GPR);
        const int img = (int)fdiv((uint32_t)row, a.div_Ho), oh = row - img * a.Ho;
        nval[t] = G > G1 ? 0 : min(4, a.Wo - ow);
        ybase[t] = (int)(img * a.Rout * a.y_cs) + oh * a.Wo + ow;   // y holds fewer than 2^31 elements
        if (t % SP == SP - 1) whole[t / SP] = runs && ybase[t] == ybase[t - SP + 1] + 4 * (SP - 1) && nval[t] == 4;
    }
#pragma unroll
    for (int m = 0; m < TM; ++m) {
        const int gm = mt0 + m;
        const int gidx = a.n_groups == 1 ? 0 : gm / a.mt_per_group;
        const int rig = (gm - gidx * a.mt_per_group) * kMT + (lane & 15);
        const int crow = gidx * a.group_rows + rig;
        const bool row_ok = rig < a.group_rows && crow < a.R;
        if (!row_ok) continue;
        int orow = crow;
        if constexpr (MAP) orow = ok ? min(max(a.rowmap[crow], 0), a.Rout - 1) : min(crow, a.Rout - 1);
        const float bv = a.bias ? a.bias[orow] : 0.f;
        const int yrow = orow * (int)a.y_cs;
#pragma unroll
        for (int r = 0; r < NT / SP; ++r) {
            float o[SP][4];
#pragma unroll
            for (int t = 0; t < SP; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) o[t][i] = ok ? epi(acc[m][r * SP + t][i], bv, a.relu) : qnan;
            store_run<SP>(a.y, a.out_bf16, 0, o, ybase + r * SP, nval + r * SP, yrow, whole[r]);
        }
    }
}

typedef void (*cv_fn)(CvArgs);

template <int SW, int NT>
cv_fn cv_pick(int TM, int TPG, bool map) {
    if (map && TPG != TM) return nullptr;
    switch (TM * 16 + TPG) {
        case 0x11: return map ? k_cv<SW, 1, 1, NT, true> : k_cv<SW, 1, 1, NT, false>;
        case 0x21: if constexpr (2 * NT <= kCvMaxAcc) return k_cv<SW, 2, 1, NT, false>; return nullptr;
        case 0x22:
            if constexpr (2 * NT <= kCvMaxAcc) return map ? k_cv<SW, 2, 2, NT, true> : k_cv<SW, 2, 2, NT, false>;
            return nullptr;
        case 0x41: if constexpr (4 * NT <= kCvMaxAcc) return k_cv<SW, 4, 1, NT, false>; return nullptr;
        case 0x42: if constexpr (4 * NT <= kCvMaxAcc) return k_cv<SW, 4, 2, NT, false>; return nullptr;
        case 0x44:
            if constexpr (4 * NT <= kCvMaxAcc) return map ? k_cv<SW, 4, 4, NT, true> : k_cv<SW, 4, 4, NT, false>;
            return nullptr;
        default: return nullptr;
    }
}

}  // namespace cv
}  // namespace bsp
