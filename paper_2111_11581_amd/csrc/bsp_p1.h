// Forward kernel of bf16 pointwise layers (1x1 convolutions without padding at stride 1
// or 2, fully connected layers; Sec. 4.2: the GEMM form of a 1x1 layer has one column per
// input channel).  Template; instantiated in bsp_p1_*.hip.
//
// As the kernel of 3-wide convs (bsp_cv.h), with output pixels as the MFMA rows and
// filters as its columns, for patches that need no shifted copies:
//  * output pixels are taken in groups of 4 (stride 1: of an image's run of pixels, two
//    groups per 16-byte granule; stride 2: of an output row); a workgroup (8 waves)
//    computes 16 NT x 2^lg_wp consecutive pixels for TM x 8 / 2^lg_wp m-tiles;
//  * a chunk's patch holds, per channel, the tile's pixels: a thread loads granules of one
//    position for channels a fixed distance apart, so it keeps one offset and the scalar
//    base moves; at stride 2 it keeps the even pixels of each granule;
//  * identity lists (IDENT: row blocks stored with zeros, dense and unstructured layers)
//    run SPC 32-channel steps per chunk and need no offsets; per-block-row lists take
//    chunks (windows of CC channels) and 16-bit offsets from the packed tables;
//  * two LDS buffers: the next chunk's input is in flight while this one multiplies, then
//    it is written to the other buffer; one barrier per chunk;
//  * a K loop split over ks workgroups stores fp32 partial sums (summed by k_splitk_sum).
//
// What bounds it: a chunk's chain of load, staging, barrier and multiply, and on layers that
// write much more than they read the stores: vector memory retires in order, so a wait for
// the next chunk's input also waits for the stores issued before it (64 -> 256 at 56x56, 103
// MB of output: 49 us where stores alone take 20; that layer stays with k_pw, 46 us).  One
// tile per workgroup and persistent workgroups measured about the same.  Against the kernels
// that ran these layers before (cold cache): stride 2, 64 images: 256 -> 512 at 56x56 82 ->
// 61 us, 512 -> 1024 at 28x28 63 -> 52; stride 1, 64 images: 512 -> 2048 at 7x7 27 -> 22, 5
// images: 256 -> 1024 at 14x14 20 -> 6.7.
#pragma once

#include "bsp_cv.h"

namespace bsp {
namespace p1 {

using cv::barrier_lds;
using cv::lds_s16x4;
using cv::Raw;
using cv::s16x4;
using fwd::epi;
using fwd::lds_addr;
using fwd::uni;

template <int SW, int TM, int TPG, int NT, bool MAP, bool IDENT>
__global__ __launch_bounds__(kCvThreads, cv_wps(TM, NT)) void k_p1(P1Args a) {
    constexpr int GW = TM / TPG;              // lists of a wave
    constexpr int SMAX = p1_smax(TM, NT);     // steps of a chunk
    constexpr int UPT = kP1Upt;               // granules a thread holds
    extern __shared__ __attribute__((aligned(256))) unsigned char lds[];

    const int per = gridDim.x >> 3;
    const int lid0 = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (lid0 >= a.grid_valid) return;
    const int kp = a.ks > 1 ? (int)fdiv((uint32_t)lid0, a.div_kpart) : 0;
    const int lid = lid0 - kp * a.kpart_wgs;
    const int jr = (int)fdiv((uint32_t)lid, a.div_nmb);   // walks tiles jr, jr + n_walk, ...
    const int mb = lid - jr * a.n_mb;

    const TileHeader *hdr = (const TileHeader *)a.tiles;
    const bool ok = hdr->magic == kMagic && hdr->fp_lo == a.fp_lo && hdr->fp_hi == a.fp_hi;
    const int nch_all = !ok ? 0 : IDENT ? (a.S + a.SPC - 1) / a.SPC : uni(hdr->n_chunks);
    const int c_begin = a.ks > 1 ? nch_all * kp / a.ks : 0, c_end = a.ks > 1 ? nch_all * (kp + 1) / a.ks : nch_all;
    const const_int *table = (const const_int *)(a.tiles + a.off_chunks);
    const unsigned char *A_g = a.tiles + a.off_a;
    const uint32_t *desc = (const uint32_t *)(a.tiles + a.off_desc16);

    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int wp = wave & ((1 << a.lg_wp) - 1), wm = wave >> a.lg_wp;
    const int mt0 = mb * a.MBT + wm * TM;     // the wave's first m-tile
    int grp[GW];                              // its lists
#pragma unroll
    for (int g = 0; g < GW; ++g) grp[g] = IDENT ? 0 : (mt0 + g * TPG) / a.mt_per_group;

    // chunk c: first step, end step, first channel
    auto chunk = [&](int c) {
        if constexpr (IDENT) return make_int4(c * a.SPC, min((c + 1) * a.SPC, a.S), c * a.SPC * kKS, 0);
        else return fwd::chunk_at(table, c);
    };

    // ---- weights and gather offsets of a chunk (always SMAX steps; steps past the end
    // repeat the last one and are not multiplied) ----
    uint4 wr[SMAX][TM];
    uint32_t of[IDENT ? 1 : SMAX][GW];
    auto load_w = [&](int4 cd) {
#pragma unroll
        for (int k = 0; k < SMAX; ++k) {
            const int s = min(cd.x + k, cd.y - 1);
            if constexpr (!IDENT) {
#pragma unroll
                for (int g = 0; g < GW; ++g)
                    of[k][g] = desc[(size_t)(grp[g] * a.S + s) * 16 + (lane >> 4) * 4 + ((lane >> 2) & 3)];
            }
#pragma unroll
            for (int t = 0; t < TM; ++t)
                wr[k][t] = *(const uint4 *)(A_g + ((size_t)(mt0 + t) * a.S + s) * 1024 + lane * 16);
        }
    };

    // ---- staging: this thread's granule position of the tile and first channel ----
    const int TG = (4 * NT) << a.lg_wp;
    const int lgp = 2 + (NT == 2 ? 1 : NT == 4 ? 2 : 3) + a.lg_wp - (SW == 1 ? 1 : 0);   // log2 of the positions
    const int gpos = tid & ((1 << lgp) - 1), c0 = tid >> lgp;
    const int cstep = kCvThreads >> lgp;      // channels between a thread's granules
    const int n_it = (a.CC + cstep - 1) >> (9 - lgp);   // granules of a thread per chunk
    int off = 0;                              // its element offset at channel 0
    bool tail = false;                        // the tile's last channels may reach past x
    auto set_tile = [&](int pt) {
        const int G0 = pt * TG, G1 = min(G0 + TG, a.n_groups_total) - 1;
        const int G = min(G0 + gpos * (SW == 1 ? 2 : 1), SW == 1 ? G1 & ~1 : G1);
        const int row = (int)fdiv((uint32_t)G, a.div_GPR), gi = G - row * a.GPR;
        const int img = (int)fdiv((uint32_t)row, a.div_Ho), oh = row - img * a.Ho;
        off = img * a.x_is + oh * a.in_row + gi * 4 * SW;
        tail = G1 >= a.tail_group;
    };
    const uint32_t c_off = (uint32_t)(c0 * a.x_cs);
    uint32_t u_dst = (uint32_t)(c0 * a.CH_STRIDE + gpos * (SW == 1 ? 8 : 4)) * 2u;
    auto load_one = [&](int c_first, int i, bool safe) {
        // identity lists: channels past the last one hold zeros (their weights are zero)
        const int c = c_first + c0 + i * cstep;
        Raw<4> v = {{0, 0, 0, 0}};
        if (!safe) {
            v = *(const Raw<4> *)((const char *)(a.x + (int64_t)(c_first + i * cstep) * a.x_cs) + ((uint32_t)off + c_off) * 2u);
        } else if (c < a.Cin && c < c_first + a.CC) {
            const int64_t e = (int64_t)off + (int64_t)c * a.x_cs;
            if (e + 8 <= a.x_total) {
                v = *(const Raw<4> *)(a.x + e);
            } else {
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const uint32_t lo = e + 2 * d < a.x_total ? a.x[e + 2 * d] : 0;
                    const uint32_t hi = e + 2 * d + 1 < a.x_total ? a.x[e + 2 * d + 1] : 0;
                    v.d[d] = lo | hi << 16;
                }
            }
        }
        return v;
    };
    auto put = [&](unsigned char *buf, int i, const Raw<4> &v) {
        unsigned char *p = buf + u_dst + (uint32_t)(i * cstep * a.CH_STRIDE) * 2u;
        if (c0 + i * cstep >= a.CC) return;
        if constexpr (SW == 1) *(uint4 *)p = make_uint4(v.d[0], v.d[1], v.d[2], v.d[3]);
        else *(uint2 *)p = make_uint2(fwd::perm(v.d[1], v.d[0], 0x05040100u), fwd::perm(v.d[3], v.d[2], 0x05040100u));
    };
    Raw<4> st[UPT];
    // a chunk is loaded without checks when all its granules' channels exist inside x
    auto is_safe = [&](int4 cd) {
        const int after = a.Cin - cd.z - n_it * cstep;   // channels behind the ones loaded
        return after < 0 || (tail && (int64_t)after * a.x_cs < 8);
    };
    auto load_x = [&](int4 cd) {
        const bool safe = is_safe(cd);
#pragma unroll
        for (int i = 0; i < UPT; ++i)
            if (i < n_it) st[i] = load_one(cd.z, i, safe);
    };
    auto write_x = [&](int4 cd, unsigned char *buf) {
#pragma unroll
        for (int i = 0; i < UPT; ++i)
            if (i < n_it) put(buf, i, st[i]);
        for (int i = UPT; i < n_it; ++i) put(buf, i, load_one(cd.z, i, is_safe(cd)));   // past the registers
    };

    // ---- the lane's pixel groups (as in k_cv): tile t's group q ----
    constexpr int SP = 2;
    const bool runs = SW == 1 || (a.Wo & 3) == 0;
    const int Gw = wp * (4 * NT);
    auto group = [&](int t, int q) { return Gw + t / SP * (4 * SP) + (runs ? q * SP + t % SP : t % SP * 4 + q); };
    const uint32_t patch0 = lds_addr(lds);
    uint32_t pixb[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        pixb[t] = patch0 + (uint32_t)(group(t, lane & 3) * 8);
        if constexpr (IDENT) pixb[t] += (uint32_t)((8 * (lane >> 4) + ((lane >> 2) & 3)) * a.CH_STRIDE) * 2u;
    }

    f32x4 acc[TM][NT];
    auto clear = [&]() {
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    clear();

    auto compute = [&](int ns, uint32_t b) {
#pragma unroll
        for (int k = 0; k < SMAX; ++k) {
            if (k >= ns) break;
#pragma unroll
            for (int g = 0; g < GW; ++g) {
                uint32_t o0, o1;
                if constexpr (IDENT) {
                    o0 = b + (uint32_t)(k * kKS * a.CH_STRIDE) * 2u;
                    o1 = o0 + (uint32_t)(4 * a.CH_STRIDE) * 2u;
                } else {
                    o0 = b + ((of[k][g] & 0xffffu) << 1);
                    o1 = b + ((of[k][g] >> 16) << 1);
                }
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

    // ---- bias, ReLU, rounding, stores: lane = filter lane % 16, pixel group lane / 16 ----
    auto epilogue = [&](int pt) {
        const int G0 = pt * TG, G1 = min(G0 + TG, a.n_groups_total) - 1;
        const float qnan = __builtin_nanf("");
        const bool part = a.ks > 1;               // partial sums: fp32, no bias, ReLU or rounding
        const int64_t pbase = part ? (int64_t)kp * a.part_stride : 0;
        int ybase[NT], nval[NT];
        bool whole[NT / SP];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int G = G0 + group(t, lane >> 4);
            const int row = (int)fdiv((uint32_t)min(G, G1), a.div_GPR);
            const int ow = 4 * (min(G, G1) - row * a.GPR);
            const int img = (int)fdiv((uint32_t)row, a.div_Ho), oh = row - img * a.Ho;
            nval[t] = G > G1 ? 0 : min(4, a.Wo - ow);
            ybase[t] = img * a.y_is + oh * a.Wo + ow;   // y holds fewer than 2^31 elements
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
            const float bv = a.bias && !part ? a.bias[orow] : 0.f;
            const int yrow = orow * (int)a.y_cs;
#pragma unroll
            for (int r = 0; r < NT / SP; ++r) {
                float o[SP][4];
#pragma unroll
                for (int t = 0; t < SP; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        o[t][i] = !ok ? qnan : part ? acc[m][r * SP + t][i] : epi(acc[m][r * SP + t][i], bv, a.relu);
                cv::store_run<SP>(a.y, a.out_bf16 && !part, pbase, o, ybase + r * SP, nval + r * SP, yrow, whole[r]);
            }
        }
    };

    // ---- pipeline over (tile, chunk) items, buffers in turn: the next item's input is loaded
    // while this one multiplies (and a finished tile is stored), then its weights (kept when
    // the K loop is one chunk), then it goes to the other buffer ----
    if (c_begin >= c_end) {   // no steps for this part, or tiles of another plan
        for (int pt = jr; pt < a.n_pt; pt += a.n_walk) epilogue(pt);
        return;
    }
    int pt = jr, c = c_begin, b = 0;
    int4 cd = chunk(c);
    set_tile(pt);
    load_x(cd);
    load_w(cd);
    write_x(cd, lds);
    barrier_lds();
    for (;;) {
        asm volatile("" : "+v"(u_dst));   // keep derived offsets out of the loop's registers
        int npt = pt, nc = c + 1;
        if (nc == c_end) {
            nc = c_begin;
            npt += a.n_walk;
        }
        const bool more = npt < a.n_pt;
        int4 nd = cd;
        if (more) {
            nd = chunk(nc);
            if (npt != pt) set_tile(npt);
            load_x(nd);
        }
        compute(cd.y - cd.x, (uint32_t)(b * a.lds_buf));
        if (c + 1 == c_end) {
            epilogue(pt);
            clear();
        }
        if (!more) break;
        if (c_end - c_begin > 1) load_w(nd);
        b ^= 1;
        write_x(nd, lds + b * a.lds_buf);
        barrier_lds();
        pt = npt; c = nc; cd = nd;
    }
}

typedef void (*p1_fn)(P1Args);

template <int SW, int NT>
p1_fn p1_pick(int TM, int TPG, bool map, bool ident) {
    if (map && (TPG != TM || !ident)) return nullptr;
    if (ident) {   // one list: every m-tile of a wave shares it
        if (TPG != TM) return nullptr;
        switch (TM) {
            case 1: return map ? k_p1<SW, 1, 1, NT, true, true> : k_p1<SW, 1, 1, NT, false, true>;
            case 2:
                if constexpr (2 * NT <= kCvMaxAcc)
                    return map ? k_p1<SW, 2, 2, NT, true, true> : k_p1<SW, 2, 2, NT, false, true>;
                return nullptr;
            case 4:
                if constexpr (4 * NT <= kCvMaxAcc)
                    return map ? k_p1<SW, 4, 4, NT, true, true> : k_p1<SW, 4, 4, NT, false, true>;
                return nullptr;
            default: return nullptr;
        }
    }
    switch (TM * 16 + TPG) {
        case 0x11: return k_p1<SW, 1, 1, NT, false, false>;
        case 0x21: if constexpr (2 * NT <= kCvMaxAcc) return k_p1<SW, 2, 1, NT, false, false>; return nullptr;
        case 0x22: if constexpr (2 * NT <= kCvMaxAcc) return k_p1<SW, 2, 2, NT, false, false>; return nullptr;
        case 0x42: if constexpr (4 * NT <= kCvMaxAcc) return k_p1<SW, 4, 2, NT, false, false>; return nullptr;
        case 0x44: if constexpr (4 * NT <= kCvMaxAcc) return k_p1<SW, 4, 4, NT, false, false>; return nullptr;
        default: return nullptr;
    }
}

}  // namespace p1
}  // namespace bsp
