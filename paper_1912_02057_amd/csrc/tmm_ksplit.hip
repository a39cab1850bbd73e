// The contraction on small grids: every wave of a block computes the block's whole output tile over a
// share of K, and the shares meet in LDS.
//
// A layer of a few images, or a GEMM of a few rows, has fewer output tiles than the chip has CUs, and
// k_tmm's time there is the serial chain of one block: 0.3 us per 64-byte K-step of its 64 x 64 tile (wait,
// barrier, fragment reads, MFMAs one after the other), whatever the depth of its ring.  Here the K-steps are
// dealt out in W contiguous shares to the W waves of a block.  Each wave loads its own operand stages (the
// direct global -> LDS loads, swizzle and fragment addressing of k_tmm) into a ring of its own and waits for its
// own loads only, so there is no barrier until the sums meet, and the W chains run side by side.  D is a sum of
// integers (int32, or below 2^24 in fp32), so its order does not matter, and the epilogue repeats k_tmm's
// operations: the outputs are the same bits whichever kernel runs.
//
// Operands straight into registers (no LDS): 1.1 to 2.1 times slower from 60 K-steps on.  An MFMA operand has
// 32 rows in consecutive lanes, so every lane of such a load touches a cache line of its own, where a direct load
// takes 64 bytes of each of 16 rows.
//
// RUN (conv, stride 1, centred window): the input pixels of the tile are loaded into LDS once, for all waves and
// taps, and only the weights go through the rings: the operand traffic L2 -> LDS, which bounds a block of many
// K-steps, falls to about half.  int8, 7 images of 27 x 27, 96 channels, 256 filters, 5 x 5 (320 tiles of 64 x 64, 50
// K-steps): k_tmm 19.1, without RUN 18.1, with it 15.3 us; no gain below some 18 K-steps, where its barrier counts.
//
// Parameters, thresholds and residual values are fetched before the K loop.  What is left of a launch: 3.1 us
// (GEMM) to 3.7 us (conv) with one K-step -- launch, first load, meeting, store -- and from 250 tiles on the
// operand traffic L2 -> LDS.  us, k_tmm 64 x 64 -> here (times of back-to-back launches):
//   conv, FP4, one image, 512 filters on 7 x 7, 36 K-steps     11.5 -> 5.0
//   conv, FP4, one image, 256 filters on 14 x 14, 18 K-steps    8.0 -> 4.8, block tail 4.7
//   conv, FP4, one image, 64 filters on 56 x 56, 9 K-steps      5.8 -> 4.5, block tail 7.5 -> 4.6
//   GEMM, int8, 661 x 174 x 5600, 88 K-steps                   14.5 -> 6.8
//   GEMM, FP4, 2 x 8144 x 300, 3 K-steps                        3.6 -> 3.1
#include "tmm_kernel.h"

namespace rtn {

namespace {

struct KsplitParams {
    TmmParams t;
    FastDiv div_spt, div_kw;  // by the K-steps per tap and the window's width
    FastDiv div_tp;           // by the tiles along P
    int xcd_tiles;            // tiles of an XCD
    FastDiv div_upr;          // RUN: by the 16-byte units of a pixel's LDS row
    int runb;                 // RUN: LDS bytes of the pixel run, whole KiB
    int main;                 // LDS bytes in front of the pixel sums
};

template <int TP, int TQ, int W, int NS, bool CONV, int TERN, int DT, bool RUN>
__global__ __launch_bounds__(64 * W) void k_ksplit(KsplitParams kp)
{
    constexpr int BP = 32 * TP, BQ = 32 * TQ, T = TP * TQ;
    constexpr int LP = BP / 16, LQ = RUN ? 0 : BQ / 16, LQA = LQ ? LQ : 1, DPS = LP + LQ;  // loads per step
    constexpr int STAGE = (BP + (RUN ? 0 : BQ)) * 64, RING = NS * STAGE;
    constexpr int REDB = RUN ? T * 4096 : RING;  // bytes between the waves' accumulators
    static_assert(RUN || RING >= T * 4096, "a wave's accumulators lie over its ring");
    static_assert(CONV || !RUN, "a conv's window");
    static_assert(NS >= 2 && NS <= 4 && 3 * DPS < 64, "vmcnt range");
    constexpr int V = 16 * T / W;              // outputs per thread
    constexpr int QV = V < 4 ? V : 4;          // ... of which so many are consecutive rows
    constexpr int NQ = V / QV;
    static_assert(V >= 1 && V * W == 16 * T, "every thread has outputs");
    static_assert(16 / QV % NQ == 0, "a thread's outputs lie in one 32 x 32 tile");
    static_assert(DT == 0 || DT == 2, "codes");
    const TmmParams& prm = kp.t;
    const ConvGeom& g = prm.g;
    using AccV = std::conditional_t<DT == 2, v16f, v16i>;
    using AccS = std::conditional_t<DT == 2, float, int>;
    typedef AccS AccQ __attribute__((ext_vector_type(QV == 1 ? 2 : QV)));

    // [W][T][4][64 lanes][4] accumulators, [W][BQ] pixel sums, conv: the epilogue table; the code
    // bytes of a ternarizing epilogue lie over the accumulators
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    AccS* red = (AccS*)smem;
    // (RUN: [W rings][pixel run][16 zero bytes], all under the accumulators)
    const int main_bytes = RUN ? kp.main : W * RING;
    AccS* red_sa = (AccS*)(smem + main_bytes);
    const int toff = main_bytes + (CONV ? W * BQ * 4 : 0);
    const int pitch = g.Cpad + 16, zoff = W * RING + kp.runb;
    const unsigned lds0 = (unsigned)(uintptr_t)smem;

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // One contiguous run of tiles per XCD.  conv: all filters of a pixel tile follow each other, the inputs are read by one
    // XCD.  GEMM: in bands, as k_tmm, so that rows that the kernel before wrote are fetched by one or two XCDs, not by
    // half of them (pack and GEMM, FP4, 2048 x 124 x 2460: 11.9 us without the bands, 10.0).
    const int bid = (int)(blockIdx.x & 7) * kp.xcd_tiles + (int)(blockIdx.x >> 3);
    if (bid >= prm.ntiles) return;
    int tileP, tileQ;
    if (CONV) {
        tileQ = (int)fastdiv_flat((uint32_t)bid, kp.div_tp), tileP = bid - tileQ * prm.tilesP;
    } else {
        band_tile(bid, prm.tilesP, prm.band_tiles, [&](int n) { return (int)fastdiv_flat((uint32_t)n, prm.div_band); },
                  [&](int n) { return (int)fastdiv_flat((uint32_t)n, prm.div_lastband); }, tileP, tileQ);
    }
    const int p0 = tileP * BP, q0 = tileQ * BQ;
    const bool want_ep = TERN || prm.y != nullptr;
    const int ohw = g.OH * g.OW;

    const int nax = CONV ? conv_axis_classes(g) : 0;

    // ---- operand loads: as in k_tmm, but by one wave for itself ------------------------------------------
    // load j of a step covers 16 rows of an operand: lane l fetches row l >> 2, chunk (l & 3) ^ swz(row)
    const int lrow = lane >> 2, lchunk = (lane & 3) ^ swz(lrow);
    const int8_t* baseP = prm.P + (int64_t)p0 * prm.ldP;
    const int8_t* baseQ = CONV ? prm.Q : prm.Q + (int64_t)q0 * prm.ldQ;
    unsigned offP[LP], offQ[LQA];
    const int8_t* gQ[LQA];
    int vmask[LQA];  // conv: bit kh = row tap in the image, bit (8 + kw) = column tap in the image
#pragma unroll
    for (int i = 0; i < LP; ++i) {
        int row = p0 + 16 * i + lrow;
        row = row < prm.RP ? row : prm.RP - 1;  // tail rows: any valid data, never stored
        offP[i] = (unsigned)(row - p0) * (unsigned)prm.ldP + lchunk * 16;
    }
    // conv: where output pixel q0 + 32 j + (lane & 31) is, its first tap's pixel and its taps in the image
    int dnb[TQ], dpix[TQ], dih[TQ], diw[TQ], dcorner[TQ], dmask[TQ];
#pragma unroll
    for (int j = 0; j < TQ; ++j) {
        dnb[j] = dpix[j] = dih[j] = diw[j] = dcorner[j] = dmask[j] = 0;
        if (CONV) {
            int m = q0 + j * 32 + (lane & 31);
            m = m < prm.RQ ? m : prm.RQ - 1;
            dnb[j] = (int)fastdiv_flat((uint32_t)m, g.div_ohw), dpix[j] = m - dnb[j] * ohw;
            const int oh = (int)fastdiv_flat((uint32_t)dpix[j], g.div_ow), ow = dpix[j] - oh * g.OW;
            dih[j] = oh * g.stride - g.pad, diw[j] = ow * g.stride - g.pad;
            dcorner[j] = (dnb[j] * g.H + dih[j]) * g.W + diw[j];
            dmask[j] = tap_mask(dih[j], g.KH, g.H) | tap_mask(diw[j], g.KW, g.W) << 8;
        }
    }
#pragma unroll
    for (int j = 0; j < LQ; ++j) {
        vmask[j] = 0;
        offQ[j] = 0;
        gQ[j] = nullptr;
        if (CONV) {
            // (row 16 j + lrow of the tile: the lane that looked at it knows)
            const int src = 16 * (j & 1) + lrow;
            gQ[j] = prm.Q + (int64_t)__shfl(dcorner[j >> 1], src, 64) * g.Cpad + lchunk * 16;
            vmask[j] = __shfl(dmask[j >> 1], src, 64);
        } else {
            int row = q0 + 16 * j + lrow;
            row = row < prm.RQ ? row : prm.RQ - 1;
            offQ[j] = (unsigned)(row - q0) * (unsigned)prm.ldQ + lchunk * 16;
        }
    }
    // this wave's share of the K-steps, and the position of the next step to load (wave-uniform)
    const int first = (int)((unsigned)prm.nk * (unsigned)wave / W), end = (int)((unsigned)prm.nk * (unsigned)(wave + 1) / W);
    const int n = end - first;
    int kh = 0, kw = 0, cc = 0;
    int64_t koffP = (int64_t)first * 64, koffQ = koffP;
    const int spt = CONV ? g.Cpad >> 6 : prm.nk;  // steps per tap
    if (CONV) {
        const int tap = (int)fastdiv_flat((uint32_t)first, kp.div_spt);
        cc = first - tap * spt;
        kh = (int)fastdiv_flat((uint32_t)tap, kp.div_kw);
        kw = tap - kh * g.KW;
        koffQ = (int64_t)(kh * g.W + kw) * g.Cpad + cc * 64;
    }
    int f_kh = kh, f_kw = kw, f_cc = cc;  // RUN: the same of the step being multiplied
    const int64_t rowskip = CONV ? (int64_t)(g.W - g.KW) * g.Cpad : 0;
    const unsigned ring = lds0 + (unsigned)(wave * RING);
    const int8_t* zero_page = (const int8_t*)g_zero16;
    auto issue = [&](int slot) {
        const unsigned dst = ring + (unsigned)(slot * STAGE);
        auto load_p = [&](auto i) { dma16_base<i * 1024>(uniform_ptr(baseP + koffP), offP[i], dst); };
        auto load_q = [&](auto j) {
            if (CONV) {
                const bool ok = ((vmask[j] >> kh) & (vmask[j] >> (8 + kw)) & 1) != 0;
                dma16<BP * 64 + j * 1024>(ok ? gQ[j] + koffQ : zero_page, dst);
            } else {
                dma16_base<BP * 64 + j * 1024>(uniform_ptr(baseQ + koffQ), offQ[j], dst);
            }
        };
        for_each_index(load_p, std::make_integer_sequence<int, LP>{});
        for_each_index(load_q, std::make_integer_sequence<int, LQ>{});
        koffP += 64;
        koffQ += 64;
        if (CONV && ++cc == spt) {
            cc = 0;
            if (++kw == g.KW) {
                kw = 0;
                ++kh;
                koffQ += rowskip;
            }
        }
    };
    int fragP[TP][2], fragQ[TQ][2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
        for (int i = 0; i < TP; ++i) {
            const int row = i * 32 + (lane & 31);
            fragP[i][ks] = row * 64 + (((ks * 2 + half) ^ swz(row)) << 4);
        }
#pragma unroll
        for (int j = 0; j < TQ; ++j) {
            const int row = j * 32 + (lane & 31);
            fragQ[j][ks] = BP * 64 + row * 64 + (((ks * 2 + half) ^ swz(row)) << 4);
        }
    }
    // RUN: stride 1 and a centred window, so output pixel m reads input pixel m + (kh - pad) W + (kw - pad) of the
    // same flattened index space: the tile's inputs are one run of pixels, loaded once, and a tap is a row offset.
    // An LDS row is the pixel's codes and 16 bytes more: an odd number of 16-byte units, so that 16 consecutive
    // rows lie in different banks whatever the channels.
    if (RUN) {
        const int total_px = g.Nb * g.H * g.W, first_px = q0 - g.pad * (g.W + 1), upr = pitch >> 4;
        for (int u = wave; u < kp.runb >> 10; u += W) {
            const int lin = u * 64 + lane, row = (int)fastdiv((uint32_t)lin, kp.div_upr), c = lin - row * upr;
            int px = first_px + row;
            px = px < 0 ? 0 : (px < total_px ? px : total_px - 1);  // past the tensor: only taps outside an image point there
            dma16(c < upr - 1 ? prm.Q + (int64_t)px * g.Cpad + c * 16 : zero_page, lds0 + (unsigned)(W * RING + u * 1024));
        }
        if (tid == 0) *(uint4*)(smem + zoff) = make_uint4(0, 0, 0, 0);
    }
    AccV acc[TP][TQ];
    v4f sa4[TQ];
    int sa1[TQ];
#pragma unroll
    for (int j = 0; j < TQ; ++j) {
        sa4[j] = v4f{0.f, 0.f, 0.f, 0.f};
        sa1[j] = 0;
#pragma unroll
        for (int i = 0; i < TP; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
    }
    // pixel sums on the matrix cores, as in k_tmm: pixels 0 .. 15 in row 0, 16 .. 31 in row 1
    const int sa_ones = ((lane & 15) < 2 && ((lane >> 4) & 1) == (lane & 15)) ? 0x22222222 : 0;
    const v8i SA8 = {sa_ones, sa_ones, sa_ones, sa_ones, 0, 0, 0, 0};
    (void)SA8;
    auto multiply = [&](const v4i (&fa)[TP], const v4i (&fb)[TQ]) {
#pragma unroll
        for (int j = 0; j < TQ; ++j) {
            const v4i q = fb[j];
            if constexpr (DT == 2) {
                const v8i B8 = {q[0], q[1], q[2], q[3], 0, 0, 0, 0};
#pragma unroll
                for (int i = 0; i < TP; ++i) {
                    const v4i p = fa[i];
                    const v8i A8 = {p[0], p[1], p[2], p[3], 0, 0, 0, 0};
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A8, B8, acc[i][j], 4, 4, 0, 0, 0, 0);
                }
                if (CONV) sa4[j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(SA8, B8, sa4[j], 4, 4, 0, 0, 0, 0);
            } else {
#pragma unroll
                for (int i = 0; i < TP; ++i) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[i], q, acc[i][j], 0, 0, 0);
                if (CONV)
#pragma unroll
                    for (int e = 0; e < 4; ++e) sa1[j] = __builtin_amdgcn_sdot4(q[e], 0x01010101, sa1[j], false);
            }
        }
    };

    for (int s = 0; s < NS && s < n; ++s) issue(s);
    // ---- epilogue table (conv): rows g1, c2, bn scale, bn shift, then the classes that can occur -----
    if (CONV && want_ep) {
        const int nrows = 4 + conv_classes(g.pad), opitch = (g.O + 1) & ~1;
        const bool compact = conv_compact(g);
        const int lrows = 4 + nax * nax, pp = (g.pad + 1) * (g.pad + 1);
        const int kib = (conv_table_bytes(BP, g) + 1023) >> 10;
        for (int n = wave; n < kib; n += W) {
            const int lin = n * 64 + lane;  // 16-byte unit = 2 doubles
            int row = lin / (BP / 2);
            const int u = lin - row * (BP / 2);
            row = row < lrows ? row : lrows - 1;
            if (row >= 4) {
                const int c = row - 4, ra = (int)fastdiv_flat((uint32_t)c, prm.div_nax), ca = c - ra * nax;
                row = 4 + conv_axis_global(compact, g.pad, ra) * pp + conv_axis_global(compact, g.pad, ca);
            }
            int64_t idx = (int64_t)row * opitch + p0 + 2 * u;
            const int64_t last = (int64_t)nrows * opitch - 2;
            idx = idx < last ? idx : last;  // columns past O are never used
            dma16(prm.cst_cls + idx, lds0 + (unsigned)(toff + n * 1024));
        }
    }

    // ---- this thread's outputs: QV consecutive rows at t0[n] of column q ------------------------------
    // thread = (lane, units): unit wave NQ + n holds rows 8 r4 + 4 half + QV sub ... of 32 x 32 tile ij
    constexpr int SUBS = 4 / QV;
    auto unit_sub = [&](int n) { return (wave * NQ + n) % SUBS; };
    auto unit_r4 = [&](int n) { return (wave * NQ + n) / SUBS % 4; };
    auto unit_ij = [&](int n) { return (wave * NQ + n) / (SUBS * 4); };
    auto row_of = [&](int n) { return unit_ij(n) / TQ * 32 + 8 * unit_r4(n) + 4 * half + QV * unit_sub(n); };
    const int jq = unit_ij(0) % TQ;  // the same for every n
    const int q = q0 + jq * 32 + (lane & 31);
    const bool qok = q < prm.RQ;
    const int qq = qok ? q : prm.RQ - 1;
    // parameters and residual values, fetched beside the operands
    float f_aa[V], f_ba[V], f_lo[V], f_hi[V], f_res[V];
    int f_sa[V];
    float f_aw = 0.f, f_bw = 0.f, f_bs = 1.f, f_bh = 0.f;
    int f_sw = 0, cls = 0;
    int64_t obase = 0;
    const EpiArgs& ep = prm.ep;
    if (!CONV && want_ep) {
        f_aw = ep.alpha_w.ptr ? ep.alpha_w.ptr[qq] : ep.alpha_w.s;
        f_bw = ep.beta_w.ptr ? ep.beta_w.ptr[qq] : ep.beta_w.s;
        f_sw = ep.sum_tw[qq];
        if (ep.bn_scale) {
            f_bs = ep.bn_scale[qq];
            if (ep.bn_shift) f_bh = ep.bn_shift[qq];
        }
#pragma unroll
        for (int n = 0; n < NQ; ++n)
#pragma unroll
            for (int e = 0; e < QV; ++e) {
                int m = p0 + row_of(n) + e;
                m = m < prm.RP ? m : prm.RP - 1;
                f_aa[n * QV + e] = ep.alpha_a.ptr ? ep.alpha_a.ptr[m] : ep.alpha_a.s;
                f_ba[n * QV + e] = ep.beta_a.ptr ? ep.beta_a.ptr[m] : ep.beta_a.s;
                f_sa[n * QV + e] = ep.sum_ta[m];
            }
    }
    if (CONV) {
        const int nb = TQ == 2 && jq ? dnb[TQ - 1] : dnb[0], pix = TQ == 2 && jq ? dpix[TQ - 1] : dpix[0];
        obase = (int64_t)nb * g.O * ohw + pix;
        if (want_ep && !g.code_zero_pad) {
            const int ih0 = TQ == 2 && jq ? dih[TQ - 1] : dih[0], iw0 = TQ == 2 && jq ? diw[TQ - 1] : diw[0];
            const int bh = ih0 + g.KH - g.H, bw = iw0 + g.KW - g.W;  // taps cut off at the far ends
            const bool compact = conv_compact(g);
            cls = conv_axis_class(compact, g.pad, ih0 < 0 ? -ih0 : 0, bh > 0 ? bh : 0) * nax +
                  conv_axis_class(compact, g.pad, iw0 < 0 ? -iw0 : 0, bw > 0 ? bw : 0);
        }
        if (TERN)
#pragma unroll
            for (int n = 0; n < NQ; ++n)
#pragma unroll
                for (int e = 0; e < QV; ++e) {
                    int o = p0 + row_of(n) + e;
                    o = o < prm.RP ? o : prm.RP - 1;
                    f_lo[n * QV + e] = prm.thr_lo.ptr ? prm.thr_lo.ptr[o] : prm.thr_lo.s;
                    f_hi[n * QV + e] = prm.thr_hi.ptr ? prm.thr_hi.ptr[o] : prm.thr_hi.s;
                    if (TERN == 2) f_res[n * QV + e] = prm.res ? prm.res[obase + (int64_t)o * ohw] : 0.0f;
                }
    }

    // ---- this wave's share of K ----------------------------------------------------------------------
    if (RUN) {  // everybody's share of the pixel run
        wait_vm<0>();
        __syncthreads();
    }
    int slot = 0;
    for (int s = 0; s < n; ++s) {
        wait_groups<DPS>(n - 1 - s < NS - 1 ? n - 1 - s : NS - 1);
        const int8_t* st = smem + wave * RING + slot * STAGE;
        v4i fa[2][TP], fb[2][TQ];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int i = 0; i < TP; ++i) fa[ks][i] = *(const v4i*)(st + fragP[i][ks]);
#pragma unroll
            for (int j = 0; j < TQ; ++j) {
                if constexpr (RUN) {
                    const int row = j * 32 + (lane & 31) + f_kh * g.W + f_kw;
                    const bool ok = ((dmask[j] >> f_kh) & (dmask[j] >> (8 + f_kw)) & 1) != 0;
                    fb[ks][j] = *(const v4i*)(smem + (ok ? W * RING + row * pitch + f_cc * 64 + (ks * 2 + half) * 16 : zoff));
                } else {
                    fb[ks][j] = *(const v4i*)(st + fragQ[j][ks]);
                }
            }
        }
        if (RUN && ++f_cc == spt) {
            f_cc = 0;
            if (++f_kw == g.KW) f_kw = 0, ++f_kh;
        }
        if (s + NS < n) {
            wait_lgkm0();
            issue(slot);
        }
        multiply(fa[0], fb[0]);
        multiply(fa[1], fb[1]);
        slot = slot + 1 == NS ? 0 : slot + 1;
    }
    wait_lgkm0();
    if (RUN) __syncthreads();  // the accumulators go over everybody's ring and the run

    // ---- the shares meet -------------------------------------------------------------------------------
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
        for (int j = 0; j < TQ; ++j)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                typedef AccS V4 __attribute__((ext_vector_type(4)));
                const V4 v = {acc[i][j][4 * r4], acc[i][j][4 * r4 + 1], acc[i][j][4 * r4 + 2], acc[i][j][4 * r4 + 3]};
                *(V4*)(red + wave * (REDB / 4) + (((i * TQ + j) * 4 + r4) * 64 + lane) * 4) = v;
            }
    if (CONV && want_ep) {
#pragma unroll
        for (int j = 0; j < TQ; ++j) {
            if constexpr (DT == 2) {
                if (lane < 16) {
                    red_sa[wave * BQ + j * 32 + lane] = sa4[j][0];
                    red_sa[wave * BQ + j * 32 + 16 + lane] = sa4[j][1];
                }
            } else {
                const int s = sa1[j] + __shfl_xor(sa1[j], 32, 64);
                if (lane < 32) red_sa[wave * BQ + j * 32 + lane] = s;
            }
        }
        wait_vm<0>();  // the epilogue table's direct loads
    }
    __syncthreads();
    AccS D[V], Sa = 0;
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
        const AccS* src = red + ((unit_ij(n) * 4 + unit_r4(n)) * 64 + lane) * 4 + unit_sub(n) * QV;
#pragma unroll
        for (int e = 0; e < QV; ++e) D[n * QV + e] = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            if constexpr (QV == 1) {
                D[n] += src[w * (REDB / 4)];
            } else {
                const AccQ v = *(const AccQ*)(src + w * (REDB / 4));
#pragma unroll
                for (int e = 0; e < QV; ++e) D[n * QV + e] += v[e];
            }
        }
    }
    if (CONV && want_ep)
#pragma unroll
        for (int w = 0; w < W; ++w) Sa += red_sa[w * BQ + jq * 32 + (lane & 31)];

    // ---- epilogue: the arithmetic of k_tmm's, operation by operation -----------------------------------
    if constexpr (!CONV) {
        const bool has_bn = ep.bn_scale != nullptr;
        const double floor = __builtin_canonicalize(ep.relu ? 0.0 : (has_bn ? -__builtin_inf() : __builtin_nan("")));
        const double aw = f_aw, bw = f_bw, sw = f_sw, bs = f_bs, bh = has_bn ? (double)f_bh : -0.0;
#pragma unroll
        for (int n = 0; n < NQ; ++n)
#pragma unroll
            for (int e = 0; e < QV; ++e) {
                const int m = p0 + row_of(n) + e;
                if (m >= prm.RP || !qok) continue;
                const int64_t idx = (int64_t)m * prm.RQ + q;
                const int x = n * QV + e;
                if (prm.acc) prm.acc[idx] = (int)D[x];
                if (prm.y) {
                    const double aa = f_aa[x], ba = f_ba[x], r2 = aa * (double)f_sa[x] + (double)prm.Klogical * ba;
                    const double v = aw * (aa * (double)D[x] + ba * sw) + bw * r2;
                    prm.y[idx] = (float)(bs * __builtin_fmax(v, floor) + bh);
                }
            }
        return;
    } else {
        const double* tab = (const double*)(smem + toff);
        const double* ctab = tab + (4 + cls) * BP;
        const double floor = __builtin_canonicalize(ep.relu ? 0.0 : -__builtin_inf());
        const float out_floor = __builtin_canonicalizef(prm.relu_out ? 0.0f : -__builtin_inff());
        uint8_t code[V];
#pragma unroll
        for (int n = 0; n < NQ; ++n)
#pragma unroll
            for (int e = 0; e < QV; ++e) {
                const int t = row_of(n) + e, o = p0 + t, x = n * QV + e;
                const bool ok = o < prm.RP && qok;
                const int64_t idx = obase + (int64_t)o * ohw;
                float z = 0.0f;
                if (want_ep) {
                    double v = tab[t] * (double)D[x] + (tab[BP + t] * (double)Sa + ctab[t]);
                    v = __builtin_fmax(v, floor);
                    z = (float)(tab[2 * BP + t] * v + tab[3 * BP + t]);
                }
                if (TERN == 2) z = __builtin_fmaxf(z + f_res[x], out_floor);
                if (TERN != 1 && prm.y && ok) prm.y[idx] = z;
                if (!TERN && prm.acc && ok) prm.acc[idx] = (int)D[x];
                if (TERN) {
                    const bool pos1 = z > f_hi[x], neg = z < f_lo[x];
                    if (DT == 2)
                        code[x] = o < prm.RP ? (uint8_t)(((unsigned)(pos1 | neg) << 1) | ((unsigned)neg << 3)) : 0;
                    else
                        code[x] = o < prm.RP ? (uint8_t)((int)pos1 - (int)neg) : 0;
                }
            }
        if constexpr (TERN != 0) {
            // codes as bytes [pixel][BP], then packed into the channel-innermost output rows
            __syncthreads();  // the accumulators are read
            uint8_t* cb = (uint8_t*)smem + (jq * 32 + (lane & 31)) * BP;
#pragma unroll
            for (int n = 0; n < NQ; ++n)
#pragma unroll
                for (int e = 0; e < QV; ++e) cb[row_of(n) + e] = code[n * QV + e];
            __syncthreads();
            constexpr int CPD = DT == 2 ? 8 : 4;        // codes per dword
            constexpr int DPR = BP / CPD;               // dwords of a pixel of this tile
            for (int d = tid; d < BQ * DPR; d += 64 * W) {
                const int px = d / DPR, c = d % DPR, m = q0 + px;
                const uint8_t* s = (const uint8_t*)smem + px * BP + c * CPD;
                unsigned word;
                if constexpr (DT == 2) {
                    const uint2 v = *(const uint2*)s;  // a nibble per byte
                    const unsigned a = v.x | (v.x >> 4), b2 = v.y | (v.y >> 4);
                    word = (a & 0xff) | ((a >> 8) & 0xff00) | ((b2 & 0xff) << 16) | ((b2 << 8) & 0xff000000u);
                } else {
                    word = *(const unsigned*)s;
                }
                const int off = p0 / (DT == 2 ? 2 : 1) + c * 4;  // byte of the code row
                if (m < prm.RQ && off < prm.ldc) *(unsigned*)(prm.codes + (int64_t)m * prm.ldc + off) = word;
            }
            // the zero codes of the row's padding, by the last tile along the channels
            const int from = (p0 + BP) / (DT == 2 ? 2 : 1);
            if (p0 + BP >= prm.RP && from < prm.ldc) {
                const int units = (prm.ldc - from) / 16;
                for (int d = tid; d < BQ * units; d += 64 * W) {
                    const int px = d / units, m = q0 + px;
                    if (m < prm.RQ)
                        *(uint4*)(prm.codes + (int64_t)m * prm.ldc + from + (d - px * units) * 16) = make_uint4(0, 0, 0, 0);
                }
            }
        }
    }
}

template <int FORM, bool CONV, int TERN, int DT>
hipError_t launch(KsplitParams& kp, const KsplitShape& s, hipStream_t st)
{
    constexpr KsplitForm f = kKsplitForms[FORM];
    if (!ksplit_fits(FORM, s)) return hipErrorInvalidValue;
    if (f.run) {
        kp.runb = (int)ksplit_run_bytes(f, s);
        kp.div_upr = make_fastdiv((uint32_t)(s.pixel_bytes / 16 + 1));
    }
    kp.main = (int)ksplit_main_bytes(f, s);
    auto kern = k_ksplit<f.tp, f.tq, f.waves, f.stages, CONV, TERN, DT, f.run>;
    static LdsLimit lds;
    const hipError_t e = lds.raise((const void*)kern, (int)kMaxLds);
    if (e != hipSuccess) return e;
    const unsigned grid = tile_grid(kp.t, 32 * f.tp, 32 * f.tq);
    if (!grid) return hipErrorInvalidValue;
    kp.div_tp = make_fastdiv((uint32_t)kp.t.tilesP);
    kp.xcd_tiles = (int)(grid / 8);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * f.waves), (size_t)ksplit_lds_bytes(f, s), st, kp);
    return hipGetLastError();
}

template <bool CONV, int TERN, int DT>
hipError_t launch_form(int form, KsplitParams& kp, const KsplitShape& s, hipStream_t st)
{
    static_assert(kKsplitGemmForms == 3 && kNumKsplitForms == 8, "every form has a case");
    switch (form) {
        case 0: return launch<0, CONV, TERN, DT>(kp, s, st);
        case 1: return launch<1, CONV, TERN, DT>(kp, s, st);
        case 2: return launch<2, CONV, TERN, DT>(kp, s, st);
        default: break;
    }
    if constexpr (CONV) {
        switch (form) {
            case 3: return launch<3, CONV, TERN, DT>(kp, s, st);
            case 4: return launch<4, CONV, TERN, DT>(kp, s, st);
            case 5: return launch<5, CONV, TERN, DT>(kp, s, st);
            case 6: return launch<6, CONV, TERN, DT>(kp, s, st);
            case 7: return launch<7, CONV, TERN, DT>(kp, s, st);
            default: break;
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace

KsplitShape ksplit_shape(const TmmParams& prm, bool conv)
{
    KsplitShape s = {};
    s.rp = prm.RP, s.rq = prm.RQ, s.nk = prm.nk;
    if (conv) {
        const ConvGeom& g = prm.g;
        s.KH = g.KH, s.KW = g.KW, s.stride = g.stride, s.pad = g.pad, s.W = g.W, s.pixel_bytes = g.Cpad;
        s.table_rows = 4 + conv_lds_classes(g);
    }
    return s;
}

template <bool CONV, int TERN, int DT>
hipError_t launch_ksplit(int form, const TmmParams& prm, hipStream_t st)
{
    KsplitParams kp = {};
    kp.t = prm;
    kp.div_spt = make_fastdiv((uint32_t)(CONV ? prm.g.Cpad >> 6 : 1));
    kp.div_kw = make_fastdiv((uint32_t)(CONV ? prm.g.KW : 1));
    return launch_form<CONV, TERN, DT>(form, kp, ksplit_shape(prm, CONV), st);
}
template hipError_t launch_ksplit<false, 0, 0>(int, const TmmParams&, hipStream_t);
template hipError_t launch_ksplit<false, 0, 2>(int, const TmmParams&, hipStream_t);
template hipError_t launch_ksplit<true, 0, 0>(int, const TmmParams&, hipStream_t);
template hipError_t launch_ksplit<true, 0, 2>(int, const TmmParams&, hipStream_t);
template hipError_t launch_ksplit<true, 1, 0>(int, const TmmParams&, hipStream_t);
template hipError_t launch_ksplit<true, 1, 2>(int, const TmmParams&, hipStream_t);
template hipError_t launch_ksplit<true, 2, 0>(int, const TmmParams&, hipStream_t);
template hipError_t launch_ksplit<true, 2, 2>(int, const TmmParams&, hipStream_t);

}  // namespace rtn
