// Depthwise ternary convolution (one k x k ternary filter per channel; the 3x3 layers of
// MobileNet, one of the networks the paper evaluates) with the per-channel four-term
// reparameterization.  A dot product here has only k*k terms: the kernels are streaming ones, 1 byte
// read and 4 bytes written per output.  Three of them: 3 x 3 windows on the matrix cores, 3 x 3
// windows on the vector ALU where the first does not apply, and any window.  In the last one a block
// owns 64 consecutive output pixels x 64 channels.  In the compute phase
// lanes run along channels -- the codes are channel-innermost, so a thread's dword is 4
// channels of one input pixel and 16 threads read 64 contiguous bytes -- and a thread forms
// its 4 pixels x 4 channels; the results cross an LDS tile so that in the store phase lanes
// run along pixels, where the NCHW output of a channel is contiguous.
#include <cmath>
#include <type_traits>

#include "tmm_kernel.h"

namespace rtn {

namespace {

constexpr int DW_PX = 64, DW_CH = 64, DW_PITCH = DW_PX + 1;  // LDS tile [channel][pixel], padded

// Byte e of each of four dwords -> one dword (a 4 x 4 byte transpose, one row of it).
__device__ __forceinline__ int gather_byte(int w0, int w1, int w2, int w3, int e)
{
    const unsigned sel = 0x04000400u + 0x00000101u * (unsigned)e;  // bytes: lo[e], hi[e] of each pair
    const unsigned p01 = __builtin_amdgcn_perm((unsigned)w1, (unsigned)w0, 0x0c0c0400u + 0x00000101u * (unsigned)e);
    const unsigned p23 = __builtin_amdgcn_perm((unsigned)w3, (unsigned)w2, 0x0c0c0400u + 0x00000101u * (unsigned)e);
    (void)sel;
    return (int)(p01 | (p23 << 16));
}

// KS = 3: the 3 x 3 window unrolled.  The nine taps of a channel are gathered into three dwords
// (byte transposes of the fetched code words), so that D, Sa and Sw of a channel are three
// 4-way byte dot products each: against the channel's filter codes, against ones, and of the
// filter codes against the per-pixel mask of taps that count.  KS = 0: any window, one tap and
// one channel at a time.
template <int KS>
__global__ __launch_bounds__(256) void k_dwconv(DwConvArgs a)
{
    __shared__ int tD[DW_CH * DW_PITCH];
    __shared__ float tY[DW_CH * DW_PITCH];
    const ConvGeom& g = a.g;
    const int tid = threadIdx.x;
    const int64_t ohw = (int64_t)g.OH * g.OW, total = (int64_t)g.Nb * ohw;
    const int64_t m0 = (int64_t)blockIdx.x * DW_PX;
    const int cb = (int)blockIdx.y * DW_CH;  // first channel of this block's slab
    const EpiArgs& ep = a.ep;
    const bool has_bn = ep.bn_scale != nullptr;
    const double aa = (double)ep.alpha_a.s, ba = (double)ep.beta_a.s;
    {
        const int cq = tid & 15, pg = tid >> 4;  // channels cb + 4 cq .. + 3, pixels m0 + 4 pg .. + 3
        const int c0 = cb + 4 * cq;
        const int KH = KS ? KS : g.KH, KW = KS ? KS : g.KW;
        // 3 x 3: the filter codes of each channel as three dwords (taps 0-3, 4-7, 8), read from the
        // channel's row of tap codes (the row is padded with zeros)
        int wq[4][3];
        if (KS) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = c0 + e < g.C ? c0 + e : g.C - 1;
                const int* wr = (const int*)(a.w + (int64_t)c * a.Kp);
                const bool cok = c0 + e < g.C;
                wq[e][0] = cok ? wr[0] : 0;
                wq[e][1] = cok ? wr[1] : 0;
                wq[e][2] = cok ? (wr[2] & 0xff) : 0;
            }
        }
        double awv[4], bwv[4], bsv[4], bhv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int c = c0 + e < g.C ? c0 + e : g.C - 1;
            awv[e] = pval(ep.alpha_w, c);
            bwv[e] = pval(ep.beta_w, c);
            bsv[e] = has_bn ? (double)ep.bn_scale[c] : 1.0;
            bhv[e] = (has_bn && ep.bn_shift) ? (double)ep.bn_shift[c] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int pl = 4 * pg + q;
            const int64_t m = m0 + pl;
            const bool mok = m < total;
            const int64_t mm = mok ? m : 0;
            // (Nb*OH*OW < 2^31: divisions by host-made magic numbers)
            const int nb = (int)fastdiv((uint32_t)mm, g.div_ohw), pix = (int)(mm - (int64_t)nb * ohw);
            const int oh = (int)fastdiv((uint32_t)pix, g.div_ow), ow = pix - oh * g.OW;
            const int ih0 = oh * g.stride - g.pad, iw0 = ow * g.stride - g.pad;
            const int8_t* img = a.a + (int64_t)nb * g.H * g.W * g.Cpad + c0;
            int d[4] = {0, 0, 0, 0}, sa[4] = {0, 0, 0, 0}, sw[4] = {0, 0, 0, 0};
            int kv = 0;
            if (KS) {
                // All taps are fetched first, from coordinates clamped into the image (every load is
                // in bounds and nothing waits between them); a tap outside the image is zeroed after.
                int words[12];
                unsigned cnt[3] = {0, 0, 0};  // byte t of cnt[t / 4]: 1 if tap t counts for Sw and Kv
#pragma unroll
                for (int kh = 0; kh < 3; ++kh)
#pragma unroll
                    for (int kw = 0; kw < 3; ++kw) {
                        const int ih = min(max(ih0 + kh, 0), g.H - 1), iw = min(max(iw0 + kw, 0), g.W - 1);
                        words[kh * 3 + kw] = *(const int*)(img + ((int64_t)ih * g.W + iw) * g.Cpad);
                    }
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    const int kh = t / 3, kw = t % 3;
                    const bool inb = (unsigned)(ih0 + kh) < (unsigned)g.H && (unsigned)(iw0 + kw) < (unsigned)g.W;
                    words[t] = inb ? words[t] : 0;
                    const bool counts = inb || g.code_zero_pad;
                    kv += counts;
                    cnt[t >> 2] |= (unsigned)counts << (8 * (t & 3));
                }
                words[9] = words[10] = words[11] = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
#pragma unroll
                    for (int h = 0; h < 3; ++h) {
                        const int av = gather_byte(words[4 * h], words[4 * h + 1], words[4 * h + 2], words[4 * h + 3], e);
                        d[e] = __builtin_amdgcn_sdot4(av, wq[e][h], d[e], false);
                        sa[e] = __builtin_amdgcn_sdot4(av, 0x01010101, sa[e], false);
                        sw[e] = __builtin_amdgcn_sdot4(wq[e][h], (int)cnt[h], sw[e], false);
                    }
                }
            } else {
                for (int kh = 0; kh < KH; ++kh)
                    for (int kw = 0; kw < KW; ++kw) {
                        const bool inb = (unsigned)(ih0 + kh) < (unsigned)g.H && (unsigned)(iw0 + kw) < (unsigned)g.W;
                        const int ih = min(max(ih0 + kh, 0), g.H - 1), iw = min(max(iw0 + kw, 0), g.W - 1);
                        int word = *(const int*)(img + ((int64_t)ih * g.W + iw) * g.Cpad);
                        word = inb ? word : 0;
                        const bool counts = inb || g.code_zero_pad;
                        kv += counts;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int w_ = c0 + e < g.C ? (int)a.w[(int64_t)(c0 + e) * a.Kp + kh * KW + kw] : 0;
                            const int a_ = (int)(int8_t)(word >> (8 * e));
                            d[e] += a_ * w_;
                            sa[e] += a_;
                            sw[e] += counts ? w_ : 0;
                        }
                    }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                tD[(4 * cq + e) * DW_PITCH + pl] = d[e];
                if (a.y)
                    tY[(4 * cq + e) * DW_PITCH + pl] =
                        reparam(aa, ba, awv[e], bwv[e], d[e], sa[e], sw[e], kv, ep.relu, has_bn, bsv[e], bhv[e]);
            }
        }
    }
    __syncthreads();
    // store phase: lane = pixel, the four waves take the channels round-robin
    const int lane = tid & 63, wave = tid >> 6;
    const int64_t m = m0 + lane;
    if (m >= total) return;
    const int nb = (int)fastdiv((uint32_t)m, g.div_ohw), pix = (int)(m - (int64_t)nb * ohw);
    for (int cl = wave; cl < DW_CH; cl += 4) {
        const int c = cb + cl;
        if (c >= g.C) break;
        const int64_t i = ((int64_t)nb * g.C + c) * ohw + pix;
        if (a.acc) a.acc[i] = tD[cl * DW_PITCH + lane];
        if (a.y) a.y[i] = tY[cl * DW_PITCH + lane];
    }
}

// ---- 3 x 3, pad <= 1: the common case with the per-output work cut down ---------------
// The kernel above spends its time in the vector ALU: coordinate and clamp arithmetic per tap
// and thread, and the four-term formula in fp64 with its products formed per output.  Here
//  * the addressing is prepared once per pixel (one thread each, kept in LDS): the 32-bit byte
//    offsets of the nine taps, with an out-of-range offset for a tap outside the image (the
//    codes are read through a buffer resource, whose out-of-range loads return 0), and the
//    border class (which of the first / last window row and column are cut off: 4 x 4
//    classes; class 0 when the pad mode counts every tap);
//  * Eq.9's constant C = beta_a*alpha_w*Sw + Kv*beta_a*beta_w is prepared once per block for
//    every (class, channel);
//  * a thread forms D and Sa of its 4 pixels x 4 channels from the nine code dwords by two
//    4 x 4 byte transposes (8 byte-permutes each) and byte dot products, and evaluates
//    y = g1*D + c2*Sa + C[class] in fp64 (ReLU, BN, one rounding) with its four channels'
//    factors held in registers; results cross the [channel][pixel] LDS tile;
//  * a block walks several consecutive pixel tiles, so the per-channel set-up is paid once;
//  * the store phase (lanes along pixels, NCHW-contiguous) only copies.
// CHB = channels per block (64, or 32 for layers with at most 32 channels, whose blocks then
// own 128 pixels); offsets are 32-bit: the code tensor must be below 2 GiB.  NT: fp32 outputs
// above 128 MiB are stored with the non-temporal hint, as the matrix-core conv does.
// Dynamic LDS: one tile (CHB x (PXB + 1) dwords) per requested output, y first.
template <int CHB, bool NT>
__global__ __launch_bounds__(256) void k_dwconv3(DwConvArgs a)
{
    constexpr int NCQ = CHB / 4, PXB = 4096 / CHB, PITCH = PXB + 1;
    __shared__ __attribute__((aligned(16))) unsigned po[PXB][12];  // byte offsets of the 9 taps (3 pad words)
    __shared__ int pm[PXB];                                          // border class
    __shared__ __attribute__((aligned(16))) double cst[16][CHB];
    extern __shared__ int dw_tiles[];
    float* tY = (float*)dw_tiles;
    int* tD = dw_tiles + (a.y ? CHB * PITCH : 0);
    const ConvGeom& g = a.g;
    const int tid = threadIdx.x;
    const int64_t ohw = (int64_t)g.OH * g.OW, total = (int64_t)g.Nb * ohw;
    const int cb = (int)blockIdx.y * CHB;
    const EpiArgs& ep = a.ep;
    const bool has_bn = ep.bn_scale != nullptr;
    const double aa = (double)ep.alpha_a.s, ba = (double)ep.beta_a.s;
    // ---- once per block: the class constants and this thread's channel factors ----------
    if (a.y) {
        // (pad <= 1 and an image at least as long as the window: a window is cut at one end of an
        // axis at most, 3 x 3 classes; the others exist only for images shorter than 3)
        const bool tiny = g.H < 3 || g.W < 3;  // only then both ends of an axis can be cut
        const int nax = tiny ? 4 : 3;
        for (int idx = tid; idx < nax * nax * CHB; idx += 256) {
            const int k = idx / CHB, cl = idx - k * CHB;
            const int c = cb + cl < g.C ? cb + cl : g.C - 1;
            const int* wr = (const int*)(a.w + (int64_t)c * a.Kp);
            const int rc = k / nax, cc = k - rc * nax;
            const int cls = rc * 4 + cc;
            unsigned cnt[3] = {0, 0, 0};
            int kv = 0;
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const int kh = t / 3, kw = t % 3;
                const bool out = (kh == 0 && (rc & 1)) || (kh == 2 && (rc & 2)) || (kw == 0 && (cc & 1)) || (kw == 2 && (cc & 2));
                kv += !out;
                cnt[t >> 2] |= (unsigned)!out << (8 * (t & 3));
            }
            int sw = __builtin_amdgcn_sdot4(wr[0], (int)cnt[0], 0, false);
            sw = __builtin_amdgcn_sdot4(wr[1], (int)cnt[1], sw, false);
            sw = __builtin_amdgcn_sdot4(wr[2] & 0xff, (int)cnt[2], sw, false);
            const double aw = pval(ep.alpha_w, c), bw = pval(ep.beta_w, c);
            cst[cls][cl] = ba * aw * (double)sw + (double)kv * ba * bw;
        }
    }
    const int cq = tid % NCQ, pg = tid / NCQ;
    const int c0 = cb + 4 * cq;
    int wq[4][3];
    double g1[4], c2[4], bs[4], bh[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const bool cok = c0 + e < g.C;
        const int c = cok ? c0 + e : g.C - 1;
        const int* wr = (const int*)(a.w + (int64_t)c * a.Kp);
        wq[e][0] = cok ? wr[0] : 0;
        wq[e][1] = cok ? wr[1] : 0;
        wq[e][2] = cok ? (wr[2] & 0xff) : 0;
        g1[e] = c2[e] = bh[e] = 0.0;
        bs[e] = 1.0;
        if (a.y) {
            g1[e] = aa * pval(ep.alpha_w, c);
            c2[e] = aa * pval(ep.beta_w, c);
            bs[e] = has_bn ? (double)ep.bn_scale[c] : 1.0;
            bh[e] = (has_bn && ep.bn_shift) ? (double)ep.bn_shift[c] : 0.0;
        }
    }
    const double relu_floor = __builtin_canonicalize(ep.relu ? 0.0 : -__builtin_inf());
    // A block walks tiles_per_block consecutive pixel tiles of its channel slab, so the
    // preparation above is paid once; two barriers per tile (a thread reaches the first one
    // of the next tile only after its copies of this one).
    for (int tt = 0; tt < a.tiles_per_block; ++tt) {
    const int64_t m0 = ((int64_t)blockIdx.x * a.tiles_per_block + tt) * PXB;
    if (m0 >= total) break;  // block-uniform
    // ---- phase 0: per-pixel preparation, the nine taps of a pixel dealt out over the block's
    // wave groups (so that the work spreads over the CU's four SIMDs) -----------------------
    {
        constexpr int PARTS = 256 / PXB;
        const int px = tid % PXB, part = tid / PXB;
        int64_t m = m0 + px;
        m = m < total ? m : total - 1;  // pixels past the end repeat the last one; never stored
        const int nb = (int)fastdiv((uint32_t)m, g.div_ohw), pix = (int)(m - (int64_t)nb * ohw);
        const int oh = (int)fastdiv((uint32_t)pix, g.div_ow), ow = pix - oh * g.OW;
        const int ih0 = oh * g.stride - g.pad, iw0 = ow * g.stride - g.pad;
        unsigned rowin = 0, colin = 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            rowin |= (unsigned)((unsigned)(ih0 + k) < (unsigned)g.H) << k;
            colin |= (unsigned)((unsigned)(iw0 + k) < (unsigned)g.W) << k;
        }
        // a tap outside the image gets an offset past the end of the buffer: the buffer load
        // returns 0 for it (no clamping, no masking of the loaded word)
        const unsigned corner = (unsigned)(((nb * g.H + ih0) * g.W + iw0) * g.Cpad);
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            if (t % PARTS != part) continue;
            const int kh = t / 3, kw = t % 3;
            const bool inb = ((rowin >> kh) & (colin >> kw) & 1u) != 0;
            po[px][t] = inb ? corner + (unsigned)((kh * g.W + kw) * g.Cpad) : 0x80000000u;
        }
        if (part == 0) {
            // pad <= 1: only the first or the last window row / column can be outside
            const unsigned rc = ((rowin & 1u) ^ 1u) | (((rowin >> 2) & 1u) ^ 1u) << 1;
            const unsigned cc = ((colin & 1u) ^ 1u) | (((colin >> 2) & 1u) ^ 1u) << 1;
            pm[px] = (int)(g.code_zero_pad ? 0u : rc * 4u + cc);
        }
    }
    __syncthreads();
    // ---- phase 1: 4 pixels x 4 channels per thread ---------------------------------------
    {
        if (c0 < g.C) {
            // the code tensor as a raw buffer: 32-bit lane offsets on a uniform base, and loads past
            // num_records (the out-of-image taps' offsets, 2^31 + channel) return 0
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
                (void*)a.a, 0, (int)((int64_t)g.Nb * g.H * g.W * g.Cpad), 0x00020000);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int pl = 4 * pg + q;
                const uint4 o0 = *(const uint4*)&po[pl][0], o1 = *(const uint4*)&po[pl][4], o2 = *(const uint4*)&po[pl][8];
                const unsigned off[9] = {o0.x, o0.y, o0.z, o0.w, o1.x, o1.y, o1.z, o1.w, o2.x};
                int w[9];
#pragma unroll
                for (int t = 0; t < 9; ++t) w[t] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, off[t] + (unsigned)c0, 0, 0);
                // two 4 x 4 byte transposes: out[e] = byte e of (w0, w1, w2, w3)
                int av[2][4];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const unsigned x0 = (unsigned)w[4 * h], x1 = (unsigned)w[4 * h + 1], x2 = (unsigned)w[4 * h + 2],
                                   x3 = (unsigned)w[4 * h + 3];
                    // perm(hi, lo, sel): selector byte values 0-3 pick from lo, 4-7 from hi
                    const unsigned t01l = __builtin_amdgcn_perm(x1, x0, 0x05010400u);  // x0.0 x1.0 x0.1 x1.1
                    const unsigned t01h = __builtin_amdgcn_perm(x1, x0, 0x07030602u);  // x0.2 x1.2 x0.3 x1.3
                    const unsigned t23l = __builtin_amdgcn_perm(x3, x2, 0x05010400u);
                    const unsigned t23h = __builtin_amdgcn_perm(x3, x2, 0x07030602u);
                    av[h][0] = (int)__builtin_amdgcn_perm(t23l, t01l, 0x05040100u);  // x0.0 x1.0 x2.0 x3.0
                    av[h][1] = (int)__builtin_amdgcn_perm(t23l, t01l, 0x07060302u);
                    av[h][2] = (int)__builtin_amdgcn_perm(t23h, t01h, 0x05040100u);
                    av[h][3] = (int)__builtin_amdgcn_perm(t23h, t01h, 0x07060302u);
                }
                const double* crow = &cst[pm[pl]][4 * cq];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int a8 = (int)__builtin_amdgcn_ubfe((unsigned)w[8], 8 * e, 8);  // tap 8 of channel e, low byte
                    int d = __builtin_amdgcn_sdot4(av[0][e], wq[e][0], 0, false);
                    d = __builtin_amdgcn_sdot4(av[1][e], wq[e][1], d, false);
                    d = __builtin_amdgcn_sdot4(a8, wq[e][2], d, false);
                    if (a.acc) tD[(4 * cq + e) * PITCH + pl] = d;
                    if (a.y) {
                        int sa = __builtin_amdgcn_sdot4(av[0][e], 0x01010101, 0, false);
                        sa = __builtin_amdgcn_sdot4(av[1][e], 0x01010101, sa, false);
                        sa = __builtin_amdgcn_sdot4(a8, 0x00000001, sa, false);
                        double y = g1[e] * (double)d + c2[e] * (double)sa + crow[e];
                        y = __builtin_fmax(y, relu_floor);
                        y = bs[e] * y + bh[e];
                        tY[(4 * cq + e) * PITCH + pl] = (float)y;
                    }
                }
            }
        }
    }
    __syncthreads();
    // ---- phase 2: lanes along pixels, channels round-robin over the wave groups; copy only
    const int pl = tid % PXB;
    const int64_t m = m0 + pl;
    if (m < total) {
    const int nb = (int)fastdiv((uint32_t)m, g.div_ohw), pix = (int)(m - (int64_t)nb * ohw);
    constexpr int STEP = 256 / PXB;  // wave groups that share the channels
    const int nch = g.C - cb < CHB ? g.C - cb : CHB;
    const int cl0 = tid / PXB;
    const int64_t i0 = ((int64_t)nb * g.C + cb + cl0) * ohw + pix;
    const int64_t istep = (int64_t)STEP * ohw;
    if (a.y) {
        float* yp = a.y + i0;
        const float* tp = tY + cl0 * PITCH + pl;
#pragma unroll 4
        for (int cl = cl0; cl < nch; cl += STEP) {
            const float v = *tp;
            if (NT)
                __builtin_nontemporal_store(v, yp);
            else
                *yp = v;
            yp += istep;
            tp += STEP * PITCH;
        }
    }
    if (a.acc) {
        int* dp = a.acc + i0;
        const int* tp = tD + cl0 * PITCH + pl;
#pragma unroll 4
        for (int cl = cl0; cl < nch; cl += STEP) {
            *dp = *tp;
            dp += istep;
            tp += STEP * PITCH;
        }
    }
    }  // m < total
    }  // tiles
}

// ---- 3 x 3, pad <= 1, stride 1 and 2: on the int8 matrix cores ----------------------------
// Streaming: 1 byte read and 4 written per output.  The kernel above is held by its vector instructions (MobileNet's 13
// layers within its pass, batch 256: 1096 us; here 855, at 3.2 TB/s).  Here the dot products go to the matrix cores, idle otherwise: v_mfma_i32_16x16x64_i8 multiplies 16 pixels by 16 channels over K = 4 taps x
// 16 channels, with filter codes on the diagonal of each tap's 16 x 16 block.  15 of 16 products are with
// zeros, and still the nine taps of 256 outputs are 3 instructions of 16 cycles.
//  * The output pixels of a tile are consecutive, so their inputs are one run of consecutive pixels (tap (0, 0) of the first
//    to tap (2, 2) of the last): loaded into LDS once, as it lies in memory.  An operand is 16 bytes per lane, 16
//    channels of one tap of one pixel; a tap outside the image reads 16 zero bytes.  A lane looks after 3 taps of
//    one pixel, not 9.  (Operands straight from memory: 1.9 times slower, a lane's 16 bytes are a line of their own.)
//  * Pixels are the rows of the product, so a lane gets 4 consecutive pixels of one channel: a 16-byte
//    store into NCHW without another turn through LDS, and the channel's factors are the lane's own registers.
// BW: there is a weight offset, so that the pixel sums of the codes count (3 more matrix instructions, against ones).
template <int NCG, bool BW, bool NT>
__global__ __launch_bounds__(256, BW && NCG == 4 ? 3 : 4) void k_dwconv3_mm(DwConvArgs a)
{
    typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));
    typedef int v4iu __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int CHB = 16 * NCG, RB = 16 * NCG;  // channels of a block = bytes of a pixel in LDS
    // LDS: [run of pixels][16 zero bytes][classes][CHB] constants
    extern __shared__ __attribute__((aligned(16))) int8_t dw_smem[];
    const ConvGeom& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned lds0 = (unsigned)(uintptr_t)dw_smem;
    const int zoff = a.run * RB;
    double* cst = (double*)(dw_smem + zoff + 16);
    const int ohw = g.OH * g.OW, total = g.Nb * ohw, total_in = g.Nb * g.H * g.W;  // (below 2^31)
    const int cb = (int)blockIdx.y * CHB;
    const EpiArgs& ep = a.ep;
    const bool has_bn = ep.bn_scale != nullptr;
    const double aa = (double)ep.alpha_a.s, ba = (double)ep.beta_a.s;
    // input pixel of tap (0, 0) of output pixel m, and the window's first row and column
    auto corner = [&](int m, int& ih0, int& iw0) {
        const int nb = (int)fastdiv((uint32_t)m, g.div_ohw), pix = m - nb * ohw;
        const int oh = (int)fastdiv((uint32_t)pix, g.div_ow), ow = pix - oh * g.OW;
        ih0 = oh * g.stride - g.pad;
        iw0 = ow * g.stride - g.pad;
        return (nb * g.H + ih0) * g.W + iw0;
    };
    // chunk swizzle of a pixel's LDS row: the 16-byte reads of 16 consecutive rows hit all banks
    auto swizzle = [](int row) { return NCG == 4 ? swz(row) : (row >> 3) & 1; };
    // each XCD gets one contiguous run of pixels (grid.x is a multiple of 8), so that window rows meet in its L2;
    // the groups of 16 pixels are dealt out evenly
    const int chunk = (int)(gridDim.x >> 3);
    const int bid = (int)(blockIdx.x & 7) * chunk + (int)(blockIdx.x >> 3);
    const int64_t ngroups = ((int64_t)total + 15) >> 4;
    const int first = (int)(ngroups * bid / gridDim.x) * 16;
    const int last = (int)(ngroups * (bid + 1) / gridDim.x) * 16;
    // loads the run of tile t0 and returns its first pixel
    auto load_run = [&](int t0) {
        int t1 = t0 + a.tile < last ? t0 + a.tile : last, d0, d1;
        t1 = t1 < total ? t1 : total;
        const int run0 = corner(t0, d0, d1), rows = corner(t1 - 1, d0, d1) + 2 * g.W + 3 - run0;
        for (int n = wave; n * (64 / NCG) < rows; n += 4) {
            const int lin = n * 64 + lane, row = lin / NCG, q = lin % NCG;
            int px = run0 + row;
            px = px < 0 ? 0 : (px < total_in ? px : total_in - 1);  // past the tensor: only taps outside an image point there
            dma16(a.a + (int64_t)px * g.Cpad + cb + ((q ^ swizzle(row)) << 4), lds0 + (unsigned)(n * 1024));
        }
        return run0;
    };
    if (first >= last) return;
    // (pad <= 1 and an image at least as long as the window: a window is cut at one end of an
    // axis at most, 3 x 3 classes; the others exist only for images shorter than 3)
    const int nax = g.H < 3 || g.W < 3 ? 4 : 3;
    if (tid < 4) ((int*)(dw_smem + zoff))[tid] = 0;
    if (a.y) {
        for (int idx = tid; idx < nax * nax * CHB; idx += 256) {
            const int k = idx / CHB, cl = idx - k * CHB;
            const int c = cb + cl < g.C ? cb + cl : g.C - 1;
            const int* wr = (const int*)(a.w + (int64_t)c * a.Kp);
            const int rc = k / nax, cc = k - rc * nax;
            unsigned cnt[3] = {0, 0, 0};
            int kv = 0;
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const int kh = t / 3, kw = t % 3;
                const bool out = (kh == 0 && (rc & 1)) || (kh == 2 && (rc & 2)) || (kw == 0 && (cc & 1)) || (kw == 2 && (cc & 2));
                kv += !out;
                cnt[t >> 2] |= (unsigned)!out << (8 * (t & 3));
            }
            int sw = __builtin_amdgcn_sdot4(wr[0], (int)cnt[0], 0, false);
            sw = __builtin_amdgcn_sdot4(wr[1], (int)cnt[1], sw, false);
            sw = __builtin_amdgcn_sdot4(wr[2] & 0xff, (int)cnt[2], sw, false);
            const double aw = pval(ep.alpha_w, c), bw = pval(ep.beta_w, c);
            cst[idx] = ba * aw * (double)sw + (double)kv * ba * bw;
        }
    }
    // ---- once per wave: filter operands, channel factors, this lane's taps ----------------
    // B operand: column = channel l15, k = 16 lk + byte: tap 4 h + lk, channel = byte, so a lane's only non-zero byte is l15
    v4i wd[NCG][3], ones;
    double g1[NCG], c2[NCG], bs[NCG], bh[NCG];
#pragma unroll
    for (int j = 0; j < 4; ++j) ones[j] = l15 >> 2 == j ? 1 << (8 * (l15 & 3)) : 0;
#pragma unroll
    for (int i = 0; i < NCG; ++i) {
        const bool cok = cb + 16 * i + l15 < g.C;
        const int c = cok ? cb + 16 * i + l15 : g.C - 1;
#pragma unroll
        for (int h = 0; h < 3; ++h) {
            const int t = 4 * h + lk;
            const int v = cok && t < 9 ? (int)(uint8_t)a.w[(int64_t)c * a.Kp + (t < 9 ? t : 0)] : 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) wd[i][h][j] = l15 >> 2 == j ? v << (8 * (l15 & 3)) : 0;
        }
        g1[i] = c2[i] = bh[i] = 0.0;
        bs[i] = 1.0;
        if (a.y) {
            g1[i] = aa * pval(ep.alpha_w, c);
            if (BW) c2[i] = aa * pval(ep.beta_w, c);
            bs[i] = has_bn ? (double)ep.bn_scale[c] : 1.0;
            bh[i] = (has_bn && ep.bn_shift) ? (double)ep.bn_shift[c] : 0.0;
        }
    }
    const double relu_floor = __builtin_canonicalize(ep.relu ? 0.0 : -__builtin_inf());
    int tkh[3], tkw[3];
#pragma unroll
    for (int h = 0; h < 3; ++h) {
        const int t = 4 * h + lk;
        tkh[h] = t / 3;
        tkw[h] = t - 3 * tkh[h];
    }
    for (int t0 = first; t0 < last; t0 += a.tile) {
        const int t1 = t0 + a.tile < last ? t0 + a.tile : last;  // pixels t0 .. t1 - 1
        if (t0 != first) __syncthreads();  // the run of the tile before has been read
        const int run0 = load_run(t0);     // (issued before the set-up it only delays the set-up's own loads)
        wait_vm<0>();
        __syncthreads();
        for (int m0 = t0 + wave * 16; m0 < t1; m0 += 64) {
            // the pixel whose taps this lane multiplies (pixels past the end repeat the last one; never stored)
            const int m = m0 + l15 < total ? m0 + l15 : total - 1;
            int ih0, iw0;
            const int row0 = corner(m, ih0, iw0) - run0;
            int addr[3];
#pragma unroll
            for (int h = 0; h < 3; ++h) {
                const bool inb = (unsigned)(ih0 + tkh[h]) < (unsigned)g.H && (unsigned)(iw0 + tkw[h]) < (unsigned)g.W && tkh[h] < 3;
                const int row = row0 + tkh[h] * g.W + tkw[h];
                addr[h] = inb ? row * RB + (swizzle(row) << 4) : -1;
            }
            // border class of that pixel; a lane stores pixels 4 lk .. + 3
            const unsigned rc = (unsigned)(ih0 < 0) | (unsigned)(ih0 + 2 >= g.H) << 1, cc = (unsigned)(iw0 < 0) | (unsigned)(iw0 + 2 >= g.W) << 1;
            const int cls = g.code_zero_pad ? 0 : (int)(rc * nax + cc) * CHB;
            const double* crow[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) crow[r] = cst + __shfl(cls, 4 * lk + r, 64) + l15;
            const int mq = m0 + 4 * lk;
            auto base_of = [&](int p) {  // output offset of pixel p, channel 0
                const int n = (int)fastdiv((uint32_t)p, g.div_ohw);
                return (int64_t)n * g.C * ohw + (p - n * ohw);
            };
            // a quad of pixels that lies in one image is stored with one instruction (16 bytes on any multiple of 4)
            const int nbq = (int)fastdiv((uint32_t)(mq < total ? mq : 0), g.div_ohw), pixq = mq - nbq * ohw;
            const bool quad = pixq + 4 <= ohw && mq < total;
            const int64_t obase = (int64_t)nbq * g.C * ohw + pixq;
#pragma unroll
            for (int i = 0; i < NCG; ++i) {
                v4i d = {0, 0, 0, 0}, s = {0, 0, 0, 0};
#pragma unroll
                for (int h = 0; h < 3; ++h) {
                    const v4i x = *(const v4i*)(dw_smem + (addr[h] < 0 ? zoff : addr[h] ^ (16 * i)));
                    d = __builtin_amdgcn_mfma_i32_16x16x64_i8(x, wd[i][h], d, 0, 0, 0);
                    if (BW) s = __builtin_amdgcn_mfma_i32_16x16x64_i8(x, ones, s, 0, 0, 0);
                }
                v4f y = {0.f, 0.f, 0.f, 0.f};
                if (a.y)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        double v = BW ? g1[i] * (double)d[r] + c2[i] * (double)s[r] + crow[r][16 * i] : g1[i] * (double)d[r] + crow[r][16 * i];
                        v = __builtin_fmax(v, relu_floor);
                        y[r] = (float)(bs[i] * v + bh[i]);
                    }
                const int c = cb + 16 * i + l15;
                if (c >= g.C || mq >= total) continue;
                const int64_t coff = (int64_t)c * ohw;
                if (quad) {
                    if (a.y) {
                        if (NT)
                            __builtin_nontemporal_store(y, (v4fu*)(a.y + obase + coff));
                        else
                            *(v4fu*)(a.y + obase + coff) = y;
                    }
                    if (a.acc) *(v4iu*)(a.acc + obase + coff) = d;
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (mq + r >= total) break;
                        const int64_t o = base_of(mq + r) + coff;
                        if (a.y) {
                            if (NT)
                                __builtin_nontemporal_store(y[r], a.y + o);
                            else
                                a.y[o] = y[r];
                        }
                        if (a.acc) a.acc[o] = d[r];
                    }
                }
            }
        }
    }
}

// Input pixels of the run of `t` consecutive output pixels, at most
int64_t dw_run(const ConvGeom& g, int t) { return conv_span(g.H, g.W, g.OH, g.OW, 3, 3, g.stride, t); }

}  // namespace

hipError_t launch_dwconv(const DwConvArgs& a, hipStream_t st)
{
    const int64_t total = (int64_t)a.g.Nb * a.g.OH * a.g.OW;
    const bool big = total * a.g.C * 4 > ((int64_t)128 << 20);
    const std::true_type yes{};
    const std::false_type no{};
    // The run of a tile's inputs decides: 64 pixels and more have to have it in 48 KB, so that three blocks fit a CU beside
    // their constants (longer tiles where 32 KB hold them, for four), and it has to be no more than four times the
    // inputs that belong to the tile.  MobileNet's 64 channels of 112 wide, stride 2, 44 KB and 2.7 times: 122 -> 89 us; but
    // 4 x 64 x 60 x 340, stride 1, 11.7 times: 16.3 -> 19.8, and 2 x 32 x 300 x 330, stride 2, 5.7 times: 8.8 -> 9.4.
    // Elsewhere (wide images, strides whose runs are mostly skipped) the kernel without it.
    const int64_t rb = a.g.C <= 32 ? 32 : 64;
    int tile = 0;
    if (a.g.KH == 3 && a.g.KW == 3 && a.g.pad <= 1 && a.g.stride <= 2) {
        for (tile = 256; tile > 64 && dw_run(a.g, tile) * rb > 32 * 1024; tile /= 2) {}
        const int64_t run = dw_run(a.g, tile);
        if (run * rb > 48 * 1024 || run > 4 * tile * a.g.stride * a.g.stride) tile = 0;
    }
    // (the hint only for whole 64-byte halves of lines: 128 x 463 x 13 x 98 134 us without, 305 with it)
    const bool halves = (a.g.OH * a.g.OW) % 16 == 0 && ((uintptr_t)a.y & 63) == 0;
    const bool vector = a.g.KH == 3 && a.g.KW == 3 && a.g.pad <= 1 && (int64_t)a.g.Nb * a.g.H * a.g.W * a.g.Cpad < ((int64_t)1 << 31);
    if (tile && a.y && vector && !halves && dw_vector_stores(a.g.C, a.g.stride, total * a.g.C * 4, a.acc != nullptr)) tile = 0;
    if (tile) {
        // (an infinite alpha_a makes c2 = alpha_a * 0 a NaN: kept by the form with the sums)
        const bool bw = a.ep.beta_w.ptr || a.ep.beta_w.s != 0.0f || !std::isfinite(a.ep.alpha_a.s);
        const bool nt = big && halves;
        DwConvArgs b = a;
        b.tile = tile;
        b.run = (int)((dw_run(a.g, tile) + 31) / 32 * 32);  // whole KiB of LDS
        const size_t lds = (size_t)(b.run * rb + 16 + 16 * rb * 8);
        const int64_t slabs = (a.g.C + rb - 1) / rb;
        // four blocks per CU, all of them resident, each with an even share of the pixels: the set-up is paid once.  MobileNet's
        // 13 layers at batch 256, each in a loop of its own: 732 us, with two rounds of them 744, with three 767.  A wave takes 16 pixels at a time.
        // (8 blocks a slab at least, one per XCD, however many channels there are: at most 2^22 / 9)
        const int64_t most = (total + 63) / 64;
        int64_t nb = 1024 / slabs < most ? 1024 / slabs : most;
        nb = nb < 1 ? 8 : (nb + 7) / 8 * 8;
        const dim3 grid((unsigned)nb, (unsigned)slabs);
        auto launch = [&](auto ncg, auto w, auto n) {
            hipLaunchKernelGGL((k_dwconv3_mm<decltype(ncg)::value, decltype(w)::value, decltype(n)::value>), grid, dim3(256), lds, st, b);
        };
        auto pick = [&](auto ncg) {
            if (bw)
                nt ? launch(ncg, yes, yes) : launch(ncg, yes, no);
            else
                nt ? launch(ncg, no, yes) : launch(ncg, no, no);
        };
        if (rb == 32)
            pick(std::integral_constant<int, 2>{});
        else
            pick(std::integral_constant<int, 4>{});
        return hipGetLastError();
    }
    if (vector) {
        const bool nt = big;
        const size_t ntile = (a.y ? 1 : 0) + (a.acc ? 1 : 0);  // LDS tiles
        DwConvArgs b = a;
        // enough blocks for a dozen per CU, each walking up to 16 pixel tiles
        const int chb = a.g.C <= 32 ? 32 : 64;
        const int64_t tiles = (total + 4096 / chb - 1) / (4096 / chb) * ((a.g.C + chb - 1) / chb);
        int64_t tpb = tiles / (256 * 12);
        b.tiles_per_block = (int)(tpb < 1 ? 1 : (tpb > 16 ? 16 : tpb));
        if (a.g.C <= 32) {
            const int64_t nb = ((total + 127) / 128 + b.tiles_per_block - 1) / b.tiles_per_block;
            if (nb <= 0 || nb > 0x7fffffff) return hipErrorInvalidValue;
            const dim3 grid((unsigned)nb, (unsigned)((a.g.C + 31) / 32));
            if (nt)
                hipLaunchKernelGGL((k_dwconv3<32, true>), grid, dim3(256), ntile * 32 * 129 * 4, st, b);
            else
                hipLaunchKernelGGL((k_dwconv3<32, false>), grid, dim3(256), ntile * 32 * 129 * 4, st, b);
        } else {
            const int64_t nb = ((total + 63) / 64 + b.tiles_per_block - 1) / b.tiles_per_block;
            if (nb <= 0 || nb > 0x7fffffff) return hipErrorInvalidValue;
            const dim3 grid((unsigned)nb, (unsigned)((a.g.C + 63) / 64));
            if (nt)
                hipLaunchKernelGGL((k_dwconv3<64, true>), grid, dim3(256), ntile * 64 * 65 * 4, st, b);
            else
                hipLaunchKernelGGL((k_dwconv3<64, false>), grid, dim3(256), ntile * 64 * 65 * 4, st, b);
        }
        return hipGetLastError();
    }
    const int64_t blocks = (total + DW_PX - 1) / DW_PX;
    if (blocks <= 0 || blocks > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks, (unsigned)(a.g.Cpad / DW_CH));
    if (a.g.KH == 3 && a.g.KW == 3)
        hipLaunchKernelGGL(k_dwconv<3>, grid, dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL(k_dwconv<0>, grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace rtn
