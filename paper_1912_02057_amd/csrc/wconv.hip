// Weight-only ternary convolution: fp32 activations (NCHW) x ternary weights, on the bf16 matrix
// cores, in one kernel.
//
//   y[n][o][oh][ow] = BN(relu(alpha_w[o] * sum x * t_w))
//
// Every fp32 activation is split exactly into three bf16 terms by truncation, x = hi + mid + lo (8
// significand bits each; both residuals are exact in fp32), and each term is multiplied with the
// weights (-1, 0, +1, exact in bf16) into the same fp32 accumulators.
//
// The contraction runs in chunks of 16 CS channels.  A block loads, for one chunk, the fp32 inputs
// its BQ output pixels need -- straight from the NCHW tensor, lanes along pixels, so a load is 256
// contiguous bytes -- splits and transposes them in registers and keeps the three bf16 images
// [term][row][16 channels] in LDS while all taps of the window are multiplied from it:
//   RUN     output pixel m reads input pixel i(m) + kh W + kw of the flattened (image, row, column)
//           index space, so the tile needs one contiguous run of input pixels; LDS row = place in
//           the run, a tap is a row offset, a tap outside the image reads the zero row.
//   GATHER  (every window; the only form of those other than 3 x 3 and 5 x 5 and of runs that do not
//           fit) LDS row = output pixel, one tap at a time; a chunk is then (16 CS channels, one tap).
// Which of the forms runs is estimated from measured constants (kForms).
// The next chunk's inputs are loaded into registers while this chunk is multiplied.  Weights are
// read from global memory in the order the matrix instruction takes them (k_codes_to_frag), PD
// steps ahead; they are shared by all blocks and stay in L2.  KG > 1: groups of four waves take
// every KG-th chunk each, with LDS images of their own, and add up at the end -- for grids too
// small to fill the chip.  The order of the fp32 sums, and with it the last bits of a result, is the
// form's: the same layer may round differently at another batch size.
//
// What it replaced wrote the three terms to memory (6 bytes per activation) in a pass of its own
// and re-read them once per tap and filter tile through LDS, with the weights fetched again for
// each term.  ResNet-18's 19 layer shapes, GPU time (before -> this kernel with 64-bit addresses): batch 256
// 4.48 -> 2.44 ms, batch 64 1.73 -> 0.85 ms, batch 1 1.01 -> 0.16 ms; with buffer resources (a scalar base, the lane's
// offset, a scalar one: no address arithmetic per load) and whole tiles stored without tests batch 256 takes 0.935 times
// that (2599 -> 2429 us on one machine; machines differ by 5 %).  GATHER re-reads and re-splits its inputs once per tap, which
// the split pass did not: over 857 random geometries with windows of 1 to 7 and strides of 1 to 4 this
// kernel takes 0.43 times the time at the median and more than 1.02 times on 7, 1.14 times at worst: nearly
// all windows of 4 and more that are strided or 5 and more wide, at some 10000 output pixels and more.
#include "tmm_kernel.h"

namespace rtn {

namespace {

struct WcParams {
    TmmParams t;        // RP = O, RQ = output pixels, g, y, cst_cls, ep, nt_out and the tiling
    const float* x;
    const int8_t* w;    // fragment-ordered bf16 weights
    int nchunk;         // chunks of 16 CS channels (GATHER: times taps)
    int span;           // RUN: rows of the image a tile may use
    FastDiv div_hw;     // by H W
    FastDiv div_tap;    // GATHER: by the taps
    int dc, dtap;       // GATHER: KG chunks on = dc channel chunks and dtap taps
    unsigned kw_inv;    // tap / KW = tap * kw_inv >> 16 for the 49 taps there are at most
};

// Two floats -> their bf16 terms, packed; exact by truncation.
__device__ __forceinline__ void split2(float a, float b, unsigned& h, unsigned& m, unsigned& l)
{
    const unsigned ua = __float_as_uint(a), ub = __float_as_uint(b);
    h = __builtin_amdgcn_perm(ub, ua, 0x07060302u);
    const float ra = a - __uint_as_float(ua & 0xffff0000u), rb = b - __uint_as_float(ub & 0xffff0000u);
    const unsigned va = __float_as_uint(ra), vb = __float_as_uint(rb);
    m = __builtin_amdgcn_perm(vb, va, 0x07060302u);
    const float sa = ra - __uint_as_float(va & 0xffff0000u), sb = rb - __uint_as_float(vb & 0xffff0000u);
    l = __builtin_amdgcn_perm(__float_as_uint(sb), __float_as_uint(sa), 0x07060302u);
}

// A second image, so that a chunk costs one barrier instead of two, where the LDS leaves room for as
// many blocks as without it.
template <bool GATHER, int KG, int BQ>
constexpr int wc_images()
{
    return GATHER && KG == 1 && BQ == 128 ? 2 : 1;
}

// NTAP: taps of the window, 0 = GATHER.  RMAX: LDS rows per image (a multiple of 64).  BIG (GATHER): the
// input offsets within a tile do not fit 32 bits.
template <int BP, int BQ, int WGP, int WGQ, int KG, int MINW, int NTAP, int CS, int RMAX, bool BIG>
__global__ __launch_bounds__(64 * WGP * WGQ * KG, MINW) void k_wconv(WcParams prm)
{
    constexpr bool GATHER = NTAP == 0;
    constexpr int WP = BP / WGP, WQ = BQ / WGQ, TP = WP / 32, TQ = WQ / 32;
    constexpr int KK = NTAP == 9 ? 3 : (NTAP == 25 ? 5 : 1);      // window side (RUN)
    constexpr int NSTEP = GATHER ? CS : CS * NTAP;                // steps of 16 channels x one tap per chunk
    constexpr int PD = NTAP == 9 ? 3 : (NTAP == 25 ? 5 : CS);     // weight prefetch distance
    constexpr int PLANE = (RMAX + 1) * 32;                        // bytes of one term's image (last row: zeros)
    constexpr int IMG = CS * 3 * PLANE;
    constexpr int NBUF = wc_images<GATHER, KG, BQ>();              // images per group
    constexpr int NW = WGP * WGQ;                                 // waves per group
    constexpr int NU = 2 * CS * RMAX / (64 * NW);                 // (row, 8 channels) units per thread
    static_assert((NW == 4 || NW == 1) && TP >= 1 && TQ >= 1, "four waves or one per group");
    static_assert(NSTEP % PD == 0 && RMAX % 64 == 0 && (2 * CS * RMAX) % (64 * NW) == 0 && (!GATHER || RMAX == BQ), "chunk shape");
    static_assert(NTAP == 0 || (!BIG && (NTAP == 9 || NTAP == 25)), "window");

    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave16 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wave16 % NW, kg = wave16 / NW;
    const int wp = wave / WGQ, wq = wave % WGQ;
    const ConvGeom& g = prm.t.g;
    int tileP, tileQ;
    if (!block_tile(prm.t, tileP, tileQ)) return;
    const int p0 = tileP * BP, q0 = tileQ * BQ;
    int8_t* img = smem + kg * IMG;  // NBUF 2 (one group): this chunk's image
    const int HW = g.H * g.W, ntap = g.KH * g.KW;

    // output pixel -> flattened index of its tap (0, 0) (may be negative), and the in-image taps
    auto origin = [&](int m, int& ih0, int& iw0, int& nb) {
        const int ohw = g.OH * g.OW;
        nb = (int)fastdiv((uint32_t)m, g.div_ohw);
        const int pix = m - nb * ohw;
        const int oh = (int)fastdiv((uint32_t)pix, g.div_ow), ow = pix - oh * g.OW;
        ih0 = oh * g.stride - g.pad, iw0 = ow * g.stride - g.pad;
    };
    int oh0, ow0, onb;
    origin(q0, oh0, ow0, onb);
    // (Nb H W < 2^31, so flattened indices are ints; windows reach at most a few rows past the ends)
    const int imin = (onb * g.H + oh0) * g.W + ow0;  // RUN: flattened index of row 0
    const int total_px = g.Nb * HW;
    const int nb0 = (int)fastdiv((uint32_t)(imin < 0 ? 0 : imin), prm.div_hw);
    const float* xbase = prm.x + (int64_t)(GATHER ? onb : nb0) * g.C * HW;

    // ---- this thread's units: rows of the image and which 8 channels of a chunk ----------------
    // unit i of a wave: 64 consecutive rows (lanes) x channels 8 hs .. 8 hs + 7
    using Off = std::conditional_t<BIG, int64_t, uint32_t>;
    constexpr int NSEG = RMAX / 64;
    Off voff[NU];
    int tmask[GATHER ? NU : 1];
    (void)tmask;
#pragma unroll
    for (int i = 0; i < NU; ++i) {
        const int r = ((wave + NW * i) % NSEG) * 64 + lane;
        if (GATHER) {
            const int m = q0 + r < prm.t.RQ ? q0 + r : prm.t.RQ - 1;
            int ih0, iw0, nb;
            origin(m, ih0, iw0, nb);
            tmask[i] = tap_mask(ih0, g.KH, g.H) | tap_mask(iw0, g.KW, g.W) << 8;
            if (BIG)  // (+ the tap's offset: in range when the tap is in the image)
                voff[i] = (Off)(((int64_t)(nb - onb) * g.C * HW + (int64_t)ih0 * g.W + iw0) * 4);
            else
                voff[i] = (Off)((unsigned)(nb - onb) * (unsigned)(g.C * HW) + (unsigned)(ih0 * g.W + iw0)) * 4u;
        } else {
            int f = imin < total_px - r ? imin + r : total_px - 1;
            f = f < 0 ? 0 : f;
            const int nb = (int)fastdiv((uint32_t)f, prm.div_hw);
            voff[i] = (Off)((unsigned)(nb - nb0) * (unsigned)(g.C * HW) + (unsigned)(f - nb * HW)) * 4u;
        }
    }
    // The chunks of this group of waves: every KG-th, channels outermost.  (Counted, not divided out:
    // a scalar division is a chain of some 25 dependent instructions, and GATHER took seven a chunk.)
    struct Chunk {
        int c, tap;  // channels 16 CS c and up; GATHER: the tap
    };
    const int nch = prm.nchunk;
    auto next_chunk = [&](Chunk& ck) {  // (past the last one: RUN repeats it, GATHER has no channels to load)
        ck.c += GATHER ? prm.dc : KG;
        if (GATHER && (ck.tap += prm.dtap) >= ntap) ck.tap -= ntap, ++ck.c;
        if (!GATHER && ck.c >= nch) ck.c = nch - 1;
    };
    float xr[NU][8];
    unsigned xtok = 0;  // GATHER, bit i: unit i's tap is in the image
    auto load_x = [&](const Chunk& ck) {
        const int c0 = ck.c * 16 * CS;
        const int kh = GATHER ? (int)((unsigned)ck.tap * prm.kw_inv >> 16) : 0, kw = GATHER ? ck.tap - kh * g.KW : 0;
        const int64_t toff = GATHER ? (int64_t)kh * g.W + kw : 0;
        xtok = 0;
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            const int hs = (wave + NW * i) / NSEG, c = c0 + 8 * hs;
            const char* xc = (const char*)(xbase + (int64_t)c * HW);
            if constexpr (GATHER) {
                // Loads only: using a value here (a select, say) would wait for it and leave nothing in
                // flight behind the matrix work.  What must not count -- a tap outside the image, a
                // channel past the last -- is loaded from somewhere valid and zeroed in store_x.
                const bool tok = ((tmask[i] >> kh) & (tmask[i] >> (8 + kw)) & 1) != 0;
                xtok |= (unsigned)tok << i;
                if (c >= g.C) continue;  // (wave-uniform)
                const Off o = tok ? (Off)(voff[i] + (Off)(toff * 4)) : (Off)0;  // outside: the tile's first element
                const int last = g.C - 1 - c;
#pragma unroll
                for (int e = 0; e < 8; ++e) xr[i][e] = *(const float*)(xc + (Off)(e < last ? e : last) * (Off)HW * 4 + o);
            } else {
                if (((wave + NW * i) % NSEG) * 64 >= prm.span) continue;  // (wave-uniform, like the channel tail)
                // (a scalar base, the lane's offset and a scalar one: nothing to add per load)
                const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)xc, 0, -1, 0x00020000);
                auto load = [&](int e) { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)voff[i], (int)(4u * e * (unsigned)HW), 0)); };
                if (c + 8 <= g.C) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) xr[i][e] = load(e);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) xr[i][e] = c + e < g.C ? load(e) : 0.0f;
                }
            }
        }
    };
    auto store_x = [&](const Chunk& ck) {
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            if (!GATHER && ((wave + NW * i) % NSEG) * 64 >= prm.span) continue;
            const int r = ((wave + NW * i) % NSEG) * 64 + lane, hs = (wave + NW * i) / NSEG;
            if constexpr (GATHER) {
                const int left = g.C - ck.c * 16 * CS - 8 * hs;
                if (left < 8) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) xr[i][e] = e < left ? xr[i][e] : 0.0f;
                }
                if (ntap > 1) {  // (a single tap is never padded)
#pragma unroll
                    for (int e = 0; e < 8; ++e) xr[i][e] = (xtok >> i & 1) ? xr[i][e] : 0.0f;
                }
            }
            unsigned h[4], m[4], l[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) split2(xr[i][2 * e], xr[i][2 * e + 1], h[e], m[e], l[e]);
            int8_t* d = img + (hs >> 1) * 3 * PLANE + r * 32 + ((((r >> 3) ^ hs) & 1) << 4);
            *(uint4*)d = make_uint4(h[0], h[1], h[2], h[3]);
            *(uint4*)(d + PLANE) = make_uint4(m[0], m[1], m[2], m[3]);
            *(uint4*)(d + 2 * PLANE) = make_uint4(l[0], l[1], l[2], l[3]);
        }
    };

    // ---- weights: fragment (32-filter tile, 16-channel slice, tap) is rows x 2 halves x 16 bytes ---
    const int nslice = g.Cpad >> 4;  // 16-channel slices the weights hold per tap
    // (through buffer resources: a scalar base per 32-filter tile, of at most 2^28 bytes, a lane offset and a scalar offset)
    __amdgpu_buffer_rsrc_t wrsrc[TP];
    unsigned wlane[TP], wstep[TP];
    const int lastpt = (prm.t.RP - 1) >> 5;
#pragma unroll
    for (int t = 0; t < TP; ++t) {
        int pt = (p0 + wp * WP) / 32 + t;
        pt = pt < lastpt ? pt : lastpt;
        const int rows = prm.t.RP - pt * 32 < 32 ? prm.t.RP - pt * 32 : 32;
        const int row = (lane & 31) < rows ? (lane & 31) : rows - 1;
        wrsrc[t] = __builtin_amdgcn_make_buffer_rsrc((void*)(prm.w + (int64_t)pt * 32 * ntap * g.Cpad * 2), 0, 0x7fffffff, 0x00020000);
        wlane[t] = (unsigned)(half * rows + row) * 16;
        wstep[t] = (unsigned)rows * 32;
    }
    v4i pw[PD][TP];
    // step s of a chunk
    auto load_w = [&](const Chunk& ck, int s, v4i* dst) {
        if constexpr (!GATHER && CS == 1) {  // a chunk's steps follow each other
            const unsigned idx = (unsigned)(ck.c * NTAP);
#pragma unroll
            for (int t = 0; t < TP; ++t)
                dst[t] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wrsrc[t], (int)wlane[t], (int)(idx * wstep[t] + s * wstep[t]), 0));
            return;
        }
        int slice = ck.c * CS + (GATHER ? s : s / (NTAP ? NTAP : 1));
        const int tap = GATHER ? ck.tap : s % (NTAP ? NTAP : 1);
        slice = slice < nslice ? slice : nslice - 1;  // past the end: multiplied with zero activations
        const unsigned idx = (unsigned)(slice * ntap + tap);
#pragma unroll
        for (int t = 0; t < TP; ++t)
            dst[t] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wrsrc[t], (int)wlane[t], (int)(idx * wstep[t]), 0));
    };

    // ---- fragment rows of this lane's output pixels ------------------------------------------
    int row0[TQ];
    unsigned vm[TQ];
#pragma unroll
    for (int j = 0; j < TQ; ++j) {
        const int ml = wq * WQ + j * 32 + (lane & 31);
        row0[j] = ml;
        vm[j] = 0;
        if (!GATHER) {
            const int m = q0 + ml < prm.t.RQ ? q0 + ml : prm.t.RQ - 1;
            int ih0, iw0, nb;
            origin(m, ih0, iw0, nb);
            row0[j] = (nb * g.H + ih0) * g.W + iw0 - imin;
            vm[j] = (unsigned)(tap_mask(ih0, KK, g.H) | tap_mask(iw0, KK, g.W) << 8);
        }
    }
    // the channels' epilogue factors: rows alpha, BN scale, BN shift of the prepared table
    constexpr int RED = (KG - 1) * BP * BQ * 4;                   // the groups' sums, over the images
    double* tab = (double*)(smem + (KG * NBUF * IMG > RED ? KG * NBUF * IMG : RED));
    for (int e = tid; e < 3 * BP; e += 64 * NW * KG) {
        const int k = e / BP, o = p0 + e % BP;
        tab[e] = prm.t.cst_cls[(k ? k + 1 : 0) * ((g.O + 1) & ~1) + (o < prm.t.RP ? o : prm.t.RP - 1)];
    }
    // every image's zero row
    if (tid < KG * CS * 3 * 2) *(uint4*)(smem + (tid / (CS * 6)) * IMG + ((tid / 2) % (CS * 3)) * PLANE + RMAX * 32 + (tid & 1) * 16) = make_uint4(0, 0, 0, 0);

    v16f acc[TP][TQ];
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
        for (int j = 0; j < TQ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    // a group of one wave needs no barrier: its LDS accesses execute in order
    auto group_sync = [&]() {
        if constexpr (NW == 1) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
    };
    __syncthreads();  // the zero rows
    const int niter = (nch + KG - 1) / KG;
    const int kgc = GATHER ? (int)fastdiv((uint32_t)kg, prm.div_tap) : (kg < nch ? kg : nch - 1);
    Chunk cur = {kgc, GATHER ? kg - kgc * ntap : 0}, nxt = cur;
#pragma unroll
    for (int s = 0; s < PD; ++s) load_w(cur, s, pw[s]);
    load_x(cur);
    for (int it = 0; it < niter; ++it) {
        if (NBUF == 1 && it) group_sync();  // everybody is done with the previous chunk's image
        if (NBUF == 2) img = smem + (it & 1) * IMG;
        store_x(cur);
        next_chunk(nxt);
        if (it + 1 < niter) load_x(nxt);
        const bool live = it * KG + kg < nch;
        group_sync();
        if (KG == 1 || live) {
#pragma unroll
            for (int s = 0; s < NSTEP; ++s) {
                const int cs = GATHER ? s : s / (NTAP ? NTAP : 1), tap = GATHER ? 0 : s % (NTAP ? NTAP : 1);
                const int kh = tap / KK, kw = tap % KK;
                v4i fq[TQ][3];
#pragma unroll
                for (int j = 0; j < TQ; ++j) {
                    const int rr = GATHER ? row0[j] : row0[j] + kh * g.W + kw;
                    int a = rr * 32 + ((((rr >> 3) ^ half) & 1) << 4);
                    if (!GATHER) a = ((vm[j] >> kh) & (vm[j] >> (8 + kw)) & 1) ? a : RMAX * 32;
#pragma unroll
                    for (int q = 0; q < 3; ++q) fq[j][q] = *(const v4i*)(img + cs * 3 * PLANE + q * PLANE + a);
                }
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int i = 0; i < TP; ++i)
#pragma unroll
                        for (int j = 0; j < TQ; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, pw[s % PD][i]),
                                                                               __builtin_bit_cast(v8bf, fq[j][q]), acc[i][j], 0, 0, 0);
                if (s + PD < NSTEP)
                    load_w(cur, s + PD, pw[s % PD]);
                else
                    load_w(nxt, s + PD - NSTEP, pw[s % PD]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        cur = nxt;
    }

    // ---- KG groups -> one sum ------------------------------------------------------------------
    __syncthreads();
    if constexpr (KG > 1) {
        float* red = (float*)smem;  // [KG - 1][NW waves][TP * TQ * 16][64]
        constexpr int NR = TP * TQ * 16;
        if (kg > 0) {
#pragma unroll
            for (int i = 0; i < TP; ++i)
#pragma unroll
                for (int j = 0; j < TQ; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) red[(((kg - 1) * NW + wave) * NR + (i * TQ + j) * 16 + r) * 64 + lane] = acc[i][j][r];
        }
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int k = 1; k < KG; ++k)
#pragma unroll
            for (int i = 0; i < TP; ++i)
#pragma unroll
                for (int j = 0; j < TQ; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][j][r] += red[(((k - 1) * NW + wave) * NR + (i * TQ + j) * 16 + r) * 64 + lane];
    }

    // ---- epilogue: y = bn_scale * relu(alpha * D) + bn_shift in fp64, one rounding --------------
    const int ohw = g.OH * g.OW;
    const double relu_floor = __builtin_canonicalize(prm.t.ep.relu ? 0.0 : -__builtin_inf());
    float* yp[TQ];
    bool mok[TQ];
#pragma unroll
    for (int j = 0; j < TQ; ++j) {
        const int m = q0 + wq * WQ + j * 32 + (lane & 31);
        mok[j] = m < prm.t.RQ;
        const int mm = mok[j] ? m : 0;
        const int nb = (int)fastdiv((uint32_t)mm, g.div_ohw);
        yp[j] = prm.t.y + ((int64_t)nb * g.O * ohw + (mm - nb * ohw));
    }
    auto run = [&](auto full, auto nt) {
        constexpr bool FULL = decltype(full)::value;
#pragma unroll
        for (int i = 0; i < TP; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int tr = wp * WP + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3), o = p0 + tr;
                const bool ook = o < prm.t.RP;
                const double g1 = tab[tr], bs = tab[BP + tr], bh = tab[2 * BP + tr];
#pragma unroll
                for (int j = 0; j < TQ; ++j) {
                    const double v = __builtin_fmax(g1 * (double)acc[i][j][r], relu_floor);
                    const float z = (float)(bs * v + bh);
                    if (FULL || (ook && mok[j])) {
                        if constexpr (decltype(nt)::value)
                            __builtin_nontemporal_store(z, yp[j] + (int64_t)o * ohw);
                        else
                            yp[j][(int64_t)o * ohw] = z;
                    }
                }
                if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
    };
    const std::true_type yes{};
    const std::false_type no{};
    if (p0 + BP <= prm.t.RP && q0 + BQ <= prm.t.RQ)
        prm.t.nt_out ? run(yes, yes) : run(yes, no);
    else
        prm.t.nt_out ? run(no, yes) : run(no, no);
}

// int8 codes [O][taps][Cpad] -> bf16 weights in fragment order: for every 32-filter tile (the last
// one holds the remaining `rows`), 16-channel slice and tap, [half][row][8 channels], so that a
// wave's matrix operand is one run of memory.  The same number of elements as the row-major form.
__global__ __launch_bounds__(256) void k_codes_to_frag(const int8_t* codes, int O, int ntap, int Cpad, uint16_t* out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;  // 8 codes each
    const int c8 = Cpad >> 3;
    if (i >= (int64_t)O * ntap * c8) return;
    const int o = (int)(i / ((int64_t)ntap * c8)), rem = (int)(i - (int64_t)o * ntap * c8), tap = rem / c8, cb = rem - tap * c8;
    const uint2 c = *(const uint2*)(codes + i * 8);
    const unsigned w[2] = {c.x, c.y};
    unsigned d[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int t0 = (int8_t)(w[e >> 1] >> (16 * (e & 1))), t1 = (int8_t)(w[e >> 1] >> (16 * (e & 1) + 8));
        const unsigned b0 = t0 > 0 ? 0x3f80u : (t0 < 0 ? 0xbf80u : 0u), b1 = t1 > 0 ? 0x3f80u : (t1 < 0 ? 0xbf80u : 0u);
        d[e] = b0 | (b1 << 16);
    }
    const int pt = o >> 5, rows = O - pt * 32 < 32 ? O - pt * 32 : 32;
    const int64_t u = (int64_t)pt * 32 * ntap * c8 + (((int64_t)(cb >> 1) * ntap + tap) * 2 + (cb & 1)) * rows + (o & 31);
    ((uint4*)out)[u] = make_uint4(d[0], d[1], d[2], d[3]);
}

template <int BP, int BQ, int WGP, int WGQ, int KG, int MINW, int NTAP, int CS, int RMAX, bool BIG = false>
hipError_t launch_wc(WcParams& prm, hipStream_t st)
{
    constexpr int img = KG * wc_images<NTAP == 0, KG, BQ>() * CS * 3 * (RMAX + 1) * 32, red = (KG - 1) * BP * BQ * 4;
    constexpr int smem = (img > red ? img : red) + 3 * BP * 8;  // the groups' sums over the images, the epilogue table behind
    static_assert(smem <= kMaxLds, "LDS");
    const ConvGeom& g = prm.t.g;
    prm.nchunk = (g.C + 16 * CS - 1) / (16 * CS) * (NTAP ? 1 : g.KH * g.KW);
    prm.dc = KG / (g.KH * g.KW);
    prm.dtap = KG % (g.KH * g.KW);
    auto kern = k_wconv<BP, BQ, WGP, WGQ, KG, MINW, NTAP, CS, RMAX, BIG>;
    static LdsLimit lds;
    const hipError_t e = lds.raise((const void*)kern, smem);
    if (e != hipSuccess) return e;
    const unsigned grid = tile_grid(prm.t, BP, BQ);
    if (!grid) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * WGP * WGQ * KG), (size_t)smem, st, prm);
    return hipGetLastError();
}

// Rows of the flattened input a tile of bq output pixels reaches over at most; 0: the pixels'
// windows do not start in ascending order, the tile has no run.
int64_t run_rows(const ConvGeom& g, int bq)
{
    const int64_t s = g.stride, n = bq - 1;
    const int64_t row_step = s * g.W - (int64_t)(g.OW - 1) * s;                                  // last pixel of a row -> next row
    const int64_t img_step = (int64_t)g.H * g.W - (int64_t)(g.OH - 1) * s * g.W - (int64_t)(g.OW - 1) * s;
    if (row_step < 0 || img_step < 0) return 0;
    const int64_t nrow = n / g.OW + 1, nimg = n / ((int64_t)g.OH * g.OW) + 1;
    const int64_t over_row = row_step > s ? row_step - s : 0, over_img = img_step > row_step ? img_step - row_step : 0;
    return n * s + nrow * over_row + nimg * over_img + (int64_t)(g.KH - 1) * g.W + g.KW;
}

// The kernel's forms and what a launch of each costs, in us:
//   base + n round + steps u max(lat ceil(n / occ), n tp),   u = 1 + slope x
// with n = blocks of the most loaded CU (256 CUs, rounded up), steps = chunks a group of waves takes,
// x = rows of the run / 64 (GATHER: stride - 1, at most 3).  A chunk's latency counts once for every
// occ blocks that run side by side, its throughput for each.  The constants are fitted to the times of all
// forms on 857 geometries (windows 1 to 7, strides 1 to 4, 3 to 512 channels, 7 to 500 pixels wide, batch 1
// to 256), each where no form of its tile with a smaller image fits; those stand first, and the roomier
// ones are passed over there.  The cheapest form by this estimate takes 1.006 times the fastest one's
// time on average, more than 1.15 times it on 12 of them, 1.45 times at worst.
// The 64 x 64 gathering form is held to 64 registers (8 waves a SIMD): two of its blocks of 16 waves on a CU.  With 68, one:
// 24 x 16 x 48 x 48 to 29 filters, 7 x 7, 65.1 us instead of 51.4.
struct WcForm {
    int bp, bq, kg, window, rmax;  // window: side of a run's window, 0: GATHER
    hipError_t (*launch)(WcParams&, hipStream_t);
    float lat, tp, base, round, slope;
    int occ;
};
template <int BP, int BQ, int WGP, int WGQ, int KG, int MINW, int NTAP, int CS, int RMAX>
constexpr WcForm wc_form(float lat, float tp, float base, float round, float slope, int occ)
{
    return {BP, BQ, KG, NTAP == 9 ? 3 : (NTAP == 25 ? 5 : 0), RMAX, launch_wc<BP, BQ, WGP, WGQ, KG, MINW, NTAP, CS, RMAX>,
            lat, tp, base, round, slope, occ};
}
const WcForm kForms[] = {
    wc_form<128, 256, 1, 4, 1, 2, 9, 1, 384>(3.76, 3.4, 11.4, 0.982, 0.0582, 2),
    wc_form<64, 256, 1, 4, 1, 2, 9, 1, 384>(1.94, 1.76, 6.9, 1, 0.0728, 2),
    wc_form<64, 256, 1, 4, 1, 2, 9, 1, 512>(2.35, 1.48, 5.75, 2.48, 0.0288, 1),
    wc_form<64, 256, 1, 4, 1, 2, 9, 1, 768>(2.35, 1.48, 5.75, 2.48, 0.0288, 1),
    wc_form<128, 128, 2, 2, 1, 2, 9, 1, 256>(0.588, 2.28, 5.99, 1.94, 0, 4),
    wc_form<128, 128, 2, 2, 1, 2, 9, 1, 768>(1.3, 0.814, 2.21, 4.34, 0.253, 2),
    wc_form<64, 64, 2, 2, 4, 4, 9, 1, 256>(0.0333, 3.11, 1.7, 3.92, 0.0102, 4),
    wc_form<64, 64, 2, 2, 2, 2, 9, 1, 512>(1.89, 0.519, 1.79, 2.66, 0.0789, 1),
    wc_form<32, 32, 1, 1, 16, 4, 9, 1, 64>(2.39, 2.11, 0.358, 4.22, 0.798, 2),
    wc_form<32, 32, 1, 1, 8, 2, 9, 1, 128>(1.86, 0.372, 1.49, 3.17, 0.322, 1),
    wc_form<32, 32, 1, 1, 8, 2, 9, 1, 192>(1.86, 0.372, 1.49, 3.17, 0.322, 1),
    wc_form<32, 32, 1, 1, 4, 1, 9, 1, 384>(0.506, 1.55, 1.18, 2.51, 0.402, 4),
    wc_form<128, 128, 2, 2, 1, 2, 25, 1, 384>(4.95, 1.39, 7.67, 0.992, 0.0475, 1),
    wc_form<64, 64, 2, 2, 4, 4, 25, 1, 256>(5.79, 0.372, 0.891, 4.87, 0.0322, 1),
    wc_form<64, 64, 2, 2, 2, 2, 25, 1, 512>(0.518, 4.33, 3.26, 2.75, 0, 4),
    wc_form<64, 256, 1, 4, 1, 2, 0, 2, 256>(1.76, 0.982, 5.76, 1.74, 0.251, 3),
    wc_form<128, 128, 2, 2, 1, 2, 0, 2, 128>(1.17, 0.701, 5.29, 2.14, 0.12, 3),
    wc_form<128, 128, 2, 2, 2, 4, 0, 2, 128>(1.78, 1.43, 5.36, 2.76, 0.17, 3),
    wc_form<64, 64, 2, 2, 4, 8, 0, 2, 64>(1.34, 1.04, 4.56, 1.25, 0.218, 3),
};

}  // namespace

// table position behind wn bf16 weights
static double* wconv_table(uint16_t* wb, int64_t wn) { return (double*)(((uintptr_t)(wb + wn) + 15) & ~(uintptr_t)15); }

hipError_t launch_wconv_prepare(const int8_t* w, const ConvGeom& g0, const EpiArgs& ep, void* prepared, hipStream_t st)
{
    uint16_t* wb = (uint16_t*)prepared;
    const int64_t wn = (int64_t)g0.O * g0.KH * g0.KW * g0.Cpad;
    hipLaunchKernelGGL(k_codes_to_frag, dim3((unsigned)((wn / 8 + 255) / 256)), dim3(256), 0, st, w, g0.O, g0.KH * g0.KW, g0.Cpad, wb);
    ConvArgs c = {};
    c.g = g0;
    c.ep = ep;
    return launch_conv_class_consts(c, wconv_table(wb, wn), st);  // g1 = alpha_w, BN rows; the class constants are 0
}

hipError_t launch_wconv(const WConvArgs& a, hipStream_t st)
{
    const ConvGeom& g = a.g;
    const int64_t wn = (int64_t)g.O * g.KH * g.KW * g.Cpad;
    // one-call form: the weight side is prepared in the workspace
    uint16_t* wb = (uint16_t*)(a.prepared ? a.prepared : a.workspace);
    if (!a.prepared) {
        const hipError_t e = launch_wconv_prepare(a.w, g, a.ep, wb, st);
        if (e != hipSuccess) return e;
    }
    WcParams prm = {};
    TmmParams& t = prm.t;
    t.g = g;
    t.RP = g.O;
    t.RQ = (int)((int64_t)g.Nb * g.OH * g.OW);
    t.y = a.y;
    t.cst_cls = wconv_table(wb, wn);
    t.ep = a.ep;
    t.nt_out = (int64_t)g.O * t.RQ * 4 > (int64_t)128 << 20;
    prm.x = a.x;
    prm.w = (const int8_t*)wb;
    prm.div_hw = make_fastdiv((uint32_t)(g.H * g.W));
    prm.div_tap = make_fastdiv((uint32_t)(g.KH * g.KW));
    prm.kw_inv = 65536u / (unsigned)g.KW + 1;

    // offsets within a tile: at most `images` images of C * HW elements
    auto big = [&](int64_t images) { return images * g.C * g.H * g.W * 4 >= (int64_t)1 << 32; };
    const bool run = g.KH == g.KW && (g.KH == 3 || g.KH == 5);
    int64_t reach[4] = {};  // of 32, 64, 128, 256 pixels
    for (int i = 0; run && i < 4; ++i) reach[i] = run_rows(g, 32 << i);
    auto rows = [&](const WcForm& f) { return f.window ? reach[__builtin_ctz(f.bq) - 5] : f.bq; };
    auto fits = [&](const WcForm& f) {
        if (!f.window) return !big(256 / ((int64_t)g.OH * g.OW) + 2);
        const int64_t r = rows(f);
        return run && f.window == g.KH && r > 0 && r <= f.rmax && !big(r / ((int64_t)g.H * g.W) + 2);
    };
    auto cost = [&](const WcForm& f) {
        const int64_t blocks = (((int64_t)t.RP + f.bp - 1) / f.bp) * (((int64_t)t.RQ + f.bq - 1) / f.bq), n = (blocks + 255) / 256;
        const int64_t chunks = f.window ? (g.C + 15) / 16 : (int64_t)((g.C + 31) / 32) * g.KH * g.KW;
        const double u = 1 + f.slope * (f.window ? (double)rows(f) / 64 : (g.stride < 4 ? g.stride : 4) - 1);
        const double lat = f.lat * (double)((n + f.occ - 1) / f.occ), tp = f.tp * (double)n;
        return f.base + f.round * (double)n + (double)((chunks + f.kg - 1) / f.kg) * u * (lat > tp ? lat : tp);
    };
    auto pick = [&](auto&& admits) {
        const WcForm* best = nullptr;
        double least = 0;
        const WcForm* tighter = nullptr;  // the last form that fits
        for (const WcForm& f : kForms)
            if (admits(f) && fits(f)) {
                if (tighter && f.window && f.window == tighter->window && f.bp == tighter->bp && f.bq == tighter->bq) continue;
                tighter = &f;
                const double c = cost(f);
                if (!best || c < least) best = &f, least = c;
            }
        return best;
    };
    const WcForm* f;
    if (const int forced = forced_tile_config(); forced >= 0) {
        // 8, 9, 10, 12: a gathering form; else the tile's run, the smallest run, or gathering if none fits
        const bool gather = forced == 8 || forced == 9 || forced == 10 || forced == 12, wide = forced == 4 || forced == 13 || forced == 19;
        const int bp = forced == 11 ? 32 : (forced == 10 ? 64 : kTileBP[forced] >= 128 ? 128 : 64);
        const int bq = forced == 11 ? 32 : (forced == 0 || forced == 10 ? 64 : bp == 128 && !wide ? 128 : 256);
        f = pick([&](const WcForm& k) { return !k.window == gather && k.bp == bp && k.bq == bq && (!gather || (k.kg == 2) == (forced == 12)); });
        if (!f) f = pick([&](const WcForm& k) { return k.window && k.bp == 64 && k.bq == 64; });
        if (!f) f = pick([&](const WcForm& k) { return !k.window && k.kg != 2 && (bp == 32 || bq == 64 ? k.bq == 64 : k.bq == bq); });
    } else {
        f = pick([](const WcForm&) { return true; });
    }
    if (!f) return launch_wc<64, 64, 2, 2, 4, 8, 0, 2, 64, true>(prm, st);
    prm.span = (int)rows(*f);
    return f->launch(prm, st);
}

}  // namespace rtn
