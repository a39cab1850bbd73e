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
//   GATHER  (1 x 1 windows, and every geometry whose run does not fit) LDS row = output pixel, one
//           tap at a time; a chunk is then (16 CS channels, one tap).
// The next chunk's inputs are loaded into registers while this chunk is multiplied.  Weights are
// read from global memory in the order the matrix instruction takes them (k_codes_to_frag), PD
// steps ahead; they are shared by all blocks and stay in L2.  KG > 1: groups of four waves take
// every KG-th chunk each, with LDS images of their own, and add up at the end -- for grids too
// small to fill the chip.
//
// What it replaced wrote the three terms to memory (6 bytes per activation) in a pass of its own
// and re-read them once per tap and filter tile through LDS, with the weights fetched again for
// each term.  ResNet-18's 19 layer shapes (before -> now): batch 256 4.54 -> 2.74 ms, batch 40 1.57
// -> 0.66 ms, batch 1 1.04 -> 0.19 ms.  The 3 x 3 stride-1 layers run at 1.0 to 1.2 PFLOP/s of
// bf16 (a library matrix product reaches 1.41 on this card) and are bound by the matrix cores
// at that clock; the stride-2 layers, which split four inputs per output, and the 64-channel
// layers, whose blocks live for four chunks only, by load latency beside it.
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

// NTAP: taps of the window, 0 = GATHER.  RMAX: LDS rows per image (a multiple of 64).  BIG: the
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
    constexpr int NW = WGP * WGQ;                                 // waves per group
    constexpr int NU = 2 * CS * RMAX / (64 * NW);                 // (row, 8 channels) units per thread
    static_assert((NW == 4 || NW == 1) && TP >= 1 && TQ >= 1, "four waves or one per group");
    static_assert(NSTEP % PD == 0 && RMAX % 64 == 0 && (2 * CS * RMAX) % (64 * NW) == 0 && (!GATHER || RMAX == BQ), "chunk shape");
    static_assert(NTAP == 0 || NTAP == 9 || NTAP == 25, "window");

    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave16 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wave16 % NW, kg = wave16 / NW;
    const int wp = wave / WGQ, wq = wave % WGQ;
    const ConvGeom& g = prm.t.g;
    int tileP, tileQ;
    if (!block_tile(prm.t, tileP, tileQ)) return;
    const int p0 = tileP * BP, q0 = tileQ * BQ;
    int8_t* img = smem + kg * IMG;
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
            int ih0, iw0, nb, v = 0;
            origin(m, ih0, iw0, nb);
            for (int k = 0; k < g.KH; ++k) v |= ((unsigned)(ih0 + k) < (unsigned)g.H) << k;
            for (int k = 0; k < g.KW; ++k) v |= ((unsigned)(iw0 + k) < (unsigned)g.W) << (8 + k);
            tmask[i] = v;
            if (BIG)  // (+ the tap's offset: in range when the tap is in the image)
                voff[i] = (Off)(((int64_t)(nb - onb) * g.C * HW + (int64_t)ih0 * g.W + iw0) * 4);
            else
                voff[i] = (Off)((unsigned)(nb - onb) * (unsigned)(g.C * HW) + (unsigned)(ih0 * g.W + iw0)) * 4u;
        } else {
            int f = imin < total_px - r ? imin + r : total_px - 1;
            f = f < 0 ? 0 : f;
            const int nb = (int)fastdiv((uint32_t)f, prm.div_hw);
            if (BIG)
                voff[i] = (Off)(((int64_t)(nb - nb0) * g.C * HW + (f - nb * HW)) * 4);
            else
                voff[i] = (Off)((unsigned)(nb - nb0) * (unsigned)(g.C * HW) + (unsigned)(f - nb * HW)) * 4u;
        }
    }
    float xr[NU][8];
    auto load_x = [&](int ci) {
        int c0 = ci * 16 * CS, tap = 0;
        int64_t toff = 0;
        if (GATHER && ntap > 1) {
            tap = ci % ntap;
            c0 = (ci / ntap) * 16 * CS;
        }
        const int kh = GATHER ? tap / g.KW : 0, kw = tap - kh * g.KW;
        toff = GATHER ? (int64_t)kh * g.W + kw : 0;
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            const int hs = (wave + NW * i) / NSEG;
            const bool live = GATHER || ((wave + NW * i) % NSEG) * 64 < prm.span;
            const int c = c0 + 8 * hs;
            const bool tok = !GATHER || ((tmask[GATHER ? i : 0] >> kh) & (tmask[GATHER ? i : 0] >> (8 + kw)) & 1) != 0;
            // a tap outside the image: load the tile's first element and drop it
            const Off o = tok ? (Off)(voff[i] + (Off)(toff * 4)) : (Off)0;
            if (!live) continue;  // (wave-uniform, like the channel tail)
            const char* xc = (const char*)(xbase + (int64_t)c * HW);
            if (c + 8 <= g.C) {
#pragma unroll
                for (int e = 0; e < 8; ++e) xr[i][e] = *(const float*)(xc + (int64_t)e * HW * 4 + o);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) xr[i][e] = c + e < g.C ? *(const float*)(xc + (int64_t)e * HW * 4 + o) : 0.0f;
            }
            if (GATHER) {
#pragma unroll
                for (int e = 0; e < 8; ++e) xr[i][e] = tok ? xr[i][e] : 0.0f;
            }
        }
    };
    auto store_x = [&]() {
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            if (!GATHER && ((wave + NW * i) % NSEG) * 64 >= prm.span) continue;
            const int r = ((wave + NW * i) % NSEG) * 64 + lane, hs = (wave + NW * i) / NSEG;
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
    int64_t wbase[TP];
    unsigned wlane[TP], wstep[TP];
    const int lastpt = (prm.t.RP - 1) >> 5;
#pragma unroll
    for (int t = 0; t < TP; ++t) {
        int pt = (p0 + wp * WP) / 32 + t;
        pt = pt < lastpt ? pt : lastpt;
        const int rows = prm.t.RP - pt * 32 < 32 ? prm.t.RP - pt * 32 : 32;
        const int row = (lane & 31) < rows ? (lane & 31) : rows - 1;
        wbase[t] = (int64_t)pt * 32 * ntap * g.Cpad * 2;
        wlane[t] = (unsigned)(half * rows + row) * 16;
        wstep[t] = (unsigned)rows * 32;
    }
    v4i pw[PD][TP];
    // step s of chunk ci
    auto load_w = [&](int ci, int s, v4i* dst) {
        int slice, tap;
        if (GATHER) {
            tap = ntap > 1 ? ci % ntap : 0;
            slice = (ntap > 1 ? ci / ntap : ci) * CS + s;
        } else {
            slice = ci * CS + s / (NTAP ? NTAP : 1);
            tap = s % (NTAP ? NTAP : 1);
        }
        slice = slice < nslice ? slice : nslice - 1;  // past the end: multiplied with zero activations
        const int64_t idx = (int64_t)slice * ntap + tap;
#pragma unroll
        for (int t = 0; t < TP; ++t) dst[t] = *(const v4i*)(prm.w + (wbase[t] + idx * wstep[t]) + wlane[t]);
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
            unsigned v = 0;
#pragma unroll
            for (int k = 0; k < KK; ++k)
                v |= (unsigned)((unsigned)(ih0 + k) < (unsigned)g.H) << k | (unsigned)((unsigned)(iw0 + k) < (unsigned)g.W) << (8 + k);
            vm[j] = v;
        }
    }
    // the channels' epilogue factors: rows alpha, BN scale, BN shift of the prepared table
    double* tab = (double*)(smem + KG * IMG);
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
    const int nch = prm.nchunk;
    const int niter = (nch + KG - 1) / KG;
    auto chunk_of = [&](int it) {
        const int ci = it * KG + kg;
        return ci < nch ? ci : nch - 1;
    };
#pragma unroll
    for (int s = 0; s < PD; ++s) load_w(chunk_of(0), s, pw[s]);
    load_x(chunk_of(0));
    for (int it = 0; it < niter; ++it) {
        if (it) group_sync();  // everybody is done with the previous chunk's image
        store_x();
        const bool live = it * KG + kg < nch;
        const int ci = chunk_of(it), cn = chunk_of(it + 1 < niter ? it + 1 : it);
        if (it + 1 < niter) load_x(cn);
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
                    load_w(ci, s + PD, pw[s % PD]);
                else
                    load_w(cn, s + PD - NSTEP, pw[s % PD]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
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
    auto run = [&](auto nt) {
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
                    if (ook && mok[j]) {
                        if constexpr (decltype(nt)::value)
                            __builtin_nontemporal_store(z, yp[j] + (int64_t)o * ohw);
                        else
                            yp[j][(int64_t)o * ohw] = z;
                    }
                }
                if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
    };
    if (prm.t.nt_out)
        run(std::true_type{});
    else
        run(std::false_type{});
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
    constexpr int img = KG * CS * 3 * (RMAX + 1) * 32, red = (KG - 1) * BP * BQ * 4;
    static_assert(red <= img, "the groups' sums over the images, the epilogue table behind them");
    constexpr int smem = img + 3 * BP * 8;
    static_assert(smem <= kMaxLds, "LDS");
    const ConvGeom& g = prm.t.g;
    prm.nchunk = (g.C + 16 * CS - 1) / (16 * CS) * (NTAP ? 1 : g.KH * g.KW);
    auto kern = k_wconv<BP, BQ, WGP, WGQ, KG, MINW, NTAP, CS, RMAX, BIG>;
    static bool attr_done = false;
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        if (e != hipSuccess) return e;
        attr_done = true;
    }
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
    // one-call form: the weight side goes behind what earlier forms of the workspace held
    uint16_t* wb = a.prepared ? (uint16_t*)a.prepared : (uint16_t*)a.workspace + 3 * (int64_t)g.Nb * g.H * g.W * g.Cpad;
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

    // offsets within a tile: at most `images` images of C * HW elements
    auto big = [&](int64_t rows) { return (rows / ((int64_t)g.H * g.W) + 2) * g.C * g.H * g.W * 4 >= (int64_t)1 << 32; };
    const int ntap = g.KH == g.KW ? g.KH * g.KW : 0;
    const int64_t r256 = run_rows(g, 256), r128 = run_rows(g, 128), r64 = run_rows(g, 64);
    auto blocks = [&](int bp, int bq) { return (((int64_t)t.RP + bp - 1) / bp) * (((int64_t)t.RQ + bq - 1) / bq); };
    auto fits = [&](int64_t rows, int rmax) { return rows > 0 && rows <= rmax && !big(rows); };
    // Estimated cycles of the K loop, by tile: the matrix-core work of the most loaded CU over the
    // tile's efficiency (small tiles read more LDS per MFMA, long runs are more work per output),
    // but no less than the chunks' load latency one after another.  The constants fit the times of
    // the ten ResNet-18 layer shapes at batch 1, 4, 16, 64 and 256: the choice is the fastest tile or
    // within 15 % of it on all of them.
    const double nchunk = (g.C + 15) / 16, slices = nchunk * g.KH * g.KW;
    auto cost = [&](int bp, int bq, int kg, double eff, int64_t rows) {
        const double work = (double)((blocks(bp, bq) + 255) / 256) * (bp * bq / 1024) * slices * 3 * 32 / 4 / eff *
                            (1 + 0.15 * ((double)rows / bq - 1));
        const double lat = nchunk / kg * (rows == bq ? 1500 : 3000);
        return work > lat ? work : lat;
    };
    const int forced = forced_tile_config();
    const int fbp = forced >= 0 ? kTileBP[forced] : 0;
    auto pick = [&](double c0, double c1, double c2, double c3, double c4) {  // 128x256, 64x256, 128x128, 64x64, 32x32
        if (forced >= 0)
            return forced == 13 || forced == 4 || forced == 19 ? 0 : (fbp >= 128 ? 2 : (forced == 0 ? 3 : (forced == 11 ? 4 : 1)));
        const double c[5] = {c0, c1, c2, c3, c4};
        int b = 0;
        for (int i = 1; i < 5; ++i) b = c[i] < c[b] ? i : b;
        return b;
    };
    const double inf = 1e300;
    const int64_t r32 = run_rows(g, 32);
    if (ntap == 9 && fits(r64, 512)) {
        const int kg32 = r32 <= 64 ? 16 : (r32 <= 192 ? 8 : 4);  // what LDS holds
        switch (pick(fits(r256, 384) ? cost(128, 256, 1, 0.40, r256) : inf, fits(r256, 512) ? cost(64, 256, 1, 0.45, r256) : inf,
                     fits(r128, 768) ? cost(128, 128, 1, 0.45, r128) : inf, cost(64, 64, 4, 0.3, r64),
                     fits(r32, 384) ? cost(32, 32, kg32, 0.2, r32) : inf)) {
            case 0:
                prm.span = (int)r256;
                if (fits(r256, 384)) return launch_wc<128, 256, 1, 4, 1, 2, 9, 1, 384>(prm, st);
                break;
            case 1:
                prm.span = (int)r256;
                if (fits(r256, 384)) return launch_wc<64, 256, 1, 4, 1, 2, 9, 1, 384>(prm, st);
                if (fits(r256, 512)) return launch_wc<64, 256, 1, 4, 1, 2, 9, 1, 512>(prm, st);
                break;
            case 2:
                prm.span = (int)r128;
                if (fits(r128, 256)) return launch_wc<128, 128, 2, 2, 1, 2, 9, 1, 256>(prm, st);
                if (fits(r128, 768)) return launch_wc<128, 128, 2, 2, 1, 2, 9, 1, 768>(prm, st);
                break;
            case 4:
                prm.span = (int)r32;
                if (fits(r32, 64)) return launch_wc<32, 32, 1, 1, 16, 4, 9, 1, 64>(prm, st);
                if (fits(r32, 128)) return launch_wc<32, 32, 1, 1, 8, 2, 9, 1, 128>(prm, st);
                if (fits(r32, 192)) return launch_wc<32, 32, 1, 1, 8, 2, 9, 1, 192>(prm, st);
                if (fits(r32, 384)) return launch_wc<32, 32, 1, 1, 4, 1, 9, 1, 384>(prm, st);
                break;
            default: break;
        }
        prm.span = (int)r64;
        if (fits(r64, 256)) return launch_wc<64, 64, 2, 2, 4, 4, 9, 1, 256>(prm, st);
        return launch_wc<64, 64, 2, 2, 2, 2, 9, 1, 512>(prm, st);
    }
    if (ntap == 25 && fits(r64, 512)) {
        if (fits(r128, 384) && pick(inf, inf, cost(128, 128, 1, 0.45, r128), cost(64, 64, 4, 0.3, r64), inf) == 2) {
            prm.span = (int)r128;
            return launch_wc<128, 128, 2, 2, 1, 2, 25, 1, 384>(prm, st);
        }
        prm.span = (int)r64;
        if (fits(r64, 256)) return launch_wc<64, 64, 2, 2, 4, 4, 25, 1, 256>(prm, st);
        return launch_wc<64, 64, 2, 2, 2, 2, 25, 1, 512>(prm, st);
    }
    // (GATHER: a tile's outputs lie in at most 256 / (OH OW) + 2 images)
    if ((256 / ((int64_t)g.OH * g.OW) + 2) * g.C * g.H * g.W * 4 >= (int64_t)1 << 32)
        return launch_wc<64, 64, 2, 2, 4, 4, 0, 2, 64, true>(prm, st);
    switch (pick(inf, cost(64, 256, 1, 0.40, 256), cost(128, 128, 1, 0.45, 128), cost(64, 64, 4, 0.3, 64), inf)) {
        case 0:
        case 1: return launch_wc<64, 256, 1, 4, 1, 2, 0, 2, 256>(prm, st);
        case 2: return launch_wc<128, 128, 2, 2, 1, 2, 0, 2, 128>(prm, st);
        default: return launch_wc<64, 64, 2, 2, 4, 4, 0, 2, 64>(prm, st);
    }
}

}  // namespace rtn
