// Ternary contraction on the gfx950 int8 matrix cores, with implicit-GEMM
// convolution addressing and the fused reparameterization epilogue.
//
//   D[p][q] = sum_k P[p][k] * Q[q][k]        (codes are int8 in {-1,0,+1})
//
// One kernel serves both entry points through its two operands:
//   GEMM:  P = activation codes (rows m), Q = weight codes (rows n);
//          output [M][N] row-major, lanes run along n.
//   conv:  P = weight codes [O][KH*KW*Cpad], Q = the *virtual* im2col matrix of
//          the channel-innermost activation codes (row = output pixel
//          m = (nb, oh, ow), column = (kh, kw, c)); output NCHW, lanes run
//          along pixels.  A 64-byte K-step never straddles a tap because
//          Cpad % 64 == 0, so a Q row of a K-step is 64 contiguous bytes of one
//          input pixel, or 64 zero bytes when the tap falls outside the image.
//
// Tiling (wave64, v_mfma_i32_32x32x32_i8): a 256-thread block owns a BP x BQ
// output tile, its 4 waves a WGP x WGQ grid of (BP/WGP) x (BQ/WGQ) sub-tiles
// made of 32x32 MFMA tiles.  K advances 64 bytes per step (two MFMA k-slices).
//
// Data movement: operand tiles go global -> LDS directly (buffer_load ... lds,
// 16 bytes per lane, no register staging) into NS ring stages, NS steps ahead
// of the MFMAs; completion is tracked by hand with s_waitcnt vmcnt and ONE
// workgroup barrier per K-step placed between the two k-slices, so that the
// fragments of the next slice are always in flight behind 16 MFMAs.  A wave's
// direct load writes 1 KiB of LDS, lane l at +16*l, i.e. 16 rows of 64 bytes;
// which global 16-byte chunk a lane fetches is permuted (XOR swizzle by row) so
// that the 16-byte fragment reads of 16 consecutive rows hit all 64 banks.
//
// Variants of the same kernel (template parameters of k_tmm):
//   HC   conv tiles that keep their run of input pixels in LDS (stride 1, centred window);
//   TERN conv whose epilogue ternarizes its output for the next layer (1), also after
//        the residual add and second ReLU of a block tail (2);
//   DT   1: bf16 operands with fp32 accumulators (v_mfma_f32_32x32x16_bf16) for the
//        weight-only ternary GEMM, whose fp32 activations are split exactly
//        into three bf16 terms laid along K;
//        2: codes stored as FP4 (E2M1) nibbles, two per byte, multiplied by
//        v_mfma_f32_32x32x64_f8f6f4 with fp32 accumulators.  -1, 0, +1 are exact in
//        E2M1 (0xA, 0x0, 0x2), every product is exact and the fp32 sums are integers
//        below 2^24, so D is the same integer the int8 form produces -- at twice the
//        matrix-core rate and half the operand bytes (a 64-byte K-step is 128 codes).
// This header holds the kernel template and its launcher; the instantiations are spread
// over several translation units (tmm_inst_*.hip) so that they compile in parallel.
#pragma once
#include <type_traits>
#include <utility>

#include "choice.h"
#include "conv_offsets.h"
#include "epilogue_math.h"
#include "lds_limit.h"
#include "rtn_kernels.h"

namespace rtn {

struct TmmParams {
    const int8_t* P;
    const int8_t* Q;
    int RP, RQ;        // valid rows of the P / Q operand
    int64_t ldP, ldQ;  // row pitch in bytes (dense operands)
    int nk;            // number of 64-byte K-steps
    int tilesP;        // number of tiles along P
    int ntiles;        // tilesP * tilesQ
    int band_tiles;    // 8 * tilesQ
    FastDiv div_band;
    FastDiv div_lastband;  // by the P-tiles of the last band
    FastDiv div_nax;       // conv: by the axis classes of the epilogue table in LDS
    int Klogical;      // K of the epilogue's constant term (GEMM)
    int hrows;         // halo variant: input pixels held in LDS (multiple of 16)
    ConvGeom g;        // conv only
    int32_t* acc;
    float* y;
    const double* cst_cls;  // conv: [class][O] constants (see k_conv_class_consts)
    EpiArgs ep;
    // conv, ternarizing epilogue: the output is the next layer's code tensor
    // [pixel][ldc] (int8, channel-innermost) instead of acc / y
    int8_t* codes;
    int ldc;
    Param thr_lo, thr_hi;  // vector: per output channel
    // ... optionally after a residual add (res, fp32 NCHW, nullable) and a second
    // ReLU; the fp32 value that is ternarized is also stored when y is given
    const float* res;
    int relu_out;
    int nt_out;  // store the outputs with the non-temporal hint (conv: fp32 / int32, GEMM: y of the 256 x 256 tile)
    // bf16 operands (DT = 1): the weight rows (Q) are wwrap bytes long and are walked again
    // from the start each time the K offset passes their end
    unsigned wwrap;
};

// Launch of tile configuration `cfg` (the numbering rtn_set_tile_config() documents) of the
// kernel on int8 (DT = 0) or FP4 (DT = 2) codes, GEMM (CONV = false) or conv with the plain
// (TERN = 0), ternarizing (1) or block-tail (2) epilogue.  hipErrorInvalidValue: the
// configuration does not fit this problem.  Defined in tmm_dispatch.inc, instantiated one
// (CONV, TERN, DT) triple per translation unit.
template <bool CONV, int TERN, int DT>
hipError_t tmm_launch_index_raw(int cfg, TmmParams& prm, hipStream_t st);
// The kernel for small grids (tmm_ksplit.hip) in form `form` of kKsplitForms, as pick_ksplit() chooses it.
KsplitShape ksplit_shape(const TmmParams& prm, bool conv);
template <bool CONV, int TERN, int DT>
hipError_t launch_ksplit(int form, const TmmParams& prm, hipStream_t st);
// The bf16-operand variants of the weight-only GEMM: 0 = 64x64, 1 = 128x128, 2 = 256x256.
hipError_t tmm_launch_bf16(int variant, TmmParams& prm, hipStream_t st);

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// 16 zero bytes every out-of-image tap reads from.
__device__ __attribute__((aligned(16))) int g_zero16[4] = {0, 0, 0, 0};
// Border classes of a conv window and the LDS bytes of the epilogue table of a
// BP-channel tile: rows g1, c2, bn scale, bn shift, then one row per class.
__host__ __device__ inline int conv_classes(int pad)
{
    const int p1 = pad + 1;
    return p1 * p1 * p1 * p1;
}
// The copy of that table a block keeps in LDS holds only the classes that can occur.
// Along one axis a window is cut by tcut taps at the low end and bcut at the high end;
// when the image is at least as long as the window it is never cut at both ends, which
// leaves 2 pad + 1 axis classes (0 = uncut, 1 .. pad = tcut, pad + 1 .. 2 pad = pad + bcut)
// instead of (pad+1)^2 (tcut + (pad+1) bcut, the numbering of the prepared table).
__host__ __device__ inline bool conv_compact(const ConvGeom& g) { return g.H >= g.KH && g.W >= g.KW; }
__host__ __device__ inline int conv_axis_classes(const ConvGeom& g)
{
    return conv_compact(g) ? 2 * g.pad + 1 : (g.pad + 1) * (g.pad + 1);
}
__host__ __device__ inline int conv_lds_classes(const ConvGeom& g)
{
    return conv_axis_classes(g) * conv_axis_classes(g);
}
__host__ __device__ inline int conv_axis_class(bool compact, int pad, int tcut, int bcut)
{
    return compact ? (bcut ? pad + bcut : tcut) : tcut + (pad + 1) * bcut;
}
// axis class of the LDS copy -> axis class of the prepared table
__host__ __device__ inline int conv_axis_global(bool compact, int pad, int a)
{
    return compact ? (a <= pad ? a : (pad + 1) * (a - pad)) : a;
}
__host__ __device__ inline int conv_table_bytes(int bp, const ConvGeom& g) { return (4 + conv_lds_classes(g)) * bp * 8; }

// Taps of a window at i0 of an axis that lie in the image, one bit each.  (Closed form: a lane has this to do for
// each of its pixels before it can load, and a launch on few blocks costs about 5 cycles per instruction of a wave.)
__device__ __forceinline__ int tap_mask(int i0, int ksize, int extent)
{
    const int lo = i0 < 0 ? -i0 : 0;
    int hi = extent - i0 < ksize ? extent - i0 : ksize;
    hi = hi > lo ? hi : lo;
    return (1 << hi) - (1 << lo);
}

// chunk swizzle of a 64-byte LDS row (depends on row & 15 only)
__device__ __forceinline__ int swz(int row) { return ((row >> 1) & 3) ^ ((row >> 3) & 1); }

// Byte of 16-byte chunk q of pixel row `row` of the halo image (rows of HC bytes, HC/16 chunks): the chunk is XOR-ed with
// the row so that 16 consecutive rows hit 16 different bank groups.
template <int HC>
__device__ __forceinline__ int halo_byte(int row, int q)
{
    return row * HC | (((row << (HC == 64 ? 2 : 3)) ^ (q << 4)) & (HC - 16));
}

// Direct global -> LDS load: every lane fetches 16 bytes at gptr; the wave's
// 1 KiB lands at LDS byte offset lds_off (wave-uniform) + 16 * lane.
// The statements overwrite M0.  It cannot be named as a clobber (the compiler keeps M0
// reserved and warns that a clobber of it is not honoured); it is safe because on this
// target the compiler itself writes M0 only immediately before an instruction that
// reads it, never across other code, so no value of its own lives in M0 here.
// The wait states are these statements' own, too: gfx9 wants one between a scalar write of M0 and a load to LDS, and the
// compiler does not look for it in here.  Nor for the five between a vector instruction's write of a scalar register
// (v_readfirstlane) and a load that reads it: scalar operands are kept in scalar registers, except where a kernel runs out
// of those, which waits itself (dma_buf).  (A scalar copy of the operand instead of the s_nop would need no such care, but
// the compiler puts a wait state of its own between two statements that write one register.)
// OFF is added on the way to M0: loads that follow each other in LDS share one address.
template <int OFF = 0>
__device__ __forceinline__ void dma16(const void* gptr, unsigned lds_off)
{
    asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, off" ::"s"(__builtin_amdgcn_readfirstlane(lds_off)), "n"(OFF),
                 "v"(gptr)
                 : "memory", "scc");
}
// 4 bytes per lane
template <int OFF = 0>
__device__ __forceinline__ void dma4(const void* gptr, unsigned lds_off)
{
    asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %2, off" ::"s"(__builtin_amdgcn_readfirstlane(lds_off)), "n"(OFF),
                 "v"(gptr)
                 : "memory", "scc");
}

// The same, with the address split into a wave-uniform 64-bit base (SGPR pair) and
// a per-lane unsigned 32-bit byte offset: nothing to add per lane per K-step.
template <int OFF = 0>
__device__ __forceinline__ void dma16_base(const void* sbase, unsigned voff, unsigned lds_off)
{
    asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3" ::"s"(__builtin_amdgcn_readfirstlane(lds_off)), "n"(OFF),
                 "v"(voff), "s"(sbase)
                 : "memory", "scc");
}
template <int OFF = 0>
__device__ __forceinline__ void dma4_base(const void* sbase, unsigned voff, unsigned lds_off)
{
    asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %2, %3" ::"s"(__builtin_amdgcn_readfirstlane(lds_off)), "n"(OFF),
                 "v"(voff), "s"(sbase)
                 : "memory", "scc");
}

// Pin a wave-uniform pointer into scalar registers (the "s" operands above must
// not be handed a vector register pair, which instruction selection may
// otherwise choose for a uniform value).
__device__ __forceinline__ const int8_t* uniform_ptr(const int8_t* p)
{
    const uint64_t v = (uint64_t)(uintptr_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const int8_t*)(uintptr_t)(((uint64_t)hi << 32) | lo);
}

// Direct global -> LDS load through a buffer resource: lane byte offset `voff` (32 bits) plus the wave-uniform `soff` on a
// scalar base.  Nothing is added per lane and load, the LDS address is one scalar addition, and a lane with an offset from
// kOutside on reads nothing: zeros land in its 16 bytes.
constexpr unsigned kOutside = 0x80000000u;
__device__ __forceinline__ v4i buffer_base(const int8_t* p)
{
    const uint64_t v = (uint64_t)(uintptr_t)p;
    return v4i{(int)__builtin_amdgcn_readfirstlane((uint32_t)v), (int)(__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32)) & 0xffff),
               (int)kOutside, 0x00020000};
}
// VECTOR: `soff` may come out of a vector register just before.
template <int OFF, bool VECTOR = false>
__device__ __forceinline__ void dma_buf(v4i rsrc, unsigned voff, unsigned soff, unsigned lds_off)
{
    asm volatile("s_add_u32 m0, %0, %1\n\ts_nop %5\n\tbuffer_load_dwordx4 %2, %3, %4 offen lds" ::"s"(__builtin_amdgcn_readfirstlane(lds_off)),
                 "n"(OFF), "v"(voff), "s"(rsrc), "s"(__builtin_amdgcn_readfirstlane(soff)), "n"(VECTOR ? 4 : 0)
                 : "memory", "scc");
}

// Keeps the computation of v here: the compiler would put off selects until their result is used, and hold all
// their operands until then.
__device__ __forceinline__ void pin(unsigned& v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(v));
#endif
}

template <class F, int... N>
__device__ __forceinline__ void for_each_index(F&& f, std::integer_sequence<int, N...>)
{
    (f(std::integral_constant<int, N>{}), ...);
}

template <int N>
__device__ __forceinline__ void wait_vm()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lgkm0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// Workgroup barrier that the compiler may not move memory accesses across.
__device__ __forceinline__ void block_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Wait until at most `groups` of this wave's K-step load groups (DPS loads
// each) are still in flight.
template <int DPS>
__device__ __forceinline__ void wait_groups(int groups)
{
    if (groups <= 0)
        wait_vm<0>();
    else if (groups == 1)
        wait_vm<DPS>();
    else if (groups == 2)
        wait_vm<2 * DPS>();
    else
        wait_vm<3 * DPS>();
}

// Output tile of this workgroup (false: none).  Workgroups are dealt to the 8 XCDs round-robin by
// blockIdx; give each XCD (and so each L2) one contiguous run of tiles, P-tile index fastest, so
// tiles that share operand rows and conv halo pixels share an L2.  Within that run, tiles are
// visited in bands of up to 8 P-tiles, P fastest, so the 32 co-resident tiles of an XCD form an
// 8 x 4 patch of the output (12 operand row-blocks per K-step instead of 18 for a 16 x 2 strip).
__device__ __forceinline__ bool block_tile(const TmmParams& prm, int& tileP, int& tileQ)
{
    const int chunk = (int)(gridDim.x >> 3);  // grid is padded to a multiple of 8
    const int bid = (int)(blockIdx.x & 7) * chunk + (int)(blockIdx.x >> 3);
    if (bid >= prm.ntiles) return false;
    band_tile(bid, prm.tilesP, prm.band_tiles, [&](int n) { return (int)fastdiv((uint32_t)n, prm.div_band); },
              [&](int n) { return (int)fastdiv((uint32_t)n, prm.div_lastband); }, tileP, tileQ);
    return true;
}

// The GEMM's epilogue on a wave's TP x TQ accumulator tiles at rows p0 + wrow, columns q0 + wcol:
//   y = aw*(aa*D + ba*Sw) + bw*r2 with r2 = aa*Sa + K*ba per row m (Eq.9 with a weight offset),
// ReLU and BN, one rounding to fp32; `tab` is LDS for [3][BP] doubles and may lie over the
// operand stages.  value(acc) is the integer D as the accumulator's type.  SUMS: the side sums
// exist (not for the weight-only form, whose beta_a and beta_w are 0).
// The element loops exist in straight-line variants -- (interior / ragged tile) x (acc only / y
// only / both), and y without ReLU and BN on interior tiles, which needs 4 fp64 operations per
// output instead of 6 and fewer registers -- picked once per block.
// Bound by the stores: a 256 x 256 tile of the FP4 GEMM takes 7.6 us (4096 x 4096 x 512; 9.1 at K = 4096), of which
// the stores alone need 7.1 (8.5).  The fp64 operations of its one wave per SIMD pass beside them as long as nothing
// spills (with 16 registers spilled: 14.3).
// NT: y is stored with the non-temporal hint.  The GEMM's tiles finish together, and a burst that the memory-side
// cache holds is absorbed faster without it (and is there for the next kernel); a larger one is written back while
// the next tiles are multiplied: 1610 cycles per K-step instead of 1316, against 12.8 us of epilogue instead of 9.8
// (16384 x 8192 x 8192; gemm_nt_hint() decides).
// ABREAST: interior tiles with y alone take one operation at a time over four outputs and more.  For the bit planes:
// 4096 x 4096 x 4096 with the pack 64.2 us, 64.5 one output after the other.  Not for the FP4 GEMM: 4096 x 4096 x 512 20.3
// against 18.8, 16384 x 8192 x 8192 509 against 505 and hinted 465 against 460.
template <int BP, int TP, int TQ, bool SUMS, bool ABREAST = false, bool NT = false, class Acc, class Value>
__device__ __forceinline__ void gemm_epilogue(const TmmParams& prm, double* tab, int p0, int q0, int wrow, int wcol,
                                              bool full_tile, const Acc& acc, Value value)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const EpiArgs& ep = prm.ep;
    const bool has_bn = ep.bn_scale != nullptr;
    // ReLU and BN are applied with neutral parameters where they are not asked for, so the element
    // code has no selects: max(v, -inf) = v and 1*v - 0 = v.  A NaN turns into the floor, 0 or -inf,
    // except where neither is asked for: there the floor is a NaN (max(v, NaN) = v), so that the variants
    // with this tail return for a NaN what the one without it does.  (A variant without for ragged tiles
    // and for acc too: 66.7 against 60.3 us at 4096^3, by the registers of the 256 x 256 tile.)
    const double relu_floor = __builtin_canonicalize(ep.relu ? 0.0 : (has_bn ? -__builtin_inf() : __builtin_nan("")));
    __syncthreads();  // all waves are done with the operand stages
    if (prm.y) {
        for (int t = tid; t < BP; t += 256) {
            const int m = p0 + t;
            double aa = 0.0, ba = 0.0, r2 = 0.0;
            if (m < prm.RP) {
                aa = pval(ep.alpha_a, m);
                ba = pval(ep.beta_a, m);
                if (SUMS) r2 = aa * (double)ep.sum_ta[m] + (double)prm.Klogical * ba;
            }
            tab[t] = aa;
            tab[BP + t] = ba;
            tab[2 * BP + t] = r2;
        }
    }
    __syncthreads();
    const int64_t N = prm.RQ;
    auto run = [&](auto full, auto want_acc, auto want_y, auto want_tail) {
        constexpr bool FULL = decltype(full)::value, ACC = decltype(want_acc)::value, Y = decltype(want_y)::value;
        constexpr bool TAIL = decltype(want_tail)::value;
        // per lane: its TQ output columns, their factors and base pointers.  Set up
        // inside each variant so that a variant holds only what it uses.
        bool nok[TQ];
        double aw[TQ], bw[TQ], bs[TQ], bh[TQ], sw[TQ];
        int32_t* accp[TQ];
        float* yp[TQ];
#pragma unroll
        for (int j = 0; j < TQ; ++j) {
            const int ncol = q0 + wcol + j * 32 + (lane & 31);
            nok[j] = FULL || ncol < prm.RQ;
            aw[j] = bw[j] = sw[j] = 0.0;
            bs[j] = 1.0;
            bh[j] = -0.0;
            if (Y && nok[j]) {
                aw[j] = pval(ep.alpha_w, ncol);
                bw[j] = pval(ep.beta_w, ncol);
                if (SUMS) sw[j] = (double)ep.sum_tw[ncol];
                if (TAIL && has_bn) {
                    bs[j] = ep.bn_scale[ncol];
                    bh[j] = ep.bn_shift ? (double)ep.bn_shift[ncol] : 0.0;
                }
            }
            accp[j] = ACC ? prm.acc + (nok[j] ? ncol : 0) : nullptr;
            yp[j] = Y ? prm.y + (nok[j] ? ncol : 0) : nullptr;
        }
        if constexpr (ABREAST && FULL && Y && !ACC) {
            constexpr int RG = TQ >= 4 ? 1 : 4 / TQ;  // rows at a time
#pragma unroll
            for (int i = 0; i < TP; ++i)
#pragma unroll
                for (int r0 = 0; r0 < 16; r0 += RG) {
                    double v[RG][TQ], aa[RG], ba[RG], r2[RG];
                    int64_t rowoff[RG];
#pragma unroll
                    for (int r = 0; r < RG; ++r) {
                        const int t = wrow + i * 32 + 8 * ((r0 + r) >> 2) + 4 * (lane >> 5) + ((r0 + r) & 3);
                        rowoff[r] = (int64_t)(p0 + t) * N;
                        aa[r] = tab[t];
                        ba[r] = tab[BP + t];
                        r2[r] = tab[2 * BP + t];
                    }
                    auto each = [&](auto&& f) {
#pragma unroll
                        for (int r = 0; r < RG; ++r)
#pragma unroll
                            for (int j = 0; j < TQ; ++j) f(r, j);
                        __builtin_amdgcn_sched_barrier(0);
                    };
                    // (operation by operation what the compiler makes of the expression below)
                    each([&](int r, int j) { v[r][j] = (double)value(acc[i][j][r0 + r]); });
                    each([&](int r, int j) { v[r][j] = aa[r] * v[r][j]; });
                    each([&](int r, int j) { v[r][j] = __builtin_fma(ba[r], sw[j], v[r][j]); });
                    each([&](int r, int j) { v[r][j] = aw[j] * v[r][j]; });
                    each([&](int r, int j) { v[r][j] = __builtin_fma(bw[j], r2[r], v[r][j]); });
                    if (TAIL) {
                        each([&](int r, int j) { v[r][j] = __builtin_fmax(v[r][j], relu_floor); });
                        each([&](int r, int j) { v[r][j] = __builtin_fma(bs[j], v[r][j], bh[j]); });
                    }
                    each([&](int r, int j) { yp[j][rowoff[r]] = (float)v[r][j]; });
                }
            return;
        }
#pragma unroll
        for (int i = 0; i < TP; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int t = wrow + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                const int m = p0 + t;
                const bool mok = FULL || m < prm.RP;
                double aa = 0.0, ba = 0.0, r2 = 0.0;
                if (Y) {
                    aa = tab[t];
                    ba = tab[BP + t];
                    r2 = tab[2 * BP + t];
                }
                const int64_t rowoff = (int64_t)m * N;
#pragma unroll
                for (int j = 0; j < TQ; ++j) {
                    if (FULL || (mok && nok[j])) {
                        const auto D = value(acc[i][j][r]);
                        if (ACC) accp[j][rowoff] = (int)D;
                        if (Y) {
                            double v = aw[j] * (aa * (double)D + ba * sw[j]) + bw[j] * r2;
                            if (TAIL) v = bs[j] * __builtin_fmax(v, relu_floor) + bh[j];
                            if constexpr (NT)
                                __builtin_nontemporal_store((float)v, yp[j] + rowoff);
                            else
                                yp[j][rowoff] = (float)v;
                        }
                    }
                }
                // keep the scheduler from hoisting every later load up here (every 4 rows let the FP4
                // 256 x 256 tile spill: 60 against 54 us at 4096^3 with ReLU and BN; the bf16 one still
                // spills 16 registers, the bit planes' 3)
                if ((r & 1) == 1) __builtin_amdgcn_sched_barrier(0);
            }
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    if (!prm.y)
        full_tile ? run(yes, yes, no, no) : run(no, yes, no, no);
    else if (prm.acc)
        full_tile ? run(yes, yes, yes, yes) : run(no, yes, yes, yes);
    else if (!full_tile)
        run(no, no, yes, yes);
    else
        ep.relu || has_bn ? run(yes, no, yes, yes) : run(yes, no, yes, no);
}

// MINW = waves per SIMD the register allocation must leave room for.
//
// HC != 0 selects the halo variant of the conv (stride 1, KH = 2 pad + 1,
// KW = 2 pad + 1, Cpad = HC in {64, 128}).  There output pixel m reads input
// pixel m + (kh - pad) W + (kw - pad) of the same flattened (image, row,
// column) index space, so the BQ output pixels of a tile need the contiguous
// run of BQ + 2 pad (W + 1) input pixels around them.  The block loads that
// run once into LDS and every tap reads its fragments from there: the input
// crosses L2 -> LDS about 1.4 times instead of KH KW times, and only the
// weight tile still streams through the ring.
//
// TERN != 0 selects the conv whose epilogue ternarizes its own output (codes for
// the next layer instead of acc / y); 2 is the block-tail form of it (residual
// add, second ReLU, fp32 copy of the result).  Each is a kernel of its own so
// that its epilogue does not enter the register budget of the others.
//
// DT = 1 multiplies bf16 operands into fp32 accumulators (v_mfma_f32_32x32x16_bf16; a
// lane's 16 operand bytes are 8 bf16 of the same row, so tiles, ring and fragment
// addressing are those of the int8 form): the weight-only ternary GEMM, whose
// activations are fp32 values split into three bf16 terms laid side by side along K.
// DT = 2 multiplies FP4 (E2M1) codes (v_mfma_f32_32x32x64_f8f6f4, both operands FP4,
// no scaling): a lane's 16 operand bytes are 32 codes of one row, everything else is
// byte for byte the int8 form.  Which 32 of a K-step's 128 codes a lane holds, and in
// which nibble order, is the same for both operands, so the sum over k is unaffected.
template <int BP, int BQ, int WGP, int WGQ, int NS, int MINW, bool CONV, int TERN = 0, int HC = 0, int DT = 0, bool NT = false, bool BIG = false>
__global__ __launch_bounds__(256, MINW) void k_tmm(TmmParams prm)
{
    static_assert(DT != 1 || !CONV, "bf16 operands: GEMM only");
    static_assert(!TERN || CONV, "the ternarizing epilogue belongs to the conv");
    static_assert(WGP * WGQ == 4, "4 waves per block");
    constexpr bool HALO = HC != 0;
    static_assert(!HALO || (CONV && (HC == 64 || HC == 128)), "halo variant: conv with Cpad 64 or 128");
    constexpr int WP = BP / WGP, WQ = BQ / WGQ, TP = WP / 32, TQ = WQ / 32;
    constexpr int LP = BP / 64, LQ = HALO ? 0 : BQ / 64;  // direct loads per wave per K-step
    constexpr int LQA = LQ ? LQ : 1;                       // array extent
    constexpr int DPS = LP + LQ;
    constexpr int NM = TP * TQ;  // MFMAs per k-slice
    static_assert(TP >= 1 && TQ >= 1 && LP >= 1, "tile too small");
    static_assert(NS >= 2 && (NS - 2) * DPS < 64 && 3 * DPS < 64, "vmcnt range");
    constexpr int STAGE = (BP + (HALO ? 0 : BQ)) * 64;  // bytes; P tile first, then Q tile

    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    const unsigned lds0 = (unsigned)(uintptr_t)smem;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform, lives in an SGPR
    const int wp = wave / WGQ, wq = wave % WGQ;
    int tileP, tileQ;
    if (!block_tile(prm, tileP, tileQ)) return;
    const int p0 = tileP * BP, q0 = tileQ * BQ;
    const ConvGeom& g = prm.g;
    // Wave priority falls along a block's life: the waves that still have to get
    // their operand loads into the memory pipeline go first, those in the K loop
    // next, those that only have output left to store last (measured: 2-5 % on the
    // conv layers, because a new block's loads no longer queue behind other blocks'
    // stores as often).
    __builtin_amdgcn_s_setprio(3);
    // LDS: [halo pixels hrows x HC][128 zero bytes][operand ring][conv: epilogue table]
    // [ternarizing conv: BP threshold pairs]; the GEMM builds its small table over the ring
    const int zoff = HALO ? prm.hrows * HC : 0;
    const int roff = HALO ? zoff + 128 : 0;
    const int toff = roff + NS * STAGE;
    const int tab_kib = CONV ? (conv_table_bytes(BP, g) + 1023) >> 10 : 0;
    const bool want_ep = TERN || prm.y != nullptr;

    // ---- loader state ------------------------------------------------------
    // Load j of a wave covers tile rows 16*(wave + 4*j) .. +15; lane l fetches
    // row (l >> 2), logical chunk (l & 3) ^ swz(row) and lands at physical
    // chunk (l & 3) of that row.
    const int lrow = lane >> 2;
    const int lchunk = (lane & 3) ^ swz(lrow);
    // A block-uniform base and a 32-bit offset per lane (at most 256 rows of at most 2^22 bytes).  The conv's Q operand
    // is counted from `bias` bytes before the first tap of the tile's first pixel, so that no offset is negative (counted
    // from its image, images of 2 GiB would not fit 32 bits); a tap outside the image gets one that reads nothing.
    // BIG: image rows for which 32 bits do not suffice (and the 64 x 64 tile, which is always there) take a pointer per
    // lane, the zero page for such a tap, and five more instructions per load.
    const v4i rsrcP = buffer_base(prm.P + (int64_t)p0 * prm.ldP);
    unsigned offP[LP];
#pragma unroll
    for (int j = 0; j < LP; ++j) {
        int row = p0 + 16 * (wave + 4 * j) + lrow;
        row = row < prm.RP ? row : prm.RP - 1;  // tail rows: any valid data, never stored
        offP[j] = (unsigned)(row - p0) * (unsigned)prm.ldP + lchunk * 16;
    }
    const int8_t* gQ[LQA];
    unsigned offQ[LQA];
    int vout[LQA];  // conv: bit kh = row tap outside the image, bit (8 + kw) = column tap outside
    int bias = 0, first_px = 0;  // (the pixel may lie before the tensor)
    if (CONV && !HALO && !BIG) {
        const int nb = (int)fastdiv((uint32_t)q0, g.div_ohw), pix = q0 - nb * (g.OH * g.OW);
        const int oh = (int)fastdiv((uint32_t)pix, g.div_ow), ow = pix - oh * g.OW;
        first_px = (nb * g.H + oh * g.stride - g.pad) * g.W + ow * g.stride - g.pad;
        bias = (int)conv_reach_back(g.pad, g.W) * g.Cpad;
    }
    const v4i rsrcQ = buffer_base(CONV ? prm.Q + (int64_t)first_px * g.Cpad - bias : prm.Q + (int64_t)q0 * prm.ldQ);
#pragma unroll
    for (int j = 0; j < LQ; ++j) {
        int row = q0 + 16 * (wave + 4 * j) + lrow;
        row = row < prm.RQ ? row : prm.RQ - 1;
        gQ[j] = nullptr;
        offQ[j] = 0;
        vout[j] = 0;
        if (CONV) {
            const int ohw = g.OH * g.OW;
            const int nb = (int)fastdiv((uint32_t)row, g.div_ohw), pix = row - nb * ohw;
            const int oh = (int)fastdiv((uint32_t)pix, g.div_ow), ow = pix - oh * g.OW;
            const int ih0 = oh * g.stride - g.pad, iw0 = ow * g.stride - g.pad;
            vout[j] = ~(tap_mask(ih0, g.KH, g.H) | tap_mask(iw0, g.KW, g.W) << 8);
            if (BIG)
                gQ[j] = prm.Q + (((int64_t)nb * g.H + ih0) * g.W + iw0) * g.Cpad + lchunk * 16;
            else
                offQ[j] = (unsigned)((nb * g.H + ih0) * g.W + iw0 - first_px) * (unsigned)g.Cpad + (unsigned)(bias + lchunk * 16);
        } else {
            offQ[j] = (unsigned)(row - q0) * (unsigned)prm.ldQ + lchunk * 16;
        }
    }
    // K position of the next step to issue: byte offset into a P row and, for Q, into a dense row or of the tap
    // (kh, kw) and its 64 channels from a pixel's first tap.
    using KOff = ConvOff<BIG>;
    unsigned n_kP = 0, n_slot = 0, is_kP = 0, is_base = 0;
    KOff is_kQ = 0;
    TapWalk<KOff> n_q;
    int is_shr = 31, is_shc = 23;  // shifts that bring bits kh, 8 + kw to the sign
    const unsigned ring0 = lds0 + (unsigned)(roff + wave * 1024);
    const KOff rowskip = CONV ? TapWalk<KOff>::row_skip(g.W, g.KW, g.Cpad) : 0;
    const int8_t* zero_page = (const int8_t*)g_zero16;
    auto issue_begin = [&]() {
        is_base = ring0 + n_slot;
        is_kP = n_kP;
        is_kQ = n_q.off;
        n_slot = n_slot + STAGE == NS * STAGE ? 0u : n_slot + STAGE;
        n_kP += 64;
        if (CONV && !HALO) {
            is_shr = n_q.shr;
            is_shc = 23 - n_q.kw;
            n_q.step(g.Cpad, g.KW, rowskip);
        } else {
            n_q.off += 64;
        }
        if (DT == 1) n_q.off = n_q.off == prm.wwrap ? 0u : n_q.off;
    };
    // (the 256 x 256 conv tile: its offsets live in vector registers)
    constexpr bool FULL_SGPRS = CONV && BP == 256 && BQ == 256;
    // the idx-th of the DPS direct loads of the step set up by issue_begin()
    auto issue_one = [&](auto index) {
        constexpr int idx = decltype(index)::value;
        if constexpr (idx < LP) {
            dma_buf<4096 * idx, FULL_SGPRS>(rsrcP, offP[idx], is_kP, is_base);
        } else if constexpr (LQ != 0) {
            constexpr int j = idx - LP;
            if constexpr (CONV) {
                const int out = vout[j] << is_shr | vout[j] << is_shc;
                if constexpr (BIG)
                    dma16<BP * 64 + 4096 * j>(out < 0 ? zero_page : gQ[j] + is_kQ, is_base);
                else
                    dma_buf<BP * 64 + 4096 * j, FULL_SGPRS>(rsrcQ, offQ[j] | ((unsigned)out & kOutside), is_kQ, is_base);
            } else {
                dma_buf<BP * 64 + 4096 * j>(rsrcQ, offQ[j], is_kQ, is_base);
            }
        }
    };
    auto issue_some = [&](auto from, auto to) {  // loads from .. to - 1
        constexpr int f = decltype(from)::value, n = decltype(to)::value - f;
        if constexpr (n > 0) issue_one(std::integral_constant<int, f>{});
        if constexpr (n > 1) issue_one(std::integral_constant<int, f + 1>{});
        if constexpr (n > 2) issue_one(std::integral_constant<int, f + 2>{});
        if constexpr (n > 3) issue_one(std::integral_constant<int, f + 3>{});
        static_assert(n <= 4, "loads behind one matrix instruction");
    };
    auto issue = [&]() {
        issue_begin();
        issue_some(std::integral_constant<int, 0>{}, std::integral_constant<int, (DPS < 4 ? DPS : 4)>{});
        issue_some(std::integral_constant<int, (DPS < 4 ? DPS : 4)>{}, std::integral_constant<int, DPS>{});
    };

    // ---- fragment addressing ------------------------------------------------
    // Lane l of an MFMA operand holds row (l & 31), 16 consecutive k-bytes of
    // the k-slice at chunk (l >> 5); both operands use the same k pairing.
    int fragP[TP][2], fragQ[TQ][2];
#pragma unroll
    for (int t = 0; t < TP; ++t) {
        const int row = wp * WP + t * 32 + (lane & 31);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) fragP[t][ks] = row * 64 + (((ks * 2 + (lane >> 5)) ^ swz(row)) << 4);
    }
#pragma unroll
    for (int t = 0; t < TQ; ++t) {
        const int row = wq * WQ + t * 32 + (lane & 31);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
            fragQ[t][ks] = BP * 64 + row * 64 + (((ks * 2 + (lane >> 5)) ^ swz(row)) << 4);
    }
    // Halo variant: the Q fragment of tap (kh, kw), channel offset cc is row
    // ml + kh W + kw of the pixel run (ml = the lane's output pixel within the
    // tile), 16 bytes at chunk q = cc/16 + 2 ks + (l >> 5); a tap outside the image reads the zero bytes
    // behind the run.  The two slices of a step differ in one bit of the address, so it is formed once per step.
    int mlb[TQ];
    int vmq[TQ];  // bit kh = row tap outside the image, bit (8 + kw) = column tap outside
    int fq[TQ];
#pragma unroll
    for (int j = 0; j < TQ; ++j) {
        mlb[j] = wq * WQ + j * 32 + (lane & 31);
        vmq[j] = fq[j] = 0;
        if (HALO) {
            int m = q0 + mlb[j];
            m = m < prm.RQ ? m : prm.RQ - 1;
            const int nb = (int)fastdiv((uint32_t)m, g.div_ohw), pix = m - nb * (g.OH * g.OW);
            const int oh = (int)fastdiv((uint32_t)pix, g.div_ow), ow = pix - oh * g.OW;
            vmq[j] = ~(tap_mask(oh - g.pad, g.KH, g.H) | tap_mask(ow - g.pad, g.KW, g.W) << 8);
        }
    }
    // K position of the fragments being read: chunk, tap as a row offset and as shifts of the masks above
    int f_q = 0, f_kw = 0, f_shr = 31, f_tapoff = 0;
    auto frag_step_advance = [&]() {
        f_q += 4;
        const bool tap = f_q == HC / 16;
        f_q = tap ? 0 : f_q;
        f_kw += tap ? 1 : 0;
        f_tapoff += tap ? 1 : 0;
        const bool end = f_kw == g.KW;
        f_kw = end ? 0 : f_kw;
        f_shr -= end ? 1 : 0;
        f_tapoff += end ? g.W - g.KW : 0;
    };
    v4i fa[2][TP], fb[2][TQ];
    constexpr int NF = TP + TQ;  // fragments per k-slice
    // idx-th fragment of slice ks of the step in stage `slot` (its offset in the ring): P fragments first, then Q
    auto load_frag = [&](unsigned slot, int ks, int idx) {
        const int8_t* st = smem + roff + slot;
        if (idx < TP) {
            fa[ks][idx] = *(const v4i*)(st + fragP[idx][ks]);
        } else if (!HALO) {
            fb[ks][idx - TP] = *(const v4i*)(st + fragQ[idx - TP][ks]);
        } else {
            const int j = idx - TP;
            if (ks == 0) {
                const int out = vmq[j] << f_shr | vmq[j] << (23 - f_kw);
                fq[j] = out < 0 ? zoff : halo_byte<HC>(mlb[j] + f_tapoff, f_q + (lane >> 5));
            }
            fb[ks][j] = *(const v4i*)(smem + (fq[j] ^ (32 * ks)));
        }
    };
    auto load_frags = [&](unsigned slot, int ks) {
#pragma unroll
        for (int i = 0; i < NF; ++i) load_frag(slot, ks, i);
    };

    // conv: Sa of an output pixel -- the sum of t_a over its in-bounds taps -- is the
    // sum of all code bytes of its row of the patch matrix (out-of-image taps are zero
    // bytes), i.e. of the Q fragments this lane multiplies anyway: 4 byte-sum dot
    // products per fragment, added up beside the MFMAs.  A lane holds half of a
    // row's bytes (the other k-chunks sit in lane ^ 32); the halves meet in the epilogue.
    // FP4 codes: the row sums come from the matrix cores as well, which have cycles to spare
    // while the vector ALU does not: one 16x16x128 FP4 MFMA per Q fragment with a constant
    // operand of +1 codes.  That instruction reads lane l's 16 bytes as row l & 15, k-block
    // l >> 4, whereas the fragment holds pixel l & 31, k-chunk l >> 5: k-blocks 0 and 2 are
    // the two chunks of pixel l & 15, k-blocks 1 and 3 those of pixel 16 + (l & 15).  With
    // ones in row 0 over k-blocks 0, 2 and in row 1 over k-blocks 1, 3, output row 0 is the
    // sum of pixels 0..15 and row 1 that of pixels 16..31 (registers 0 and 1 of lanes 0..15).
    int sa_part[TQ];
    v4f sa_acc[DT == 2 ? TQ : 1];
#pragma unroll
    for (int j = 0; j < TQ; ++j) sa_part[j] = 0;
#pragma unroll
    for (int j = 0; j < (DT == 2 ? TQ : 1); ++j) sa_acc[j] = v4f{0.f, 0.f, 0.f, 0.f};
    const int sa_ones = ((lane & 15) < 2 && ((lane >> 4) & 1) == (lane & 15)) ? 0x22222222 : 0;
    const v8i SA8 = {sa_ones, sa_ones, sa_ones, sa_ones, 0, 0, 0, 0};
    (void)SA8;
    using AccV = std::conditional_t<DT != 0, v16f, v16i>;
    AccV acc[TP][TQ];
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
        for (int j = 0; j < TQ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
    // One k-slice of MFMAs in a fixed issue order: after the n-th MFMA come its
    // share of the next slice's fragment reads (slice fks of the step in stage fslot) and, if
    // ISSUE, of the next step's direct loads; a scheduling fence after each
    // group keeps the compiler from sinking the reads back to their first use,
    // so LDS and load-issue latency hide behind matrix-core time.
    auto slice = [&](auto with_frags, auto with_issue, int ks, unsigned fslot, int fks) {
        constexpr bool FRAGS = decltype(with_frags)::value, ISSUE = decltype(with_issue)::value;
        if (ISSUE && NM > 1) issue_begin();
        if (HALO && FRAGS && fks == 0) frag_step_advance();
        auto group = [&](auto index) {
            constexpr int n = decltype(index)::value;
            if constexpr (DT == 1)
                acc[n / TQ][n % TQ] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(v8bf, fa[ks][n / TQ]), __builtin_bit_cast(v8bf, fb[ks][n % TQ]),
                    acc[n / TQ][n % TQ], 0, 0, 0);
            else if constexpr (DT == 2) {
                // cbsz = blgp = 4: both operands FP4; the upper half of the 8-register operand is unused
                const v4i pa = fa[ks][n / TQ], pb = fb[ks][n % TQ];
                const v8i A8 = {pa[0], pa[1], pa[2], pa[3], 0, 0, 0, 0}, B8 = {pb[0], pb[1], pb[2], pb[3], 0, 0, 0, 0};
                acc[n / TQ][n % TQ] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A8, B8, acc[n / TQ][n % TQ], 4, 4, 0,
                                                                                      0, 0, 0);
                if constexpr (CONV && n < TQ)
                    sa_acc[n] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(SA8, B8, sa_acc[n], 4, 4, 0, 0, 0, 0);
            } else
                acc[n / TQ][n % TQ] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[ks][n / TQ], fb[ks][n % TQ],
                                                                            acc[n / TQ][n % TQ], 0, 0, 0);
            if (FRAGS) {
                // front-loaded: one read per MFMA when there are enough MFMAs,
                // so the last read is long done at the end of the slice
                constexpr int PER = (NF + NM - 1) / NM;
#pragma unroll
                for (int f = n * PER; f < (n + 1) * PER && f < NF; ++f) load_frag(fslot, fks, f);
            }
            if constexpr (ISSUE)
                issue_some(std::integral_constant<int, n * DPS / NM>{}, std::integral_constant<int, (n + 1) * DPS / NM>{});
            __builtin_amdgcn_sched_barrier(0);
        };
        for_each_index(group, std::make_integer_sequence<int, NM>{});
        if (CONV && DT == 0) {
#pragma unroll
            for (int j = 0; j < TQ; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) sa_part[j] = __builtin_amdgcn_sdot4(fb[ks][j][e], 0x01010101, sa_part[j], false);
        }
    };
    const std::true_type yes{};
    const std::false_type no{};

    // ---- prologue: start the first NS steps, then per-lane epilogue terms -----
    const int nk = prm.nk;
    const int npro = nk < NS ? nk : NS;
    if (TERN) {
        // thresholds of this tile's channels, (lo, hi) pairs behind the table
        // (visible to every wave after the first barrier of the main loop)
        if (tid < BP) {
            const int o = p0 + tid < prm.RP ? p0 + tid : prm.RP - 1;
            ((float2*)(smem + toff + tab_kib * 1024))[tid] = make_float2((float)pval(prm.thr_lo, o), (float)pval(prm.thr_hi, o));
        }
    }
    if (CONV && want_ep) {
        // epilogue table: rows [g1, c2, bn scale, bn shift, class constants...] of the
        // prepared per-layer table, columns p0 .. p0+BP-1, copied as they are
        // (the class rows that can occur here, see conv_lds_classes)
        const int nrows = 4 + conv_classes(g.pad), opitch = (g.O + 1) & ~1;
        const bool compact = conv_compact(g);
        const int nax = conv_axis_classes(g), lrows = 4 + nax * nax, pp = (g.pad + 1) * (g.pad + 1);
        for (int n = wave; n < tab_kib; n += 4) {
            const int lin = n * 64 + lane;  // 16-byte unit = 2 doubles
            int row = lin / (BP / 2);
            const int u = lin - row * (BP / 2);
            row = row < lrows ? row : lrows - 1;
            if (row >= 4) {
                const int c = row - 4, ra = (int)fastdiv((uint32_t)c, prm.div_nax), ca = c - ra * nax;
                row = 4 + conv_axis_global(compact, g.pad, ra) * pp + conv_axis_global(compact, g.pad, ca);
            }
            int64_t idx = (int64_t)row * opitch + p0 + 2 * u;
            const int64_t last = (int64_t)nrows * opitch - 2;
            idx = idx < last ? idx : last;  // columns past O are never used
            dma16(prm.cst_cls + idx, lds0 + (unsigned)(toff + n * 1024));
        }
    }
    if (HALO) {
        // the pixel run: 1 KiB per load, lane l lands at 16-byte unit n*64 + l; which chunk
        // of its row a lane fetches is permuted as halo_byte() has it.  Runs past either
        // end of the tensor re-read the end pixel (only out-of-image taps point there).
        const int total_px = g.Nb * g.H * g.W;
        const int first_px = q0 - g.pad * (g.W + 1);
        const int ninstr = prm.hrows * HC / 1024;
        for (int n = wave; n < ninstr; n += 4) {
            const int lin = n * 64 + lane;
            const int row = lin / (HC / 16), qp = lin % (HC / 16);
            int px = first_px + row;
            px = px < 0 ? 0 : (px < total_px ? px : total_px - 1);
            dma16(prm.Q + (int64_t)px * HC + (halo_byte<HC>(row, qp) & (HC - 1)), lds0 + (unsigned)(n * 1024));
        }
        if (tid < 8) *(uint4*)(smem + zoff + tid * 16) = make_uint4(0, 0, 0, 0);
    }
    for (int s = 0; s < npro; ++s) issue();

    // Block-tail form: where this lane's output pixels lie in the residual and in y, in bytes from channel p0 + wp WP of the
    // image of pixel q0 (the rows of a tile that lie 4 apart are lane halves): an access is then a scalar pointer per
    // row and a 32-bit lane offset (with a 64-bit lane address each, and bounds tests on whole tiles, the 64
    // loads of a lane were 900 instructions).
    using Off = std::conditional_t<BIG, int64_t, uint32_t>;
    const bool full_tile = p0 + BP <= prm.RP && q0 + BQ <= prm.RQ;
    Off yoff[TERN == 2 ? TQ : 1];
    int64_t ybase = 0;
    if constexpr (TERN == 2) {
        const int ohw = g.OH * g.OW, nbq = (int)fastdiv((uint32_t)q0, g.div_ohw);
        ybase = ((int64_t)nbq * g.O + p0 + wp * WP) * ohw;
#pragma unroll
        for (int j = 0; j < TQ; ++j) {
            int m = q0 + wq * WQ + j * 32 + (lane & 31);
            m = m < prm.RQ ? m : prm.RQ - 1;
            const int nb = (int)fastdiv((uint32_t)m, g.div_ohw), pix = m - nb * ohw;
            yoff[j] = ((Off)(nb - nbq) * (Off)g.O * (Off)ohw + (Off)pix + (Off)(lane >> 5) * 4 * (Off)ohw) * 4;
        }
    }
    // row 8 (r >> 2) + 4 half + (r & 3) of 32-row tile i, of a tensor at `t`
    auto row_of = [&](auto* t, int i, int r) {
        return t + ybase + (int64_t)(i * 32 + 8 * (r >> 2) + (r & 3)) * (g.OH * g.OW);
    };
    auto at = [](auto* row, Off off) { return (decltype(row))((char*)row + off); };
    (void)row_of, (void)at, (void)ybase;
    // The residual values this lane will add, fetched now so that their
    // HBM latency passes behind the K loop (tiles whose accumulators leave the registers
    // for it; the larger tiles fetch them in the epilogue, 16 at a time).
    constexpr bool RES_EARLY = TERN == 2 && TP * TQ <= 4;
    float rv_all[RES_EARLY ? TQ : 1][RES_EARLY ? TP : 1][16];
    if constexpr (RES_EARLY) {
        auto load_res = [&](auto full) {
#pragma unroll
            for (int i = 0; i < TP; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float* row = row_of((float*)prm.res, i, r);
                    const int o = p0 + wp * WP + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
#pragma unroll
                    for (int j = 0; j < TQ; ++j) {
                        rv_all[j][i][r] = 0.0f;
                        if (decltype(full)::value || (q0 + wq * WQ + j * 32 + (lane & 31) < prm.RQ && o < prm.RP))
                            rv_all[j][i][r] = __builtin_nontemporal_load(at(row, yoff[j]));
                    }
                }
        };
        if (!prm.res) {
#pragma unroll
            for (int j = 0; j < TQ; ++j)
#pragma unroll
                for (int i = 0; i < TP; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) rv_all[j][i][r] = 0.0f;
        } else if (full_tile) {
            load_res(std::true_type{});
        } else {
            load_res(std::false_type{});
        }
    }

    // conv: the border class of each of this lane's TQ output pixels,
    //   class = rid * (pad+1)^2 + cid,  rid = khl + (pad+1)*(KH-1-khh), cid likewise;
    //   class 0 is the interior (all taps in bounds).
    int pixcls[TQ];
#pragma unroll
    for (int j = 0; j < TQ; ++j) pixcls[j] = 0;
    if (CONV && want_ep && !g.code_zero_pad) {
        const int ohw = g.OH * g.OW;
#pragma unroll
        for (int j = 0; j < TQ; ++j) {
            int m = q0 + wq * WQ + j * 32 + (lane & 31);
            m = m < prm.RQ ? m : prm.RQ - 1;
            const int nb = (int)fastdiv((uint32_t)m, g.div_ohw), pix = m - nb * ohw;
            const int oh = (int)fastdiv((uint32_t)pix, g.div_ow), ow = pix - oh * g.OW;
            int khl, khh, kwl, kwh;
            tap_range(oh, g.stride, g.pad, g.KH, g.H, khl, khh);
            tap_range(ow, g.stride, g.pad, g.KW, g.W, kwl, kwh);
            const bool compact = conv_compact(g);
            pixcls[j] = conv_axis_class(compact, g.pad, khl, g.KH - 1 - khh) * conv_axis_classes(g) +
                        conv_axis_class(compact, g.pad, kwl, g.KW - 1 - kwh);
        }
    }
    __builtin_amdgcn_s_setprio(2);
    // ---- main loop ------------------------------------------------------------
    // Steps kt .. kt+NS-1 are in flight or resident while step kt is multiplied.
    wait_groups<DPS>(npro - 1);
    wait_lgkm0();  // the prologue's plain LDS stores (halo zero bytes, threshold pairs)
    block_barrier();
    load_frags(0, 0);
    int kt = 0;
    unsigned cur = 0, nxt = STAGE;  // stages of steps kt and kt + 1
    auto after = [&](unsigned slot) { return slot + STAGE == NS * STAGE ? 0u : slot + STAGE; };
    auto advance = [&]() {
        cur = nxt;
        nxt = after(nxt);
    };
    // Steady state: between the two k-slices, stage kt is fully in registers
    // (slice-1 fragments waited for), step kt+1 has landed for this wave
    // (all but the NS-2 younger load groups done) and, after the barrier, for
    // every wave; the freed stage is refilled with step kt+NS.
    for (; kt + NS < nk; ++kt) {
        slice(yes, no, 0, cur, 1);
        unsigned third = after(nxt);
        if (NM == 1) {
            // (one matrix instruction per slice: a step is a chain of LDS reads, and this bookkeeping passes behind the
            // first of them; behind the second one the loads do)
            issue_begin();
            __builtin_amdgcn_sched_barrier(0);
        }
        wait_lgkm0();
        wait_vm<(NS - 2) * DPS>();
        block_barrier();
        slice(yes, yes, 1, nxt, 0);
        cur = nxt, nxt = third;
    }
    // Drain: nothing left to issue.
    for (; kt + 1 < nk; ++kt) {
        slice(yes, no, 0, cur, 1);
        wait_lgkm0();
        wait_vm<0>();
        block_barrier();
        slice(yes, no, 1, nxt, 0);
        advance();
    }
    slice(yes, no, 0, cur, 1);
    slice(no, no, 1, 0, 0);

    __builtin_amdgcn_s_setprio(0);
    // ---- epilogue ---------------------------------------------------------------
    // Large conv outputs are written with the non-temporal hint, small ones plainly.  A plain
    // store leaves its dirty lines in the cache hierarchy; when the output is larger than
    // what the memory-side cache holds they are written back while the *next* kernel
    // runs and slow it more than the hint slows this one (205 MB stored, then 205 MB
    // read: 92 us plain, 75 us with the hint).  An output that fits is stored about twice
    // as fast without the hint, and the kernel after it is not slowed (51 MB: 25 us
    // against 39 us for the pair).  The launch code decides (prm.nt_out).
    // (a tag type, not a run-time test at the store: the compiler merges the two arms of such
    // a test into one plain store)
    const bool nt_out = CONV && prm.nt_out;
    auto put = [&](auto nt, auto value, auto* ptr) {
        if constexpr (decltype(nt)::value)
            __builtin_nontemporal_store(value, ptr);
        else
            *ptr = value;
    };
    const EpiArgs& ep = prm.ep;
    // ReLU and BN with neutral parameters when off, as in gemm_epilogue
    const double relu_floor = __builtin_canonicalize(ep.relu ? 0.0 : -__builtin_inf());
    double* tab = (double*)(smem + (CONV ? toff : 0));
    // The element loops exist in 6 straight-line variants (interior / ragged
    // tile) x (acc only / y only / both), picked once per block.
    auto dispatch3 = [&](auto&& run, auto nt) {
        if (full_tile) {
            if (!prm.y)
                run(std::true_type{}, std::true_type{}, std::false_type{}, nt);
            else if (!prm.acc)
                run(std::true_type{}, std::false_type{}, std::true_type{}, nt);
            else
                run(std::true_type{}, std::true_type{}, std::true_type{}, nt);
        } else {
            if (!prm.y)
                run(std::false_type{}, std::true_type{}, std::false_type{}, nt);
            else if (!prm.acc)
                run(std::false_type{}, std::false_type{}, std::true_type{}, nt);
            else
                run(std::false_type{}, std::true_type{}, std::true_type{}, nt);
        }
    };
    auto dispatch = [&](auto&& run) {
        if (nt_out)
            dispatch3(run, std::true_type{});
        else
            dispatch3(run, std::false_type{});
    };
    if constexpr (!CONV) {
        gemm_epilogue<BP, TP, TQ, DT != 1, false, NT>(prm, (double*)smem, p0, q0, wp * WP, wq * WQ, full_tile, acc,
                                            [](auto d) { return d; });
    } else {
        // y = g1[o]*D + c2[o]*Sa[m] + Cst[class(m)][o],  g1 = aa*aw, c2 = aa*bw;
        // tab = [4 + ncls][BP]: g1, c2, bn scale, bn shift, then the class constants.
        const int ohw = g.OH * g.OW;
        const int p1 = g.pad + 1;
        (void)p1;
        // (the table was copied into LDS by the prologue's direct loads)
        int sa_full[TQ];
#pragma unroll
        for (int j = 0; j < TQ; ++j) {
            if constexpr (DT == 2) {
                const float s0 = __shfl(sa_acc[j][0], lane & 15, 64), s1 = __shfl(sa_acc[j][1], lane & 15, 64);
                sa_full[j] = (int)((lane & 16) ? s1 : s0);
            } else {
                const int mine = sa_part[j];
                sa_full[j] = mine + __shfl_xor(mine, 32, 64);
            }
        }
        if constexpr (TERN) {
            // Ternarizing epilogue (Eq.1 / Eq.3 applied to the activation of Eq.9): the
            // fp32 value z is formed exactly as below, compared with the channel's
            // thresholds, and only the code leaves the chip.  A lane's accumulator
            // registers 4 r4 .. 4 r4 + 3 are 4 consecutive channels of one pixel: one
            // dword of the channel-innermost code tensor.  Channels O .. ldc-1 get code 0.
            const float2* thr = (const float2*)(smem + toff + tab_kib * 1024);
            // STREAM: the block-tail form -- z + residual (fp32 add, as a separate add
            // kernel would do it), a second ReLU, and the fp32 result stored as well.
            const float relu_out_floor = __builtin_canonicalizef(prm.relu_out ? 0.0f : -__builtin_inff());
            // A channel's factors are read from LDS once for the lane's TQ pixels: pixel by pixel (48 bytes per output
            // and lane, at 128 bytes a cycle for the CU) those reads were more than the arithmetic: 64 filters on 56 x 56,
            // 256 images, ternarizing, 67.1 -> 60.1 us (with the halo addresses above).
            auto run_codes = [&](auto full, auto stream, auto nt) {
                constexpr bool FULL = decltype(full)::value, STREAM = decltype(stream)::value;
                bool mok[TQ];
                int8_t* cp[TQ];
                double Sa[TQ];
                const double* ctab[TQ];
#pragma unroll
                for (int j = 0; j < TQ; ++j) {
                    const int m = q0 + wq * WQ + j * 32 + (lane & 31);
                    mok[j] = FULL || m < prm.RQ;
                    cp[j] = prm.codes + (int64_t)(mok[j] ? m : 0) * prm.ldc;
                    Sa[j] = (double)sa_full[j];
                    ctab[j] = tab + (4 + pixcls[j]) * BP;
                }
#pragma unroll
                for (int i = 0; i < TP; ++i) {
                    // residual values of this lane's 16 channels, fetched ahead of their use
                    float rv[STREAM ? TQ : 1][16];
                    if constexpr (RES_EARLY) {
#pragma unroll
                        for (int j = 0; j < TQ; ++j)
#pragma unroll
                            for (int r = 0; r < 16; ++r) rv[j][r] = rv_all[j][i][r];
                    } else if constexpr (STREAM) {
#pragma unroll
                        for (int j = 0; j < TQ; ++j)
#pragma unroll
                            for (int r = 0; r < 16; ++r) {
                                const int o = p0 + wp * WP + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                                rv[j][r] = 0.0f;
                                if (prm.res && (FULL || (mok[j] && o < prm.RP)))
                                    rv[j][r] = __builtin_nontemporal_load(at(row_of((float*)prm.res, i, r), yoff[j]));
                            }
                    }
                    unsigned half4[TQ][4];  // FP4 output: this lane's 4 nibbles of each channel group
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        const int t0 = wp * WP + i * 32 + 8 * r4 + 4 * (lane >> 5);
                        const int o0 = p0 + t0;
                        unsigned word[TQ];
#pragma unroll
                        for (int j = 0; j < TQ; ++j) word[j] = 0;
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            const int t = t0 + b;
                            const bool ook = FULL || o0 + b < prm.RP;
                            const double g1 = tab[t], c2 = tab[BP + t], bs = tab[2 * BP + t], bh = tab[3 * BP + t];
                            const float2 th = thr[t];
                            float* yrow = STREAM ? row_of(prm.y, i, 4 * r4 + b) : nullptr;
                            (void)yrow;
#pragma unroll
                            for (int j = 0; j < TQ; ++j) {
                                const auto D = acc[i][j][4 * r4 + b];
                                double v = g1 * (double)D + (c2 * Sa[j] + ctab[j][t]);
                                v = __builtin_fmax(v, relu_floor);
                                float z = (float)(bs * v + bh);
                                if constexpr (STREAM) {
                                    z = __builtin_fmaxf(z + rv[j][4 * r4 + b], relu_out_floor);
                                    if (prm.y && (FULL || (mok[j] && ook))) put(nt, z, at(yrow, yoff[j]));
                                }
                                if constexpr (DT == 2) {
                                    // E2M1 nibble: +1 -> 0x2, -1 -> 0xA
                                    unsigned c = z > th.y ? 0x2u << (4 * b) : 0u;
                                    c = z < th.x ? 0xAu << (4 * b) : c;
                                    if (!FULL && !ook) c = 0;
                                    word[j] |= c;
                                } else {
                                    int code = (int)(z > th.y) - (int)(z < th.x);
                                    if (!FULL && !ook) code = 0;
                                    word[j] |= (unsigned)(code & 0xff) << (8 * b);
                                }
                            }
                        }
#pragma unroll
                        for (int j = 0; j < TQ; ++j) {
                            if constexpr (DT == 2) {
                                pin(word[j]);
                                half4[j][r4] = word[j];
                            } else {
                                if (FULL || (mok[j] && o0 < prm.ldc)) *(unsigned*)(cp[j] + o0) = word[j];
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if constexpr (DT == 2) {
                        // A dword of the FP4 code tensor is 8 consecutive channels: the 4 of this
                        // lane and the 4 of lane ^ 32 (same pixel).  The lower lane half assembles
                        // channel groups 0 and 2, the upper half groups 1 and 3; each sends the
                        // other the two 16-bit halves it needs in one cross-lane move.
                        const bool upper = (lane >> 5) != 0;
                        const int c0 = p0 + wp * WP + i * 32 + (upper ? 8 : 0);  // first channel of word wa
#pragma unroll
                        for (int j = 0; j < TQ; ++j) {
                            const unsigned(&h)[4] = half4[j];
                            const unsigned send = upper ? (h[0] | (h[2] << 16)) : (h[1] | (h[3] << 16));
                            const unsigned recv = (unsigned)__shfl_xor((int)send, 32, 64);
                            const unsigned wa = upper ? ((recv & 0xffffu) | (h[1] << 16)) : (h[0] | (recv << 16));
                            const unsigned wb = upper ? ((recv >> 16) | (h[3] << 16)) : (h[2] | (recv & 0xffff0000u));
                            if (FULL || (mok[j] && (c0 >> 1) < prm.ldc)) *(unsigned*)(cp[j] + (c0 >> 1)) = wa;
                            if (FULL || (mok[j] && ((c0 + 16) >> 1) < prm.ldc)) *(unsigned*)(cp[j] + ((c0 + 16) >> 1)) = wb;
                        }
                    }
                }
                if constexpr (DT == 2) {
                    // a 64-row tile covers half of a 128-code row: the last tile along the
                    // channels also writes the zero codes of the other half
                    if (BP == 64 && wp == 0 && (p0 + BP) / 2 < prm.ldc && p0 + BP >= prm.RP)
#pragma unroll
                        for (int j = 0; j < TQ; ++j)
                            if (mok[j]) *(uint4*)(cp[j] + (p0 + BP) / 2 + 16 * (lane >> 5)) = make_uint4(0, 0, 0, 0);
                }
            };
            constexpr std::integral_constant<bool, TERN == 2> tail{};
            if (TERN == 2 && nt_out) {
                if (full_tile)
                    run_codes(std::true_type{}, tail, std::true_type{});
                else
                    run_codes(std::false_type{}, tail, std::true_type{});
            } else {
                if (full_tile)
                    run_codes(std::true_type{}, tail, std::false_type{});
                else
                    run_codes(std::false_type{}, tail, std::false_type{});
            }
            return;
        }
        dispatch([&](auto full, auto want_acc, auto want_y, auto nt) {
            constexpr bool FULL = decltype(full)::value, ACC = decltype(want_acc)::value,
                           Y = decltype(want_y)::value;
            // per lane: its TQ output pixels -> Sa, class constants, output base pointers
            bool mok[TQ];
            double Sa[TQ];
            const double* ctab[TQ];
            int32_t* accp[TQ];
            float* yp[TQ];
#pragma unroll
            for (int j = 0; j < TQ; ++j) {
                const int m = q0 + wq * WQ + j * 32 + (lane & 31);
                mok[j] = FULL || m < prm.RQ;
                const int mm = mok[j] ? m : 0;
                const int nb = (int)fastdiv((uint32_t)mm, g.div_ohw), pix = mm - nb * ohw;
                const int64_t obase = (int64_t)nb * g.O * ohw + pix;
                accp[j] = ACC ? prm.acc + obase : nullptr;
                yp[j] = Y ? prm.y + obase : nullptr;
                Sa[j] = (double)sa_full[j];
                ctab[j] = tab + (4 + pixcls[j]) * BP;
            }
#pragma unroll
            for (int i = 0; i < TP; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int t = wp * WP + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                    const int o = p0 + t;
                    const bool ook = FULL || o < prm.RP;
                    double g1 = 0.0, c2 = 0.0, bs = 1.0, bh = 0.0, cc[TQ];
                    if (Y) {
                        g1 = tab[t];
                        c2 = tab[BP + t];
                        bs = tab[2 * BP + t];
                        bh = tab[3 * BP + t];
#pragma unroll
                        for (int j = 0; j < TQ; ++j) cc[j] = ctab[j][t];
                    }
                    const int64_t rowoff = (int64_t)o * ohw;
#pragma unroll
                    for (int j = 0; j < TQ; ++j) {
                        if (FULL || (ook && mok[j])) {
                            const auto D = acc[i][j][r];
                            if (ACC) put(nt, (int)D, accp[j] + rowoff);
                            if (Y) {
                                double v = g1 * (double)D + (c2 * Sa[j] + cc[j]);
                                v = __builtin_fmax(v, relu_floor);
                                put(nt, (float)(bs * v + bh), yp[j] + rowoff);
                            }
                        }
                    }
                    if ((r & 1) == 1) __builtin_amdgcn_sched_barrier(0);
                }
        });
    }
}

// LDS bytes of the epilogue tables of a BP-row tile.
inline int64_t table_bytes(int bp, bool conv, const ConvGeom& g)
{
    return conv ? (int64_t)conv_table_bytes(bp, g) : (int64_t)3 * bp * 8;
}

// Halo variant: stride 1, window centred on the output pixel, HC-byte pixel rows.
inline bool halo_eligible(const TmmParams& prm, int hc)
{
    const ConvGeom& g = prm.g;
    return g.stride == 1 && g.KH == 2 * g.pad + 1 && g.KW == 2 * g.pad + 1 && g.Cpad == hc && g.OH == g.H &&
           g.OW == g.W;
}

// Fills in the tile counts of a BP x BQ tiling; the grid size, or 0 if it is out of range.
inline unsigned tile_grid(TmmParams& prm, int bp, int bq)
{
    prm.tilesP = (prm.RP + bp - 1) / bp;
    const int64_t tilesQ = ((int64_t)prm.RQ + bq - 1) / bq;
    const int64_t blocks = (int64_t)prm.tilesP * tilesQ;
    if (blocks <= 0 || blocks > 0x7fffff00 || tilesQ * 8 > 0x7fffffff) return 0;
    prm.ntiles = (int)blocks;
    prm.band_tiles = (int)(8 * tilesQ);
    prm.div_band = make_fastdiv((uint32_t)prm.band_tiles);
    prm.div_lastband = make_fastdiv((uint32_t)(prm.tilesP & 7 ? prm.tilesP & 7 : 8));
    prm.div_nax = make_fastdiv((uint32_t)conv_axis_classes(prm.g));
    return (unsigned)((blocks + 7) / 8 * 8);
}

// (the pixel-run tiles, halo, take 64-bit pointers to their codes)
inline bool conv_offsets_fit(const ConvGeom& g, int bq, bool halo, bool tail)
{
    return (halo || conv_codes_fit(g.H, g.W, g.OH, g.OW, g.KH, g.KW, g.stride, g.pad, g.Cpad, bq)) &&
           (!tail || conv_outputs_fit(g.Nb, g.O, (int64_t)g.OH * g.OW, bq));
}

template <int BP, int BQ, int WGP, int WGQ, int NS, int MINW, bool CONV, int TERN = 0, int HC = 0, int DT = 0, bool NT = false, bool BIG = false>
hipError_t launch_cfg(TmmParams& prm, hipStream_t st)
{
    constexpr int ring_bytes = NS * (BP + (HC ? 0 : BQ)) * 64;
    int64_t stage_bytes = ring_bytes;
    if (CONV && !BIG && !conv_offsets_fit(prm.g, BQ, HC != 0, TERN == 2)) return hipErrorInvalidValue;
    if (HC) {
        if (!halo_eligible(prm, HC)) return hipErrorInvalidValue;
        const int64_t rows = halo_rows(BQ, prm.g.pad, prm.g.W);
        prm.hrows = (int)rows;
        stage_bytes += rows * HC + 128;
    }
    int64_t smem;
    if (CONV) {
        // ring (+ halo), then the epilogue table in whole KiB
        smem = stage_bytes + ((table_bytes(BP, true, prm.g) + 1023) & ~(int64_t)1023);
        if (TERN) smem += BP * 8;  // threshold pairs of the ternarizing epilogue
    } else {
        const int64_t tb = table_bytes(BP, false, prm.g);
        smem = stage_bytes > tb ? stage_bytes : tb;
    }
    if (smem > kMaxLds) return hipErrorInvalidValue;
    auto kern = k_tmm<BP, BQ, WGP, WGQ, NS, MINW, CONV, TERN, HC, DT, NT, BIG>;
    static LdsLimit lds;
    const hipError_t e = lds.raise((const void*)kern, (int)kMaxLds);
    if (e != hipSuccess) return e;
    const unsigned grid = tile_grid(prm, BP, BQ);
    if (!grid) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), (size_t)smem, st, prm);
    return hipGetLastError();
}

// Tile configurations, indexed as rtn_set_tile_config() documents: BP of each.
constexpr int kNumTileConfigs = 20;
constexpr int kTileBP[kNumTileConfigs] = {64, 128, 256, 64,  128, 256, 64, 64, 128, 64,
                                           64, 64,  128, 128, 64,  64,  64, 64, 128, 128};

}  // namespace

}  // namespace rtn
