// Ternary GEMM on bit planes (RTN_CODE_BITPLANE) with the FP4 matrix cores.
//
// The operands stay in the paper's 2-bit storage in memory, in L2 and in LDS -- 0.25 byte per
// code -- and become FP4 nibbles only in registers, right before the MFMA.  The kernel the
// method's own pattern gives (AND / XOR / popcount, k_gemm_popc) is bound by the vector ALU: about
// 12 instructions per 64 products of a lane, 407 us at M = N = K = 4096.  Here a
// fragment of 32 codes costs 10 vector instructions once and feeds TP or TQ MFMAs:
//
//   * E2M1 is (sign, exponent 2 bits, mantissa): sign bit over the *upper* exponent bit is +-2.0
//     (0x4, 0xC), and those are adjacent bits.  So mask and sign bits are interleaved into 2-bit
//     fields (two bit-selects per 16 codes, one plane shifted by 1) and a dword of 8 nibbles is
//     one AND, every second one after a shift by 2.  Both operands are 2 t, D is the sum / 4,
//     exact: |sum| <= 4 * 2^22 = 2^24.
//   * a zero may carry a sign (-0.0): it adds nothing.  Both operands use the stored sign bit
//     (1 <=> +1) as the number's sign, i.e. both are negated, which their product undoes.
//   * which k a nibble position stands for is the same in both operands, so the order of a
//     fragment's codes is free: lane half h takes 16-byte chunk 2 g + h of a row, and its four
//     dwords are four k-slices.
//
// A stage is 64 bytes of each plane of every tile row (512 codes, 8 MFMA k-slices), loaded global
// -> LDS directly, two stages, one barrier per stage.  EB = bytes a lane loads at once: 16, or 4
// when the rows' byte length is not a multiple of 16 (an odd number of plane words); what lies
// behind a row's end is read from the zero page.
//
// M = N = K = 4096: 48 us against 407 us for k_gemm_popc (and 37.5 us for the FP4 GEMM, which has nothing to
// expand); with an odd number of words, 4096 x 4096 x 4160, 57 us.  Bound by vector-instruction issue: per k-slice a
// wave of the 256 x 256 tile runs 80 expanding instructions for 16 MFMAs, at one wave per SIMD.  A wave tile of
// 128 x 128 halves that share against 64 x 64, hence the largest tile as soon as it gives every CU a block.
// The expansion of a slice is dealt out behind the MFMAs of the slice before, and a load costs a 32-bit lane
// offset on a scalar base (not a pointer per lane, and 271 scalar registers spilled in the 4-byte form): without the
// two, 51.5 and 72.5 us.
#include "tmm_kernel.h"

namespace rtn {

namespace {

__device__ __forceinline__ unsigned bitsel(unsigned m, unsigned a, unsigned b) { return (a & m) | (b & ~m); }

// 32 codes of one row (mask and sign dword) as an FP4 fragment of values +-2, 0
__device__ __forceinline__ v8i planes_to_fp4(unsigned m, unsigned s)
{
    const unsigned lo = bitsel(0x55555555u, m, s << 1), hi = bitsel(0x55555555u, m >> 1, s);
    return v8i{(int)(lo & 0xccccccccu), (int)((lo << 2) & 0xccccccccu), (int)(hi & 0xccccccccu),
               (int)((hi << 2) & 0xccccccccu), 0, 0, 0, 0};
}

template <int BP, int BQ, int WGP, int WGQ, int MINW, int EB>
__global__ __launch_bounds__(256, MINW) void k_gemm_planes(TmmParams prm, const int8_t* Psign, const int8_t* Qsign)
{
    constexpr int WP = BP / WGP, WQ = BQ / WGQ, TP = WP / 32, TQ = WQ / 32;
    constexpr int ROWS = 2 * (BP + BQ);          // LDS rows of a stage: P mask, P sign, Q mask, Q sign
    constexpr int STAGE = ROWS * 64;
    constexpr int RPL = EB, NL = ROWS / (4 * RPL);  // rows a wave's load covers (64 EB / 64), loads per wave
    static_assert(EB == 16 || EB == 4, "16- or 4-byte lanes");
    static_assert(BP % 64 == 0 && BQ % 64 == 0 && NL >= 1, "tile too small");

    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    const unsigned lds0 = (unsigned)(uintptr_t)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wp = wave / WGQ, wq = wave % WGQ;
    int tileP, tileQ;
    if (!block_tile(prm, tileP, tileQ)) return;
    const int p0 = tileP * BP, q0 = tileQ * BQ;
    const unsigned rowb = (unsigned)prm.ldP;  // bytes of a plane row (both operands)

    // ---- loader: load j of a wave covers stage rows RPL * (wave + 4 j) .. + RPL - 1 ----------
    // (4 RPL divides BP and BQ: which operand and plane a load belongs to is known when compiling, and so
    // a load is a scalar base and a 32-bit lane offset, shared by the two planes)
    static_assert(BP % (4 * RPL) == 0 && BQ % (4 * RPL) == 0, "a load lies in one plane");
    const int lpos = (lane * EB) & 63;                     // byte position within the 64-byte LDS row
    const int lrow = RPL * wave + lane * EB / 64;          // row of load 0
    const int limP = prm.RP - 1 - p0, limQ = prm.RQ - 1 - q0;
    const unsigned kb0 = (unsigned)((((lpos >> 4) ^ swz(lrow)) << 4) + (lpos & 15));  // swz: by row & 15, the same for every j
    const int8_t* const bases[4] = {prm.P + (int64_t)p0 * rowb, Psign + (int64_t)p0 * rowb, prm.Q + (int64_t)q0 * rowb,
                                    Qsign + (int64_t)q0 * rowb};
    auto issue = [&](int st) {
        const unsigned dst0 = lds0 + (unsigned)((st & 1) * STAGE + RPL * wave * 64);
        auto all = [&](auto whole) {
            const unsigned kb = (unsigned)st * 64 + kb0;
            auto load = [&](auto j) {
                constexpr int rr = 4 * RPL * decltype(j)::value;  // first row of this load, without the wave's share
                constexpr bool isP = rr < 2 * BP;
                constexpr int r0 = isP ? rr : rr - 2 * BP, half = isP ? BP : BQ, sgn = r0 >= half;
                int row = r0 - (sgn ? half : 0) + lrow;
                const int lim = isP ? limP : limQ;
                row = row < lim ? row : lim;  // rows past the end: any valid row, never stored
                const int8_t* base = uniform_ptr(bases[(isP ? 0 : 2) + sgn]);
                const unsigned off = (unsigned)row * rowb + kb;
                if constexpr (decltype(whole)::value) {
                    if constexpr (EB == 16)
                        dma16_base<rr * 64>(base, off, dst0);
                    else
                        dma4_base<rr * 64>(base, off, dst0);
                } else {  // the stage that reaches past the rows' end
                    const int8_t* src = kb < rowb ? base + off : (const int8_t*)g_zero16;
                    if constexpr (EB == 16)
                        dma16<rr * 64>(src, dst0);
                    else
                        dma4<rr * 64>(src, dst0);
                }
            };
            for_each_index(load, std::make_integer_sequence<int, NL>{});
        };
        if ((unsigned)(st + 1) * 64 <= rowb)
            all(std::true_type{});
        else
            all(std::false_type{});
    };

    v16f acc[TP][TQ];
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
        for (int j = 0; j < TQ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    const int nst = prm.nk;
    issue(0);
    for (int st = 0; st < nst; ++st) {
        // this wave's loads of stage st have landed; after the barrier everybody's have, and
        // every wave is done with the other stage, which the next loads overwrite
        wait_vm<0>();
        wait_lgkm0();
        block_barrier();
        if (st + 1 < nst) issue(st + 1);
        const int8_t* sb = smem + (st & 1) * STAGE;
        constexpr int NM = TP * TQ, NF = TP + TQ;
        v4i raw[2][NF][2];  // [half of the stage][fragment][mask, sign]
        v8i frag[2][NF];
        auto fetch = [&](int h, int f, int plane) {
            const bool isP = f < TP;
            const int row = (isP ? wp * WP + f * 32 : wq * WQ + (f - TP) * 32) + (lane & 31), ch = 2 * h + (lane >> 5);
            raw[h][f][plane] = *(const v4i*)(sb + (isP ? plane * BP : (2 * BP + plane * BQ)) * 64 + row * 64 + ((ch ^ swz(row)) << 4));
        };
        auto expand = [&](int s, int f) {
            frag[s & 1][f] = planes_to_fp4((unsigned)raw[s >> 2][f][0][s & 3], (unsigned)raw[s >> 2][f][1][s & 3]);
        };
        auto product = [&](int s, int n) {
            const int i = n / TQ, j = n % TQ;
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(frag[s & 1][i], frag[s & 1][TP + j], acc[i][j], 4, 4, 0, 0, 0, 0);
        };
        // The 8 k-slices in a fixed issue order: behind every MFMA of a slice its share of the next slice's
        // expansion, behind those of the first one also the second half's LDS reads.
#pragma unroll
        for (int f = 0; f < NF; ++f) fetch(0, f, 0), fetch(0, f, 1);
#pragma unroll
        for (int f = 0; f < NF; ++f) expand(0, f);
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int n = 0; n < NM; ++n) {
                product(s, n);
                if (s == 0) {
#pragma unroll
                    for (int x = n * 2 * NF / NM; x < (n + 1) * 2 * NF / NM; ++x) fetch(1, x / 2, x % 2);
                }
                if (s < 7) {
#pragma unroll
                    for (int f = n * NF / NM; f < (n + 1) * NF / NM; ++f) expand(s + 1, f);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
    }
    const bool full_tile = p0 + BP <= prm.RP && q0 + BQ <= prm.RQ;
    gemm_epilogue<BP, TP, TQ, true, true>(prm, (double*)smem, p0, q0, wp * WP, wq * WQ, full_tile, acc,
                                    [](float s) { return 0.25f * s; });
}

template <int BP, int BQ, int WGP, int WGQ, int MINW, int EB>
hipError_t launch_planes(TmmParams& prm, const int8_t* ps, const int8_t* qs, hipStream_t st)
{
    constexpr int smem = 2 * 2 * (BP + BQ) * 64;  // two stages; the epilogue's [3][BP] doubles fit in one
    static_assert(3 * BP * 8 <= smem, "epilogue table over the stages");
    auto kern = k_gemm_planes<BP, BQ, WGP, WGQ, MINW, EB>;
    static LdsLimit lds;
    const hipError_t e = lds.raise((const void*)kern, smem);
    if (e != hipSuccess) return e;
    const unsigned grid = tile_grid(prm, BP, BQ);
    if (!grid) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), (size_t)smem, st, prm, ps, qs);
    return hipGetLastError();
}

template <int EB>
hipError_t launch_planes_eb(TmmParams& prm, const int8_t* ps, const int8_t* qs, hipStream_t st)
{
    auto tiles = [&](int bp, int bq) { return (((int64_t)prm.RP + bp - 1) / bp) * (((int64_t)prm.RQ + bq - 1) / bq); };
    if (tiles(256, 256) >= 256) return launch_planes<256, 256, 2, 2, 1, EB>(prm, ps, qs, st);
    if (tiles(128, 128) >= 192) return launch_planes<128, 128, 2, 2, 2, EB>(prm, ps, qs, st);
    return launch_planes<64, 64, 2, 2, 4, EB>(prm, ps, qs, st);
}

}  // namespace

hipError_t launch_gemm_planes(const PopcArgs& a, hipStream_t st)
{
    TmmParams prm = {};
    prm.P = (const int8_t*)a.a_mask;
    prm.Q = (const int8_t*)a.w_mask;
    prm.RP = (int)a.M;
    prm.RQ = (int)a.N;
    prm.ldP = a.words * 8;
    prm.nk = (int)((a.words + 7) / 8);
    prm.Klogical = (int)a.K;
    prm.acc = a.acc;
    prm.y = a.y;
    prm.ep = a.ep;
    const int8_t *ps = (const int8_t*)a.a_sign, *qs = (const int8_t*)a.w_sign;
    return a.words % 2 == 0 ? launch_planes_eb<16>(prm, ps, qs, st) : launch_planes_eb<4>(prm, ps, qs, st);
}

}  // namespace rtn
