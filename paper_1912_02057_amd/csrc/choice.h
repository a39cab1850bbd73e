// Choices of a launch that follow from its sizes alone: host code without HIP, so that tests can ask it on the CPU.
#pragma once
#include <cstdint>

namespace rtn {

// The form of the row packs: waves that share a row, steps whose loads a wave has in flight (its turn), elements of a step.
struct PackRowsForm {
    int waves, steps, step;
};

// Codes.  One wave per row while its one or two steps are the row, and where the rows alone give every CU 8 waves;
// else the four of a block, with turns so short that at most one of them has no work.  us, one wave -> four:
//   FP4, 16 x 1536  3.29 -> 2.84     int8, 2000 x 1536  5.28 -> 5.09     int8, 2100 x 1536  5.52 -> 5.60, not taken
//   FP4, 16 x 8192  8.08 -> 3.91     int8, 2000 x 576   3.17 -> 3.65, not taken
// Turns of one step up to 2048 elements, of two beyond: FP4, 16 x 2048 2.85 against 3.10, 16 x 8192 4.18 against 3.91
// (four steps: 3.71 and 3.82, and 16 x 576 to 2000 x 2048 take 1.1 to 1.5 times as long: one wave has the row).  Of
// many rows, short ones take steps of 256: int8, 5000 x 1100 7.03 against 7.54, FP4 7.02 against 7.59; int8, 5000 x
// 2048 9.90 against 9.64, not taken.
inline PackRowsForm pack_rows_form(int64_t rows, int64_t Kpad)
{
    if (Kpad <= 256) return {1, 1, 256};
    if (Kpad <= 512) return {1, 1, 512};
    if (rows >= 2048) return {1, 2, Kpad <= 1280 ? 256 : 512};
    if (Kpad <= 1024) return {1, 2, 512};
    return {4, Kpad <= 2048 ? 1 : 2, 512};
}

// Bit planes: a step is a 64-element word.  us, one wave -> four: 2000 x 512 2.89 -> 3.26, not taken; 2000 x 576
// 3.64 -> 3.56, 16 x 2048 4.51 -> 2.91.  Turns of four words against eight: 2000 x 576 3.56, 4.16; 500 x 4096 4.75, 4.23.
inline PackRowsForm pack_rows_planes_form(int64_t rows, int64_t Kpad)
{
    if (Kpad <= 256) return {1, 4, 64};
    if (rows >= 2048 || Kpad <= 512) return {1, 8, 64};
    return {4, Kpad <= 2048 ? 4 : 8, 64};
}

// NCHW packs of few pixels and many channels, with scalar thresholds and no sums: does k_pack_nchw_small run?  `flat`: the
// kernel with one block per image could (its LDS holds the image).  us, FP4, what runs otherwise -> this one:
//   quads of pixels that lie in one image: everywhere
//     64 x 1024 x 8 x 8  8.1 -> 4.2     1 x 948 x 62 x 62  10.8 -> 7.9     20 x 1024 x 14 x 14  9.8 -> 8.5
//   else its time grows with the images: up to 17 of them or 800 pixels, and always beyond 1000 channels, where the
//   general kernel takes twice the LDS
//     9 x 513 x 9 x 9  13.6 -> 8.9      19 x 513 x 9 x 9  13.8 -> 13.1     49 x 513 x 9 x 9  15.0 -> 19.1
//     88 x 513 x 3 x 3  15.3 -> 11.8    16 x 513 x 7 x 7  13.6 -> 11.7     177 x 513 x 3 x 3  15.3 -> 17.4
//     33 x 768 x 11 x 11  18.7 -> 20.2  81 x 1021 x 7 x 7  24.4 -> 24.7    83 x 2048 x 7 x 7  46.0 -> 30.5
//   against a block per image, whose time grows with the image: (int8) 1 x 516 x 9 x 9  6.9 -> 4.8
//     1 x 1024 x 7 x 7  7.1 -> 5.4      2 x 1024 x 7 x 7  7.2 -> 6.4       2 x 768 x 7 x 7  5.7 -> 6.0
//     83 x 576 x 7 x 7  5.3 -> 21.8     8 x 1280 x 7 x 7  8.6 -> 12.7      9 x 768 x 9 x 9  8.5 -> 9.6
inline bool pack_nchw_few_pixels(int64_t N, int64_t K, int64_t HW, bool flat)
{
    if (N * HW > 4096 || K <= 512 || HW < 4) return false;
    if (HW % 4 == 0) return true;
    if (flat) return K * HW >= 26000 + 11000 * N;
    return K > 1000 || N <= 17 || N * HW <= 800;
}

// Lanes of k_pack_nchw that share a channel's run of pixels (4 each, 16 / 32 / 64 lanes): a block takes 64 to 256 pixels
// and its groups are 256 to 64 channels.  The widest run that still gives every CU several blocks:
// fewer lanes mean more blocks and fewer rounds over the channels, but masked channels and a vector address per
// load where the channels are no multiple of the group.  So multiples of 64 take the run whose group divides them, if
// that is blocks enough.  us, int8, a masked group of 256 -> a group that divides:
//   multiples of 128, from 11264 pixels on
//     256 x 384 x 14 x 14  23.2 -> 18.4   64 x 640 x 28 x 28  34.8 -> 29.6   46 x 1152 x 14 x 14  14.0 -> 12.9, not taken
//   of 64, images up to 1024 pixels, where the last round of blocks, of four at most, has one for more than half of the CUs,
//   or, with more than a third of the channels masked, in any number of rounds
//     256 x 320 x 14 x 14  20.3 -> 16.6   256 x 576 x 14 x 14  34.1 -> 27.3  64 x 576 x 28 x 28  29.6 -> 26.2
//     408 x 320 x 14 x 14  28.1 -> 25.0   1327 x 192 x 14 x 14  46.2 -> 42.3
//     16 x 448 x 28 x 28   8.3 -> 13.2,   16 x 320 x 56 x 56   20.0 -> 20.6 and 256 x 448 x 28 x 28  80 -> 105: not taken
inline int pack_nchw_lanes(int64_t K, int64_t Kpad, int64_t px, int64_t HW)
{
    if (K % 256 && K % 128 == 0 && px >= 11264) return px < 4096 * 256 ? 32 : 64;
    if (K % 128 && K % 64 == 0) {
        const int64_t blocks = (px + 255) / 256, masked = (K + 255) / 256 * 256 - K;
        if (HW <= 1024 && ((blocks <= 1024 && (blocks - 1) % 256 >= 128) || (blocks > 256 && 2 * masked > K))) return 64;
    }
    if (Kpad >= 256 && px < 2048 * 256) return 16;
    return Kpad >= 128 && K > 64 && px < 4096 * 256 ? 32 : 64;
}

// Do 32-bit offsets from a block's first image reach all elements of its at most 256 pixels?
inline bool pack_nchw_offsets_fit(int64_t N, int64_t K, int64_t HW)
{
    const int64_t spanned = 255 / HW + 2, images = N < spanned ? N : spanned;
    return images * K * HW < (int64_t)1 << 30;
}

// Depthwise 3 x 3, outputs that the memory-side cache does not hold, in planes that are no whole 64-byte halves of lines: where
// the stores themselves are what a launch takes, the vector kernel's runs of 64 pixels with the non-temporal hint are faster
// than the matrix-core kernel's parts of lines, which cannot take it.  us, matrix cores -> vector (odd planes of 27 to
// 137 wide, 32 to 256 channels, 150 to 400 MiB of y: 165 launches)
//   y and acc, stride 1  256 x 1024 x 13 x 13 (169 MiB) 181 -> 121   256 x 512 x 24 x 21 (252) 204 -> 189, 400 MiB 0.9 times, not taken
//   y and acc, stride 2  256 x 64 x 113 x 113 (203) 238 -> 232       188 x 372 x 42 x 42 (117) 131 -> 143, at 230 MiB 1.0, not taken
//   y, stride 2          256 x 64 x 113 x 113 (203) 136 -> 113       600 x 128 x 60 x 72 (316) 248 -> 239, 400 MiB 0.9 times, not taken
//   up to 48 channels    200 x 32 x 93 x 136 (308) 143 -> 123        100 x 48 x 93 x 136 (231) 119 -> 106
//   y, stride 1          256 x 512 x 24 x 21 (252) 88 -> 118, not taken
inline bool dw_vector_stores(int64_t C, int stride, int64_t y_bytes, bool acc)
{
    const int64_t mib = y_bytes >> 20;
    if (C <= 48) return acc ? mib > 128 && (C <= 32 || mib <= 280) : mib > (stride == 2 ? 128 : 220);
    if (acc) return mib > 128 && mib <= (stride == 2 ? 200 : 280);
    return stride == 2 && mib > 128 && mib <= 320;
}

// Does a GEMM store y [M][N] with the non-temporal hint?  A burst of stores that the memory-side cache (256 MiB) absorbs
// and writes back later slows the K loops of the tiles behind it, and hinted ones do not.  But a hinted store of a
// part of a line goes to memory as it is, and the next kernel finds nothing in the cache.  us, plain -> hinted, two
// inputs and outputs in turn; pack + GEMM, and the same with a pack of y behind it:
//   FP4, 16384 x 8192 x 2048 (512 MiB)  271 -> 239    396 -> 365    16384 x 4096 x 2048 (256)  152 -> 117    197 -> 186
//   int8, 16384 x 8192 x 4096           590 -> 557    712 -> 687    16384 x 2048 x 4096 (128)  199 -> 176    223 -> 216
// Up to 256 MiB not for fewer than 8 K-steps, where no K loop is worth the reader's loss:
//   FP4, 8192 x 4096 x 256 (128)         38 ->  42     64 ->  73    8192 x 8192 x 512 (256)     98 ->  99    140 -> 160
//   int8, 8192 x 4096 x 256              40 ->  45     70 ->  77    8192 x 6144 x 256 (192)     58 ->  53     99 -> 103
// and only for rows of whole 128-byte lines; beyond, of whole 64-byte halves:
//   FP4, 12000 x 3000 x 2048 (137)      106 -> 112    132 -> 150    12000 x 2992 x 2048 (137)  102 -> 102    131 -> 137
//   FP4, 16384 x 8191 x 2048 (512)      300 -> 326    429 -> 457    16384 x 8176 x 2048 (511)  298 -> 239    429 -> 396
//   FP4, 16384 x 8188 x 2048 (511)      299 -> 248    429 -> 441    16384 x 8188 x 512         198 -> 208    331 -> 338
//   int8, 16384 x 8191 x 512            227 -> 273    375 -> 397
inline bool gemm_nt_hint(int64_t M, int64_t N, uintptr_t y, int nk)
{
    const int64_t bytes = M * N * 4, mib = (int64_t)1 << 20;
    if (bytes < 128 * mib || (bytes <= 256 * mib && nk < 8)) return false;
    const int64_t line = bytes <= 256 * mib ? 128 : 64;
    return N * 4 % line == 0 && (int64_t)(y % (uintptr_t)line) == 0;
}

constexpr int64_t kMaxLds = 160 * 1024;

inline int64_t nblocks(int64_t rp, int64_t rq, int bp, int bq)
{
    return ((rp + bp - 1) / bp) * ((rq + bq - 1) / bq);
}

// Tile `bid` of a grid in bands of 8 tiles along P, all columns of a band and along P first: a run of tiles, as an XCD has
// it, is a block of rows and columns.  `band_tiles` 8 x columns; the divisions by that and by the height of the last band are
// the caller's (multiplications on the device).
template <class DivBand, class DivLast>
constexpr void band_tile(int bid, int tilesP, int band_tiles, DivBand div_band, DivLast div_last, int& tileP, int& tileQ)
{
    const int band = div_band(bid), inband = bid - band * band_tiles, left = tilesP - band * 8;
    tileQ = left >= 8 ? inband >> 3 : div_last(inband);
    tileP = band * 8 + inband - tileQ * (left < 8 ? left : 8);
}

// The forms of k_ksplit: tiles of 32 along P and Q, waves that share K, ring stages, pixel run in LDS (convs).
struct KsplitForm {
    int tp, tq, waves, stages;
    bool run;
};
constexpr KsplitForm kKsplitForms[] = {{1, 1, 4, 4, false}, {1, 1, 8, 2, false}, {2, 1, 8, 3, false}, {2, 2, 8, 2, false},
                                       {2, 2, 4, 2, false}, {2, 1, 8, 2, true},  {2, 2, 8, 2, true},  {2, 2, 4, 2, true}};
constexpr int kKsplitGemmForms = 3, kNumKsplitForms = 8;

// What the choice depends on.  GEMM: rows of P (M) and Q (N) and K-steps, the rest 0.  conv: P = filters, Q = output
// pixels; a pixel's code bytes; rows of the epilogue table in LDS.
struct KsplitShape {
    int64_t rp, rq;
    int nk, KH, KW, stride, pad, W, pixel_bytes, table_rows;
};

// LDS of the pixel run of a tile: rows of the pixel's codes and 16 bytes more, whole KiB
inline int64_t ksplit_run_bytes(const KsplitForm& f, const KsplitShape& s)
{
    const int64_t rows = 32 * f.tq + 2 * (int64_t)s.pad * (s.W + 1);
    return (rows * (s.pixel_bytes + 16) + 1023) & ~(int64_t)1023;
}
// rings, pixel run and its zero bytes, or the accumulators over them
inline int64_t ksplit_main_bytes(const KsplitForm& f, const KsplitShape& s)
{
    const int64_t rings = f.waves * f.stages * (f.tp + (f.run ? 0 : f.tq)) * 2048;
    if (!f.run) return rings;
    const int64_t a = rings + ksplit_run_bytes(f, s) + 16, b = f.waves * f.tp * f.tq * 4096;
    return a > b ? a : b;
}
// ... and a conv's pixel sums and epilogue table
inline int64_t ksplit_lds_bytes(const KsplitForm& f, const KsplitShape& s)
{
    if (!s.KH) return ksplit_main_bytes(f, s);
    return ksplit_main_bytes(f, s) + f.waves * f.tq * 128 + (((int64_t)s.table_rows * 32 * f.tp * 8 + 1023) & ~(int64_t)1023);
}
inline bool ksplit_fits(int form, const KsplitShape& s)
{
    const KsplitForm& f = kKsplitForms[form];
    if (f.run && (s.stride != 1 || s.KH != 2 * s.pad + 1 || s.KW != 2 * s.pad + 1)) return false;
    // (the four-wave form with a pixel run is for grids of more than a block per CU: two have to fit)
    return ksplit_lds_bytes(f, s) <= (f.run && f.waves == 4 ? kMaxLds / 2 : kMaxLds);
}

// The form of k_ksplit for a grid too small for k_tmm, or -1.
// K's share of the time decides between the forms, the number of 32 x 32 tiles whether to cut K at all; past
// these lines the small tiles' operand traffic (L2 to LDS) costs more than the cut saves.
// k_tmm's time over this kernel's, geometric mean (least) over 680 random geometries (GEMM M 1 to 4096, N and K 64 to
// 8192; convs of 24 to 1024 channels and filters, 7 to 112 wide, windows 1, 3, 5, stride 1, 2, every epilogue; FP4, int8):
//   K-steps           1-3          4-8          9-16         17-32        33-64        65-128
//   GEMM, <= 256   1.23 (1.13)  1.38 (1.20)  1.45 (1.29)  1.67 (1.52)  1.91 (1.60)  2.26 (1.56)
//   GEMM, <= 512   1.19 (1.11)  1.22 (1.15)  1.21 (1.11)  1.20 (1.12)  1.25 (1.10)  1.22 (1.03)
//   GEMM, <= 1024, not taken, the best of the forms of 32 and 64:  0.86 (0.78), 0.94 (0.75), 0.95 (0.87)
//   conv, <= 256   1.15 (1.02)  1.30 (1.12)  1.44 (1.35)  1.89 (1.74)  2.47 (2.10)  3.01 (2.69)
//   conv, <= 512   1.09 (0.97)  1.22 (1.08)  1.26 (1.05)  1.48 (1.26)  1.72 (1.41)  2.00 (1.51)
//   conv, <= 1024, with the pixel run's forms:             1.11 (1.00)  1.26 (1.01)  1.62 (1.48)
//   conv, 64 x 64 tiles in 257 .. 512: 1.00 at 33-64 K-steps, not taken, 1.3 (1.03) beyond
// A conv of 257 to 512 tiles takes four waves up to 8 K-steps (with eight 1.09, least 0.91: a ternarizing conv was slower
// than with k_tmm), and 64 x 32 tiles, if they are no more than 256, from 9 on: 1.04 to 1.14 times as fast at 9 to 36,
// 1.1 to 1.2 beyond.
inline int pick_ksplit_plain(const KsplitShape& s)
{
    const bool conv = s.KH != 0;
    const int64_t tiles = nblocks(s.rp, s.rq, 32, 32);
    if (tiles <= 512) {
        if (s.nk <= (conv && tiles > 256 ? 8 : 3)) return 0;
        return s.nk > (conv ? 8 : 32) && tiles > 256 && nblocks(s.rp, s.rq, 64, 32) <= 256 ? 2 : 1;
    }
    if (!conv) return -1;
    if (s.nk > 32 && nblocks(s.rp, s.rq, 64, 64) <= 256) return 3;
    return s.nk > 64 && nblocks(s.rp, s.rq, 64, 64) <= 512 ? 4 : -1;
}

// The same for convs whose pixels are one run of the input; these forms come first.  Against the best of the others, 121
// random convs with windows 3 and 5: 64 x 32 tiles 1.05 to 1.15 times as fast beyond 64 K-steps (0.95 to 1.04 below);
// 64 x 64 tiles, up to 256, 1.05 to 1.2 times from 18 to 25, 1.05 to 1.15 beyond; up to 512 of them 1.1 to 1.25 at 36 to
// 50 (0.9 to 1.06 at 18 to 27) where two blocks fit a CU, 0.7 to 0.85 where they do not.
inline int pick_ksplit_run(const KsplitShape& s)
{
    if (s.KH < 3) return -1;
    if (nblocks(s.rp, s.rq, 32, 32) <= 512)
        return s.nk > 64 && nblocks(s.rp, s.rq, 32, 32) > 256 && nblocks(s.rp, s.rq, 64, 32) <= 256 ? 5 : -1;
    if (nblocks(s.rp, s.rq, 64, 64) <= 256) return s.nk >= 18 ? 6 : -1;
    return s.nk > 32 && nblocks(s.rp, s.rq, 64, 64) <= 512 ? 7 : -1;
}

// The form that runs: with a pixel run where there is one and it fits (a long run or the table of a large pad can
// exceed the LDS), else without; -1: k_tmm's tiles.
inline int pick_ksplit(const KsplitShape& s)
{
    const int run = pick_ksplit_run(s), plain = pick_ksplit_plain(s);
    if (run >= 0 && ksplit_fits(run, s)) return run;
    return plain >= 0 && ksplit_fits(plain, s) ? plain : -1;
}

}  // namespace rtn
