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
// (four steps: 3.71 and 3.82, and 16 x 576 to 2000 x 2048 take 1.1 to 1.45 times as long: one wave has the row).  Of
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
//   int8, 16384 x 8191 x 512            227 -> 273    375 -> 397    16384 x 8188 x 2048 (511)  299 -> 248    429 -> 441
inline bool gemm_nt_hint(int64_t M, int64_t N, uintptr_t y, int nk)
{
    const int64_t bytes = M * N * 4, mib = (int64_t)1 << 20;
    if (bytes < 128 * mib || (bytes <= 256 * mib && nk < 8)) return false;
    const int64_t line = bytes <= 256 * mib ? 128 : 64;
    return N * 4 % line == 0 && (int64_t)(y % (uintptr_t)line) == 0;
}

}  // namespace rtn
