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

}  // namespace rtn
