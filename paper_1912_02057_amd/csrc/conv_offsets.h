// A conv's offsets into its input codes, in bytes: code without HIP, so that tests can ask it on the CPU.
#pragma once
#include <cstdint>
#include <type_traits>

namespace rtn {

// Offsets that are added to a pixel's first tap: 32 bits, or (BIG: images that they do not hold) 64.
template <bool BIG>
using ConvOff = std::conditional_t<BIG, int64_t, uint32_t>;

// The walk over a window's K-steps of 64 bytes: (kh W + kw) Cpad + cc as a running sum, + 64 per step, which also carries
// over from the last chunk of a tap to the next tap of the row, and + (W - KW) Cpad at the end of a window row.
// No multiplications, no branches: scalar instructions in the K loop cost matrix-core time.
template <class Off>
struct TapWalk {
    Off off = 0;
    int cc = 0, kw = 0, shr = 31;  // 31 - kh: the shift that brings bit kh to the sign
    static constexpr Off row_skip(int W, int KW, int Cpad) { return (Off)(W - KW) * (Off)Cpad; }
    constexpr void step(int Cpad, int KW, Off skip)
    {
        off += 64;
        cc += 64;
        const bool tap = cc == Cpad;
        cc = tap ? 0 : cc;
        kw += tap ? 1 : 0;
        const bool end = kw == KW;
        kw = end ? 0 : kw;
        shr -= end ? 1 : 0;
        off += end ? skip : (Off)0;
    }
};

// Does a conv's tile of bq pixels lie within 32-bit offsets from its first image, of codes (with the window's reach before
// and behind an image) and, for a block tail, of outputs?  `ohw` output pixels of an image, `pixel` bytes of its codes.
// The pixel-run tiles (halo) take 64-bit pointers to their codes.
inline bool conv_offsets_fit(int64_t Nb, int64_t H, int64_t W, int64_t pixel, int64_t O, int64_t ohw, int bq, bool halo, bool tail)
{
    const int64_t spanned = (bq - 1) / ohw + 2, images = Nb < spanned ? Nb : spanned;
    if (tail && ((images - 1) * O + 8) * ohw * 4 > (int64_t)0xffffffffu) return false;
    return halo || (images * H + 16) * W * pixel < (int64_t)0x80000000u;
}

// Input pixels that a pixel-run tile of bq pixels holds, a multiple of 16
inline int64_t halo_rows(int bq, int pad, int W) { return (bq + 2 * (int64_t)pad * ((int64_t)W + 1) + 15) & ~(int64_t)15; }

}  // namespace rtn
