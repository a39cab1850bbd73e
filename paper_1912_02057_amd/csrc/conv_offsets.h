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

// Input pixels between tap (0, 0) of the first and the last tap of the last of t consecutive output pixels, at most: each
// step is `stride` pixels, and some are the ends of a row or of an image.
inline int64_t conv_span(int64_t H, int64_t W, int64_t OH, int64_t OW, int64_t KH, int64_t KW, int64_t stride, int64_t t)
{
    const int64_t row = stride * (W - OW), img = (H - (OH - 1) * stride) * W - OW * stride;
    const int64_t nrow = (t - 2) / OW + 1, nimg = (t - 2) / (OH * OW) + 1;
    return (t - 1) * stride + nrow * (row > 0 ? row : 0) + nimg * (img > 0 ? img : 0) + (KH - 1) * W + KW;
}

// A padded window's corner lies at most this many pixels before that of an earlier output pixel (of the image before,
// where the padding at its end and at the start of the next are more than the window).
constexpr int64_t conv_reach_back(int64_t pad, int64_t W) { return pad * (W + 1); }

// Does a conv's tile of bq pixels lie within 32-bit offsets from that far before its first window?  `pixel` bytes of codes.
inline bool conv_codes_fit(int64_t H, int64_t W, int64_t OH, int64_t OW, int64_t KH, int64_t KW, int64_t stride, int64_t pad, int64_t pixel, int bq)
{
    return (conv_span(H, W, OH, OW, KH, KW, stride, bq) + conv_reach_back(pad, W)) * pixel + 128 < (int64_t)0x80000000u;
}

// Do a block tail's outputs of a tile of bq pixels, 8 channels of all its images, lie within 32-bit offsets?
inline bool conv_outputs_fit(int64_t Nb, int64_t O, int64_t ohw, int bq)
{
    const int64_t spanned = (bq - 1) / ohw + 2, images = Nb < spanned ? Nb : spanned;
    return ((images - 1) * O + 8) * ohw * 4 <= (int64_t)0xffffffffu;
}

// Input pixels that a pixel-run tile of bq pixels holds, a multiple of 16
inline int64_t halo_rows(int bq, int pad, int W) { return (bq + 2 * (int64_t)pad * ((int64_t)W + 1) + 15) & ~(int64_t)15; }

}  // namespace rtn
