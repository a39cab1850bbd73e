// Ternarize + pack kernels (Eq.1 / Eq.3 thresholds, Table 1 encoding) for gfx950.
//
// t = (x > hi) - (x < lo) on the stored fp32 value.  The kernels are pure
// streaming: coalesced fp32 reads, code writes, and the side sum of t per GEMM
// row / per pixel taken with wavefront reductions (64-wide ballots and
// cross-lane adds).  They are HBM-bound: 4 B read per element, 1 B (int8) or
// 0.25 B (two bit planes) written.
#include <mutex>
#include <type_traits>

#include "choice.h"
#include "lds_limit.h"
#include "rtn_kernels.h"

namespace rtn {

namespace {

__device__ __forceinline__ float thr(const Param& p, int64_t i) { return p.ptr ? p.ptr[i] : p.s; }

__device__ __forceinline__ int tern(float v, float lo, float hi) { return (int)(v > hi) - (int)(v < lo); }

// FP4 (E2M1) code of a ternary value: +1 -> 0x2, -1 -> 0xA, 0 -> 0x0.
__device__ __forceinline__ uint32_t nib(int t) { return (uint32_t)((t & 1) << 1) | (uint32_t)((t >> 28) & 8); }
// Four int8 codes in a dword (bytes 0x00, 0x01, 0xFF) -> their four FP4 nibbles in 16 bits,
// element 0 in the lowest nibble.
__device__ __forceinline__ uint32_t i8x4_to_fp4(uint32_t w)
{
    const uint32_t t = ((w << 1) & 0x02020202u) | ((w >> 4) & 0x08080808u);  // one nibble per byte
    const uint32_t r = (t | (t >> 4)) & 0x00ff00ffu;
    return (r | (r >> 8)) & 0xffffu;
}

__device__ __forceinline__ int wave_sum(int v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// ---- rows layout -----------------------------------------------------------
// WPR waves per row: 1, or the 4 of a block where the rows alone would leave most of the chip without a wave.
// A wave that waits for each step's loads before the next is bound by their latency, so it asks for up to 4 quads
// (codes) or 8 words' worth (planes) of its row at a time, and the waves of a row take turns in runs of that size
// (choice.h).  Quads are loaded as 16 bytes at any K and row address: a global load of several dwords needs 4-byte
// alignment only.
//   us, before (one wave per row, one step's loads in flight; K % 4 != 0: 4-byte loads) -> now:
//     int8, 1000 x 2187  10.4 -> 4.4     FP4, 16 x 8192  10.7 -> 3.9     FP4, 4096 x 4096  14.3 -> 14.2
//     int8, 4096 x 4095  25.4 -> 15.2    FP4, 16384 x 8191  182 -> 120 (5.0 TB/s), 16384 x 8192  127 -> 121
//     planes, 16 x 8192  15.9 -> 4.9, 4096 x 4096  16.8 -> 14.2
// elements k .. k + 3 of a row, k = k0 + 4 lane; NaN, whose code is 0, past its end
__device__ __forceinline__ void load_quad(const float* xr, unsigned k0, unsigned lane, unsigned K, float (&v)[4])
{
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = __builtin_nanf("");
    if (k0 >= K) return;  // the whole wave
    const unsigned k = k0 + 4 * lane;
    if (k + 4 <= K) {
        const f4 q = *(const f4*)(xr + k);
        v[0] = q[0], v[1] = q[1], v[2] = q[2], v[3] = q[3];
    } else if (k < K) {  // one lane
        v[0] = xr[k];
        if (k + 1 < K) v[1] = xr[k + 1];
        if (k + 2 < K) v[2] = xr[k + 2];
    }
}

// The row sum from the waves' shares: every wave of a row (WPR > 1: the block) calls it.
template <int WPR>
__device__ __forceinline__ void store_row_sum(int32_t* sum_t, int64_t row, int sum, int sub, int lane)
{
    if constexpr (WPR == 1) {
        if (lane == 0) sum_t[row] = sum;
    } else {
        __shared__ int part[WPR];
        if (lane == 0) part[sub] = sum;
        __syncthreads();
        if (threadIdx.x == 0) {
            sum = 0;
#pragma unroll
            for (int w = 0; w < WPR; ++w) sum += part[w];
            sum_t[row] = sum;
        }
    }
}

// Codes.  A step covers 512 elements: every lane loads elements 4l .. 4l+3 of the first and of the second 256
// (NP = 2 coalesced 1 KiB reads per wave; rows of up to 256 take one).  int8: a dword per quad.  FP4: 16 bits per quad; a dword of output is 8
// consecutive elements, i.e. the quads of lanes 2j and 2j+1: the even lane assembles the dword of the first
// half, the odd lane that of the second half, after one exchange with its neighbour.
template <bool FP4, int WPR, int UN, int NP = 2>
__global__ __launch_bounds__(256) void k_pack_rows(PackArgs a)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = wave % WPR;
    const int64_t row = (int64_t)blockIdx.x * (4 / WPR) + wave / WPR;
    if (row >= a.rows) return;
    const float lo = thr(a.lo, row), hi = thr(a.hi, row);
    const float* xr = a.x + row * a.K;
    uint8_t* cr = (uint8_t*)a.codes + row * (FP4 ? a.Kpad >> 1 : a.Kpad);
    const bool odd = lane & 1;
    const unsigned K = (unsigned)a.K, Kpad = (unsigned)a.Kpad;
    constexpr unsigned STEP = 256 * NP;
    int sum = 0;
    for (unsigned k1 = sub * STEP * UN; k1 < Kpad; k1 += STEP * UN * WPR) {
        float v[UN][NP][4];
#pragma unroll
        for (int u = 0; u < UN; ++u)
#pragma unroll
            for (int part = 0; part < NP; ++part) load_quad(xr, k1 + STEP * u + 256 * part, lane, K, v[u][part]);
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const unsigned k0 = k1 + STEP * u;
            if (k0 >= Kpad) break;
            uint32_t h[NP];
#pragma unroll
            for (int part = 0; part < NP; ++part) {
                int t[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) t[e] = tern(v[u][part][e], lo, hi), sum += t[e];
                if (FP4) {
                    h[part] = nib(t[0]) | (nib(t[1]) << 4) | (nib(t[2]) << 8) | (nib(t[3]) << 12);
                } else {
                    const unsigned k = k0 + 256 * part + 4 * lane;
                    if (k < Kpad)
                        *(uint32_t*)(cr + k) = (uint32_t)(t[0] & 0xff) | ((uint32_t)(t[1] & 0xff) << 8) |
                                               ((uint32_t)(t[2] & 0xff) << 16) | ((uint32_t)(t[3] & 0xff) << 24);
                }
            }
            if (FP4) {
                // even lane: needs the neighbour's first-half quad; odd lane: the neighbour's second-half quad
                const uint32_t h1 = NP == 2 ? h[NP - 1] : 0;  // (one half: the odd lanes have nothing to store)
                const uint32_t recv = (uint32_t)__shfl_xor((int)(odd ? h[0] : h1), 1, 64);
                const uint32_t word = odd ? (recv | (h1 << 16)) : (h[0] | (recv << 16));
                if (NP == 1 && odd) continue;
                const unsigned kw = k0 + (odd ? 256 + 4 * (lane - 1) : 4 * lane);  // first element of the dword
                if (kw < Kpad) *(uint32_t*)(cr + (kw >> 1)) = word;
            }
        }
    }
    if (a.sum_t) store_row_sum<WPR>(a.sum_t, row, wave_sum(sum), sub, lane);
}

// Bit planes.  Lane l reads element 64*w + l, so one 64-wide ballot of (x > hi) / (x < lo) *is* plane word w; the
// row sum is popcount(pos) - popcount(neg) on the scalar unit.  Eight words are produced per step and written by
// lanes 0..7 as one 64-byte store.
template <int WPR, int UN>
__global__ __launch_bounds__(256) void k_pack_rows_planes(PackArgs a)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = wave % WPR;
    const int64_t row = (int64_t)blockIdx.x * (4 / WPR) + wave / WPR;
    if (row >= a.rows) return;
    const float lo = thr(a.lo, row), hi = thr(a.hi, row);
    const float* xr = a.x + row * a.K;
    const int64_t words = a.Kpad >> 6;
    uint64_t* mrow = (uint64_t*)a.codes + row * words;
    uint64_t* srow = (uint64_t*)a.codes + a.rows * words + row * words;
    int sum = 0;
    for (int64_t w0 = sub * UN; w0 < words; w0 += UN * WPR) {
        float v[UN];
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            const int64_t k = (w0 + i) * 64 + lane;
            v[i] = k < a.K ? xr[k] : __builtin_nanf("");
        }
        uint64_t mword = 0, sword = 0;
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            const uint64_t pos = __ballot(v[i] > hi);
            const uint64_t neg = __ballot(v[i] < lo);
            sum += __popcll(pos) - __popcll(neg);
            if (lane == i) {
                mword = pos | neg;
                sword = pos;
            }
        }
        if (lane < UN && w0 + lane < words) {
            mrow[w0 + lane] = mword;
            srow[w0 + lane] = sword;
        }
    }
    if (a.sum_t) store_row_sum<WPR>(a.sum_t, row, sum, sub, lane);
}

// ---- NCHW layout, int8 codes, channel-innermost output -------------------
// A block owns 64 consecutive pixels of the flattened (image, pixel) index, so
// its output -- 64 rows of Cpad bytes -- is one contiguous run of the
// [N][H][W][Cpad] tensor, whatever H*W is.  lane <-> pixel: every load (fixed
// channel, 64 pixels) is a coalesced 256-byte read.  Wave w owns the 16-channel
// groups g = w, w+4, ...; a lane packs its 16 codes of a group into 16 bytes
// and parks them in an LDS image of the output run, which the block then
// streams out with consecutive lanes writing consecutive 16-byte chunks (full
// cache lines).  Channel sums are combined through LDS.
template <bool FP4>
__global__ __launch_bounds__(256) void k_pack_nchw_i8(PackArgs a)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t tile[];  // [64][Cpad], FP4: [64][Cpad / 2]
    __shared__ int part[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t total = a.N * a.HW;
    const int64_t q0 = (int64_t)blockIdx.x * 64, q = q0 + lane;
    const bool pin = q < total;
    const int64_t n = pin ? q / a.HW : 0;
    const int64_t p = pin ? q - n * a.HW : 0;
    const float lo = thr(a.lo, n), hi = thr(a.hi, n);
    const float* xn = a.x + n * a.K * a.HW + p;
    const int groups = (int)(a.Kpad >> 4);
    const int64_t rowb = FP4 ? a.Kpad >> 1 : a.Kpad;  // bytes of a pixel's code row
    int sum = 0;
    for (int g = wave; g < groups; g += 4) {
        uint32_t w4[4] = {0, 0, 0, 0};
        float v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int64_t c = (int64_t)g * 16 + j;
            v[j] = (pin && c < a.K) ? xn[c * a.HW] : 0.0f;
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int64_t c = (int64_t)g * 16 + j;
            const int t = (pin && c < a.K) ? tern(v[j], lo, hi) : 0;
            sum += t;
            w4[j >> 2] |= (uint32_t)(t & 0xff) << (8 * (j & 3));
        }
        if (FP4)
            *(uint2*)(tile + (size_t)lane * rowb + g * 8) =
                make_uint2(i8x4_to_fp4(w4[0]) | (i8x4_to_fp4(w4[1]) << 16), i8x4_to_fp4(w4[2]) | (i8x4_to_fp4(w4[3]) << 16));
        else
            *(uint4*)(tile + (size_t)lane * rowb + g * 16) = make_uint4(w4[0], w4[1], w4[2], w4[3]);
    }
    part[wave][lane] = sum;
    __syncthreads();
    if (a.sum_t && wave == 0 && pin) a.sum_t[q] = part[0][lane] + part[1][lane] + part[2][lane] + part[3][lane];
    const int64_t valid = total - q0 < 64 ? total - q0 : 64;
    const int chunks = (int)(valid * (rowb >> 4));
    uint8_t* out = (uint8_t*)a.codes + q0 * rowb;
    for (int e = threadIdx.x; e < chunks; e += 256) *(uint4*)(out + (size_t)e * 16) = *(const uint4*)(tile + (size_t)e * 16);
}

// ---- NCHW layout, 16-byte loads ---------------------------------------------------
// For H*W % 4 == 0.  A block owns
// PB = 4*LPR consecutive pixels; LPR lanes read one channel's run of them with
// one 16-byte load each (lane l: pixels 4q..4q+3, q = l % LPR; a load of several dwords needs 4-byte alignment
// only), and the SUBS = 64/LPR lane groups of a wave read channels 16 apart.  Channels go in
// groups of CG = 64*SUBS: wave w, lane group s take channels 16*(w*SUBS+s) .. +15 of
// the group, so a lane ends up with, for each of its 4 pixels, 16 codes
// that are contiguous in the channel-innermost output.  They are parked in a
// PB-pixel LDS image (always 16 KiB, FP4 8; slots of 16 codes, XOR-swizzled by
// the pixel quad to spread banks) and streamed out with consecutive lanes
// writing consecutive pieces of a pixel's contiguous bytes.
// LPR = 64 gives the widest pixel runs; the smaller ones trade them for more
// blocks (a tensor with few pixels and many channels) and fewer passes.
// HBM-bound, as long as little is done per element: a lane's byte offset fits 32
// bits and is added to a wave-uniform base, so that a load costs no vector instruction
// besides itself; two
// compares, two selects and an OR into the code word when the thresholds are
// ordered (ORDERED: scalar thresholds, lo <= hi checked by the entry point, so
// x > hi and x < lo exclude each other), else the subtract form.  The side sum is
// taken from the packed words (SUM).
//  PART: the channels are not a multiple of CG; those past the last read the last and get code 0.  us, FP4, against the
//  kernel with bounds selects and 64-bit addresses per element that it replaced: 64 x 32 x 112 x 112 38.0 -> 24.9,
//  50 x 25 x 64 x 64 13.2 -> 8.2, 70 x 107 x 42 x 42 13.9 -> 12.0.
//  Off: of a lane's elements from the block's first image; 64 bits where 32 do not reach (pack_nchw_offsets_fit()).
template <int LPR, bool FP4, bool SUM, bool ORDERED, bool PART, class Off = uint32_t>
__global__ __launch_bounds__(256) void k_pack_nchw(PackArgs a)
{
    static_assert(PART || sizeof(Off) == 4, "64-bit offsets: the form with a vector address per load");
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int SUBS = 64 / LPR, PB = 4 * LPR, SLOT = FP4 ? 8 : 16, NSLOT = 4 * SUBS, RB = SLOT * NSLOT;
    constexpr int CG = 64 * SUBS;
    constexpr int NW = FP4 ? 2 : 4;  // code words per pixel and lane
    __shared__ __attribute__((aligned(16))) uint8_t tile[PB * RB];
    __shared__ int part[SUM ? 4 * SUBS : 1][SUM ? PB : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int quad = lane % LPR, cblk = wave * SUBS + lane / LPR;
    const int total = (int)(a.N * a.HW);
    const int q0 = (int)blockIdx.x * PB;
    int q = q0 + 4 * quad;
    q = q < total ? q : total - 4;  // total % 4 == 0; lanes past the end redo the last quad, never stored
    const int HW = (int)a.HW, K = (int)a.K;
    const int n = (int)fastdiv_flat((uint32_t)q, a.div_hw), p = q - n * HW;
    const int n0 = (int)fastdiv_flat((uint32_t)q0, a.div_hw);  // the block's first image: offsets are from there
    const float* const x0 = a.x + (int64_t)n0 * K * HW;
    const float lo = thr(a.lo, n), hi = thr(a.hi, n);
    const Off off = ((Off)((n - n0) * K + (PART ? 0 : cblk * 16)) * (Off)HW + (Off)p) * 4u;
    const int ngroup = PART ? (K + CG - 1) / CG : K / CG;
    const int valid = total - q0 < PB ? total - q0 : PB;
    const int rowb = (int)(FP4 ? a.Kpad >> 1 : a.Kpad);
    uint8_t* out = (uint8_t*)a.codes + (int64_t)q0 * rowb;
    int sum[4] = {0, 0, 0, 0}, usum[4] = {0, 0, 0, 0};
    (void)usum;
    for (int cg = 0; cg < ngroup; ++cg) {
        f4 v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            if (PART) {
                const int c = cg * CG + cblk * 16 + j;
                v[j] = *(const f4*)((const char*)x0 + (off + (Off)(c < K ? c : K - 1) * (Off)HW * 4u));
            } else {
                const float* base = x0 + (int64_t)(cg * CG + j) * HW;  // wave-uniform
                v[j] = *(const f4*)((const char*)base + off);
            }
        }
        uint32_t w[4][NW];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int k = 0; k < NW; ++k) w[i][k] = 0;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int sh = FP4 ? 4 * (j & 7) : 8 * (j & 3);
            const bool cok = !PART || cg * CG + cblk * 16 + j < K;
            const uint32_t cp = cok ? (FP4 ? 0x2u : 0x01u) << sh : 0u, cn = cok ? (FP4 ? 0xAu : 0xFFu) << sh : 0u;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t c;
                if (ORDERED) {
                    c = v[j][i] > hi ? cp : 0u;
                    c = v[j][i] < lo ? cn : c;
                } else {
                    // t in {-1, 0, 1}: the int8 code is t's low byte, the FP4 code (t << 1) & 0xA
                    c = ((uint32_t)tern(v[j][i], lo, hi) << (FP4 ? sh + 1 : sh)) & cn;
                }
                w[i][FP4 ? j >> 3 : j >> 2] |= c;
            }
        }
        if (SUM) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int k = 0; k < NW; ++k) {
                    if (FP4) {
                        sum[i] = __builtin_amdgcn_sdot8((int)w[i][k], 0x11111111, sum[i], false);
                        usum[i] = (int)__builtin_amdgcn_udot8(w[i][k], 0x11111111u, (unsigned)usum[i], false);
                    } else {
                        sum[i] = __builtin_amdgcn_sdot4((int)w[i][k], 0x01010101, sum[i], false);
                    }
                }
        }
        if (cg > 0) __syncthreads();  // previous group fully streamed out
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint8_t* slot = tile + (4 * quad + i) * RB + (cblk ^ (quad & (NSLOT - 1))) * SLOT;
            if (FP4)
                *(uint2*)slot = make_uint2(w[i][0], w[i][1]);
            else
                *(uint4*)slot = make_uint4(w[i][0], w[i][1], w[i][2], w[i][3]);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PB * NSLOT / 256; ++k) {
            const int e = tid + 256 * k, px = e / NSLOT, pp = e % NSLOT;
            const int logical = pp ^ ((px >> 2) & (NSLOT - 1));
            const int cbyte = cg * RB + logical * SLOT;  // (PART: the last group may overhang the row)
            if (px < valid && (!PART || cbyte < rowb)) {
                if (FP4)
                    *(uint2*)(out + (size_t)px * rowb + cbyte) = *(const uint2*)(tile + e * SLOT);
                else
                    *(uint4*)(out + (size_t)px * rowb + cbyte) = *(const uint4*)(tile + e * SLOT);
            }
        }
    }
    // the zero codes behind the last group (FP4 rows are padded to 128 codes)
    const int donebytes = ngroup * RB, padu = (rowb - donebytes) >> 4;  // 16-byte units per pixel
    for (int e = tid; e < PB * padu; e += 256) {
        const int px = e / padu, u = e - px * padu;
        if (px < valid) *(uint4*)(out + (size_t)px * rowb + donebytes + 16 * u) = make_uint4(0, 0, 0, 0);
    }
    if (SUM && (sizeof(Off) == 4 || a.sum_t)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int t = sum[i];
            if (FP4) {
                // nibbles as integers: +1 is 2 signed and unsigned, -1 is -6 signed and 10 unsigned
                const int neg = (usum[i] - sum[i]) >> 4, pos = (sum[i] + 6 * neg) >> 1;
                t = pos - neg;
            }
            part[cblk][4 * quad + i] = t;
        }
        __syncthreads();
        if (tid < valid && tid < PB) {
            int s = 0;
#pragma unroll
            for (int b = 0; b < 4 * SUBS; ++b) s += part[b][tid];
            a.sum_t[q0 + tid] = s;
        }
    }
}

// ---- NCHW layout, few pixels -----------------------------------------------------------
// One image is a handful of blocks of the kernels around, each lane with dozens of elements one after the other.  Here a
// block has 64 pixels x 64 channels and a lane 4 x 4 of them.  The blocks of the same pixels run on one XCD: their pieces of
// a line meet in its L2.  Any H*W of at least 4 (a quad that begins in one image and ends in the next reads the last
// 4 pixels of the one and the first 4 of the other and shifts them into place) and any number of channels; scalar
// thresholds, tensors below 4 GiB, no sums.
template <bool FP4>
__global__ __launch_bounds__(256) void k_pack_nchw_small(PackArgs a)
{
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int RB = FP4 ? 32 : 64;
    __shared__ __attribute__((aligned(16))) uint8_t tile[64 * RB];
    const int tid = threadIdx.x, quad = tid & 15, c4 = tid >> 4;
    const int total = (int)(a.N * a.HW), HW = (int)a.HW, K = (int)a.K, ngroup = (K + 63) >> 6;
    const int xi = (int)fastdiv_flat(blockIdx.x >> 3, a.div_groups), cg = (int)(blockIdx.x >> 3) - xi * ngroup;
    const int q0 = (xi * 8 + (int)(blockIdx.x & 7)) * 64;
    if (q0 >= total) return;
    int q = q0 + 4 * quad;
    q = q < total ? q : total - 1;  // lanes past the end read some pixel's quad, never stored
    const int n = (int)fastdiv_flat((uint32_t)q, a.div_hw), p = q - n * HW;
    const int pa = p < HW - 4 ? p : HW - 4, shift = p - pa;
    const float lo = a.lo.s, hi = a.hi.s;
    const int rowb = (int)(FP4 ? a.Kpad >> 1 : a.Kpad);
    const int valid = total - q0 < 64 ? total - q0 : 64;
    uint8_t* out = (uint8_t*)a.codes + (int64_t)q0 * rowb;
    f4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int c = cg * 64 + c4 * 4 + j;
        v[j] = *(const f4*)((const char*)a.x + (uint32_t)(((n * K + (c < K ? c : K - 1)) * HW + pa) * 4));
    }
    if (__any(shift)) {
        f4 b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int c = cg * 64 + c4 * 4 + j;
            b[j] = v[j];
            if (shift && n + 1 < (int)a.N)  // (behind the last image nothing is stored)
                b[j] = *(const f4*)((const char*)a.x + (uint32_t)((((n + 1) * K + (c < K ? c : K - 1)) * HW) * 4));
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float c[8] = {v[j][0], v[j][1], v[j][2], v[j][3], b[j][0], b[j][1], b[j][2], b[j][3]};
            float t[6];
#pragma unroll
            for (int e = 0; e < 6; ++e) t[e] = shift & 1 ? c[e + 1] : c[e];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[j][e] = shift & 2 ? t[e + 2] : t[e];
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t w = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int t = cg * 64 + c4 * 4 + j < K ? tern(v[j][i], lo, hi) : 0;
            w |= FP4 ? nib(t) << (4 * j) : (uint32_t)(t & 0xff) << (8 * j);
        }
        if (FP4)
            *(uint16_t*)(tile + (4 * quad + i) * RB + c4 * 2) = (uint16_t)w;
        else
            *(uint32_t*)(tile + (4 * quad + i) * RB + c4 * 4) = w;
    }
    __syncthreads();
    if (tid < 64 * RB / 16) {
        const int px = tid / (RB / 16), cbyte = cg * RB + tid % (RB / 16) * 16;
        if (px < valid) *(uint4*)(out + (size_t)px * rowb + cbyte) = *(const uint4*)(tile + tid * 16);
    } else if (FP4 && cg == ngroup - 1 && ngroup * RB < rowb) {
        // the zero codes behind the last group (FP4 rows are padded to 128 codes)
        const int e = tid - 64 * RB / 16;
        if (e / 2 < valid) *(uint4*)(out + (size_t)(e / 2) * rowb + ngroup * RB + e % 2 * 16) = make_uint4(0, 0, 0, 0);
    }
}

// ---- NCHW layout, int8 codes, small images whose H*W is not a multiple of 4 ---
// One 1024-thread block per image.  The image's C*H*W floats are one contiguous,
// 16-byte aligned run (C*H*W % 4 == 0), read with 16-byte loads regardless of
// where the channel rows start; element e is channel e / HW, pixel e % HW.  Codes
// are dropped byte by byte into an LDS image [HW][Cpad + 4] (the 4 pad bytes put
// consecutive pixels of a channel on consecutive banks), which is then streamed
// out in 16-byte pieces, every piece adding its 16 codes to its pixel's sum.
template <bool FP4>
__global__ __launch_bounds__(1024) void k_pack_nchw_i8_flat(PackArgs a, FastDiv div_hw)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t img[];  // [HW][Cpad + 4], then int psum[HW]
    const int tid = threadIdx.x;
    const int64_t n = blockIdx.x;
    const int HW = (int)a.HW, K = (int)a.K, Kpad = (int)a.Kpad, pitch = Kpad + 4;
    int* psum = (int*)(img + (size_t)HW * pitch);
    const float lo = thr(a.lo, n), hi = thr(a.hi, n);
    const float* xn = a.x + n * a.K * a.HW;
    for (int p = tid; p < HW; p += 1024) psum[p] = 0;
    // channels K .. Kpad-1 of every pixel are zero codes
    const int padc = Kpad - K;
    for (int e = tid; e < HW * padc; e += 1024) {
        const int p = e / padc;
        img[p * pitch + K + (e - p * padc)] = 0;
    }
    const int nvec = K * HW / 4;
    for (int v0 = tid; v0 < nvec; v0 += 4 * 1024) {
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int vi = v0 + u * 1024;
            v[u] = vi < nvec ? *(const float4*)(xn + 4 * (int64_t)vi) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int vi = v0 + u * 1024;
            if (vi < nvec) {
                int c = (int)fastdiv((uint32_t)(4 * vi), div_hw), p = 4 * vi - c * HW;
                const float e[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    img[p * pitch + c] = (uint8_t)(tern(e[i], lo, hi) & 0xff);
                    if (++p == HW) {
                        p = 0;
                        ++c;
                    }
                }
            }
        }
    }
    __syncthreads();
    const int np = Kpad / 16;
    const int rowb = FP4 ? Kpad >> 1 : Kpad;
    uint8_t* out = (uint8_t*)a.codes + n * a.HW * rowb;
    for (int e = tid; e < HW * np; e += 1024) {
        const int p = e / np, piece = e - p * np;
        const uint32_t* src = (const uint32_t*)(img + p * pitch + piece * 16);
        const uint4 w = make_uint4(src[0], src[1], src[2], src[3]);
        if (FP4)
            *(uint2*)(out + (size_t)p * rowb + piece * 8) =
                make_uint2(i8x4_to_fp4(w.x) | (i8x4_to_fp4(w.y) << 16), i8x4_to_fp4(w.z) | (i8x4_to_fp4(w.w) << 16));
        else
            *(uint4*)(out + (size_t)p * rowb + piece * 16) = w;
        if (a.sum_t) {
            int s = 0;
            s = __builtin_amdgcn_sdot4((int)w.x, 0x01010101, s, false);
            s = __builtin_amdgcn_sdot4((int)w.y, 0x01010101, s, false);
            s = __builtin_amdgcn_sdot4((int)w.z, 0x01010101, s, false);
            s = __builtin_amdgcn_sdot4((int)w.w, 0x01010101, s, false);
            atomicAdd(&psum[p], s);
        }
    }
    if (a.sum_t) {
        __syncthreads();
        for (int p = tid; p < HW; p += 1024) a.sum_t[n * a.HW + p] = psum[p];
    }
}

// ---- NCHW layout, bit planes ---------------------------------------------
// Same tiling; wave w owns the 64-channel words w, w+4, ...; a lane builds the
// mask and sign words of its pixel bit by bit.
__global__ __launch_bounds__(256) void k_pack_nchw_planes(PackArgs a)
{
    __shared__ int part[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t tiles = (a.HW + 63) >> 6;
    const int64_t n = blockIdx.x / tiles;
    const int64_t p = ((int64_t)blockIdx.x - n * tiles) * 64 + lane;
    const bool pin = p < a.HW;
    const float lo = thr(a.lo, n), hi = thr(a.hi, n);
    const float* xn = a.x + n * a.K * a.HW;
    const int64_t words = a.Kpad >> 6;
    const int64_t rows = a.N * a.HW;
    uint64_t* mrow = (uint64_t*)a.codes + (n * a.HW + p) * words;
    uint64_t* srow = (uint64_t*)a.codes + rows * words + (n * a.HW + p) * words;
    int sum = 0;
    for (int64_t w = wave; w < words; w += 4) {
        uint64_t m = 0, s = 0;
        for (int j0 = 0; j0 < 64; j0 += 16) {
            float v[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int64_t c = w * 64 + j0 + j;
                v[j] = (pin && c < a.K) ? xn[c * a.HW + p] : 0.0f;
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int64_t c = w * 64 + j0 + j;
                const bool ok = pin && c < a.K;
                const uint64_t pos = ok && v[j] > hi, neg = ok && v[j] < lo;
                m |= (pos | neg) << (j0 + j);
                s |= pos << (j0 + j);
                sum += (int)pos - (int)neg;
            }
        }
        if (pin) {
            mrow[w] = m;
            srow[w] = s;
        }
    }
    if (a.sum_t) {
        part[wave][lane] = sum;
        __syncthreads();
        if (wave == 0 && pin)
            a.sum_t[n * a.HW + p] = part[0][lane] + part[1][lane] + part[2][lane] + part[3][lane];
    }
}

}  // namespace

// pack_rows_form() says which form
template <bool FP4>
static hipError_t launch_pack_rows_codes(const PackArgs& a, hipStream_t st)
{
    const PackRowsForm f = pack_rows_form(a.rows, a.Kpad);
    auto go = [&](auto W, auto U, auto P) {
        constexpr int WPR = decltype(W)::value, UN = decltype(U)::value, NP = decltype(P)::value;
        if (f.waves != WPR || f.steps != UN || f.step != 256 * NP) return false;
        hipLaunchKernelGGL((k_pack_rows<FP4, WPR, UN, NP>), dim3((unsigned)((a.rows * WPR + 3) / 4)), dim3(256), 0, st, a);
        return true;
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I4 = std::integral_constant<int, 4>;
    if (go(I1{}, I1{}, I1{}) || go(I1{}, I1{}, I2{}) || go(I1{}, I2{}, I1{}) || go(I1{}, I2{}, I2{}) || go(I4{}, I1{}, I2{}) ||
        go(I4{}, I2{}, I2{}))
        return hipGetLastError();
    return hipErrorInvalidValue;
}
hipError_t launch_pack_rows_i8(const PackArgs& a, hipStream_t st) { return launch_pack_rows_codes<false>(a, st); }
hipError_t launch_pack_rows_fp4(const PackArgs& a, hipStream_t st) { return launch_pack_rows_codes<true>(a, st); }

hipError_t launch_pack_rows_planes(const PackArgs& a, hipStream_t st)
{
    const PackRowsForm f = pack_rows_planes_form(a.rows, a.Kpad);
    auto go = [&](auto W, auto U) {
        constexpr int WPR = decltype(W)::value, UN = decltype(U)::value;
        if (f.waves != WPR || f.steps != UN) return false;
        hipLaunchKernelGGL((k_pack_rows_planes<WPR, UN>), dim3((unsigned)((a.rows * WPR + 3) / 4)), dim3(256), 0, st, a);
        return true;
    };
    using I1 = std::integral_constant<int, 1>;
    using I4 = std::integral_constant<int, 4>;
    using I8 = std::integral_constant<int, 8>;
    if (go(I1{}, I4{}) || go(I1{}, I8{}) || go(I4{}, I4{}) || go(I4{}, I8{})) return hipGetLastError();
    return hipErrorInvalidValue;
}

template <bool FP4>
hipError_t launch_pack_nchw_codes(const PackArgs& a, hipStream_t st)
{
    const size_t smem = (size_t)64 * (FP4 ? a.Kpad / 2 : a.Kpad);  // LDS image of the block's output run
    if (smem > 128 * 1024) return hipErrorInvalidValue;
    const bool ordered = !a.lo.ptr && !a.hi.ptr, sum = a.sum_t != nullptr;
    const int64_t px = a.N * a.HW;
    PackArgs b = a;
    b.div_hw = make_fastdiv((uint32_t)a.HW);
    // small images with H*W % 4 != 0: one block per image over the flat C*H*W run
    const size_t flat_smem = (size_t)a.HW * (a.Kpad + 4) + (size_t)a.HW * 4;
    const bool flat = a.HW % 4 != 0 && (a.K * a.HW) % 4 == 0 && ((uintptr_t)a.x) % 16 == 0 && flat_smem <= 64 * 1024 && a.HW >= 4 &&
                      a.K * a.HW < ((int64_t)1 << 30) && a.N <= 0x7fffffff;
    if (ordered && !sum && a.N * a.K * a.HW < ((int64_t)1 << 30) && pack_nchw_few_pixels(a.N, a.K, a.HW, flat)) {
        const int64_t groups = (a.K + 63) / 64;
        b.div_groups = make_fastdiv((uint32_t)groups);
        hipLaunchKernelGGL(k_pack_nchw_small<FP4>, dim3((unsigned)((px + 511) / 512 * 8 * groups)), dim3(256), 0, st, b);
        return hipGetLastError();
    }
    // (At least half a million pixels.  Always with the sums, which memory hides, stored where they are wanted: FP4, 1 x 64 x
    // 4100 x 4100 1014 us, without them 1183; 1 x 37 x 5000 x 5000 965 and 948, the general kernel 1420.)
    if (a.HW % 4 == 0 && !pack_nchw_offsets_fit(a.N, a.K, a.HW)) {
        const dim3 grid((unsigned)((px + 255) / 256));
        hipLaunchKernelGGL((k_pack_nchw<64, FP4, true, false, true, uint64_t>), grid, dim3(256), 0, st, b);
        return hipGetLastError();
    }
    if (a.HW % 4 == 0) {
        const int lpr = pack_nchw_lanes(a.K, a.Kpad, px, a.HW);
        const bool part = a.K % (64 * 64 / lpr) != 0;
        const dim3 grid((unsigned)((px + 4 * lpr - 1) / (4 * lpr)));
        const std::true_type yes{};
        const std::false_type no{};
        auto go = [&](auto L, auto S, auto O, auto P) {
            hipLaunchKernelGGL((k_pack_nchw<decltype(L)::value, FP4, decltype(S)::value, decltype(O)::value, decltype(P)::value>),
                               grid, dim3(256), 0, st, b);
        };
        auto go2 = [&](auto L, auto S) {
            if (part)
                ordered ? go(L, S, yes, yes) : go(L, S, no, yes);
            else
                ordered ? go(L, S, yes, no) : go(L, S, no, no);
        };
        auto go1 = [&](auto L) { sum ? go2(L, yes) : go2(L, no); };
        if (lpr == 16)
            go1(std::integral_constant<int, 16>{});
        else if (lpr == 32)
            go1(std::integral_constant<int, 32>{});
        else
            go1(std::integral_constant<int, 64>{});
        return hipGetLastError();
    }
    if (flat) {
        hipLaunchKernelGGL(k_pack_nchw_i8_flat<FP4>, dim3((unsigned)a.N), dim3(1024), flat_smem, st, a,
                           make_fastdiv((uint32_t)a.HW));
        return hipGetLastError();
    }
    static LdsLimit lds;
    const hipError_t e = lds.raise((const void*)k_pack_nchw_i8<FP4>, 128 * 1024);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)((a.N * a.HW + 63) / 64)), block(256);
    hipLaunchKernelGGL(k_pack_nchw_i8<FP4>, grid, block, smem, st, a);
    return hipGetLastError();
}

hipError_t launch_pack_nchw_i8(const PackArgs& a, hipStream_t st) { return launch_pack_nchw_codes<false>(a, st); }
hipError_t launch_pack_nchw_fp4(const PackArgs& a, hipStream_t st) { return launch_pack_nchw_codes<true>(a, st); }

hipError_t launch_pack_nchw_planes(const PackArgs& a, hipStream_t st)
{
    const dim3 grid((unsigned)(((a.HW + 63) / 64) * a.N)), block(256);
    hipLaunchKernelGGL(k_pack_nchw_planes, grid, block, 0, st, a);
    return hipGetLastError();
}

// ---- backward of the reparameterized ternary activation (Eq.6, Eq.7) -----------
// One block: 16384 consecutive elements (64 per thread).  Writes dL/dAbar and the
// block's two partial sums (dgamma, dbeta) in double; a second single-block kernel
// adds the partials in index order, so the result does not depend on scheduling.
namespace {
constexpr int kBwdPerBlock = 16384;

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    return v;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// NT: the gradient tensor is stored with the non-temporal hint (tensors above 128 MiB, which
// the memory-side cache cannot keep for the next kernel anyway)
template <bool VEC, bool NT = false>
__global__ __launch_bounds__(256) void k_act_backward(ActBwdArgs p)
{
    __shared__ double red[2][4];
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * kBwdPerBlock;
    double sg = 0.0, sb = 0.0;
    auto one = [&](float a, float g, float& da) {
        const int t = (int)(a > p.hi) - (int)(a < p.lo);
        sg += (double)t * (double)g;
        sb += (double)g;
        const float prod = __fmul_rn(p.gamma, g);  // one fp32 product, never fused
        da = (a <= 1.0f && a >= -1.0f) ? prod : 0.0f;
    };
    if (VEC) {
#pragma unroll 4
        for (int i = 0; i < kBwdPerBlock / 1024; ++i) {
            const int64_t e = base + (int64_t)(i * 256 + tid) * 4;
            if (e + 4 <= p.n) {
                const float4 a = *(const float4*)(p.a + e), g = *(const float4*)(p.g + e);
                float4 d;
                one(a.x, g.x, d.x), one(a.y, g.y, d.y), one(a.z, g.z, d.z), one(a.w, g.w, d.w);
                if (p.da) {
                    if (NT)
                        __builtin_nontemporal_store(f32x4{d.x, d.y, d.z, d.w}, (f32x4*)(p.da + e));
                    else
                        *(float4*)(p.da + e) = d;
                }
            } else {
                for (int64_t k = e; k < p.n; ++k) {
                    float d;
                    one(p.a[k], p.g[k], d);
                    if (p.da) p.da[k] = d;
                }
            }
        }
    } else {
#pragma unroll 4
        for (int i = 0; i < kBwdPerBlock / 256; ++i) {
            const int64_t e = base + i * 256 + tid;
            if (e < p.n) {
                float d;
                one(p.a[e], p.g[e], d);
                if (p.da) p.da[e] = d;
            }
        }
    }
    sg = wave_sum(sg);
    sb = wave_sum(sb);
    if ((tid & 63) == 0) red[0][tid >> 6] = sg, red[1][tid >> 6] = sb;
    __syncthreads();
    if (tid == 0) {
        p.partials[2 * (int64_t)blockIdx.x] = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
        p.partials[2 * (int64_t)blockIdx.x + 1] = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
    }
}

// One block, UN blocks' sums of each thread in flight.
template <int THREADS, int UN>
__global__ __launch_bounds__(THREADS) void k_sum_partials(const double* partials, int64_t nblocks, double* out)
{
    constexpr int NW = THREADS / 64;
    __shared__ double red[2][NW];
    const int tid = threadIdx.x;
    double sg = 0.0, sb = 0.0;
    for (int64_t b0 = tid; b0 < nblocks; b0 += THREADS * UN) {
        double g[UN], b[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int64_t i = b0 + THREADS * u;
            g[u] = i < nblocks ? partials[2 * i] : 0.0;
            b[u] = i < nblocks ? partials[2 * i + 1] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) sg += g[u], sb += b[u];
    }
    sg = wave_sum(sg);
    sb = wave_sum(sb);
    if ((tid & 63) == 0) red[0][tid >> 6] = sg, red[1][tid >> 6] = sb;
    __syncthreads();
    if (tid < 2) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += red[tid][w];
        out[tid] = s;
    }
}

// Weight side (Section "Weight Ternarization": Wbar = k_W*W + b_W per filter, W^t = Q(Wbar),
// Wbar^t = alpha*W^t): the rules of Eq.6 / Eq.7 carried through the weight transform by the
// chain rule.  One block per filter; a lane walks the filter with stride 256 (elements, or
// groups of four where the layout allows 16-byte accesses), so a wave reads whole lines.
// The three sums are formed in double, per lane in index order, then over the wave and
// over the four waves in a fixed order: reproducible run to run.
template <bool VEC>
__global__ __launch_bounds__(256) void k_weight_backward(WeightBwdArgs p)
{
    __shared__ double red[3][4];
    const int64_t o = blockIdx.x;
    const float kw = p.kw[o], bw = p.bw[o], al = p.alpha[o];
    const float* w = p.w + o * p.K;
    const float* g = p.g + o * p.K;
    float* dw = p.dw ? p.dw + o * p.K : nullptr;
    double sa = 0.0, sk = 0.0, sb = 0.0;
    auto element = [&](float wv, float gv) -> float {
        const float wbar = __fmaf_rn(kw, wv, bw);
        const int t = (int)(wbar > p.hi) - (int)(wbar < p.lo);
        sa += (double)t * (double)gv;
        const bool inside = wbar <= 1.0f && wbar >= -1.0f;  // NaN is outside
        const float dwbar = inside ? __fmul_rn(al, gv) : 0.0f;
        if (inside) {  // a clipped (or NaN) weight adds nothing, not NaN * 0
            sk += (double)wv * (double)dwbar;
            sb += (double)dwbar;
        }
        return __fmul_rn(kw, dwbar);
    };
    if (VEC) {  // K % 4 == 0 and 16-byte aligned tensors: every filter starts on a 16-byte boundary
        // the loads of up to UN steps (4608 weights: 5) in flight together: a step at a time, the time of a
        // launch was the sum of their latencies
        constexpr int UN = 5;
        const int64_t k4n = p.K >> 2;
        for (int64_t k0 = threadIdx.x; k0 < k4n; k0 += 256 * UN) {
            float4 wv[UN], gv[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u)
                if (k0 + 256 * u < k4n) wv[u] = ((const float4*)w)[k0 + 256 * u], gv[u] = ((const float4*)g)[k0 + 256 * u];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                if (k0 + 256 * u >= k4n) break;
                float4 d;
                d.x = element(wv[u].x, gv[u].x);
                d.y = element(wv[u].y, gv[u].y);
                d.z = element(wv[u].z, gv[u].z);
                d.w = element(wv[u].w, gv[u].w);
                if (dw) ((float4*)dw)[k0 + 256 * u] = d;
            }
        }
    } else {
        for (int64_t k = threadIdx.x; k < p.K; k += 256) {
            const float d = element(w[k], g[k]);
            if (dw) dw[k] = d;
        }
    }
    sa = wave_sum(sa);
    sk = wave_sum(sk);
    sb = wave_sum(sb);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][wave] = sa;
        red[1][wave] = sk;
        red[2][wave] = sb;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int c = threadIdx.x;
        p.sums[3 * o + c] = (red[c][0] + red[c][1]) + (red[c][2] + red[c][3]);
    }
}
}  // namespace

int64_t act_backward_blocks(int64_t n) { return (n + kBwdPerBlock - 1) / kBwdPerBlock; }

hipError_t launch_act_backward(const ActBwdArgs& p, hipStream_t st)
{
    const int64_t nb = act_backward_blocks(p.n);
    const bool vec = (((uintptr_t)p.a | (uintptr_t)p.g | (uintptr_t)p.da) & 15) == 0;
    if (vec && p.da && p.n * 4 > ((int64_t)128 << 20))
        hipLaunchKernelGGL((k_act_backward<true, true>), dim3((unsigned)nb), dim3(256), 0, st, p);
    else if (vec)
        hipLaunchKernelGGL(k_act_backward<true>, dim3((unsigned)nb), dim3(256), 0, st, p);
    else
        hipLaunchKernelGGL(k_act_backward<false>, dim3((unsigned)nb), dim3(256), 0, st, p);
    // Up to 256 blocks 256 threads have a sum each: with 1024, most of them idle, the two launches took 5.1 us at
    // n = 4 where they take 4.6, and 9.3 at n = 2^20 where they take 8.8.  More: 3136 blocks in one round of loads.
    if (nb <= 256)
        hipLaunchKernelGGL((k_sum_partials<256, 1>), dim3(1), dim3(256), 0, st, p.partials, nb, p.sums);
    else
        hipLaunchKernelGGL((k_sum_partials<1024, 8>), dim3(1), dim3(1024), 0, st, p.partials, nb, p.sums);
    return hipGetLastError();
}

// The form for callers that cannot allocate: the per-block partial sums go to a fixed
// array in device memory instead of a caller workspace.  Every GPU holds its own copy of
// the array at its own address, looked up once per device (the array's name is only a
// host-side handle and is never passed to a kernel).  k_act_backward writes partials
// 0 .. nblocks-1 before k_sum_partials reads exactly those, so what an earlier call left
// in the array is never read and nothing needs clearing.
namespace {
constexpr int64_t kStaticBwdBlocks = 65536;  // 1 MiB of partial sums
__device__ __align__(256) double g_act_bwd_scratch[2 * kStaticBwdBlocks];
constexpr int kMaxDevices = 64;
double* g_act_bwd_scratch_ptr[kMaxDevices] = {};
std::mutex g_act_bwd_scratch_mutex;
}  // namespace

int64_t act_backward_static_max_n() { return kStaticBwdBlocks * kBwdPerBlock; }

hipError_t launch_act_backward_static(ActBwdArgs p, hipStream_t st)
{
    if (act_backward_blocks(p.n) > kStaticBwdBlocks) return hipErrorInvalidValue;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    {
        std::lock_guard<std::mutex> lock(g_act_bwd_scratch_mutex);
        if (!g_act_bwd_scratch_ptr[dev]) {
            double* ptr = nullptr;
            e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(g_act_bwd_scratch));
            if (e != hipSuccess) return e;
            if (!ptr) return hipErrorInvalidSymbol;
            g_act_bwd_scratch_ptr[dev] = ptr;
        }
        p.partials = g_act_bwd_scratch_ptr[dev];
    }
    return launch_act_backward(p, st);
}

hipError_t launch_weight_backward(const WeightBwdArgs& p, hipStream_t st)
{
    const bool vec = (p.K & 3) == 0 && (((uintptr_t)p.w | (uintptr_t)p.g | (uintptr_t)p.dw) & 15) == 0;
    if (vec)
        hipLaunchKernelGGL(k_weight_backward<true>, dim3((unsigned)p.O), dim3(256), 0, st, p);
    else
        hipLaunchKernelGGL(k_weight_backward<false>, dim3((unsigned)p.O), dim3(256), 0, st, p);
    return hipGetLastError();
}


}  // namespace rtn
