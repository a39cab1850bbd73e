"""The size rules of csrc/choice.h and the offsets of csrc/conv_offsets.h, compiled for the host."""
import ctypes as C
import os
import random
import subprocess

import pytest

from paper_1912_02057_amd import binding as B
from test_gpu_parity import KSPLIT_CONVS, KSPLIT_GEMMS

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1912_02057_amd", "csrc")

SHIM = r"""
#include "choice.h"
#include "conv_offsets.h"
template <bool BIG>
static void walk(int W, int Cpad, int KW, int steps, int64_t *out)
{
    using Walk = rtn::TapWalk<rtn::ConvOff<BIG>>;
    Walk w;
    for (int i = 0; i < steps; ++i, w.step(Cpad, KW, Walk::row_skip(W, KW, Cpad)))
        out[3 * i] = (int64_t)w.off, out[3 * i + 1] = 31 - w.shr, out[3 * i + 2] = w.kw;
}
extern "C" void tap_walk(int big, int W, int Cpad, int KW, int steps, int64_t *out)
{
    big ? walk<true>(W, Cpad, KW, steps, out) : walk<false>(W, Cpad, KW, steps, out);
}
extern "C" int64_t conv_span(const int64_t *v, int t) { return rtn::conv_span(v[0], v[1], v[2], v[3], v[4], v[5], v[6], t); }
extern "C" int64_t reach_back(int64_t pad, int64_t W) { return rtn::conv_reach_back(pad, W); }
extern "C" int codes_fit(const int64_t *v, int64_t pad, int64_t pixel, int bq)
{
    return rtn::conv_codes_fit(v[0], v[1], v[2], v[3], v[4], v[5], v[6], pad, pixel, bq);
}
extern "C" int outputs_fit(int64_t Nb, int64_t O, int64_t ohw, int bq) { return rtn::conv_outputs_fit(Nb, O, ohw, bq); }
extern "C" int64_t halo_rows(int bq, int pad, int W) { return rtn::halo_rows(bq, pad, W); }
extern "C" void pack_form(int planes, int64_t rows, int64_t Kpad, int *out)
{
    const rtn::PackRowsForm f = planes ? rtn::pack_rows_planes_form(rows, Kpad) : rtn::pack_rows_form(rows, Kpad);
    out[0] = f.waves, out[1] = f.steps, out[2] = f.step;
}
extern "C" int ksplit(const int64_t *v, int limit)
{
    const rtn::KsplitShape s = {v[0], v[1], (int)v[2], (int)v[3], (int)v[4], (int)v[5], (int)v[6], (int)v[7], (int)v[8], (int)v[9]};
    return limit ? (int)rtn::ksplit_lds_bytes(rtn::kKsplitForms[limit - 1], s) : rtn::pick_ksplit(s);
}
extern "C" int few_pixels(int64_t N, int64_t K, int64_t HW, int flat) { return rtn::pack_nchw_few_pixels(N, K, HW, flat); }
extern "C" int pack_lanes(int64_t K, int64_t Kpad, int64_t px, int64_t HW) { return rtn::pack_nchw_lanes(K, Kpad, px, HW); }
extern "C" int pack_offsets_fit(int64_t N, int64_t K, int64_t HW) { return rtn::pack_nchw_offsets_fit(N, K, HW); }
extern "C" int dw_vector(int64_t C, int stride, int64_t y_bytes, int acc) { return rtn::dw_vector_stores(C, stride, y_bytes, acc); }
extern "C" void band_tile(int bid, int tilesP, int tilesQ, int *out)
{
    const int last = tilesP & 7 ? tilesP & 7 : 8;
    rtn::band_tile(bid, tilesP, 8 * tilesQ, [&](int n) { return n / (8 * tilesQ); }, [&](int n) { return n / last; }, out[0], out[1]);
}
extern "C" int nt_hint(int64_t M, int64_t N, uintptr_t y, int nk) { return rtn::gemm_nt_hint(M, N, y, nk); }
"""


@pytest.fixture(scope="module")
def L(tmp_path_factory):
    d = tmp_path_factory.mktemp("choice")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "choice.so")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC, str(d / "shim.cpp"), "-o", so], check=True)
    lib = C.CDLL(so)
    lib.pack_form.argtypes = [C.c_int, C.c_int64, C.c_int64, C.c_void_p]
    lib.ksplit.argtypes = [C.c_void_p, C.c_int]
    lib.tap_walk.argtypes = [C.c_int] * 5 + [C.c_void_p]
    lib.few_pixels.argtypes = [C.c_int64, C.c_int64, C.c_int64, C.c_int]
    lib.pack_lanes.argtypes = [C.c_int64] * 4
    lib.pack_offsets_fit.argtypes = [C.c_int64] * 3
    lib.conv_span.argtypes, lib.conv_span.restype = [C.c_void_p, C.c_int], C.c_int64
    lib.reach_back.argtypes, lib.reach_back.restype = [C.c_int64] * 2, C.c_int64
    lib.codes_fit.argtypes, lib.outputs_fit.argtypes = [C.c_void_p, C.c_int64, C.c_int64, C.c_int], [C.c_int64] * 3 + [C.c_int]
    lib.halo_rows.argtypes, lib.halo_rows.restype = [C.c_int] * 3, C.c_int64
    lib.dw_vector.argtypes = [C.c_int64, C.c_int, C.c_int64, C.c_int]
    lib.nt_hint.argtypes = [C.c_int64, C.c_int64, C.c_size_t, C.c_int]
    return lib


@pytest.mark.parametrize("planes", [0, 1])
def test_row_pack_waves_have_work(L, planes):
    """Of the waves that share a row at most one has no elements of it, at any length."""
    out = (C.c_int * 3)()
    for rows in (1, 16, 500, 2047, 2048, 100000):
        for Kpad in list(range(64, 9000, 64)) + [1 << 20]:
            L.pack_form(planes, rows, Kpad, out)
            waves, turn = out[0], out[1] * out[2]
            assert waves in (1, 4) and turn > 0
            assert waves == 1 or (waves - 2) * turn < Kpad, (rows, Kpad, list(out))


def test_pack_of_few_pixels(L):
    """Both sides of each line of the rule."""
    few = lambda N, K, H, W, flat: bool(L.few_pixels(N, K, H * W, flat))
    assert few(64, 1024, 8, 8, 0) and few(1, 948, 62, 62, 0)
    assert not few(65, 1024, 8, 8, 0) and not few(1, 512, 8, 8, 0) and not few(100, 600, 1, 3, 0)
    assert few(17, 513, 9, 9, 0) and few(88, 513, 3, 3, 0) and few(83, 2048, 7, 7, 0)
    assert not few(18, 513, 9, 9, 0) and not few(89, 513, 3, 3, 0) and not few(33, 768, 11, 11, 0)
    # many small images with a block each: five times as long without it
    assert few(1, 516, 9, 9, 1) and few(2, 1024, 7, 7, 1)
    for shape in ((2, 768, 7, 7), (83, 576, 7, 7), (8, 1280, 7, 7), (9, 768, 9, 9), (444, 516, 3, 3), (64, 2048, 5, 5)):
        assert not few(*shape, 1)


def test_pack_groups_divide_the_channels(L):
    """Channels that a group divides are not masked where that is blocks enough; a row of any length has its run."""
    lanes = lambda N, K, H: L.pack_lanes(K, -(-K // 64) * 64, N * H * H, H * H)
    for K in (64, 128, 256, 512, 768, 1024, 2048):
        for N, H in ((1, 8), (16, 28), (256, 28), (32, 56)):
            assert K % (4096 // lanes(N, K, H)) == 0
    for K in (384, 640, 896, 1152, 1920):
        assert lanes(256, K, 14) == lanes(64, K, 28) == lanes(32, K, 56) == 32 and lanes(14, K, 28) == 16
    for K in (192, 320, 448, 576, 960):
        assert lanes(256, K, 14) == lanes(64, K, 28) == 64 and lanes(408, K, 14) == (64 if K == 320 else 32 if K == 192 else 16)
        for N, H in ((16, 28), (16, 56), (32, 56), (160, 14)):
            assert lanes(N, K, H) == (32 if K == 192 else 16)
    assert lanes(256, 100, 14) == 32 and lanes(256, 300, 14) == 16 and lanes(256, 50, 14) == 64


def test_pack_offsets(L):
    """32-bit offsets for every block whose images they reach: the last element of 256 consecutive pixels, in bytes."""
    for N, K, HW in ((1, 64, 9000000), (1, 64, 1 << 24), (2, 64, 9000000), (2, 64, 1 << 23), (1, 2048, 1 << 19), (3, 2048, 1 << 18),
                     (1 << 20, 2048, 4), (4096, 2048, 256), (1000, 2048, 4096), (1, 1, (1 << 30) - 4), (1, 1, 1 << 30)):
        last = max(((N * HW - 1 if q + 255 >= N * HW else q + 255) // HW - q // HW) for q in (0, HW - 1, 4 * (HW // 8))) + 1
        fits = bool(L.pack_offsets_fit(N, K, HW))
        assert not fits or 4 * last * K * HW <= 1 << 32, (N, K, HW)
        assert fits or 4 * min(N, last + 1) * K * HW >= 1 << 32, (N, K, HW)


def test_depthwise_stores_in_parts_of_lines(L):
    """Both sides of each line of the rule, in MiB of y."""
    for Ch, stride, acc, yes, no in ((1024, 1, 1, (129, 169, 280), (128, 281, 400)), (128, 2, 1, (129, 200), (128, 201, 400)),
                                     (64, 2, 0, (129, 203, 320), (128, 321)), (512, 1, 0, (), (130, 252, 600)), (32, 1, 0, (221, 308, 600), (220, 130)),
                                     (48, 1, 1, (129, 280), (128, 281)), (32, 1, 1, (129, 400), (128,)), (40, 2, 0, (129, 600), (128,))):
        for mib, want in [(m, True) for m in yes] + [(m, False) for m in no]:
            assert bool(L.dw_vector(Ch, stride, mib << 20, acc)) == want, (Ch, stride, acc, mib)


def test_tiles_of_an_xcd_are_a_block(L):
    """Each tile once; the run of tiles that an XCD has lies in as few bands of 8 rows as it can."""
    out = (C.c_int * 2)()
    for tilesP, tilesQ in ((1, 1), (64, 4), (72, 4), (3, 100), (8, 9), (9, 8), (13, 17), (100, 3)):
        tiles = []
        for bid in range(tilesP * tilesQ):
            L.band_tile(bid, tilesP, tilesQ, out)
            tiles.append((out[0], out[1]))
        assert sorted(tiles) == [(p, q) for p in range(tilesP) for q in range(tilesQ)]
        share = -(-len(tiles) // 8)
        for x in range(0, len(tiles), share):
            rows = {p for p, _ in tiles[x:x + share]}
            assert len(rows) <= 8 * (-(-share // (8 * tilesQ)) + 1)


def test_gemm_store_hint(L):
    """Only whole lines are hinted, and outputs that the memory-side cache holds only behind a K loop."""
    base = 1 << 30
    assert L.nt_hint(8192, 4096, base, 8) and L.nt_hint(16384, 8192, base, 1) and L.nt_hint(16384, 8176, base, 64)
    assert not L.nt_hint(8192, 4096, base, 7) and not L.nt_hint(8191, 4096, base, 64)     # few K-steps; below 128 MiB
    assert not L.nt_hint(16384, 4096, base, 7) and L.nt_hint(16385, 4096, base, 1)        # both sides of 256 MiB
    for N in (3001, 3004, 3000, 2992):
        assert not L.nt_hint(12000, N, base, 64)
    for N in (8191, 8188, 8184):
        assert not L.nt_hint(16384, N, base, 64)
    for y in (4, 16, 32, 64):
        assert not L.nt_hint(8192, 4096, base + y, 64)
    assert L.nt_hint(16384, 8192, base + 64, 64) and not L.nt_hint(16384, 8192, base + 32, 64)


def _form(L, fmt, rp, rq, K=0, conv=None):
    """The small-grid form of a GEMM (rp x rq x K) or of a conv (filters x pixels, conv = C, H, W, k, stride, pad)."""
    codes = 128 if fmt == B.RTN_CODE_FP4 else 64        # of a K-step
    v = [rp, rq, -(-K // codes)] + [0] * 7
    if conv:
        Cc, H, W, k, stride, pad = conv
        axis = 2 * pad + 1 if min(H, W) >= k else (pad + 1) ** 2
        v[2:] = [k * k * -(-Cc // codes), k, k, stride, pad, W, 64 * -(-Cc // codes), 4 + axis * axis]
    return L.ksplit((C.c_int64 * 10)(*v), 0)


def _conv_form(L, fmt, geo):
    Cc, H, W, O, k, stride, pad, batch = geo
    OH, OW = (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1
    return _form(L, fmt, O, batch * OH * OW, conv=(Cc, H, W, k, stride, pad))


@pytest.mark.parametrize("fmt", [B.RTN_CODE_I8, B.RTN_CODE_FP4])
def test_small_grid_tests_reach_every_form(L, fmt):
    """The GPU tests of the small-grid kernel run all of its forms in both formats."""
    assert {_form(L, fmt, *g) for g in KSPLIT_GEMMS} == {0, 1, 2}
    assert {_conv_form(L, fmt, g) for g in KSPLIT_CONVS} >= set(range(8))


def test_small_grid_lines(L):
    """Both sides of each line of the rule, in tiles and in K-steps."""
    I8 = B.RTN_CODE_I8
    for nk, form in ((1, 0), (3, 0), (4, 1), (33, 1)):                   # 256 tiles of 32 x 32
        assert _form(L, I8, 512, 512, 64 * nk) == form
    for nk, form in ((3, 0), (4, 1), (32, 1), (33, 2)):                  # 512, 256 of 64 x 32
        assert _form(L, I8, 512, 1024, 64 * nk) == form
    assert _form(L, I8, 32, 16384, 64 * 33) == 1                         # 512, 512 of 64 x 32
    for nk in (1, 65):
        assert _form(L, I8, 513, 1024, 64 * nk) == -1                    # 544
    conv = lambda O, px, nk, k=1: _form(L, I8, O, px, conv=(64 * nk // (k * k), 16, 16, k, 1 if k > 1 else 2, k // 2))
    for nk, form in ((3, 0), (4, 1), (9, 1)):
        assert conv(512, 512, nk) == form
    for nk, form in ((1, 0), (4, 0), (8, 0), (9, 2)):
        assert conv(512, 1024, nk) == form
    assert conv(32, 16384, 8) == 0 and conv(32, 16384, 9) == 1
    for nk, form in ((32, -1), (33, 3)):
        assert conv(1024, 1024, nk) == form                              # 256 of 64 x 64
    for nk, form in ((64, -1), (65, 4)):
        assert conv(1024, 2048, nk) == form                              # 512
    assert conv(1024, 2049, 65) == -1
    for nk, form in ((9, -1), (18, 6)):                                  # 3 x 3, stride 1: the pixel run
        assert conv(1024, 1024, nk, 3) == form
    for nk, form in ((27, -1), (36, 7)):
        assert conv(1024, 2048, nk, 3) == form
    for nk, form in ((63, 2), (72, 5)):
        assert conv(512, 1024, nk, 3) == form


@pytest.mark.parametrize("big,W,Cpad,KH,KW", [
    (0, 56, 64, 3, 3), (0, 1, 128, 3, 3), (0, 1, 64, 5, 2), (0, 1009, 2048, 7, 7), (1, 56, 64, 3, 3), (1, 1, 128, 3, 3),
    (1, 1 << 25, 64, 3, 3), (1, (1 << 24) + 3, 64, 5, 5), (1, 1 << 30, 64, 2, 2), (1, 700001, 1024, 7, 7), (1, 1 << 24, 8192, 3, 3)])
def test_tap_offsets_of_a_window(L, big, W, Cpad, KH, KW):
    """The running offset of a window's K-steps is (kh W + kw) Cpad + cc, also where that passes 32 bits."""
    steps = [((kh * W + kw) * Cpad + cc, kh, kw) for kh in range(KH) for kw in range(KW) for cc in range(0, Cpad, 64)]
    assert big or max(steps)[0] < 1 << 32
    out = (C.c_int64 * (3 * len(steps)))()
    L.tap_walk(big, W, Cpad, KW, len(steps), out)
    assert [tuple(out[3 * i:3 * i + 3]) for i in range(len(steps))] == steps


def _conv_dims(H, W, KH, KW, stride, pad):
    OH, OW = (H + 2 * pad - KH) // stride + 1, (W + 2 * pad - KW) // stride + 1
    return OH, OW, (C.c_int64 * 7)(H, W, OH, OW, KH, KW, stride)


def test_conv_span(L):
    """Over random geometries: every window of a tile lies between the reach before its first one and the span behind it."""
    rng = random.Random(7)
    for _ in range(3000):
        KH, KW, stride = rng.randint(1, 7), rng.randint(1, 7), rng.choice([1, 1, 2, 3, 5, 64])
        pad = rng.randint(0, min(KH, KW, 3) - 1)
        H, W, Nb = rng.randint(max(1, KH - 2 * pad), 40), rng.randint(max(1, KW - 2 * pad), 40), rng.randint(1, 5)
        OH, OW, v = _conv_dims(H, W, KH, KW, stride, pad)

        def corner(m):
            nb, pix = divmod(m, OH * OW)
            return (nb * H + pix // OW * stride - pad) * W + pix % OW * stride - pad

        for bq in (32, 64, 256):
            q0 = rng.randrange(0, Nb * OH * OW)
            ends = [corner(m) - corner(q0) for m in range(q0, min(q0 + bq, Nb * OH * OW))]
            assert -L.reach_back(pad, W) <= min(ends)
            assert max(ends) + (KH - 1) * W + KW <= L.conv_span(v, bq)


def test_conv_offsets_fit(L):
    """Images of any size fit 32-bit offsets, rows of hundreds of millions of bytes do not; outputs fit that are not
    2^32 bytes apart."""
    for H, W, pixel, k, stride, fits in ((4096, 4096, 64, 3, 1, True), (5825, 5825, 64, 3, 64, True), (30000, 30000, 64, 3, 1, True),
                                         (2, 1 << 25, 64, 3, 1, False), (2, 1 << 23, 64, 3, 1, True), (2, 1 << 24, 64, 3, 1, False),
                                         (1, 1 << 25, 64, 1, 1, True), (5, 1 << 20, 1024, 5, 1, False), (1, 1 << 18, 64, 1, 64, True)):
        _, _, v = _conv_dims(H, W, k, min(k, W), stride, k // 2)
        for bq in (64, 128, 256):
            assert bool(L.codes_fit(v, k // 2, pixel, bq)) == fits, (H, W, bq)
    assert L.outputs_fit(1, 128, 4096 ** 2, 64) and not L.outputs_fit(2, 128, 4096 ** 2, 64) and not L.outputs_fit(1, 8, 1 << 27, 64)
    assert L.outputs_fit(256, 512, 49, 64) and L.outputs_fit(2, 128, 2800 ** 2, 256) and L.outputs_fit(1 << 20, 4096, 49, 256)


def test_halo_rows(L):
    """The pixel run of a tile is counted in 64 bits, whole multiples of 16."""
    assert L.halo_rows(128, 1, 56) == 256 and L.halo_rows(256, 2, 13) == 320
    assert L.halo_rows(128, 2, (1 << 31) - 1025) == (128 + 4 * ((1 << 31) - 1024) + 15) // 16 * 16


LDS_SHIM = r"""
#include "lds_limit.h"
static int device, calls[70], fail;
extern "C" hipError_t hipGetDevice(int *d) { *d = device; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int)
{
    ++calls[device];
    return fail ? hipErrorInvalidValue : hipSuccess;
}
extern "C" int launch_on(int dev, int failing)
{
    static rtn::LdsLimit lds;
    device = dev, fail = failing;
    return (int)lds.raise(nullptr, 1 << 17);
}
extern "C" int calls_on(int dev) { return calls[dev]; }
"""


def test_lds_limit_is_raised_on_every_device(tmp_path):
    """Once per device, again after a failure, and at every launch beyond the 64 devices that have a bit."""
    (tmp_path / "shim.cpp").write_text(LDS_SHIM)
    so = str(tmp_path / "lds.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-shared", "-fPIC", "-I" + CSRC, "-isystem", rocm + "/include",
                    str(tmp_path / "shim.cpp"), "-o", so, "-Wl,-Bsymbolic"], check=True)
    S = C.CDLL(so)
    for dev in (0, 1, 0, 1, 63, 63):
        assert S.launch_on(dev, 0) == 0
    assert [S.calls_on(d) for d in (0, 1, 63)] == [1, 1, 1]
    assert S.launch_on(2, 1) != 0 and S.launch_on(2, 0) == 0 and S.launch_on(2, 0) == 0 and S.calls_on(2) == 2
    assert S.launch_on(64, 0) == 0 and S.launch_on(64, 0) == 0 and S.calls_on(64) == 2
