"""CPU build of the HIP library's device bit logic, checked against the oracle (no GPU).

The header with the device functions is compiled for the host with g++ through a small
shim (tests/devfn_host).  This is not the parity test proper (that one runs the kernels
on the GPU through the C ABI); it checks the integer encode / decode logic the kernels
are built from on every binary32 top-13-bit pattern, every 16-bit source pattern and
random patterns, under every rounding method and option.
"""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

from oracle import hif8_oracle as orc

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "devfn_host", "devfn_host.cpp")
HDR = os.path.join(HERE, "..", "paper_2409_16626_amd", "csrc", "hif8_device.hpp")
HDR2 = os.path.join(HERE, "..", "paper_2409_16626_amd", "csrc", "hif8_gemm_split.hpp")
HDR3 = os.path.join(HERE, "..", "paper_2409_16626_amd", "csrc", "hif8_multi_plan.hpp")
HDR4 = os.path.join(HERE, "..", "paper_2409_16626_amd", "csrc", "hif8_axis_plan.hpp")
LIB = os.path.join(HERE, "devfn_host", "libdevfn_host.so")


@pytest.fixture(scope="module")
def dev():
    newest = max(os.path.getmtime(f) for f in (SRC, HDR, HDR2, HDR3, HDR4))
    if not os.path.exists(LIB) or os.path.getmtime(LIB) < newest:
        subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", LIB, SRC], check=True)
    lib = ctypes.CDLL(LIB)
    return lib


def _enc(lib, ybits, mode, srck, seed=0):
    ybits = np.ascontiguousarray(ybits, np.uint32)
    out = np.empty(ybits.shape, np.uint8)
    lib.devfn_encode_bits(ybits.ctypes.data_as(ctypes.c_void_p), out.ctypes.data_as(ctypes.c_void_p),
                          ctypes.c_size_t(ybits.size), ctypes.c_uint32(mode), ctypes.c_int(srck),
                          ctypes.c_uint64(seed))
    if (mode & 0xF) in (orc.RM_HR, orc.RM_SSR):
        # the streaming kernels' table-driven forms must agree with the generic form
        out2 = np.empty(ybits.shape, np.uint8)
        if srck == 0:
            lib.devfn_encode_bits_hr_table(ybits.ctypes.data_as(ctypes.c_void_p), out2.ctypes.data_as(ctypes.c_void_p),
                                           ctypes.c_size_t(ybits.size), ctypes.c_uint32(mode))
        else:
            # 16-bit sources: the clamped sum looked up in the truncating table
            lib.devfn_encode_bits_hr16_stream(ybits.ctypes.data_as(ctypes.c_void_p), out2.ctypes.data_as(ctypes.c_void_p),
                                              ctypes.c_size_t(ybits.size), ctypes.c_uint32(mode), ctypes.c_int(srck))
        bad = np.nonzero(out != out2)[0]
        assert bad.size == 0, [(hex(ybits[i]), hex(out[i]), hex(out2[i])) for i in bad[:8]]
    if (mode & 0xF) == orc.RM_SR:
        # the streaming kernels' add-and-truncate form of standard SR must agree as well
        out2 = np.empty(ybits.shape, np.uint8)
        lib.devfn_encode_bits_sr_table(ybits.ctypes.data_as(ctypes.c_void_p), out2.ctypes.data_as(ctypes.c_void_p),
                                       ctypes.c_size_t(ybits.size), ctypes.c_uint32(mode), ctypes.c_uint64(seed))
        bad = np.nonzero(out != out2)[0]
        assert bad.size == 0, [(hex(ybits[i]), hex(out[i]), hex(out2[i])) for i in bad[:8]]
    return out


MODES = [orc.RM_TA, orc.RM_HR, orc.RM_TA | orc.FLAG_SAT, orc.RM_HR | orc.FLAG_SAT,
         orc.RM_TA | orc.FLAG_NAN2ZERO, orc.RM_HR | orc.FLAG_SAT | orc.FLAG_NAN2ZERO,
         orc.RM_TE, orc.RM_SSR, orc.RM_SR, orc.RM_TE | orc.FLAG_SAT, orc.RM_SR | orc.FLAG_SAT | orc.FLAG_NAN2ZERO]


@pytest.mark.parametrize("mode", MODES)
def test_device_encode_logic_f32(dev, mode):
    rng = np.random.default_rng(21)
    top = np.arange(1 << 13, dtype=np.uint32) << 19
    parts = [top, top | np.uint32(0x7FFFF), top | np.uint32(1), top | np.uint32(0x2000),
             top | rng.integers(0, 1 << 19, size=top.size).astype(np.uint32)]
    yb = rng.integers(0, 2 ** 32, size=1 << 20, dtype=np.uint64).astype(np.uint32)
    ex = rng.integers(127 - 40, 127 + 18, size=yb.size).astype(np.uint32)
    yb[::2] = (yb[::2] & np.uint32(0x807FFFFF)) | (ex[::2] << 23)
    yb[::8] &= np.uint32(0xFFFFC000)
    h = np.arange(65536, dtype=np.uint16).view(np.float16).astype(np.float32).view(np.uint32)
    allb = np.concatenate(parts + [yb, h])
    allb[5::16] &= np.uint32(0xFFF80000)      # exact ties and representable values for TE
    orc.set_sr_seed(0xABCDEF0123)
    try:
        want = orc.encode_f32(allb.view(np.float32), 1.0, mode)
    finally:
        orc.set_sr_seed(0)
    got = _enc(dev, allb, mode, 0, 0xABCDEF0123)
    bad = np.nonzero(want != got)[0]
    assert bad.size == 0, [(hex(allb[i]), hex(want[i]), hex(got[i])) for i in bad[:8]]


@pytest.mark.parametrize("mode", MODES)
def test_device_encode_logic_bf16(dev, mode):
    b = np.arange(65536, dtype=np.uint16)
    for scale in (np.float32(1.0), np.float32(0.37), np.float32(1311.7), np.float32(2.0 ** -20)):
        prod = ((b.astype(np.uint32) << 16).view(np.float32) * scale).astype(np.float32)
        want = orc.encode_bf16(b, scale, mode)
        got = _enc(dev, prod.view(np.uint32), mode, 1)
        bad = np.nonzero(want != got)[0]
        assert bad.size == 0, [(hex(b[i]), hex(want[i]), hex(got[i])) for i in bad[:8]]


@pytest.mark.parametrize("mode", MODES)
def test_device_encode_logic_f16(dev, mode):
    h = np.arange(65536, dtype=np.uint16)
    for scale in (np.float32(1.0), np.float32(0.37), np.float32(2.0 ** -9)):
        prod = (h.view(np.float16).astype(np.float32) * scale).astype(np.float32)
        want = orc.encode_f16(h, scale, mode)
        got = _enc(dev, prod.view(np.uint32), mode, 2)
        bad = np.nonzero(want != got)[0]
        assert bad.size == 0, [(hex(h[i]), hex(want[i]), hex(got[i])) for i in bad[:8]]


def test_device_decode_logic(dev):
    codes = np.arange(256, dtype=np.uint8)
    out = np.empty(256, np.uint32)
    dev.devfn_decode_bits(codes.ctypes.data_as(ctypes.c_void_p), out.ctypes.data_as(ctypes.c_void_p),
                          ctypes.c_size_t(256))
    assert np.array_equal(out, orc.decode_f32(codes, 1.0).view(np.uint32))


def test_device_narrow_logic(dev):
    rng = np.random.default_rng(22)
    u = rng.integers(0, 2 ** 32, size=1 << 18, dtype=np.uint64).astype(np.uint32)
    u[::7] = (u[::7] & np.uint32(0xFFFF0000)) | np.uint32(0x8000)
    out = np.empty(u.shape, np.uint16)
    dev.devfn_narrow_bf16(u.ctypes.data_as(ctypes.c_void_p), out.ctypes.data_as(ctypes.c_void_p),
                          ctypes.c_size_t(u.size))
    assert np.array_equal(out, orc.narrow_bf16(u.view(np.float32)))


def test_device_scale_from_amax_logic(dev):
    """The scale arithmetic of the scale kernels (fl32(target / amax), optional floor to a power of two,
    degenerate amax -> 1) against the oracle, bit for bit, on special values and random patterns."""
    rng = np.random.default_rng(23)
    special = np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 1e-45, 1.1754944e-38, 3.4028235e38, 1.0, 32768.0, 32767.99,
                        5e-39, 2.5e-41, 3.0e33, 6.1e-5], np.float32)
    rnd = rng.integers(0, 2 ** 31, size=200000, dtype=np.int64).astype(np.uint32).view(np.float32)   # non-negative patterns
    amax = np.concatenate([special, rnd, np.exp2(rng.uniform(-40, 40, 50000)).astype(np.float32)])
    out = np.empty(amax.shape, np.float32)
    for target in (32768.0, 1.0, 448.0, 3.0e38, 1e-30):
        for pow2 in (0, 1):
            dev.devfn_scale_from_amax(amax.ctypes.data_as(ctypes.c_void_p), out.ctypes.data_as(ctypes.c_void_p),
                                      ctypes.c_size_t(amax.size), ctypes.c_float(target), ctypes.c_int(pow2))
            want = np.array([orc.scale_from_amax(a, target, bool(pow2)) for a in amax[:2000]], np.float32)
            assert np.array_equal(out[:2000].view(np.uint32), want.view(np.uint32)), (target, pow2)
            assert np.all(out > 0) and np.all(np.isfinite(out))
            if pow2:      # a power of two: empty mantissa field, or (subnormal) a single mantissa bit
                b = out.view(np.uint32)
                normal = (b >> 23) != 0
                assert np.all((b[normal] & 0x7FFFFF) == 0)
                sub = b[~normal]
                assert np.all((sub & (sub - 1)) == 0)


def test_gemm_ragged_round_split_plan(dev):
    """Host-side planning of the GEMM launches: a second launch of small tiles only where the last round of
    256 x 256 tiles would be at most half full and whole tile columns fill the complete rounds; the split
    column is a multiple of 256 inside the matrix and the large tiles left of it fill whole rounds or less."""
    dev.devfn_ragged_round_split.restype = ctypes.c_uint32
    dev.devfn_ragged_round_split.argtypes = [ctypes.c_size_t, ctypes.c_size_t, ctypes.c_size_t]
    f = dev.devfn_ragged_round_split
    assert f(8192, 11008, 256) == 40 * 256            # 32 x 43 tiles = 5.375 rounds: 40 tile columns = 5 rounds exactly
    assert f(8192, 8192, 256) == 0                    # 1024 tiles = 4 whole rounds
    assert f(4096, 4096, 256) == 0                    # one round exactly
    assert f(2048, 2048, 256) == 0                    # fewer tiles than compute units
    assert f(8192, 11008, 0) == 0
    assert f(8192, 12288, 256) == 0                   # 6 rounds exactly
    assert f(8192, 12800, 256) == 48 * 256            # 32 x 50 = 6.25 rounds
    assert f(8192, 14336, 256) == 0                   # 7 rounds exactly
    assert f(8192, 15000, 256) == 56 * 256            # 32 x 59 = 7.4 rounds: 3 tile columns left = 96 tiles
    assert f(8192, 16000, 256) == 0                   # 32 x 63 = 7.9 rounds: the last round is nearly full
    rng = np.random.default_rng(3)
    for _ in range(2000):
        M, N, cus = int(rng.integers(1, 40000)), int(rng.integers(1, 40000)), int(rng.choice([64, 120, 256, 304]))
        s = f(M, N, cus)
        tm, tn = (M + 255) // 256, (N + 255) // 256
        if s:
            assert s % 256 == 0 and 0 < s < N
            big = tm * (s // 256)
            assert big <= (tm * tn // cus) * cus                  # the large tiles fit the complete rounds
            assert (tn - s // 256) * tm * 2 <= cus                # what is left is at most half a round of large tiles
            assert tm * tn > cus and (tm * tn) % cus != 0


def test_codes_gemm_launches(dev):
    """Tiles of the code-operand kernel: every column in one launch, a second launch only where the large tiles of the first fill whole rounds, every tile
    shape reached, and never a price above that of any single tile."""
    f, us = dev.devfn_codes_launches, dev.devfn_codes_tile_us
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_size_t] * 4 + [ctypes.POINTER(ctypes.c_uint32)]
    us.restype, us.argtypes = ctypes.c_double, [ctypes.c_int] + [ctypes.c_size_t] * 4

    def plan(M, N, K, cus=256):
        out = (ctypes.c_uint32 * 6)()
        n = f(M, N, K, cus, out)
        return [tuple(out[3 * i:3 * i + 3]) for i in range(n)]

    assert plan(512, 4096, 4096) == [(0, 0, 4096)] and plan(1024, 8192, 4096) == [(1, 0, 8192)] and plan(100, 33000, 80) == [(2, 0, 33000)]
    assert plan(4096, 4096, 4096) == [(3, 0, 4096)] and plan(2048, 11008, 4096) == [(3, 0, 8192), (1, 8192, 11008)]
    rng = np.random.default_rng(8)
    for _ in range(3000):
        M, N, K = (int(2.0 ** rng.uniform(0, 15)) for _ in range(3))
        cus = int(rng.choice([64, 256, 304]))
        got = plan(M, N, K, cus)
        assert got[0][1] == 0 and got[-1][2] == N and all(0 <= t <= 3 and b < e for t, b, e in got)
        price = [us(t, M, N, K, cus) for t in range(4)]
        if len(got) == 2:
            assert got[0][0] == 3 and got[0][2] == got[1][1] and got[1][1] % 256 == 0
            assert us(3, M, got[0][2], K, cus) + us(got[1][0], M, N - got[0][2], K, cus) < min(price)
        else:
            assert price[got[0][0]] == min(price)


def test_gemm_tile_order_is_a_bijection_and_compact_per_die(dev):
    """Workgroup -> tile of the expanded-operand GEMM: every tile is taken exactly once, only workgroups at the
    end of the grid go without one, and the 32 workgroups that run together on one die (b = die + 8 s for 32
    consecutive s) touch few operand panels: at most 8 tile rows and, for full groups, 4 to 5 tile columns."""
    dev.devfn_tile_order.restype = ctypes.c_uint32
    dev.devfn_tile_order.argtypes = [ctypes.c_uint32] * 3
    dev.devfn_tile_order_grid.restype = ctypes.c_uint32
    dev.devfn_tile_order_grid.argtypes = [ctypes.c_uint32]
    for tm, tn in [(1, 1), (1, 7), (3, 5), (8, 4), (32, 32), (32, 43), (16, 16), (9, 100), (100, 9), (13, 1), (64, 3)]:
        n = tm * tn
        grid = dev.devfn_tile_order_grid(n)
        assert grid % 8 == 0 and n <= grid < n + 8
        got = np.array([dev.devfn_tile_order(b, tm, tn) for b in range(grid)], np.int64)
        have = got[got != 0xFFFFFFFF]
        assert np.array_equal(np.sort(have), np.arange(n))
        assert len(have) == n
    # one round of 256 workgroups on the 32 x 43 tiles of the 8192 x 11008 product: panels per die
    tm, tn = 32, 43
    for die in range(8):
        tiles = [dev.devfn_tile_order(die + 8 * s, tm, tn) for s in range(32)]
        rows = {t // tn for t in tiles}
        cols = {t % tn for t in tiles}
        assert len(rows) <= 8 and len(cols) <= 5, (die, sorted(rows), sorted(cols))


def test_small_gemm_plan(dev):
    """Small-tile GEMM kernel: only the tiles that exist, up to 16 wavefronts (more than 8 only with the tile whose kernel allows
    them), above four not twice as many as K has shares of 128, nor at all with more tiles than fit the chip, tile areas within the 160 KiB of LDS, and below
    129 rows the same K split for codes and for expanded operands, whose K is the pitch."""
    dev.devfn_small_plan.restype = ctypes.c_uint32
    dev.devfn_small_plan.argtypes = [ctypes.c_size_t] * 3 + [ctypes.c_int, ctypes.c_int, ctypes.POINTER(ctypes.c_uint32)]

    def plan(M, N, K, codes, sqerr=0):
        w = ctypes.c_uint32(0)
        return dev.devfn_small_plan(M, N, K, codes, sqerr, ctypes.byref(w)), w.value

    assert plan(8, 11008, 4096, 1) == (110, 8) and plan(8, 11008, 520, 1) == (110, 8) and plan(8, 11008, 512, 1) == (110, 4)
    assert plan(32, 200000, 64, 1) == (220, 1) and plan(32, 200000, 129, 1)[1] == 2 and plan(8, 8, 0, 1) == (110, 4)
    assert plan(32, 16384, 1024, 1) == (240, 8) and plan(128, 8192, 512, 0) == (220, 4) and plan(128, 8192, 513, 0) == plan(128, 8192, 512, 0, 1) == (240, 4)
    assert plan(32, 32768, 11008, 1) == (240, 8) and plan(32, 20480, 11008, 1) == (220, 4)
    rng = np.random.default_rng(4)
    for _ in range(3000):
        M, N, K = (int(2.0 ** rng.uniform(0, 20)) for _ in range(3))
        ld = -(-K // 64) * 64
        sqerr = int(rng.integers(2))
        got = [plan(M, N, k, c, sqerr) for c, k in ((0, ld), (1, K))]
        for codes, (t, w) in enumerate(got):
            tm, tn = t // 100, t // 10 % 10
            assert t in (110, 120, 220, 240, 440) and w in (1, 2, 4, 8, 16) and (w <= 8 or t == 220)
            per_simd = {1: 6, 2: 5, 4: 4, 8: 2 if codes else 3, 16: 2}[tm * tn]  # wavefronts, by the kernels' registers
            assert 512 + w * (tm + tn) * 2048 <= 160 * 1024
            tiles = -(-M // (16 * tm)) * -(-N // (16 * tn))
            assert w <= 4 or w // 2 < -(-ld // 128)
            assert w == 1 or tiles <= 256 * min(4 * per_simd // w, 160 * 1024 // (512 + w * (tm + tn) * 2048)) or w // 2 < -(-ld // 128)
            assert w >= min(4, -(-ld // 128))  # every share of K has a wavefront, up to the least full number of them
        if min(M, N) <= 128:  # the same tile and the same K split: an equal number, or the shares one by one in both
            assert got[0][0] == got[1][0] and (got[0][1] == got[1][1] or min(got[0][1], got[1][1]) >= -(-ld // 128))


def test_small_gemm_choice(dev):
    """Only tiles that are built, lanes and LDS within a launch's limits, wavefronts with a share of K; up to 128 rows one K split for codes and expanded
    operands, and above it the codes can be asked for the expanded operands' split; the squared error's split that of the stored product; small_problem()'s products stay, and what the workspace takes
    from the codes is what the expanded operands would take to the same kernel."""
    f, route, waves_of = dev.devfn_small_choice, dev.devfn_small_route, dev.devfn_small_codes_waves
    f.restype, f.argtypes = ctypes.c_uint32, [ctypes.c_size_t] * 3 + [ctypes.c_int, ctypes.c_int, ctypes.c_uint32, ctypes.POINTER(ctypes.c_uint32)]
    route.restype, route.argtypes = ctypes.c_int, [ctypes.c_size_t] * 3 + [ctypes.c_int, ctypes.c_int]
    waves_of.restype, waves_of.argtypes = ctypes.c_uint32, [ctypes.c_size_t] * 3
    small = dev.devfn_small_problem
    small.restype, small.argtypes = ctypes.c_int, [ctypes.c_size_t] * 3 + [ctypes.c_int, ctypes.c_int]

    def plan(M, N, K, codes, asked=0, sqerr=0):
        w = ctypes.c_uint32(0)
        return f(M, N, K, codes, sqerr, asked, ctypes.byref(w)), w.value

    assert plan(48, 10642, 8528, 1) == (340, 8) and plan(42, 816, 3693, 1)[0] == 110 and plan(64, 11008, 4096, 1) == (430, 8) and plan(32, 11008, 4096, 1) == (230, 8)
    tiles = (110, 120, 130, 220, 230, 240, 340, 430, 440)
    rng = np.random.default_rng(6)
    seen = set()
    for i in range(4000):
        M, N, K = (int(2.0 ** rng.uniform(0, 20 if i % 4 == 0 else 13)) for _ in range(3))
        ld = -(-K // 64) * 64
        got = [plan(M, N, k, c) for c, k in ((0, ld), (1, K))]
        checked = list(got)
        if min(M, N) > 128 and got[0][1] >= 4:
            checked.append(plan(M, N, K, 1, got[0][1]))
            assert checked[-1][1] == got[0][1]
        for t, w in checked:
            tm, tn = t // 100, t // 10 % 10
            assert t in tiles and w in (1, 2, 4, 8, 9, 16) and w <= (16 if tm * tn <= 4 else 9 if tm * tn <= 8 else 8)
            assert w != 9 or (tm * tn > 4 and min(M, N) > 128)
            assert 512 + w * (tm + tn) * 2048 <= 160 * 1024 and (w <= 4 or w // 2 < -(-ld // 128))
        seen.update(t for t, w in got)
        for (_, w), codes, k in zip(got, (0, 1), (ld, K)):  # the squared error of the stored product's bits
            t, we = plan(M, N, k, codes, 0, 1)
            assert t in (110, 120, 220, 240, 440) and (we == w or min(w, we) >= -(-ld // 128)) and we <= (16 if t in (110, 120, 220) else 9 if t == 240 else 8)
        if min(M, N) <= 128:
            assert got[0][1] == got[1][1] or min(got[0][1], got[1][1]) >= -(-ld // 128)
        for codes, k in ((0, ld), (1, K)):
            # the squared error leaves the small tiles with the stored product, where both had been there
            assert route(M, N, k, codes, 1) == (small(M, N, k, codes, 1) and (route(M, N, k, codes, 0) or not small(M, N, k, codes, 0)))
            if min(M, N) <= (32 if codes else 128) or k < 320 or -(-M // 128) * -(-N // 128) > (512 if codes else 256):
                assert route(M, N, k, codes, 0) == small(M, N, k, codes, 0)
            assert route(M, N, k, codes, 0) or not codes or not small(M, N, k, codes, 0)
        if min(M, N) > 128 and waves_of(M, N, K):
            assert waves_of(M, N, K) == got[0][1] >= 4
    assert seen == set(tiles)
    # both sides of the routes' lines: small tiles, tiled
    for codes, yes, no in ((1, [(370, 1071, 6608), (512, 3328, 4096)], [(1000, 7514, 5136), (512, 10419, 3392), (700, 4177, 5136), (1428, 2166, 3792)]),
                           (0, [(200, 594, 4224), (512, 1000, 8000), (300, 520, 4096)], [(512, 2006, 4096), (256, 3163, 2048), (256, 10456, 4672), (520, 2578, 9920)])):
        assert all(route(*x, codes, 0) for x in yes) and not any(route(*x, codes, 0) for x in no)
    assert all(small(*x, 0, 1) and not route(*x, 0, 1) for x in ((512, 2006, 4096), (700, 1227, 4096), (512, 2006, 8000))) and route(512, 1000, 8000, 0, 1)
    assert [plan(509, 1003, k, 1) for k in (2049, 2200, 2304, 3100)] == [(240, 9)] * 4 and all(plan(509, 1003, k, 1)[1] == 8 for k in (1024, 2048, 2305, 4100)) and plan(509, 1003, 2049, 1, 0, 1)[1] == 9
    assert waves_of(130, 900, 2730) and not waves_of(1000, 1000, 100000)


def test_small_gemm_route_brings_its_plan(dev):
    """What the route says and what it took to say so: the plan of the kernel that is launched, so that a call searches once (and once more for the codes'
    plan, where a product through the workspace is taken from them)."""
    f, choice, route = dev.devfn_small_route_plan, dev.devfn_small_choice, dev.devfn_small_route
    f.restype, f.argtypes = ctypes.c_uint32, [ctypes.c_size_t] * 3 + [ctypes.c_int, ctypes.c_int, ctypes.POINTER(ctypes.c_uint32)]
    choice.restype, choice.argtypes = ctypes.c_uint32, [ctypes.c_size_t] * 3 + [ctypes.c_int, ctypes.c_int, ctypes.c_uint32, ctypes.POINTER(ctypes.c_uint32)]
    route.restype, route.argtypes = ctypes.c_int, [ctypes.c_size_t] * 3 + [ctypes.c_int, ctypes.c_int]
    rng = np.random.default_rng(12)
    seen = set()
    for i in range(4000):
        M, N, K = (int(2.0 ** rng.uniform(0, 20 if i % 4 == 0 else 13)) for _ in range(3))
        codes, sqerr = i // 4 % 2, i // 8 % 2
        k = K if codes else -(-K // 64) * 64
        w, want = ctypes.c_uint32(0), ctypes.c_uint32(0)
        t = f(M, N, k, codes, sqerr, ctypes.byref(w))
        assert (t != 0) == route(M, N, k, codes, sqerr)
        if t:
            assert (t, w.value) == (choice(M, N, k, codes, sqerr, 0, ctypes.byref(want)), want.value)
        seen.add((codes, sqerr, t != 0))
    assert len(seen) == 8
    took, search = dev.devfn_small_route_ns, dev.devfn_small_choice_ns
    for g in (took, search):
        g.restype, g.argtypes = ctypes.c_double, [ctypes.c_size_t] * 3 + [ctypes.c_int, ctypes.c_int]
    for M, N, K, codes, most in ((40, 600, 400, 1, 1.7), (700, 700, 704, 1, 1.7), (509, 1003, 2112, 1, 1.7), (200, 400, 512, 0, 2.8), (700, 700, 704, 0, 2.8)):
        assert any(took(M, N, K, codes, 30) <= most * search(M, N, K, codes, 30) for _ in range(5))  # the machine may be busy


# (M, N, K) measured faster in small tiles, then those measured faster in the tiled kernels, in the kernels' own time
SMALL_OR_TILED = {
    ("codes", "store"): ([(8, 11008, 4096), (1, 200000, 16), (32, 8192, 64), (32, 200000, 64), (64, 8000, 64), (128, 8192, 64), (512, 2048, 64),
                          (64, 24000, 512), (128, 11008, 256), (256, 6656, 1024), (512, 3328, 4096), (509, 1003, 2048), (1024, 1664, 11008)],
                         [(64, 32000, 64), (128, 10240, 64), (512, 2560, 64), (1024, 1280, 64), (256, 10240, 1024), (512, 5120, 4096),
                          (2048, 11008, 4096), (256, 10240, 256)]),
    ("codes", "sqerr"): ([(8, 2000, 16), (8, 10240, 256), (8, 32000, 512), (8, 200000, 256), (32, 10240, 64), (32, 20480, 512), (64, 2000, 128),
                          (64, 10240, 512), (128, 8192, 512), (256, 4096, 512), (1024, 1024, 512), (64, 20480, 1024)],
                         [(8, 32000, 64), (16, 20480, 128), (32, 32000, 64), (64, 8000, 64), (64, 32000, 512), (128, 8000, 128),
                          (512, 2000, 128), (1024, 1280, 256)]),
    ("expanded", "store"): ([(8, 11008, 4096), (16, 200000, 64), (32, 8000, 64), (32, 20480, 1024), (32, 81920, 4096), (64, 8000, 512),
                             (64, 10240, 4096), (128, 2560, 512), (128, 8192, 4096), (256, 4096, 2048), (512, 2048, 4096), (1024, 1024, 4096)],
                            [(128, 11008, 4096), (64, 32000, 4096), (100, 20000, 512),
                             (256, 512, 64), (256, 2000, 512), (512, 967, 128), (512, 2560, 4096), (1000, 1153, 256), (1024, 1280, 4096)]),
    ("expanded", "sqerr"): ([(8, 512, 64), (8, 8000, 1024), (8, 10240, 2048), (16, 81920, 4096), (32, 4096, 512), (32, 10240, 4096),
                             (64, 2048, 1024), (128, 2560, 2048), (192, 1706, 2048), (512, 2048, 4096)],
                            [(8, 8000, 64), (16, 32000, 1024), (32, 20480, 1024), (64, 8000, 512), (64, 10240, 1024), (128, 8000, 1024),
                             (256, 2000, 512), (512, 2560, 4096), (1000, 1153, 256)]),
}


@pytest.mark.parametrize("operands,out", list(SMALL_OR_TILED))
def test_small_gemm_route(dev, operands, out):
    f = dev.devfn_small_problem
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_size_t] * 3 + [ctypes.c_int, ctypes.c_int]
    for want, shapes in zip((1, 0), SMALL_OR_TILED[operands, out]):
        for M, N, K in shapes:
            assert f(M, N, K, operands == "codes", out == "sqerr") == want, (M, N, K)
            assert f(N, M, K, operands == "codes", out == "sqerr") == want, (N, M, K)
    assert f(32, 1 << 30, 1 << 20, operands == "codes", out == "sqerr") == 1 and f(7, 9, 0, operands == "codes", out == "sqerr") == 1


@pytest.mark.parametrize("target", [32768.0, 1.0, 240.0, 3e38, 1e-38])
def test_scale_of_a_sample_holds_where_the_whole_gives_the_same(dev, target):
    """Never where the whole tensor's amax gives another scale; always where nothing lies above the sample, zeros, Inf and NaN among
    it; false for a part that contains the sample only where it is false for the whole."""
    dev.devfn_sample_holds.argtypes = [ctypes.c_uint32, ctypes.c_uint32, ctypes.c_float, ctypes.c_void_p]
    rng = np.random.default_rng(5)
    edge = [0, 1, 2, 3, 0x007FFFFF, 0x00800000, 0x00800001, 0x3F7FFFFF, 0x3F800000, 0x3F800001, 0x7F000000, 0x7F7FFFFF, 0x7F800000, 0x7F800001, 0x7FFFFFFF]
    near = [int(p) for e in rng.integers(0, 255, 12) for p in ((e << 23) - 1, e << 23, (e << 23) + 1) if p >= 0]
    some = sorted(set(edge + near + [int(x) for x in rng.integers(0, 0x7FC00000, 25)]))
    scales = [np.float32(orc.scale_from_amax(np.uint32(u).view(np.float32), target, True)) for u in some]
    got = ctypes.c_float()
    for i, s in enumerate(some):
        held = []
        for j in range(i, len(some)):
            held.append(dev.devfn_sample_holds(s, some[j], target, ctypes.byref(got)))
            assert np.float32(got.value) == scales[i]
            assert not held[-1] or scales[j] == scales[i], (hex(s), hex(some[j]))
        assert held[0] and held == sorted(held, reverse=True), hex(s)
        # a sample that gives a scale by the rule holds up to the amax at which the scale changes
        if 0 < s < 0x7F800000 and scales[i] != 1:
            assert all(h or scales[j] != scales[i] for h, j in zip(held, range(i, len(some)))), hex(s)


@pytest.mark.parametrize("tiles", [64, 65, 72, 84, 91, 92, 127, 128, 130, 700, 1028])
def test_every_tensor_that_is_not_read_whole_is_sampled(dev, tiles):
    """Wherever a tensor begins in the list, steps of a period meet it, and the pieces that are read there lie inside it, apart from
    each other, a sixteenth of it at most and a piece more."""
    dev.devfn_sampled_piece.restype, dev.devfn_sampled_piece.argtypes = ctypes.c_uint64, [ctypes.c_uint64] * 2
    period = dev.devfn_sample_period()
    assert period <= tiles
    for first in [*range(period), (1 << 40) + 1]:
        steps = range((first + period - 1) // period * period, first + tiles, period)
        assert sum(s - first < period for s in steps) == 1  # the first step that meets it, and no other
        at = [dev.devfn_sampled_piece(s - first, tiles) for s in steps]
        assert at and at[0] + 4 <= tiles and at[-1] + 4 <= tiles
        assert all(b - a >= 4 for a, b in zip(at[:-1], at[1:-1])) and 4 * len(at) <= tiles // 16 + 4


def test_small_gemm_shares_split_cache_lines_only_where_that_shortens_the_longest(dev):
    """Shares of K are counted in units of 64, half a cache line of codes, only where the wavefront with the most then has less to do than in
    pairs of units; each way deals out every unit once."""
    f = dev.devfn_small_by_pairs
    f.argtypes = [ctypes.c_size_t, ctypes.c_uint32]
    for waves in (1, 2, 4, 8, 16):
        for K in [*range(1, 5000, 37), 4096, 11008, 1 << 20, (1 << 32) - 64]:
            units = (K + 63) // 64
            bounds = lambda shares, size: [min(units, shares * w // waves * size) for w in range(waves + 1)]
            single, pairs = bounds(units, 1), bounds(units - units // 2, 2)
            assert single[0] == pairs[0] == 0 and single[-1] == pairs[-1] == units
            longest = lambda at: max(b - a for a, b in zip(at, at[1:]))
            if f(K, waves):
                assert longest(pairs) <= longest(single)
            else:
                assert longest(single) < longest(pairs) or units % 2 == 1, (K, waves)
    assert f(11008, 8) and f(4096, 8) and not f(2049, 8)


def test_multi_cast_ways(dev):
    """By sample only where the scales are powers of two and the list is worth it; not under the rounding methods for gradients, whose samples
    miss the largest values, unless the tensors are small and sampled whole; very many tiny tensors in four launches."""
    f = dev.devfn_multi_cast_way
    f.argtypes = [ctypes.c_size_t, ctypes.c_uint64, ctypes.c_int, ctypes.c_int, ctypes.c_uint32]
    SAMPLE, GROUPS, FOUR = range(3)
    ta, hr, te, ssr, sr = (orc.RM_TA, orc.RM_HR, orc.RM_TE, orc.RM_SSR, orc.RM_SR)
    for mode in (ta, hr, te, ssr, sr):
        for flags in (0, orc.FLAG_SAT, orc.FLAG_SAT | orc.FLAG_NAN2ZERO):
            m = mode | flags
            assert f(29, 114816, 1, 0, m) == GROUPS and f(29, 114816, 0, 0, m) == FOUR  # any scale
            assert f(64, 0, 1, 1, m) == GROUPS and f(64, 0, 0, 1, m) == FOUR  # empty tensors only
            assert f(29, 114816, 1, 1, m) == (GROUPS if mode in (hr, ssr, sr) else SAMPLE)
            assert f(29, 114816, 0, 1, m) == (FOUR if mode in (hr, ssr, sr) else SAMPLE)
            assert f(144, 144 * 72, 1, 1, m) == (FOUR if mode in (hr, ssr, sr) else SAMPLE)
            assert [f(100, t, 1, 1, m) for t in (3200, 3201)] == [SAMPLE, FOUR if mode in (hr, ssr, sr) else SAMPLE]
            assert [f(c, 2 * c - 1, h, 1, m) for c in (4096, 4097) for h in (0, 1)] == [SAMPLE, SAMPLE, FOUR, FOUR] and f(5000, 10000, 1, 1, m) == SAMPLE
            assert f(63, 1535, 0, 1, m) == FOUR and f(63, 1536, 0, 1, m) == f(63, 1600, 0, 1, m) == SAMPLE
            assert f(63, 1999, 1, 1, m) == GROUPS and f(63, 63, 1, 1, m) == GROUPS and f(64, 64, 1, 1, m) == SAMPLE
    assert f(63, 3071, 1, 1, ta) == GROUPS and f(63, 3072, 1, 1, ta) == SAMPLE


@pytest.mark.parametrize("tm,tn", [(1, 1), (3, 5), (4, 8), (5, 1), (8, 32), (13, 7), (43, 16), (8, 58), (64, 3), (32, 8), (40, 13), (16, 43), (100, 9)])
def test_gemm_tile_order_of_paired_tiles(dev, tm, tn):
    """Every tile once, and the 32 workgroups that run together on a die within as few groups of 4 tile rows as a walk along the groups
    allows: a compact block, where a group has eight columns or more 4 rows by 9 columns at most but for the seam between two groups."""
    dev.devfn_tile_order_paired.restype, dev.devfn_tile_order_paired.argtypes = ctypes.c_uint32, [ctypes.c_uint32] * 3
    grid = (tm * tn + 7) // 8 * 8
    got = [dev.devfn_tile_order_paired(b, tm, tn) for b in range(grid)]
    assert sorted(t for t in got if t != 0xFFFFFFFF) == list(range(tm * tn))
    for die in range(8):
        mine = [t for t in got[die::8] if t != 0xFFFFFFFF]
        for at in range(0, len(mine) - 31, 32):
            run = mine[at:at + 32]
            groups = sorted({t // tn // 4 for t in run})
            assert len(groups) <= 1 + -(-31 // (4 * tn)), (tm, tn, die, at)
            if tn >= 8:
                parts = [[t for t in run if t // tn // 4 == g] for g in groups]
                for part in parts:
                    rows, cols = {t // tn for t in part}, {t % tn for t in part}
                    whole = min(4, tm - 4 * (part[0] // tn // 4))  # the last group may have fewer rows
                    assert len(rows) <= 4 and len(cols) <= -(-len(part) // whole) + 1


# sum of rounds of a launch by the kernel it starts (tile, LDS stages): the measured times behind the rule, relative to each other
# from K = 1024 on, below it in tenths of a us by output (0: 16-bit, 1: binary32, 2: squared error) and K
def launch_price(tile, stages, tiles, cus, K, kind, pairs, edges):
    rnd = [130, 100, 76, 62, 40]
    if K < 1024 and pairs == 1:
        out = ([90, 70, 35, 32, 38], [125, 95, 60, 45, 42], [156, 125, 84, 55, 60])[kind]
        rnd = [o + -(-K // 64) * p // 10 for o, p in zip(out, (111, 87, 68, 59, 34))]
        rnd[0] += 40 if kind == 2 and edges else 0
    if tile != 2:
        assert stages == 2
        return -(-tiles // cus) * rnd[tile]
    if stages == 4:
        assert tiles <= cus  # a compute unit holds one workgroup of this form
        return rnd[4]
    rest = tiles % (2 * cus)
    return tiles // (2 * cus) * rnd[2] + (0 if rest == 0 else rnd[3] if rest <= cus else rnd[2])


def tile_count(tile, M, N, pairs):
    bm, bn = ((256, 256), (256, 192), (128, 128))[tile]
    return -(-M // bm) * -(-N // bn) * pairs


@pytest.fixture(scope="module")
def tile_launches(dev):
    dev.devfn_tile_launches.restype = ctypes.c_int
    dev.devfn_tile_launches.argtypes = [ctypes.c_size_t] * 5 + [ctypes.c_int, ctypes.POINTER(ctypes.c_uint32)]

    def launches(M, N, pairs=1, cus=256, K=4096, kind=0):
        out = (ctypes.c_uint32 * 8)()
        return [tuple(out[4 * i:4 * i + 4]) for i in range(dev.devfn_tile_launches(M, N, K, pairs, cus, kind, out))]
    return launches


def test_gemm_tile_plan(tile_launches):
    """Launches of the expanded-operand GEMM: they cover the columns; priced by the kernels they start, none of the single tiles
    in its best form has a shorter sum of rounds; and a split is shorter than all of them by its second launch at least."""
    assert [l[0] for l in tile_launches(4096, 4096)] == [0] and [l[0] for l in tile_launches(2048, 11008)] == [1]
    assert [l[0] for l in tile_launches(2048, 4096)] == [2] and [l[0] for l in tile_launches(2048, 4096, 100)] == [0]
    assert tile_launches(1, 1) == [(2, 4, 0, 1)]
    assert tile_launches(8192, 11008) == [(0, 2, 0, 40 * 256), (2, 2, 40 * 256, 11008)]
    assert tile_launches(4096, 5000) == [(0, 2, 0, 4096), (2, 4, 4096, 5000)]  # 256 tiles of 128 x 128 in the remainder
    # a short K: 128 x 128 tiles hide their epilogues from each other
    assert [tile_launches(8192, 8192, K=k)[0][0] for k in (128, 256, 1024)] == [2, 2, 0]
    assert [tile_launches(4096, 4096, K=256, kind=k)[0][0] for k in (0, 1, 2)] == [2, 0, 0] and tile_launches(1500, 9000, K=128, kind=2)[0][0] == 2
    rng = np.random.default_rng(6)
    splits = 0
    shapes = [(256 * int(rng.integers(1, 33)), 64 * int(rng.integers(4, 173)), 1, 256) for _ in range(2000)]
    shapes += [(int(2.0 ** rng.uniform(0, 16)), int(2.0 ** rng.uniform(0, 16)), int(rng.choice([1, 1, 16, 100])),
                int(rng.choice([64, 256, 304]))) for _ in range(2000)]
    for M, N, pairs, cus in shapes:
        K, kind = int(rng.choice([64, 100, 448, 1000, 1024, 4096])), int(rng.integers(3))
        got = tile_launches(M, N, pairs, cus, K, kind)
        assert got[0][2] == 0 and got[-1][3] == N and all(a[3] == b[2] for a, b in zip(got, got[1:]))
        price = sum(launch_price(t, st, tile_count(t, M, end - begin, pairs), cus, K, kind, pairs, M % 256 or (end - begin) % 256) for t, st, begin, end in got)
        singles = []
        for t in range(3):
            n = tile_count(t, M, N, pairs)
            singles.append(launch_price(t, 4 if t == 2 and n <= cus else 2, n, cus, K, kind, pairs, M % 256 or N % 256))
        if len(got) == 2:
            splits += 1
            assert pairs == 1 and got[0][3] % 256 == 0 and 0 < got[0][3] < N
            assert price + (25 if K < 1024 else 10) < min(singles), (M, N, cus, got)
        else:
            assert price == min(singles), (M, N, K, kind, pairs, cus, got)
    assert splits > 50


def test_gemm_tile_forms(dev, tile_launches):
    """The kernel behind each launch of a plan: the ring for large tiles, four LDS stages where every tile has a compute unit to itself, pairs
    of 128 x 128 tiles from K = 4096 on, but only where they take no more rounds than two to a compute unit."""
    form = dev.devfn_tile_form
    form.argtypes = [ctypes.c_size_t] * 5 + [ctypes.c_int] * 3
    assert form(8192, 8192, 4096, 1, 256, 0, -1, 0) == 0 and form(2048, 11008, 4096, 1, 256, 0, -1, 0) == 0
    assert [form(2048, 4096, k, 1, 256, 0, -1, 0) for k in (64, 4032, 4096, 11008)] == [2, 2, 3, 3]
    assert [form(8192, 11008, k, 1, 256, 0, -1, 1) for k in (4032, 4096)] == [2, 3] and form(4096, 5000, 4096, 1, 256, 0, -1, 1) == 4
    # three tile rows of 170 make 510 tiles, a round of two to a compute unit, but two rows of 170 pairs more than a round of them
    assert [form(m, n * 128, 4096, 1, 256, 0, 2, 0) for m, n in ((256, 128), (256, 129), (384, 128), (384, 129), (384, 170), (384, 171), (1024, 64))] == [4, 3, 3, 2, 2, 3, 3]
    assert form(512, 640, 4096, 100, 256, 2, -1, 0) == 3  # a scale search
    # a round of 256 x 192 tiles, up to a short K
    assert [form(m, n, k, 1, 256, 0, 1, 0) for m, n, k in ((4096, 3072, 768), (4096, 3072, 832), (4096, 3073, 768))] == [2, 0, 0]
    rng = np.random.default_rng(8)
    for _ in range(3000):
        M, N, pairs, cus = int(2.0 ** rng.uniform(0, 15)), int(2.0 ** rng.uniform(0, 15)), int(rng.choice([1, 1, 16, 100])), int(rng.choice([64, 256, 304]))
        K = int(rng.choice([64, 1024, 4032, 4096, 8192]))
        for i, (tile, stages, begin, end) in enumerate(tile_launches(M, N, pairs, cus, K, 2)):
            got = form(M, N, K, pairs, cus, 2, -1, i)
            cols = -(-(end - begin) // 128) * pairs
            ones, twos = -(-M // 128) * cols, -(-M // 256) * cols
            paired = K >= 4096 and -(-twos // cus) <= -(-ones // (2 * cus))
            short = tile == 1 and K <= 768 and -(-M // 256) * -(-(end - begin) // 192) * pairs <= cus
            assert got == (2 if short else 0 if tile != 2 else 4 if stages == 4 else 3 if paired else 2)
            assert got != 4 or ones <= cus


def test_small_gemm_route_of_expanded_operands_beyond_64_x_64_tiles(dev):
    """Where 64 x 64 tiles do not have a compute unit each, the lines of small_problem() hold for expanded operands (products that the price had moved, and
    slowed down, then drawn ones)."""
    route, small = dev.devfn_small_route, dev.devfn_small_problem
    for f in (route, small):
        f.restype, f.argtypes = ctypes.c_int, [ctypes.c_size_t] * 3 + [ctypes.c_int, ctypes.c_int]
    for M, N, K in ((187, 8860, 448), (146, 10754, 768), (283, 6438, 3776), (148, 10790, 6016), (258, 4012, 1024), (582, 1998, 512), (141, 6452, 5824)):
        assert not small(M, N, K, 0, 0) and not route(M, N, K, 0, 0)
    rng = np.random.default_rng(11)
    for _ in range(4000):
        M, N, K = (int(2.0 ** rng.uniform(lo, hi)) for lo, hi in ((5, 13), (5, 14), (0, 7)))
        if -(-M // 64) * -(-N // 64) > 256:
            assert route(M, N, 64 * K, 0, 0) == small(M, N, 64 * K, 0, 0)


def test_per_channel_calls_that_go_to_the_element_kernels(dev):
    """Narrow and small matrices, both sides of each line; what the vector kernels cannot take: rows shorter than a vector, launches of 2^32 lanes and more, vectors
    that may reach over the end of a standard SR block."""
    f = dev.devfn_axis_by_elements
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int, ctypes.c_int, ctypes.c_size_t, ctypes.c_size_t, ctypes.c_size_t, ctypes.c_uint64, ctypes.c_uint32, ctypes.c_int]
    AMAX, ENCODE, DECODE, TA, HR, TE, SSR, SR, Ki, Mi = 0, 1, 2, 0, 1, 2, 3, 4, 1 << 10, 1 << 20
    # columns and values of each line, by axis, call, vectors at multiples of 16 bytes or not, and vector
    lines = {(0, ENCODE, False, 0): ((384, 640 * Ki), (320, 640 * Ki)), (0, ENCODE, False, 1): ((384, 512 * Ki), (320, 512 * Ki)),
             (0, ENCODE, True, 0): ((448, 704 * Ki), (448, 704 * Ki)), (0, ENCODE, True, 1): ((384, 512 * Ki), (288, 512 * Ki)),
             (0, DECODE, False, 0): ((1024, 3 * Mi), (640, 5 * Mi // 2)), (0, DECODE, False, 1): ((704, 704 * Ki), (512, 5 * Mi // 4)),
             (1, ENCODE, False, 0): ((48, 3 * Mi // 2), (64, 9 * Mi // 4)), (1, ENCODE, False, 1): ((48, 5 * Mi // 4), (56, 2 * Mi)),
             (1, ENCODE, True, 0): ((80, 5 * Mi // 2), (128, 13 * Mi // 4)), (1, ENCODE, True, 1): ((80, 5 * Mi // 2), (96, 3 * Mi)),
             (1, DECODE, False, 0): (None, (112, 15 * Mi // 4)), (1, DECODE, False, 1): ((80, 2 * Mi), (80, 5 * Mi // 2))}
    for ve in (4, 8):
        for what in (AMAX, ENCODE, DECODE):
            for axis in (0, 1):
                assert f(what, axis, 1 << 22, ve - 1, ve, 100, TA, 1) and f(what, axis, 1 << 23, 4096, ve, 1 << 24, TA, 1)
                assert not f(what, axis, 1 << 23, 4096, ve, (1 << 24) - 1, TA | 0x30, 1)
        # maxima: up to 32 columns by rows, 16 where there are few; by columns always in vectors
        assert f(AMAX, 0, 1 << 20, 32, ve, 1, TA, 1) and not f(AMAX, 0, 1 << 20, 33, ve, 1, TA, 1) and not f(AMAX, 1, 1 << 20, 9, ve, 1, TA, 1)
        assert f(AMAX, 0, 100, 16, ve, 1, TA, 1) and not f(AMAX, 0, 100, 17, ve, 1, TA, 1)
        for (axis, what, drawn, aligned), of in lines.items():
            line = of[ve == 8]
            for mode in (HR, SR) + (SSR,) * (axis == 0 or not aligned) if drawn else (TA, TE) + (SSR,) * (axis == 1 and aligned):
                if line is None:  # binary32 by columns at any address: elements
                    assert f(what, axis, 1 << 16, 5000, ve, 1, mode, 0) and f(what, axis, 1 << 16, 5001, ve, 1, mode, 1) and not f(what, axis, 1 << 16, 5000, ve, 1, mode, 1)
                    continue
                c, n = line
                least = -(-c // ve) * ve if aligned else c
                assert f(what, axis, 1 << 17, least - (ve if aligned else 1), ve, 1, mode, aligned) and not f(what, axis, 1 << 17, least, ve, 1, mode, aligned)
                assert f(what, axis, 1 << 17, c - 1, ve, 1, mode, 1) == f(what, axis, 1 << 17, c - 1, ve, 1, mode, aligned and (c - 1) % ve == 0)  # an odd number of columns alone
                cols = 64 * ve * 16 + 32 * ve
                assert f(what, axis, n // cols, cols, ve, 1, mode, aligned) and not f(what, axis, n // cols + 1, cols, ve, 1, mode, aligned)
        for mode in (HR, SR):  # 16 bits by columns, one vector in the last wavefront of a row
            cols, n = 64 * ve + 1, 4 * Mi if ve == 8 else 5 * Mi // 2
            assert f(ENCODE, 1, n // cols, cols, ve, 1, mode, 1) and not f(ENCODE, 1, n // cols + 1, cols, ve, 1, mode, 1)
        for mode in (TA, TE, HR, SSR, SR):
            # more than 2^32 elements: whole vectors to a row, or element by element under standard SR
            assert not f(ENCODE, 0, 1 << 21, 4096, ve, 1, mode, 1) and f(ENCODE, 0, 1 << 21, 4097, ve, 1, mode, 1) == (mode == SR) == f(ENCODE, 1, 1 << 21, 4097, ve, 1, mode | 0x10, 1)
            assert not f(ENCODE, 0, (1 << 32) // 4097, 4097, ve, 1, mode, 1)


def test_finest_tile_with_a_compute_unit_each(dev):
    f = dev.devfn_fine_tile
    f.argtypes = [ctypes.c_size_t, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_size_t, ctypes.c_size_t]
    assert [f(m, b, e, p, 256) for m, b, e, p in ((1024, 0, 1024, 1), (1024, 0, 1025, 1), (1024, 64, 1088, 1), (1025, 0, 1024, 1), (1024, 0, 2048, 1), (1024, 0, 2049, 1), (1, 0, 1, 256),
                                                 (1, 0, 1, 257), (4096, 0, 1024, 1))] == [2, 1, 2, 1, 1, 0, 2, 0, 0]
    rng = np.random.default_rng(3)
    for _ in range(1000):
        M, begin, cols, pairs, cus = (int(2 ** rng.uniform(0, 13)) for _ in range(5))
        got = f(M, begin, begin + cols, pairs, cus)
        tiles = [-(-M // m) * -(-cols // n) * pairs for m, n in ((128, 128), (128, 64), (64, 64))]
        assert (got == 0 or tiles[got] <= cus) and all(t > cus for t in tiles[got + 1:])


def test_scale_search_launches_fit(dev, tile_launches):
    """A scale search takes as many pairs in a launch as its workgroups of 256 threads, counted in 32 bits, allow (the 256 x 256
    tiles of the squared error walk: one workgroup per compute unit); a row of the search, or one pair, always fits."""
    f = dev.devfn_pairs_per_launch
    f.restype, f.argtypes = ctypes.c_uint32, [ctypes.c_int] + [ctypes.c_size_t] * 3 + [ctypes.c_uint32, ctypes.c_uint32, ctypes.c_size_t]
    assert f(-1, 2048, 4096, 4096, 10, 10, 256) == 100
    assert tile_launches(116736, 1728, 4096, K=64, kind=2)[0][0] == 1 and f(-1, 116736, 1728, 64, 64, 64, 256) == 64  # 456 x 9 x 4096 > 2^24
    assert f(2, 8256, 8256, 64, 64, 64, 256) == 64 and f(0, 8256, 8256, 64, 64, 64, 256) == 4096
    assert f(2, 600000, 7000, 64, 64, 64, 256) == 64 and f(2, 600000, 17000, 64, 64, 64, 256) == 1
    rng = np.random.default_rng(9)
    seen = set()
    for _ in range(5000):
        M, N = int(2.0 ** rng.uniform(0, 27)), int(2.0 ** rng.uniform(0, 27))
        na, nb, tile = int(rng.integers(1, 65)), int(rng.integers(1, 65)), int(rng.integers(-1, 3))
        if M * N > 7e10:  # the reference would not fit the memory
            continue
        K = int(rng.choice([64, 4096]))
        some = f(tile, M, N, K, na, nb, 256)
        assert some in (na * nb, nb, 1)
        seen.add("all" if some == na * nb else "row" if some == nb else "pair")

        def fits(pairs):
            launches = [(tile, 0, 0, N)] if tile >= 0 else tile_launches(M, N, pairs, K=K, kind=2)
            return all((t == 0 and tile_count(t, M, e - b, pairs) < 2 ** 31) or (tile_count(t, M, e - b, pairs) + 7) // 8 * 8 * 256 < 2 ** 32
                       for t, _, b, e in launches)
        assert fits(some)
        assert some == na * nb or not fits(na * nb)
    assert seen == {"all", "row", "pair"}


LLVM = "/opt/rocm/llvm/bin/"


def device_code(source, tmp_path):
    """The gfx950 code object of a built source file."""
    from paper_2409_16626_amd import build
    obj = os.path.join(build.OBJDIR, source + ".o")
    if not os.path.exists(obj):
        build.build(force=False)
    fat, code = str(tmp_path / "fat"), str(tmp_path / "code")
    subprocess.run([LLVM + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, obj, str(tmp_path / "copy.o")], check=True)
    subprocess.run([LLVM + "clang-offload-bundler", "--type=o", "--unbundle", "--input=" + fat, "--output=" + code,
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    return code


def test_walking_gemm_kernels_store_as_often_as_they_count(tmp_path):
    """The kernels that walk over tiles wait for the loads of the next tile by the number of instructions behind them: the 16-byte stores of a
    tile inside the matrix.  The built code has them once for such tiles and once, each behind its own test, for edge tiles."""
    code = device_code("hif8_gemm_x.hip", tmp_path)
    asm = subprocess.run([LLVM + "llvm-objdump", "-d", "--no-show-raw-insn", code], check=True, stdout=subprocess.PIPE, text=True).stdout
    seen = 0
    for body in re.split(r"^[0-9a-f]+ <", asm, flags=re.M):
        name = re.match(r"\w*k_gemm_xILi(\d)ELi(\d)ELi(\d)ELi0E", body)  # TA, TB, output (0 binary32, 1 and 2 16 bits, 3 squared error), ring
        if not name:
            continue
        ta, tb, epi = map(int, name.groups())
        stores = 0 if epi == 3 else 16 * ta * 16 * tb // (64 * (4 if epi == 0 else 8))
        assert len(re.findall(r"\b(?:global|flat|buffer)_store_dwordx4\b", body)) == 2 * stores, name.group(0)
        assert stores == 0 or re.search(r"s_waitcnt vmcnt\(%d\)" % min(stores, 63), body), name.group(0)
        assert "scratch_" not in body  # spills would be counted as well
        seen += 1
    assert seen == 8


def test_gemm_accumulators_are_read_behind_wait_states(tmp_path):
    """The matrix instructions of k_gemm_x are assembly, which the compiler takes for ordinary instructions: where it copied an accumulator between two of
    them, the copy would not wait for the result.  In the built code no other instruction of a basic block names the accumulators that its matrix instructions
    write, but for those behind the wait states."""
    code = device_code("hif8_gemm_x.hip", tmp_path)
    asm = subprocess.run([LLVM + "llvm-objdump", "-d", "--no-show-raw-insn", code], check=True, stdout=subprocess.PIPE, text=True).stdout

    def registers(text):
        return {k + str(i) for k, a, b, k1, one in re.findall(r"\b([av])\[(\d+):(\d+)\]|\b([av])(\d+)\b", text) for k, i in
                ([(k, i) for i in range(int(a), int(b) + 1)] if k else [(k1, int(one))])}

    seen = 0
    for body in re.split(r"^[0-9a-f]+ <", asm, flags=re.M):
        if not re.match(r"\w*k_gemm_xI", body):
            continue
        for block in re.split(r"\n[^\n]*\bs_c?branch[^\n]*", body):
            lines = [line.split("//")[0].split(None, 1) for line in block.split("s_nop 15")[0].splitlines()]
            lines = [line for line in lines if len(line) == 2]
            written = set().union(*[registers(ops.split(",")[0]) for op, ops in lines if op.startswith("v_mfma")])
            first = next((i for i, (op, _) in enumerate(lines) if op.startswith("v_mfma")), 0)
            others = [(op, ops) for op, ops in lines[first:] if not op.startswith("v_mfma") and registers(ops) & written]
            assert not others, (body[:60], others[:3])
        seen += 1
    assert seen == 36


def test_small_gemm_kernel_has_no_static_lds(tmp_path):
    """k_gemm_s looks codes up in a table at LDS address 0, the start of its dynamic LDS: static LDS would come before it."""
    code = device_code("hif8_gemm_s.hip", tmp_path)
    notes = subprocess.run([LLVM + "llvm-readelf", "--notes", code], check=True, stdout=subprocess.PIPE, text=True).stdout
    sizes = re.findall(r"\.group_segment_fixed_size:\s*(\d+)", notes)
    assert notes.count("k_gemm_s") > 0 and len(sizes) >= 40 and set(sizes) == {"0"}, sizes
