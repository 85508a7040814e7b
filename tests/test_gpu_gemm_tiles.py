"""GPU tests of the expanded-operand GEMM's tiles: every tile shape on edge tiles and unaligned rows, in every output
kind, against the fp64 oracle (bound of test_gpu_gemm.py: K * 2^-23 * sum_k |a b| * descale per element) and against its
own binary32 result; launches with more tiles than workgroups; batched pairs over every tile."""
import numpy as np
import pytest
import torch

from gpu_util import dev
from oracle import hif8_oracle as orc
from test_gpu_gemm import check, h, random_codes  # noqa: F401  (h is the fixture)
from test_gpu_gemm_expanded import expand

pytestmark = pytest.mark.gpu


# K steps 1, 2, 3, 4 and more; rows that are not 16-byte aligned (N odd), shorter than a run of four or of eight columns, one
# past and one below a block; one tile, edge tiles only, whole tiles and edge tiles; more 128 x 128 tiles than compute units (two
# LDS stages there, four in all the others); 256 x 192 tiles with two LDS stages and, from K = 833 on, in the ring
@pytest.mark.parametrize("variant", [9, 10, 11])
@pytest.mark.parametrize("M,N,K", [(5, 1, 64), (300, 3, 65), (257, 7, 130), (130, 191, 200), (511, 385, 256), (256, 192, 300), (514, 770, 400),
                                   (2100, 2300, 130), (300, 3, 833), (514, 770, 900)])
def test_tiles_every_output(h, variant, M, N, K):
    rng = np.random.default_rng(variant + M + 3 * N + 7 * K)
    ca, cb = random_codes(rng, (M, K), "cast_normal"), random_codes(rng, (N, K), "cast_normal")
    (a, ld), (b, _) = expand(h, ca), expand(h, cb)
    o32 = torch.full((M * N + 8,), 7.0, dtype=torch.float32, device=dev())
    ob, oh = (torch.full((M * N + 8,), 7.0, dtype=d, device=dev()) for d in (torch.bfloat16, torch.float16))
    h.hif8_gemm_set_variant(variant)
    for call, o in ((h.hif8_gemm_expanded_f32, o32), (h.hif8_gemm_expanded_bf16, ob), (h.hif8_gemm_expanded_f16, oh)):
        call(a, b, o, M, N, K, ld, 8.0, 8.0)
        assert torch.all(o[M * N:] == 7.0)
    out = o32[:M * N].view(M, N)
    check(out.cpu().numpy(), ca, cb, 8.0, 8.0)
    assert torch.equal(ob[:M * N].view(M, N), out.to(torch.bfloat16)) and torch.equal(oh[:M * N].view(M, N), out.to(torch.float16))
    ref = (out * 1.01 + 0.5).contiguous()
    err = torch.zeros(2, dtype=torch.float64, device=dev())
    h.hif8_gemm_expanded_sqerr(a, b, ref, M, N, K, ld, 8.0, 8.0, err)
    h.hif8_gemm_set_variant(0)
    want = float(((out.double() - ref.double()) ** 2).sum())
    assert err[1].item() == 0.0 and abs(err[0].item() - want) <= 1e-12 * want


# every length of a row's last run, of 4 binary32 and of 8 16-bit values; rows and columns that end in each quarter of a tile,
# so that whole blocks of it lie outside
@pytest.mark.parametrize("variant", [9, 10, 11])
def test_tiles_row_ends(h, variant):
    rng = np.random.default_rng(variant)
    K = 64
    full, _ = expand(h, random_codes(rng, (300, K), "cast_normal"))
    b_full, _ = expand(h, random_codes(rng, (300, K), "cast_normal"))
    want = full.view(torch.bfloat16).double() @ b_full.view(torch.bfloat16).double().t() / 64.0
    sums = full.view(torch.bfloat16).double().abs() @ b_full.view(torch.bfloat16).double().abs().t() / 64.0
    h.hif8_gemm_set_variant(variant)
    for M, N in [(40 + 37 * i, n) for i, n in enumerate((1, 2, 5, 6, 33, 58, 67))] + [(70, n) for n in range(128, 137)] + [(290, 259)]:
        o32 = torch.full((M * N + 8,), 7.0, dtype=torch.float32, device=dev())
        ob, oh = (torch.full((M * N + 8,), 7.0, dtype=d, device=dev()) for d in (torch.bfloat16, torch.float16))
        for call, o in ((h.hif8_gemm_expanded_f32, o32), (h.hif8_gemm_expanded_bf16, ob), (h.hif8_gemm_expanded_f16, oh)):
            call(full, b_full, o, M, N, K, K, 8.0, 8.0)
            assert torch.all(o[M * N:] == 7.0), (M, N)
        out = o32[:M * N].view(M, N)
        assert torch.all((out.double() - want[:M, :N]).abs() <= K * 2.0 ** -23 * sums[:M, :N]), (M, N)
        assert torch.equal(ob[:M * N].view(M, N), out.to(torch.bfloat16)) and torch.equal(oh[:M * N].view(M, N), out.to(torch.float16)), (M, N)
        ref = (out * 1.01 + 0.5).contiguous()
        err = torch.zeros(1, dtype=torch.float64, device=dev())
        h.hif8_gemm_expanded_sqerr(full, b_full, ref, M, N, K, K, 8.0, 8.0, err)
        e = float(((out.double() - ref.double()) ** 2).sum())
        assert abs(err.item() - e) <= 1e-12 * e, (M, N)
    h.hif8_gemm_set_variant(0)


# the remaining columns of a split: at most one 128 x 128 tile per compute unit (four LDS stages), and more (two)
@pytest.mark.parametrize("M,N,K", [(7290, 2238, 200), (3450, 10430, 67)])
def test_column_split_equals_one_launch(h, M, N, K):
    rng = np.random.default_rng(M)
    (a, ld), (b, _) = (expand(h, random_codes(rng, (r, K), "cast_normal")) for r in (M, N))
    got = {}
    for variant in (0, 9):
        h.hif8_gemm_set_variant(variant)
        for name, d in (("f32", torch.float32), ("bf16", torch.bfloat16), ("f16", torch.float16)):
            o = torch.full((M * N + 8,), 7.0, dtype=d, device=dev())
            getattr(h, "hif8_gemm_expanded_" + name)(a, b, o, M, N, K, ld, 4.0, 2.0)
            assert torch.all(o[M * N:] == 7.0)
            assert variant == 0 or torch.equal(o, got[name])
            got[name] = o
    h.hif8_gemm_set_variant(0)
    rows = rng.integers(0, M, 40)
    want = a[rows].view(torch.bfloat16).double() @ b.view(torch.bfloat16).double().t() / 8.0
    sums = a[rows].view(torch.bfloat16).double().abs() @ b.view(torch.bfloat16).double().abs().t() / 8.0
    assert torch.all((got["f32"][:M * N].view(M, N)[rows].double() - want).abs() <= K * 2.0 ** -23 * sums)


# more tiles of 256 columns or 192 than compute units: workgroups that walk over several, inside the matrix and at its edges, rows
# that are not 16-byte aligned, K steps 1 to 5 (the first loads of a tile go out before the stores of the one before it)
@pytest.mark.parametrize("variant", [10, 11])
@pytest.mark.parametrize("M,N,K", [(4100, 5001, 64), (4100, 5001, 128), (4352, 4608, 192), (4100, 5001, 250), (8200, 4096, 320)])
def test_walk_over_tiles_equals_small_tiles(h, variant, M, N, K):
    rng = np.random.default_rng(variant + K)
    (a, ld), (b, _) = (expand(h, random_codes(rng, (r, K), "cast_normal")) for r in (M, N))
    for name, d in (("f32", torch.float32), ("bf16", torch.bfloat16), ("f16", torch.float16)):
        got = []
        for v in (9, variant):
            o = torch.full((M * N + 8,), 7.0, dtype=d, device=dev())
            h.hif8_gemm_set_variant(v)
            getattr(h, "hif8_gemm_expanded_" + name)(a, b, o, M, N, K, ld, 4.0, 2.0)
            h.hif8_gemm_set_variant(0)
            assert torch.all(o[M * N:] == 7.0)
            got.append(o)
        assert torch.equal(got[0], got[1]), name


# 128 x 128 tiles in pairs (256 x 128) from K = 4096 on, more than a round and part of one, edge tiles and whole ones: the same bits as in
# 256 x 256 tiles, and a score of them
@pytest.mark.parametrize("M,N,K", [(2048, 2304, 4096), (2100, 2301, 4100), (4400, 4203, 4096)])
def test_paired_tiles_equal_large_tiles(h, M, N, K):
    rng = np.random.default_rng(M)
    (a, ld), (b, _) = (expand(h, random_codes(rng, (r, K), "cast_normal")) for r in (M, N))
    got = {}
    for v in (9, 10):
        h.hif8_gemm_set_variant(v)
        for name, d in (("f32", torch.float32), ("bf16", torch.bfloat16), ("f16", torch.float16)):
            o = torch.full((M * N + 8,), 7.0, dtype=d, device=dev())
            getattr(h, "hif8_gemm_expanded_" + name)(a, b, o, M, N, K, ld, 4.0, 2.0)
            assert torch.all(o[M * N:] == 7.0)
            assert v == 9 or torch.equal(got[name], o), name
            got[name] = o
        out = got["f32"][:M * N]
        ref = (out * 1.01 + 0.5).contiguous()
        err = torch.zeros(1, dtype=torch.float64, device=dev())
        h.hif8_gemm_expanded_sqerr(a, b, ref, M, N, K, ld, 4.0, 2.0, err)
        h.hif8_gemm_set_variant(0)
        want = float(((out.double() - ref.double()) ** 2).sum())
        assert abs(err.item() - want) <= 1e-12 * want


# codes in 256 x 256 and 128 x 128 tiles, expanded operands in 128 x 128, 256 x 256 and 256 x 192, both in small tiles; whole runs
# of a row and shorter ones.  Sums of small integers are exact, so a result is one binary32 product and one rounding to 16 bits.
@pytest.mark.parametrize("operands,variant", [("codes", 5), ("codes", 6), ("codes", 12), ("expanded", 9), ("expanded", 10), ("expanded", 11),
                                              ("expanded", 12)])
def test_results_below_the_normal_range(h, operands, variant):
    rng = np.random.default_rng(variant)
    M, N, K = 140, 267, 192
    vals = np.array([0x00, 0x08, 0x10, 0x14, 0x20, 0x88, 0x90], np.uint8)  # 0, 1, 2, 3, 4, -1, -2
    ca, cb = rng.choice(vals, size=(M, K)), rng.choice(vals, size=(N, K))
    v = np.array([orc.decode_value(c) if np.isfinite(orc.decode_value(c)) else 0.0 for c in range(256)], np.float64)
    sums = torch.from_numpy((v[ca] @ v[cb].T).astype(np.float32))
    if operands == "codes":
        a, b, ld = torch.from_numpy(ca).to(dev()), torch.from_numpy(cb).to(dev()), ()
    else:
        (a, ld), (b, _) = expand(h, ca), expand(h, cb)
        ld = (ld,)
    prefix = "hif8_gemm_" if operands == "codes" else "hif8_gemm_expanded_"
    h.hif8_gemm_set_variant(variant)
    for name, dtype, ea, eb in (("bf16", torch.bfloat16, 66, 68), ("bf16", torch.bfloat16, 66, 70), ("bf16", torch.bfloat16, 70, 71),
                                ("f32", torch.float32, 70, 74), ("f16", torch.float16, 10, 12), ("f16", torch.float16, 14, 17)):
        out = torch.full((M, N), 7.0, dtype=dtype, device=dev())
        getattr(h, prefix + name)(a, b, out, M, N, K, *ld, 2.0 ** ea, 2.0 ** eb)
        want = (sums * torch.tensor(2.0 ** -(ea + eb), dtype=torch.float32)).to(dtype)
        assert torch.equal(out.cpu(), want), (name, ea, eb)
        least = torch.finfo(dtype).tiny
        assert ((want != 0) & (want.float().abs() < least)).float().mean() > 0.1
    h.hif8_gemm_set_variant(0)


@pytest.mark.parametrize("variant", [9, 10, 11])
def test_tiles_nan_and_inf(h, variant):
    """A NaN of either operand reaches its row or column only, as 0x7FC0 in bfloat16, and nothing past the edge of a tile."""
    rng = np.random.default_rng(3)
    M, N, K = 300, 270, 128
    ca, cb = random_codes(rng, (M, K), "cast_normal"), random_codes(rng, (N, K), "cast_normal")
    ca[7, 3], cb[100, 70], cb[269, 5] = 0x80, 0x80, 0x6F
    (a, ld), (b, _) = expand(h, ca), expand(h, cb)
    o32, ob = (torch.zeros(M, N, dtype=d, device=dev()) for d in (torch.float32, torch.bfloat16))
    ref, err = torch.zeros(M, N, device=dev()), torch.zeros(1, dtype=torch.float64, device=dev())
    h.hif8_gemm_set_variant(variant)
    h.hif8_gemm_expanded_f32(a, b, o32, M, N, K, ld, 1.0, 1.0)
    h.hif8_gemm_expanded_bf16(a, b, ob, M, N, K, ld, 1.0, 1.0)
    h.hif8_gemm_expanded_sqerr(a, b, ref, M, N, K, ld, 1.0, 1.0, err)
    h.hif8_gemm_set_variant(0)
    nan = torch.isnan(o32)
    want = torch.zeros(M, N, dtype=torch.bool, device=dev())
    want[7], want[:, 100] = True, True
    want[torch.from_numpy(np.isin(ca[:, 5], [0x00])).to(dev()), 269] = True  # 0 * Inf
    assert torch.equal(nan, want)
    assert torch.all(ob.view(torch.int16)[nan] == 0x7FC0) and torch.isnan(err).item()


def test_squared_error_of_more_tiles_than_workgroups(h):
    """The workgroups of the squared error walk over tiles: 17 x 18 tiles of 256 x 256, edges on both sides."""
    rng = np.random.default_rng(8)
    M, N, K = 4200, 4503, 192
    (a, ld), (b, _) = (expand(h, random_codes(rng, (r, K), "cast_normal")) for r in (M, N))
    out = torch.empty(M, N, dtype=torch.float32, device=dev())
    h.hif8_gemm_set_variant(10)
    h.hif8_gemm_expanded_f32(a, b, out, M, N, K, ld, 2.0, 4.0)
    ref = out + torch.randn(M, N, device=dev(), generator=torch.Generator(device=dev()).manual_seed(1))
    err = torch.zeros(1, dtype=torch.float64, device=dev())
    h.hif8_gemm_expanded_sqerr(a, b, ref, M, N, K, ld, 2.0, 4.0, err)
    h.hif8_gemm_set_variant(0)
    want = float(((out.double() - ref.double()) ** 2).sum())
    assert abs(err.item() - want) <= 1e-12 * want


@pytest.mark.parametrize("variant", [9, 10, 11])
def test_scale_search_over_every_tile(h, variant):
    """Every pair of a 10 x 7 search meets its own operands, scale and place in the table (edge tiles; with 256 x 256 tiles
    420 tiles on at most 256 workgroups): each entry against the same product made alone."""
    search_against_products_alone(h, variant, 300, 520, 130, 10, 7)


# 24 tiles of 64 x 64 (a single chain over K, and a part of K every two steps) and 162 of 128 x 64, whose 64 x 64 tiles would be more than the compute units
@pytest.mark.parametrize("M,N,K,na,nb", [(65, 40, 130, 4, 3), (65, 40, 1100, 4, 3), (128, 130, 200, 9, 6)])
def test_scale_search_in_the_finest_tiles(h, M, N, K, na, nb):
    search_against_products_alone(h, 9, M, N, K, na, nb)


def search_against_products_alone(h, variant, M, N, K, na, nb):
    rng = np.random.default_rng(5)
    x = torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)).to(dev())
    w = torch.from_numpy((rng.standard_normal((N, K)) * 0.02).astype(np.float32)).to(dev())
    ref = (x.double() @ w.double().t()).float()
    ws = torch.empty(h.hif8_calibrate_workspace_bytes(M, N, K, na, nb), dtype=torch.uint8, device=dev())
    err = torch.full((na, nb), -1.0, dtype=torch.float64, device=dev())
    best = torch.zeros(2, dtype=torch.int32, device=dev())
    h.hif8_gemm_set_variant(variant)
    h.hif8_calibrate_layer_f32(x, w, ref, M, N, K, -3, na, -2, nb, orc.RM_TA, ws, ws.numel(), err, best)
    one = torch.zeros(na, nb, dtype=torch.float64, device=dev())
    ld = h.hif8_expanded_ld(K)
    cast = []
    for t, rows, lo, count in ((x, M, -3, na), (w, N, -2, nb)):
        codes, xs = torch.empty(rows, K, dtype=torch.uint8, device=dev()), torch.zeros(count, rows, ld, dtype=torch.bfloat16, device=dev())
        for i in range(count):
            h.hif8_encode_f32(t, codes, rows * K, 2.0 ** (lo + i), orc.RM_TA)
            h.hif8_expand_bf16(codes, rows, K, xs[i], ld)
        cast.append(xs)
    for i in range(na):
        for j in range(nb):
            h.hif8_gemm_expanded_sqerr(cast[0][i], cast[1][j], ref, M, N, K, ld, 2.0 ** (-3 + i), 2.0 ** (-2 + j), one[i, j:])
    h.hif8_gemm_set_variant(0)
    assert torch.all((err - one).abs() <= 1e-12 * one)
    at = int(one.argmin())
    assert best.tolist() == [-3 + at // nb, -2 + at % nb]


@pytest.mark.parametrize("M,N,K", [(512, 640, 4096), (700, 900, 4100)])
def test_scale_search_in_paired_tiles(h, M, N, K):
    """A search whose plan takes 256 x 128 tiles: every pair against the same product made alone in 256 x 256 tiles."""
    rng = np.random.default_rng(6)
    na, nb = 10, 10
    x = torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)).to(dev())
    w = torch.from_numpy((rng.standard_normal((N, K)) * 0.02).astype(np.float32)).to(dev())
    ref = (x.double() @ w.double().t()).float()
    ws = torch.empty(h.hif8_calibrate_workspace_bytes(M, N, K, na, nb), dtype=torch.uint8, device=dev())
    best = torch.zeros(2, dtype=torch.int32, device=dev())
    got = {}
    for variant in (0, 9, 10):
        h.hif8_gemm_set_variant(variant)
        err = torch.full((na, nb), -1.0, dtype=torch.float64, device=dev())
        h.hif8_calibrate_layer_f32(x, w, ref, M, N, K, -4, na, -4, nb, orc.RM_TA, ws, ws.numel(), err, best)
        got[variant] = err
    ld = h.hif8_expanded_ld(K)
    one = torch.zeros(na, nb, dtype=torch.float64, device=dev())
    cast = []
    for t, rows in ((x, M), (w, N)):
        codes, xs = torch.empty(rows, K, dtype=torch.uint8, device=dev()), torch.zeros(10, rows, ld, dtype=torch.bfloat16, device=dev())
        for i in range(10):
            h.hif8_encode_f32(t, codes, rows * K, 2.0 ** (-4 + i), orc.RM_TA)
            h.hif8_expand_bf16(codes, rows, K, xs[i], ld)
        cast.append(xs)
    h.hif8_gemm_set_variant(10)
    for i in range(na):
        for j in range(nb):
            h.hif8_gemm_expanded_sqerr(cast[0][i], cast[1][j], ref, M, N, K, ld, 2.0 ** (-4 + i), 2.0 ** (-4 + j), one[i, j:])
    h.hif8_gemm_set_variant(0)
    for err in got.values():
        assert torch.all((err - one).abs() <= 1e-12 * one)


def test_scale_search_of_more_tiles_than_a_launch_has(h):
    """65 x 65 tiles of 128 x 128 for 64 x 64 pairs are more workgroups of 256 threads than 32 bits count: the search goes row by
    row.  Against the walking form in 256 x 256 tiles, which takes them in one launch."""
    M, N, K, n = 8256, 8256, 40, 64
    g = torch.Generator(device=dev()).manual_seed(11)
    x, w = torch.randn(M, K, device=dev(), generator=g), torch.randn(N, K, device=dev(), generator=g) * 0.02
    ref = (x.double() @ w.double().t()).float()
    ws = torch.empty(h.hif8_calibrate_workspace_bytes(M, N, K, n, n), dtype=torch.uint8, device=dev())
    got = {}
    for variant in (9, 10):
        err = torch.full((n, n), -1.0, dtype=torch.float64, device=dev())
        best = torch.zeros(2, dtype=torch.int32, device=dev())
        h.hif8_gemm_set_variant(variant)
        h.hif8_calibrate_layer_f32(x, w, ref, M, N, K, -32, n, -32, n, orc.RM_TA, ws, ws.numel(), err, best)
        torch.cuda.synchronize()
        got[variant] = (err, best)
    h.hif8_gemm_set_variant(0)
    fin = torch.isfinite(got[10][0])  # large scales overflow to infinity, and 0 * infinity is NaN
    assert fin.sum() > 1000 and torch.equal(torch.isnan(got[9][0]), torch.isnan(got[10][0]))
    assert torch.all((got[9][0] - got[10][0]).abs()[fin] <= 1e-12 * got[10][0][fin])
    for err, best in got.values():  # many scales cast to the same bits: the least entry of its own table
        at = int(torch.where(torch.isfinite(err), err, float("inf")).argmin())
        assert best.tolist() == [-32 + at // n, -32 + at % n]


# every rounding method on every kind of source: rows of whole and of odd numbers of 8-element runs, K at, below and above
# the 64-element pitch, a source off the 16-byte grid; inputs with NaN, both infinities, zeros and values of every binade
@pytest.mark.parametrize("kind", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("mode", [orc.RM_TA, orc.RM_HR, orc.RM_TE, orc.RM_SSR, orc.RM_SR, orc.RM_TA | orc.FLAG_SAT])
def test_scale_search_casts(h, kind, mode):
    dtype = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[kind]
    g = torch.Generator(device=dev()).manual_seed(mode + len(kind))
    encode, calibrate = getattr(h, "hif8_encode_" + kind), getattr(h, "hif8_calibrate_layer_" + kind)
    for M, N, K, off in ((40, 33, 64, 0), (37, 70, 61, 1), (33, 34, 200, 0), (65, 40, 3, 3)):
        mats = []
        for rows, std in ((M, 1.0), (N, 0.05)):
            v = torch.randn(rows * K + off, device=dev(), generator=g) * std * torch.exp2(torch.randint(-12, 6, (rows * K + off,), device=dev(), generator=g))
            v[off::97] = 0.0
            mats.append(v.to(dtype)[off:])
        if K == 61:  # a row of A and a column of B become NaN or Inf: so do the sums
            mats[0][5], mats[1][7] = float("nan"), float("inf")
        x, w = mats
        ref = torch.zeros(M, N, device=dev())
        na, nb, ea, ew = 3, 4, -2, 1
        ws = torch.empty(h.hif8_calibrate_workspace_bytes(M, N, K, na, nb), dtype=torch.uint8, device=dev())
        err, one = (torch.zeros(na, nb, dtype=torch.float64, device=dev()) for _ in range(2))
        best = torch.zeros(2, dtype=torch.int32, device=dev())
        calibrate(x, w, ref, M, N, K, ea, na, ew, nb, mode, ws, ws.numel(), err, best)
        ld = h.hif8_expanded_ld(K)
        cast = []
        for t, rows, lo, count in ((x, M, ea, na), (w, N, ew, nb)):
            codes, xs = torch.empty(rows * K, dtype=torch.uint8, device=dev()), torch.zeros(count, rows, ld, dtype=torch.bfloat16, device=dev())
            for i in range(count):
                encode(t, codes, rows * K, 2.0 ** (lo + i), mode)
                h.hif8_expand_bf16(codes, rows, K, xs[i], ld)
            cast.append(xs)
        # the casts themselves, where the search leaves them: behind room for one code matrix, rows of the A casts first
        at = (max(M, N) * K + 15) // 16 * 16
        got = ws[at:at + 2 * (cast[0].numel() + cast[1].numel())].view(torch.int16)
        assert torch.equal(got, torch.cat([c.reshape(-1).view(torch.int16) for c in cast]))
        for i in range(na):
            for j in range(nb):
                h.hif8_gemm_expanded_sqerr(cast[0][i], cast[1][j], ref, M, N, K, ld, 2.0 ** (ea + i), 2.0 ** (ew + j), one[i, j:])
        nan = torch.isnan(one)
        assert torch.equal(torch.isnan(err), nan) and torch.all(((err - one).abs() <= 1e-6 * one)[~nan])
        fin = torch.where(torch.isfinite(err), err, float("inf"))
        pos = int(fin.argmin()) if torch.isfinite(err).any() else 0
        assert best.tolist() == [ea + pos // nb, ew + pos % nb]


# rows of every remainder of a run of 8 codes and of 16, shorter and longer than a run; one past and one below a tile of
# 64 x 128; the matrix at the start and at an odd address of its buffer, whose next byte is NaN
@pytest.mark.parametrize("rows", [1, 5, 63, 64, 65, 130])
def test_expansions_of_every_remainder(h, rows):
    lut = torch.tensor([orc.decode_value(c) for c in range(256)], dtype=torch.float64).to(torch.bfloat16).view(torch.int16).to(dev())
    lut[0x80] = torch.tensor(0x7FC0, dtype=torch.int16)
    g = torch.Generator(device=dev()).manual_seed(rows)
    for cols in (1, 2, 3, 7, 8, 9, 13, 15, 16, 17, 23, 24, 31, 33, 63, 64, 65, 120, 127, 128, 129, 136, 200):
        for off in (0, 1):
            buf = torch.full((rows * cols + off + 16,), 0x80, dtype=torch.uint8, device=dev())
            codes = buf[off:off + rows * cols]
            codes.copy_(torch.randint(0, 256, (rows * cols,), dtype=torch.uint8, device=dev(), generator=g))
            want = lut[codes.long()].view(rows, cols)
            for call, w in ((h.hif8_expand_bf16, want), (h.hif8_expand_bf16_t, want.t())):
                r, c = w.shape
                ld = h.hif8_expanded_ld(c)
                dst = torch.full((r + 1, ld), 0x1234, dtype=torch.int16, device=dev())
                call(codes, rows, cols, dst, ld)
                assert torch.equal(dst[:r, :c], w) and torch.all(dst[:r, c:] == 0) and torch.all(dst[r] == 0x1234)


# both forms of each expansion: one step and four per lane (2^21 codes of a padded matrix), tiles of 64 and of 128 columns
# (512 tiles of 64 x 128; 64 columns and fewer), on either side of the lines
@pytest.mark.parametrize("rows,cols", [(511, 4096), (512, 4096), (513, 4095), (1024, 4096), (1024, 4097), (1025, 4096), (40000, 64), (40000, 65),
                                       (64, 65600)])
def test_expansions_on_either_side_of_their_lines(h, rows, cols):
    lut = torch.tensor([orc.decode_value(c) for c in range(256)], dtype=torch.float64).to(torch.bfloat16).view(torch.int16).to(dev())
    lut[0x80] = torch.tensor(0x7FC0, dtype=torch.int16)
    codes = torch.randint(0, 256, (rows, cols), dtype=torch.uint8, device=dev(), generator=torch.Generator(device=dev()).manual_seed(rows))
    want = lut[codes.long()]
    for call, w in ((h.hif8_expand_bf16, want), (h.hif8_expand_bf16_t, want.t())):
        r, c = w.shape
        ld = h.hif8_expanded_ld(c)
        dst = torch.full((r + 1, ld), 0x1234, dtype=torch.int16, device=dev())
        call(codes, rows, cols, dst, ld)
        assert torch.equal(dst[:r, :c], w) and torch.all(dst[:r, c:] == 0) and torch.all(dst[r] == 0x1234)


def test_workspace_product_expands_both_operands(h):
    """Both operands of hif8_gemm_ws_* are expanded in one launch: the bits of the two expansions and the product on them."""
    rng = np.random.default_rng(4)
    for M, N, K in ((1300, 1100, 67), (257, 8200, 5), (1500, 1400, 130)):
        a, b = (torch.from_numpy(random_codes(rng, (r, K), "cast_normal")).to(dev()) for r in (M, N))
        ld = h.hif8_expanded_ld(K)
        xa, xb = (torch.empty(r, ld, dtype=torch.bfloat16, device=dev()) for r in (M, N))
        h.hif8_expand_bf16(a, M, K, xa, ld)
        h.hif8_expand_bf16(b, N, K, xb, ld)
        ws = torch.full((h.hif8_gemm_workspace_bytes(M, N, K),), 0x7F, dtype=torch.uint8, device=dev())
        one, two = (torch.empty(M, N, device=dev()) for _ in range(2))
        h.hif8_gemm_ws_f32(a, b, one, M, N, K, ws, 2.0, 4.0)
        h.hif8_gemm_expanded_f32(xa, xb, two, M, N, K, ld, 2.0, 4.0)
        assert torch.equal(ws.view(torch.int16), torch.cat([xa, xb]).view(torch.int16).reshape(-1)) and torch.equal(one, two)


# tiles of 64 x 64 (one and four K steps more than its four stages, and fewer), 128 x 64 in six stages, and 128 x 128 where the finer ones are too many; edges of
# their blocks, rows at unaligned addresses
@pytest.mark.parametrize("M,N,K", [(1, 1, 64), (66, 63, 128), (129, 190, 192), (700, 1227, 256), (513, 1003, 330), (64, 64, 520), (1000, 1023, 1000),
                                   (520, 2578, 64), (1030, 1101, 256), (513, 2049, 320), (900, 1153, 384), (641, 3001, 450), (1024, 2048, 770),
                                   (1500, 2003, 200), (1030, 4001, 330)])
def test_finest_tiles_every_output(h, M, N, K):
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    (a, ld), (b, _) = expand(h, random_codes(rng, (M, K), "cast_normal")), expand(h, random_codes(rng, (N, K), "cast_normal"))
    outs = {d: torch.full((M * N + 8,), 7.0, dtype=d, device=dev()) for d in (torch.float32, torch.bfloat16, torch.float16)}
    h.hif8_gemm_set_variant(9)
    for call, o in zip((h.hif8_gemm_expanded_f32, h.hif8_gemm_expanded_bf16, h.hif8_gemm_expanded_f16), outs.values()):
        call(a, b, o, M, N, K, ld, 8.0, 8.0)
        assert torch.all(o[M * N:] == 7.0)
    out = outs[torch.float32][:M * N].view(M, N)
    x, y = a.view(torch.bfloat16).double(), b.view(torch.bfloat16).double()
    assert torch.all((out.double() - x @ y.t() / 64.0).abs() <= K * 2.0 ** -23 * (x.abs() @ y.abs().t()) / 64.0)
    for d in (torch.bfloat16, torch.float16):
        assert torch.equal(outs[d][:M * N].view(M, N), out.to(d))
    ref = (out * 1.01 + 0.5).contiguous()
    err = torch.zeros(2, dtype=torch.float64, device=dev())
    h.hif8_gemm_expanded_sqerr(a, b, ref, M, N, K, ld, 8.0, 8.0, err)
    h.hif8_gemm_set_variant(0)
    want = float(((out.double() - ref.double()) ** 2).sum())
    assert err[1].item() == 0.0 and abs(err[0].item() - want) <= 1e-12 * want


# 64 x 64 tiles from 16 K steps on: a part of K every two steps, unevenly, and with a remainder of K; 700 x 1227 and 512 x 2006 go there by price
@pytest.mark.parametrize("M,N,K,variant", [(130, 190, 1024, 9), (66, 257, 1500, 9), (310, 2751, 2160, 0), (700, 1227, 4096, 0), (512, 2006, 8000, 0)])
def test_finest_tiles_sum_over_parts_of_k(h, M, N, K, variant):
    """No less exact than eight binary32 chains, one for each eighth of K, added one after the other (the sum of these products in the small-tile
    kernel): the error against fp64 is the rounding of the chains, so the two agree to the noise of M N independent errors; one chain is 1.2
    (K = 2160) to 1.6 times (8000) as far off."""
    rng = np.random.default_rng(M + N + K)
    (a, ld), (b, _) = expand(h, random_codes(rng, (M, K), "cast_normal")), expand(h, random_codes(rng, (N, K), "cast_normal"))
    x, y = a.view(torch.bfloat16).double(), b.view(torch.bfloat16).double()
    out = torch.empty(M, N, device=dev())
    h.hif8_gemm_set_variant(variant)
    h.hif8_gemm_expanded_f32(a, b, out, M, N, K, ld, 1.0, 1.0)
    h.hif8_gemm_set_variant(0)
    want, total = x @ y.t(), None
    units = ld // 64
    for p in range(8):
        chain = torch.zeros(M, N, device=dev())
        for k in range(units * p // 8 * 64, units * (p + 1) // 8 * 64, 32):  # a matrix instruction adds 32 products to the accumulator
            chain = (chain.double() + x[:, k:k + 32] @ y[:, k:k + 32].t()).float()
        total = chain if total is None else total + chain
    off, split = ((o.double() - want).square().mean().sqrt() for o in (out, total))
    print("%dx%dx%d: %.4g of eight chains' error" % (M, N, K, off / split))
    assert off <= 1.05 * split


# products that the price takes from the small tiles to 64 x 64 tiles, and some that stay there; odd rows and a K with a remainder
@pytest.mark.parametrize("M,N,K", [(700, 1227, 4096), (512, 2006, 4096), (512, 2006, 8000), (311, 1633, 5930), (512, 1000, 8000), (200, 594, 4176)])
def test_squared_error_of_the_stored_bits(h, M, N, K):
    """Where the squared error had run in the small-tile kernel as the stored product had, both take the same kernel: against the stored result it is zero."""
    rng = np.random.default_rng(M + N + K)
    (a, ld), (b, _) = expand(h, random_codes(rng, (M, K), "cast_normal")), expand(h, random_codes(rng, (N, K), "cast_normal"))
    out, err = torch.empty(M, N, device=dev()), torch.zeros(1, dtype=torch.float64, device=dev())
    h.hif8_gemm_expanded_f32(a, b, out, M, N, K, ld, 8.0, 0.5)
    h.hif8_gemm_expanded_sqerr(a, b, out, M, N, K, ld, 8.0, 0.5, err)
    assert err.item() == 0.0
