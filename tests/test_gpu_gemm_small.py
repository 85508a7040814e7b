"""GPU parity for the small-tile GEMM kernel (few output tiles, code matrices of any K and alignment) against the
fp64 oracle, with the bound of test_gpu_gemm.py: K * 2^-23 * sum_k |a b| * descale per element."""
import numpy as np
import pytest
import torch

from oracle import gemm_oracle as go
from oracle import hif8_oracle as orc
from gpu_util import dev
from test_gpu_gemm import check, h, random_codes  # noqa: F401  (h is the fixture)

pytestmark = pytest.mark.gpu


def on_gpu(codes, off=0):
    buf = torch.zeros(codes.size + off + 1, dtype=torch.uint8, device=dev())
    buf[off:off + codes.size] = torch.from_numpy(codes.reshape(-1)).to(dev())
    return buf[off:off + codes.size]


# every tile of the plan: 1 x 1 with and without the half-row form (8 / 9 / 16 rows), 1 x 2 and 2 x 4 (17 .. 32 rows), 2 x 2
# with 16 and 4 wavefronts (33 .. 64), 2 x 4 with 8 and 4 (65 .. 128), 2 x 4 / 4 x 4 above; edges of the 16-row blocks;
# K below, at and above one 128-element share, more and fewer shares than wavefronts, remainders of 1, 15, 16, 17
SHAPES = [(1, 1, 1), (3, 2, 15), (8, 64, 128), (9, 65, 127), (16, 15, 129), (7, 8200, 144), (17, 33, 1025), (32, 8193, 17),
          (33, 40, 2047), (64, 2100, 272), (64, 9000, 130), (65, 70, 1000), (128, 1024, 400), (100, 9000, 131), (129, 300, 513),
          (300, 257, 2049), (2000, 2100, 33), (300, 12, 700), (5000, 3, 31)]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("off", [0, 1])
def test_small_gemm_codes_match_oracle(h, M, N, K, off):
    rng = np.random.default_rng(M + 5 * N + 11 * K + off)
    for kind in ("cast_normal", "uniform_codes"):
        ca, cb = random_codes(rng, (M, K), kind), random_codes(rng, (N, K), kind)
        out = torch.full((M + 1, N), 7.0, dtype=torch.float32, device=dev())
        h.hif8_gemm_set_variant(12 if off == 0 else 0)
        h.hif8_gemm_f32(on_gpu(ca, off), on_gpu(cb, off), out, M, N, K, 2.0, 0.5)
        torch.cuda.synchronize()
        h.hif8_gemm_set_variant(0)
        check(out[:M].cpu().numpy(), ca, cb, 2.0, 0.5)
        assert torch.all(out[M] == 7.0)


# shares of K in units of 64: one element to a unit and a bit, an odd number of units (a stage of one), rows whose last 16 bytes
# begin in every position before the one asked for; shares in pairs of units with one unit at the end (2885); codes and expanded operands give the same bits
@pytest.mark.parametrize("M,N", [(5, 37), (14, 20), (20, 50), (40, 70), (100, 131)])
def test_small_gemm_units_of_k(h, M, N):
    rng = np.random.default_rng(M)
    for K in (1, 7, 15, 16, 17, 31, 63, 64, 65, 77, 127, 128, 129, 190, 193, 200, 577, 641, 1027, 1088, 2049, 2885):
        ca, cb = random_codes(rng, (M, K), "uniform_codes"), random_codes(rng, (N, K), "cast_normal")
        a, b, ld = on_gpu(ca, K % 3), on_gpu(cb, K % 2), h.hif8_expanded_ld(K)
        xa, xb = (torch.empty(r, ld, dtype=torch.bfloat16, device=dev()) for r in (M, N))
        h.hif8_expand_bf16(a, M, K, xa, ld)
        h.hif8_expand_bf16(b, N, K, xb, ld)
        one, two = (torch.full((M + 1, N), 7.0, dtype=torch.float32, device=dev()) for _ in range(2))
        h.hif8_gemm_set_variant(12)
        h.hif8_gemm_f32(a, b, one, M, N, K, 8.0, 0.5)
        h.hif8_gemm_expanded_f32(xa, xb, two, M, N, K, ld, 8.0, 0.5)
        h.hif8_gemm_set_variant(0)
        check(one[:M].cpu().numpy(), ca, cb, 8.0, 0.5)
        assert torch.equal(one.view(torch.int32), two.view(torch.int32)) and torch.all(one[M] == 7.0), K


@pytest.mark.parametrize("M,N,K", [(1, 100, 100), (8, 4100, 300), (20, 70, 1001), (32, 9000, 65), (64, 2100, 272), (50, 9000, 257),
                                   (128, 700, 900), (129, 700, 900), (256, 4096, 130), (700, 40, 1111)])
def test_small_gemm_same_bits_from_codes_workspace_and_expanded(h, M, N, K):
    """hif8_gemm_ws_* takes the codes directly below 129 rows and expands first above: the bits of the expanded form."""
    rng = np.random.default_rng(M + N + K)
    ca, cb = random_codes(rng, (M, K), "cast_normal"), random_codes(rng, (N, K), "cast_normal")
    a, b, ld = on_gpu(ca), on_gpu(cb), h.hif8_expanded_ld(K)
    ws = torch.empty(h.hif8_gemm_workspace_bytes(M, N, K), dtype=torch.uint8, device=dev())
    xa, xb = (torch.empty(r, ld, dtype=torch.bfloat16, device=dev()) for r in (M, N))
    h.hif8_expand_bf16(a, M, K, xa, ld)
    h.hif8_expand_bf16(b, N, K, xb, ld)
    one, two = (torch.empty(M, N, dtype=torch.float32, device=dev()) for _ in range(2))
    h.hif8_gemm_ws_f32(a, b, one, M, N, K, ws, 8.0, 0.5)
    h.hif8_gemm_expanded_f32(xa, xb, two, M, N, K, ld, 8.0, 0.5)
    check(two.cpu().numpy(), ca, cb, 8.0, 0.5)
    assert torch.equal(one.view(torch.int32), two.view(torch.int32))
    if min(M, N) <= 128:
        h.hif8_gemm_f32(a, b, one, M, N, K, 8.0, 0.5)
        assert torch.equal(one.view(torch.int32), two.view(torch.int32))


# more tiles than the chip holds workgroups: as many wavefronts as K has shares of 128 (1, 2 and 4), in every tile; and 2 x 2
# tiles of four wavefronts for up to 128 rows with four shares or less, one element past and below that
@pytest.mark.parametrize("M,N,K", [(16, 33001, 40), (30, 70001, 17), (50, 40003, 129), (128, 9000, 200), (100, 20001, 300), (32, 20000, 385),
                                   (70, 300, 512), (70, 300, 513), (128, 10003, 449)])
def test_small_gemm_wavefronts_by_shares(h, M, N, K):
    rng = np.random.default_rng(M + N + K)
    a, b, ld = on_gpu(random_codes(rng, (M, K), "cast_normal")), on_gpu(random_codes(rng, (N, K), "cast_normal")), h.hif8_expanded_ld(K)
    xa, xb = (torch.empty(r, ld, dtype=torch.bfloat16, device=dev()) for r in (M, N))
    h.hif8_expand_bf16(a, M, K, xa, ld)
    h.hif8_expand_bf16(b, N, K, xb, ld)
    one, two = (torch.full((M * N + 8,), 7.0, dtype=torch.float32, device=dev()) for _ in range(2))
    h.hif8_gemm_set_variant(12)
    h.hif8_gemm_f32(a, b, one, M, N, K, 8.0, 0.5)
    h.hif8_gemm_expanded_f32(xa, xb, two, M, N, K, ld, 8.0, 0.5)
    h.hif8_gemm_set_variant(0)
    assert torch.equal(one.view(torch.int32), two.view(torch.int32)) and torch.all(one[M * N:] == 7.0)
    want, sums = xa.double() @ xb.double().t() / 4.0, xa.double().abs() @ xb.double().abs().t() / 4.0
    assert torch.all((one[:M * N].view(M, N).double() - want).abs() <= K * 2.0 ** -23 * sums)


def test_small_gemm_16bit_outputs_and_squared_error(h):
    rng = np.random.default_rng(21)
    for M, N, K in ((8, 96, 333), (48, 130, 512), (200, 150, 257)):
        ca, cb = random_codes(rng, (M, K), "cast_normal"), random_codes(rng, (N, K), "cast_normal")
        a, b = on_gpu(ca), on_gpu(cb)
        o32, o16 = (torch.empty(M, N, dtype=d, device=dev()) for d in (torch.float32, torch.bfloat16))
        oh = torch.empty(M, N, dtype=torch.float16, device=dev())
        for call, o in ((h.hif8_gemm_f32, o32), (h.hif8_gemm_bf16, o16), (h.hif8_gemm_f16, oh)):
            call(a, b, o, M, N, K, 8.0, 8.0)
        assert torch.equal(o16, o32.to(torch.bfloat16)) and torch.equal(oh, o32.to(torch.float16))
        ref = (o32 * 1.01 + 0.5).contiguous()
        err = torch.zeros(1, dtype=torch.float64, device=dev())
        h.hif8_gemm_sqerr(a, b, ref, M, N, K, 8.0, 8.0, err)
        want = float(((o32.double() - ref.double()) ** 2).sum())
        assert abs(err.item() - want) <= 1e-12 * want


# more tiles than the four workgroups per compute unit that the squared error walks over them with, and as many
@pytest.mark.parametrize("M,N,K", [(16, 33001, 40), (8, 16384, 130), (30, 70001, 17), (50, 40003, 129), (100, 20001, 300)])
def test_small_gemm_squared_error_of_many_tiles(h, M, N, K):
    rng = np.random.default_rng(M + N)
    a, b = (on_gpu(random_codes(rng, (r, K), "cast_normal")) for r in (M, N))
    out = torch.empty(M, N, dtype=torch.float32, device=dev())
    h.hif8_gemm_set_variant(12)
    h.hif8_gemm_f32(a, b, out, M, N, K, 2.0, 4.0)
    ref = out + torch.randn(M, N, device=dev(), generator=torch.Generator(device=dev()).manual_seed(1))
    err = torch.zeros(2, dtype=torch.float64, device=dev())
    h.hif8_gemm_sqerr(a, b, ref, M, N, K, 2.0, 4.0, err)
    h.hif8_gemm_set_variant(0)
    want = float(((out.double() - ref.double()) ** 2).sum())
    assert err[1].item() == 0.0 and abs(err[0].item() - want) <= 1e-12 * want


def test_small_gemm_special_codes_follow_ieee(h):
    rng = np.random.default_rng(22)
    for M, N in ((7, 20), (40, 50)):
        K = 150
        ca, cb = random_codes(rng, (M, K), "cast_normal"), random_codes(rng, (N, K), "cast_normal")
        ca[1, 5], ca[2, 149], ca[5, 140] = 0x6F, 0x80, 0xEF          # +Inf, NaN, -Inf (meeting a zero below)
        cb[11, 140] = 0x00
        out = torch.zeros(M, N, dtype=torch.float32, device=dev())
        h.hif8_gemm_f32(on_gpu(ca), on_gpu(cb), out, M, N, K, 1.0, 1.0)
        got, want = out.cpu().numpy(), go.gemm_hif8(ca, cb)
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.isnan(want[2]).all() and np.isnan(want[5, 11])
        assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want))


def test_small_gemm_more_tiles_than_workgroups(h):
    """2^20 workgroups walk more tiles than that (a launch counts its threads in 32 bits)."""
    M, N, K = (1 << 24) + 37, 2, 3
    rng = np.random.default_rng(23)
    vals = np.array([0x00, 0x08, 0x10, 0x14, 0x20, 0x88, 0x90], np.uint8)      # 0, 1, 2, 3, 4, -1, -2: sums exact
    ca, cb = rng.choice(vals, size=(M, K)), rng.choice(vals, size=(N, K))
    out = torch.empty(M, N, dtype=torch.float32, device=dev())
    h.hif8_gemm_f32(on_gpu(ca), on_gpu(cb), out, M, N, K, 1.0, 1.0)
    v = np.array([orc.decode_value(c) if np.isfinite(orc.decode_value(c)) else 0.0 for c in range(256)], np.float32)
    assert np.array_equal(out.cpu().numpy(), v[ca] @ v[cb].T)


# tiles of three blocks of rows or columns (two of 1 x 3, two of 2 x 3, 3 x 4, 4 x 3), then others; edges of their blocks, rows at odd addresses, a K with a remainder; codes, the
# workspace above 128 rows (from the codes) and the expanded operands give the same bits
@pytest.mark.parametrize("M,N,K", [(200, 643, 1999), (16, 10641, 4097), (130, 2001, 1500), (36, 5700, 1999), (130, 10001, 577), (100, 5701, 1999), (130, 1477, 577),
                                   (173, 2000, 577), (1266, 148, 1345), (255, 257, 2049)])
def test_small_gemm_tiles_of_three_blocks(h, M, N, K):
    rng = np.random.default_rng(M + N + K)
    a, b, ld = on_gpu(random_codes(rng, (M, K), "cast_normal"), 1), on_gpu(random_codes(rng, (N, K), "cast_normal"), 1), h.hif8_expanded_ld(K)
    xa, xb = (torch.empty(r, ld, dtype=torch.bfloat16, device=dev()) for r in (M, N))
    h.hif8_expand_bf16(a, M, K, xa, ld)
    h.hif8_expand_bf16(b, N, K, xb, ld)
    ws = torch.empty(h.hif8_gemm_workspace_bytes(M, N, K), dtype=torch.uint8, device=dev())
    want, sums = xa.double() @ xb.double().t() / 4.0, xa.double().abs() @ xb.double().abs().t() / 4.0
    got = {}
    for name, call in (("codes", lambda o: h.hif8_gemm_f32(a, b, o, M, N, K, 8.0, 0.5)), ("ws", lambda o: h.hif8_gemm_ws_f32(a, b, o, M, N, K, ws, 8.0, 0.5)),
                       ("expanded", lambda o: h.hif8_gemm_expanded_f32(xa, xb, o, M, N, K, ld, 8.0, 0.5))):
        out = torch.full((M * N + 8,), 7.0, dtype=torch.float32, device=dev())
        call(out)
        assert torch.all(out[M * N:] == 7.0)
        got[name] = out[:M * N].view(M, N)
        assert torch.all((got[name].double() - want).abs() <= K * 2.0 ** -23 * sums), name
    assert torch.equal(got["ws"].view(torch.int32), got["expanded"].view(torch.int32))
    if min(M, N) <= 128:
        assert torch.equal(got["codes"].view(torch.int32), got["ws"].view(torch.int32))


# nine wavefronts: 17, 33, 36 and 54 units of K, the last of them of one element or whole; the squared error of the same bits
@pytest.mark.parametrize("M,N,K", [(509, 1003, 1025), (509, 1000, 2049), (500, 1003, 2304), (512, 1024, 3456)])
def test_small_gemm_nine_wavefronts(h, M, N, K):
    rng = np.random.default_rng(K)
    ca, cb = random_codes(rng, (M, K), "cast_normal"), random_codes(rng, (N, K), "cast_normal")
    a, b = on_gpu(ca, 1), on_gpu(cb, 1)
    out = torch.full((M * N + 8,), 7.0, dtype=torch.float32, device=dev())
    h.hif8_gemm_f32(a, b, out, M, N, K, 8.0, 0.5)
    assert torch.all(out[M * N:] == 7.0)
    out = out[:M * N].view(M, N)
    check(out.cpu().numpy(), ca, cb, 8.0, 0.5)
    ref, err = (out * 1.01 + 0.5).contiguous(), torch.zeros(1, dtype=torch.float64, device=dev())
    h.hif8_gemm_sqerr(a, b, ref, M, N, K, 8.0, 0.5, err)
    want = float(((out.double() - ref.double()) ** 2).sum())
    assert abs(err.item() - want) <= 1e-12 * want


# more wavefronts than the lines of small_plan() give (16 for 8, 8 for 4, 9 for 8), the same number, and fewer (8 for 16)
@pytest.mark.parametrize("M,N,K,chains", [(20, 1284, 2614, 8), (18, 5345, 2592, 8), (36, 6384, 832, 4), (612, 788, 785, 4), (509, 1003, 2049, 8), (578, 1056, 2849, 4),
                                          (46, 1475, 10960, 16), (8, 4096, 4096, 8)])
def test_small_gemm_sum_is_no_less_exact_with_other_wavefronts(h, M, N, K, chains):
    """The error against fp64 is that of at most `chains` binary32 chains, one for each share of K, added one after the other; the two agree to the noise of
    M N independent errors, 2 % here at most."""
    rng = np.random.default_rng(M + N + K)
    a, b, ld = on_gpu(random_codes(rng, (M, K), "cast_normal"), 1), on_gpu(random_codes(rng, (N, K), "cast_normal"), 1), h.hif8_expanded_ld(K)
    xa, xb = (torch.empty(r, ld, dtype=torch.bfloat16, device=dev()) for r in (M, N))
    h.hif8_expand_bf16(a, M, K, xa, ld)
    h.hif8_expand_bf16(b, N, K, xb, ld)
    x, y = xa.double(), xb.double()
    want, total = x @ y.t(), None
    units = ld // 64
    for p in range(chains):
        chain = torch.zeros(M, N, device=dev())
        for k in range(units * p // chains * 64, units * (p + 1) // chains * 64, 32):  # a matrix instruction adds 32 products to the accumulator
            chain = (chain.double() + x[:, k:k + 32] @ y[:, k:k + 32].t()).float()
        total = chain if total is None else total + chain
    out = torch.empty(M, N, device=dev())
    h.hif8_gemm_f32(a, b, out, M, N, K, 1.0, 1.0)
    off, split = ((o.double() - want).square().mean().sqrt() for o in (out, total))
    print("%dx%dx%d: %.4g of %d chains' error" % (M, N, K, off / split, chains))
    assert off <= 1.02 * split
