"""GPU parity for the scale sweep (cast-and-score step of Algorithm 1 on one tensor) and the
per-channel amax / encode / decode kernels, against the CPU oracle.

Bars: codes and amax bit-exact, decoded outputs as raw bit patterns; the fp64 error sums
within 1e-12 relative (every term is exact in fp64 on both sides; only the order in which
partial sums are combined differs -- n * 2^-53 relative at worst, ~1e-9 for n = 2^24 in theory,
far less in practice because the sums are tree-shaped on both sides).
"""
import numpy as np
import pytest
import torch

from oracle import hif8_oracle as orc
from gpu_util import assert_same_bytes, bf16_bits, dev, f32_bits, to_gpu

pytestmark = pytest.mark.gpu

TA, HR, TE, SSR, SR = orc.RM_TA, orc.RM_HR, orc.RM_TE, orc.RM_SSR, orc.RM_SR
SAT = orc.FLAG_SAT
KINDS = {"f32": orc.SRC_F32, "bf16": orc.SRC_BF16, "f16": orc.SRC_F16}
SEED = 0xC0FFEE12345


@pytest.fixture(scope="module")
def h():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2409_16626_amd import hif8
    hif8.hif8_init()
    return hif8


@pytest.fixture(autouse=True)
def seeds(h):
    h.hif8_set_sr_seed(SEED)
    orc.set_sr_seed(SEED)
    yield
    h.hif8_set_sr_seed(0)
    orc.set_sr_seed(0)


def as_kind(xf, kind):
    """float32 device tensor -> (device tensor of that kind, numpy array in the oracle's container)."""
    if kind == "f32":
        return xf, xf.cpu().numpy()
    if kind == "bf16":
        t = xf.to(torch.bfloat16)
        return t, bf16_bits(t)
    t = xf.to(torch.float16)
    return t, t.view(torch.int16).cpu().numpy().view(np.uint16)


def bits16(t):
    return t.view(torch.int16).cpu().numpy().view(np.uint16)


def gpu_sweep(h, kind, x, n, e_lo, count, mode):
    err = torch.full((count,), -1.0, dtype=torch.float64, device=dev())
    getattr(h, "hif8_scale_sweep_" + kind)(x, n, e_lo, count, mode, err)
    torch.cuda.synchronize()
    return err.cpu().numpy()


@pytest.mark.parametrize("kind", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("mode", [TA, HR, TE, SSR, SR, TA | SAT])
def test_scale_sweep_matches_oracle(h, kind, mode):
    g = torch.Generator(device=dev()).manual_seed(17)
    n = (1 << 20) + 13
    xf = torch.randn(n, generator=g, device=dev()) * torch.exp2(torch.rand(n, generator=g, device=dev()) * 16 - 10)
    x, xn = as_kind(xf, kind)
    got = gpu_sweep(h, kind, x, n, -4, 10, mode)
    want = orc.scale_sweep(xn, KINDS[kind], -4, 10, mode)
    assert np.all(np.isfinite(want))
    np.testing.assert_allclose(got, want, rtol=1e-12)
    # the best scale of Algorithm 1's search is the same on both sides
    assert int(np.argmin(got)) == int(np.argmin(want))


@pytest.mark.parametrize("n,off", [(0, 0), (1, 0), (5, 0), (9, 0), (4099, 0), (10007, 1), (70001, 3)])
def test_scale_sweep_ragged_unaligned_and_ranges(h, n, off):
    g = torch.Generator(device=dev()).manual_seed(18)
    big = torch.randn(1 << 17, generator=g, device=dev()) * 3.0
    for kind in ("f32", "bf16", "f16"):
        xa, _ = as_kind(big, kind)
        x = xa[off:off + n]
        xn = x.contiguous().cpu().numpy() if kind == "f32" else bits16(x.contiguous())
        for e_lo, count, mode in ((-4, 10, TA), (0, 1, HR), (-8, 16, TE), (3, 2, SR)):
            err = torch.full((count,), -1.0, dtype=torch.float64, device=dev())
            getattr(h, "hif8_scale_sweep_" + kind)(x.data_ptr() if n else 0, n, e_lo, count, mode, err)
            torch.cuda.synchronize()
            want = orc.scale_sweep(xn, KINDS[kind], e_lo, count, mode)
            np.testing.assert_allclose(err.cpu().numpy(), want, rtol=1e-12, atol=0)


def test_scale_sweep_non_finite_terms(h):
    x = torch.tensor([3.0e4, 1.0, -2.5, 0.0] * 1000, dtype=torch.float32, device=dev())
    got = gpu_sweep(h, "f32", x, x.numel(), 0, 3, TA)
    want = orc.scale_sweep(x.cpu().numpy(), orc.SRC_F32, 0, 3, TA)
    assert np.isfinite(want[0]) and np.isposinf(want[1]) and np.isposinf(want[2])
    assert got[0] == pytest.approx(want[0], rel=1e-12) and np.isposinf(got[1]) and np.isposinf(got[2])
    gs = gpu_sweep(h, "f32", x, x.numel(), 0, 3, TA | SAT)
    np.testing.assert_allclose(gs, orc.scale_sweep(x.cpu().numpy(), orc.SRC_F32, 0, 3, TA | SAT), rtol=1e-12)
    x[777] = float("nan")
    assert np.all(np.isnan(gpu_sweep(h, "f32", x, x.numel(), -1, 4, HR)))
    # argument checks
    from paper_2409_16626_amd.hif8 import Hif8Error
    err = torch.zeros(16, dtype=torch.float64, device=dev())
    for bad in ((0, 17), (0, 0), (-127, 2), (120, 8)):
        with pytest.raises(Hif8Error):
            h.hif8_scale_sweep_f32(x, x.numel(), bad[0], bad[1], TA, err)


def test_scale_sweep_large_tensor(h):
    from paper_2409_16626_amd import workloads
    x = workloads.activation_bf16(4096, 4096, dev()).view(-1)
    got = gpu_sweep(h, "bf16", x, x.numel(), -4, 10, TA)
    want = orc.scale_sweep(bf16_bits(x), orc.SRC_BF16, -4, 10, TA)
    np.testing.assert_allclose(got, want, rtol=1e-12)


# ------------------------------------------------------------------ per-channel
SHAPES = [(37, 53), (64, 4096), (300, 1032), (1, 8), (4096, 8), (5, 8200), (1030, 264), (2, 3)]


@pytest.mark.parametrize("rows,cols", SHAPES)
@pytest.mark.parametrize("axis", [0, 1])
def test_per_channel_amax_scale_encode_decode(h, rows, cols, axis):
    g = torch.Generator(device=dev()).manual_seed(rows * 131 + cols)
    ch_shape = (rows, 1) if axis == 0 else (1, cols)
    xf = (torch.randn(rows, cols, generator=g, device=dev())
          * torch.exp2(torch.rand(ch_shape, generator=g, device=dev()) * 12 - 6)).contiguous()
    nch = rows if axis == 0 else cols
    for kind in ("f32", "bf16", "f16"):
        x, xn = as_kind(xf, kind)
        am = torch.full((nch,), 5.0, dtype=torch.float32, device=dev())
        sc = torch.zeros(nch, 2, dtype=torch.float32, device=dev())
        getattr(h, "hif8_amax_axis_" + kind)(x, rows, cols, axis, am)
        h.hif8_scale_from_amax_n(am, sc, nch, 32768.0, 1)
        torch.cuda.synchronize()
        w_am = orc.amax_axis(xn, KINDS[kind], axis)
        assert_same_bytes(f32_bits(am), w_am.view(np.uint32), "amax_axis %s" % kind)
        w_sc = np.array([orc.scale_from_amax(a, 32768.0, True) for a in w_am], np.float32)
        scn = sc.cpu().numpy()
        assert np.array_equal(scn[:, 0], w_sc) and np.array_equal(scn[:, 1], np.float32(1.0) / w_sc)
        for mode in (TA, HR, SR):
            codes = torch.zeros(rows, cols, dtype=torch.uint8, device=dev())
            getattr(h, "hif8_encode_axis_" + kind)(x, codes, rows, cols, axis, sc, mode)
            torch.cuda.synchronize()
            want = orc.encode_axis(xn, w_sc, KINDS[kind], axis, mode)
            assert_same_bytes(codes.cpu().numpy().reshape(-1), want.reshape(-1), "encode_axis %s %#x" % (kind, mode))
        out = torch.empty_like(x)
        getattr(h, "hif8_decode_axis_" + kind)(codes, out, rows, cols, axis, sc)
        torch.cuda.synchronize()
        wd = orc.decode_axis(want, w_sc, KINDS[kind], axis)
        gd = f32_bits(out) if kind == "f32" else bits16(out)
        wdb = wd.view(np.uint32) if kind == "f32" else wd
        assert_same_bytes(gd.reshape(-1), wdb.reshape(-1), "decode_axis %s" % kind)


QR_SHAPES = [(37, 56), (64, 4096), (300, 1032), (1, 8), (4096, 8), (5, 8200), (1030, 264), (2, 3), (3, 16392),
             (700, 4104), (2, 32768), (2, 32776), (9, 2048)]


@pytest.mark.parametrize("rows,cols", QR_SHAPES)
def test_quantize_rows_matches_oracle_composition(h, rows, cols):
    """The one-call per-row path (one pass where a row fits a workgroup, the three launches otherwise):
    amax, scale pair and codes bit for bit what the oracle's amax -> scale -> cast composition gives."""
    g = torch.Generator(device=dev()).manual_seed(rows * 977 + cols)
    xf = (torch.randn(rows, cols, generator=g, device=dev())
          * torch.exp2(torch.rand((rows, 1), generator=g, device=dev()) * 14 - 7)).contiguous()
    if rows > 2:
        xf[1] = 0.0                                            # an all-zero row: amax 0 -> scale 1
    for kind in ("f32", "bf16", "f16"):
        x, xn = as_kind(xf, kind)
        w_am = orc.amax_axis(xn, KINDS[kind], 0)
        for mode, pow2, target in ((TA, 1, 32768.0), (HR, 0, 32768.0), (SR | SAT, 1, 16.0), (TE, 0, 1000.0)):
            am = torch.full((rows,), 5.0, dtype=torch.float32, device=dev())
            sc = torch.full((rows, 2), -1.0, dtype=torch.float32, device=dev())
            codes = torch.full((rows, cols), 0xAA, dtype=torch.uint8, device=dev())
            getattr(h, "hif8_quantize_rows_" + kind)(x, codes, rows, cols, am, sc, target, pow2, mode)
            torch.cuda.synchronize()
            assert_same_bytes(f32_bits(am), w_am.view(np.uint32), "quantize_rows amax %s" % kind)
            w_sc = np.array([orc.scale_from_amax(a, target, bool(pow2)) for a in w_am], np.float32)
            scn = sc.cpu().numpy()
            assert np.array_equal(scn[:, 0], w_sc) and np.array_equal(scn[:, 1], np.float32(1.0) / w_sc)
            want = orc.encode_axis(xn, w_sc, KINDS[kind], 0, mode)
            assert_same_bytes(codes.cpu().numpy().reshape(-1), want.reshape(-1), "quantize_rows %s %#x" % (kind, mode))


# many narrow rows, which take three launches by elements (rows_by_elements): on both sides of the lines
@pytest.mark.parametrize("rows,cols", [(100000, 9), (60000, 16), (59999, 17), (100001, 24), (60001, 25)])
def test_quantize_rows_many_narrow_rows(h, rows, cols):
    test_quantize_rows_matches_oracle_composition(h, rows, cols)


def test_quantize_rows_no_slower_by_many_narrow_rows(h):
    """As many values in rows of eight as in rows of 1024 cost no more than four times as much (us: 15 and 6; in one pass 93)."""
    n, best = 223270 * 8, []
    x = torch.randn(n, device=dev()).to(torch.bfloat16)
    codes = torch.empty(n, dtype=torch.uint8, device=dev())
    for rows, cols in ((n // 8, 8), (n // 1024, 1024)):
        am, sc = torch.empty(rows, device=dev()), torch.empty(rows, 2, device=dev())
        took = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                h.hif8_quantize_rows_bf16(x, codes, rows, cols, am, sc, 32768.0, 0, SR)
            b.record()
            b.synchronize()
            took.append(a.elapsed_time(b))
        best.append(min(took))
    assert best[0] < 4 * best[1], best


def test_quantize_rows_unaligned_special_values_and_arguments(h):
    from paper_2409_16626_amd.hif8 import Hif8Error
    rows, cols = 19, 72
    g = torch.Generator(device=dev()).manual_seed(5)
    base = torch.randn(rows * cols + 8, generator=g, device=dev())
    x = base[1:1 + rows * cols]                                # 4-byte aligned only: the separate launches
    x[5] = float("inf"); x[cols + 3] = float("nan"); x[2 * cols:3 * cols] = 0.0
    xn = x.cpu().numpy().reshape(rows, cols)
    am = torch.zeros(rows, dtype=torch.float32, device=dev())
    sc = torch.zeros(rows, 2, dtype=torch.float32, device=dev())
    codes = torch.zeros(rows, cols, dtype=torch.uint8, device=dev())
    h.hif8_quantize_rows_f32(x.data_ptr(), codes, rows, cols, am, sc, 32768.0, 1, TA)
    torch.cuda.synchronize()
    w_am = orc.amax_axis(xn, orc.SRC_F32, 0)
    assert_same_bytes(f32_bits(am), w_am.view(np.uint32), "amax")
    w_sc = np.array([orc.scale_from_amax(a, 32768.0, True) for a in w_am], np.float32)
    assert np.array_equal(sc.cpu().numpy()[:, 0], w_sc)
    assert_same_bytes(codes.cpu().numpy().reshape(-1), orc.encode_axis(xn, w_sc, orc.SRC_F32, 0, TA).reshape(-1), "codes")
    # the same values through the aligned (single-pass) path
    xa = x.clone()
    am2, sc2, codes2 = torch.zeros_like(am), torch.zeros_like(sc), torch.zeros_like(codes)
    h.hif8_quantize_rows_f32(xa, codes2, rows, cols, am2, sc2, 32768.0, 1, TA)
    torch.cuda.synchronize()
    assert torch.equal(am.view(torch.int32), am2.view(torch.int32)) and torch.equal(sc.view(torch.int32), sc2.view(torch.int32))
    assert torch.equal(codes, codes2)
    # arguments
    h.hif8_quantize_rows_f32(0, 0, 0, 64, 0, 0)                # no rows: nothing to do
    for bad in (dict(target=0.0), dict(target=float("inf")), dict(rounding_mode=7)):
        with pytest.raises(Hif8Error):
            h.hif8_quantize_rows_f32(xa, codes2, rows, cols, am2, sc2, **bad)
    with pytest.raises(Hif8Error):
        h.hif8_quantize_rows_f32(xa, codes2, rows, cols, 0, sc2)
    with pytest.raises(Hif8Error):
        h.hif8_quantize_rows_f32(xa, codes2, rows, cols, am2, 0)


def test_per_channel_unaligned_base_and_special_values(h):
    rows, cols = 33, 64
    g = torch.Generator(device=dev()).manual_seed(3)
    buf = torch.randn(rows * cols + 8, generator=g, device=dev())
    x = buf[1:1 + rows * cols].view(rows, cols)            # 4 bytes off a 16-byte boundary
    xn = x.contiguous().cpu().numpy()
    for axis in (0, 1):
        nch = rows if axis == 0 else cols
        am = torch.zeros(nch, dtype=torch.float32, device=dev())
        h.hif8_amax_axis_f32(x.data_ptr(), rows, cols, axis, am)
        torch.cuda.synchronize()
        assert_same_bytes(f32_bits(am), orc.amax_axis(xn, orc.SRC_F32, axis).view(np.uint32), "unaligned amax")
    y = torch.randn(16, 128, generator=g, device=dev())
    y[3, 5] = float("inf")
    y[7, 9] = float("nan")
    y[9] = 0.0
    for axis in (0, 1):
        nch = 16 if axis == 0 else 128
        am = torch.zeros(nch, dtype=torch.float32, device=dev())
        sc = torch.zeros(nch, 2, dtype=torch.float32, device=dev())
        h.hif8_amax_axis_f32(y, 16, 128, axis, am)
        h.hif8_scale_from_amax_n(am, sc, nch, 32768.0, 0)
        torch.cuda.synchronize()
        w = orc.amax_axis(y.cpu().numpy(), orc.SRC_F32, axis)
        assert_same_bytes(f32_bits(am), w.view(np.uint32), "special amax")
        w_sc = np.array([orc.scale_from_amax(a, 32768.0, False) for a in w], np.float32)
        assert np.array_equal(sc.cpu().numpy()[:, 0], w_sc)   # degenerate channels (0, Inf, NaN) get scale 1


# one below, at and above a vector (4 or 8 values); a wavefront's vectors of a row (64 to 256) and one more; a workgroup's (512 to 4096) and one more,
# which takes the three launches; several chunks of a row; many short rows; strips of columns; enough rows for a wavefront each at three and four vectors a lane
@pytest.mark.parametrize("rows,cols", [(700, 1), (65, 3), (3000, 7), (33, 9), (40, 513), (9, 1021), (2500, 259), (17, 2047), (6, 2051), (5, 4099), (3, 16381),
                                       (2, 32771), (300, 1547), (1100, 1099), (1540, 1001)])
@pytest.mark.parametrize("off", [0, 1])
def test_per_channel_any_columns_and_address(h, rows, cols, off):
    """Rows that start anywhere (odd numbers of columns, a base one element or one byte off): bit for bit the oracle's, nothing
    written outside."""
    g = torch.Generator(device=dev()).manual_seed(rows * 31 + cols)
    n = rows * cols
    xf = torch.randn(rows, cols, generator=g, device=dev()) * torch.exp2(torch.rand((rows, 1), generator=g, device=dev()) * 14 - 7)
    for kind in ("f32", "bf16", "f16"):
        flat = xf.to({"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[kind]).reshape(-1)
        src = torch.full((n + 2,), 3e4, dtype=flat.dtype, device=dev())  # larger than the values: a read outside shows
        src[off:off + n] = flat
        x = src[off:off + n]
        xn = as_kind(flat.float().view(rows, cols), kind)[1]
        for axis in (0, 1):
            nch = rows if axis == 0 else cols
            am, sc = torch.full((nch,), 5.0, device=dev()), torch.empty(nch, 2, device=dev())
            getattr(h, "hif8_amax_axis_" + kind)(x.data_ptr(), rows, cols, axis, am)
            h.hif8_scale_from_amax_n(am, sc, nch, 32768.0, 1)
            w_am = orc.amax_axis(xn, KINDS[kind], axis)
            assert_same_bytes(f32_bits(am), w_am.view(np.uint32), "amax %s %d" % (kind, axis))
            w_sc = np.array([orc.scale_from_amax(a, 32768.0, True) for a in w_am], np.float32)
            for mode in (TA, HR, SR):
                codes = torch.full((n + 2,), 0xAA, dtype=torch.uint8, device=dev())
                getattr(h, "hif8_encode_axis_" + kind)(x.data_ptr(), codes.data_ptr() + off, rows, cols, axis, sc, mode)
                want = orc.encode_axis(xn, w_sc, KINDS[kind], axis, mode).reshape(-1)
                got = codes.cpu().numpy()
                assert_same_bytes(got[off:off + n], want, "encode %s %d %#x" % (kind, axis, mode))
                assert np.all(got[:off] == 0xAA) and np.all(got[off + n:] == 0xAA)
                if axis == 0:
                    am2, sc2 = torch.full((rows,), 5.0, device=dev()), torch.empty(rows, 2, device=dev())
                    codes.fill_(0xAA)
                    getattr(h, "hif8_quantize_rows_" + kind)(x.data_ptr(), codes.data_ptr() + off, rows, cols, am2, sc2, 32768.0, 1, mode)
                    assert np.array_equal(codes.cpu().numpy(), got)
                    assert torch.equal(am2.view(torch.int32), am.view(torch.int32)) and torch.equal(sc2.view(torch.int32), sc.view(torch.int32))
            out = torch.full((n + 2,), 7.0, dtype=flat.dtype, device=dev())
            getattr(h, "hif8_decode_axis_" + kind)(codes.data_ptr() + off, out[off:].data_ptr(), rows, cols, axis, sc)
            wd = orc.decode_axis(want.reshape(rows, cols), w_sc, KINDS[kind], axis)
            gd = f32_bits(out) if kind == "f32" else bits16(out)
            assert_same_bytes(gd[off:off + n], (wd.view(np.uint32) if kind == "f32" else wd).reshape(-1), "decode %s %d" % (kind, axis))
            assert torch.all(out[:off] == 7.0) and torch.all(out[off + n:] == 7.0)


# the vector kernels, which matrices that are neither narrow nor small take (axis_by_elements): several chunks of a row and one, whole vectors to a row or not; strips with a
# vector in the last wavefront; the fewest columns that go there by rows and by columns
@pytest.mark.parametrize("rows,cols,off", [(1100, 4099, 1), (1030, 4096, 0), (70, 70001, 1), (9000, 515, 0), (14000, 321, 1), (10500, 449, 1), (16500, 288, 0), (45000, 97, 1),
                                           (70000, 65, 0), (70000, 56, 0), (44000, 96, 0), (40000, 129, 1)])
def test_per_channel_vector_kernels(h, rows, cols, off):
    test_per_channel_any_columns_and_address(h, rows, cols, off)


def test_standard_sr_rows_over_the_end_of_a_threshold_block(h):
    """More than 2^32 elements in rows of an odd number of columns, so that a row, and in it a vector, reaches over element 2^32, where another key of the
    thresholds begins: that row and its neighbours, cast by rows, by columns and in one pass, against the oracle's one-element entry point."""
    cols = 32749
    row = (1 << 32) // cols  # the row that reaches over the end
    rows = row + 3
    x = torch.zeros(rows * cols, dtype=torch.bfloat16, device=dev())
    lo, hi = (row - 1) * cols, (row + 2) * cols
    g = torch.Generator(device=dev()).manual_seed(3)
    x[lo:hi] = (torch.randn(hi - lo, generator=g, device=dev()) * 40.0).to(torch.bfloat16)
    assert lo < (1 << 32) - 8 and (1 << 32) - row * cols > 8 and hi > (1 << 32) + 8 and ((1 << 32) - row * cols) % 8 != 0
    at = np.concatenate([np.arange(lo, lo + 64), np.arange(row * cols - 16, row * cols + 16), np.arange((1 << 32) - 64, (1 << 32) + 64),
                         np.arange((row + 1) * cols - 16, (row + 1) * cols + 64), np.arange(hi - 64, hi)])
    idx = torch.from_numpy(at).to(dev())
    xs = bf16_bits(x[idx])
    codes, am, sc = torch.empty(rows * cols, dtype=torch.uint8, device=dev()), torch.empty(rows, device=dev()), torch.ones(rows, 2, device=dev())
    got = {}
    h.hif8_encode_axis_bf16(x, codes, rows, cols, 0, sc, SR)
    got["rows"] = codes[idx].cpu().numpy()
    codes.fill_(0xAA)
    h.hif8_encode_axis_bf16(x, codes, rows, cols, 1, torch.ones(cols, 2, device=dev()), SR)
    got["columns"] = codes[idx].cpu().numpy()
    want = [orc.encode_one(np.array([int(b) << 16], np.uint32).view(np.float32)[0], SR, orc.SRC_BF16, orc.sr_threshold(SEED, int(i))) for b, i in zip(xs, at)]
    for name in got:
        assert got[name].tolist() == want, name
    codes.fill_(0xAA)
    h.hif8_quantize_rows_bf16(x, codes, rows, cols, am, sc, 32768.0, 1, SR)
    one = codes[idx].cpu().numpy()
    h.hif8_encode_axis_bf16(x, codes, rows, cols, 0, sc, SR)
    assert np.array_equal(one, codes[idx].cpu().numpy())


def test_standard_sr_by_columns_costs_no_more_than_twice_by_rows(h):
    """Both draw one threshold per element and read and write the same bytes (40 and 43 us for 11008 x 4096; a key selected for each element: 154)."""
    rows, cols = 8192, 4096
    x = torch.randn(rows, cols, device=dev()).to(torch.bfloat16)
    codes = torch.empty(rows, cols, dtype=torch.uint8, device=dev())
    best = []
    for axis in (0, 1):
        sc = torch.ones(rows if axis == 0 else cols, 2, device=dev())
        took = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                h.hif8_encode_axis_bf16(x, codes, rows, cols, axis, sc, SR)
            b.record()
            b.synchronize()
            took.append(a.elapsed_time(b))
        best.append(min(took))
    assert best[1] < 2 * best[0], best
