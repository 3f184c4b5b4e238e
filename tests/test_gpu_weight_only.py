"""GPU parity of the weight-only group-128 W4 linear (mquant_w4g128_gemm) against
the oracle.  The dequantised fp16 weight is checked bit for bit through one-hot
activations; the linear within
    1e-3 * |ref| + 1e-5 * sum_k |x_k W~_nk|
of the oracle's double-precision sum: the first term covers the fp16 rounding of
the result (2^-11), the second the fp32 accumulation of the matrix core (K/16
additions of relative error <= 2^-23 on partial sums of size ~ sqrt(K) terms:
below 2e-6 of the absolute sum at K = 18944)."""
import sys

import numpy as np
import pytest

from oracle import mquant_oracle as orc

torch = pytest.importorskip("torch")
from kernel_trace import traced

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mq():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2502_00425_amd import binding
    return binding


def say(msg):
    print(f"[parity-w4g128] {msg}", flush=True)
    sys.stdout.flush()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def pack_int4(wq):
    u = (wq.astype(np.int16) & 0xF).astype(np.uint8)
    return (u[:, 0::2] | (u[:, 1::2] << 4)).astype(np.uint8)


def make_weight(rng, N, K):
    """Gaussian weight with a few large entries, quantised by the oracle's group quantiser."""
    W = rng.standard_normal((N, K)) * 0.02
    W[rng.integers(0, N, 8), rng.integers(0, K, 8)] *= 12.0
    return orc.quantize_weight_groups_int4(W)


def check(y_gpu, ref, mag, what):
    y = y_gpu.astype(np.float64)
    tol = 1e-3 * np.abs(ref) + 1e-5 * mag + 2.0 ** -24
    bad = np.abs(y - ref) > tol
    assert not bad.any(), f"{what}: {int(bad.sum())} outputs out of tolerance (first {np.argwhere(bad)[:3].tolist()})"


def test_dequantised_weight_bit_exact_through_one_hot_rows(mq):
    """x = identity: y[k, n] is the dequantised weight itself, so nibble order, the +8 storage,
    the group of every channel and the single rounding are all fixed bit for bit."""
    rng = np.random.default_rng(31)
    N, K = 72, 384
    wq = rng.integers(-8, 8, size=(N, K), dtype=np.int8)
    sc = rng.uniform(0.001, 0.08, size=(N, K // 128)).astype(np.float16)
    sc[0, 0] = np.float16(1e-5)                          # a subnormal scale: subnormal products
    want = orc.dequant_weight_groups_f16(wq, sc)
    wp = mq.w4g128_prepack(dev(pack_int4(wq)), dev(sc))
    x = np.eye(K, dtype=np.float16)
    say(f"one-hot T={K} N={N} K={K}")
    y = mq.w4g128_gemm(dev(x), wp, N).cpu().numpy()
    assert (np.ascontiguousarray(y.T).view(np.uint16) == want.view(np.uint16)).all()
    assert (want[0, :128] != 0).any() and (np.abs(want[0, :128]) < 6.1e-5).any()


@pytest.mark.parametrize("T,N,K", [
    (1, 32, 128), (5, 200, 256), (9, 72, 1152),             # GEMV
    (16, 200, 640), (31, 40, 2176), (32, 136, 384),         # rows that GEMV and GEMM share by estimate
    (33, 64, 128), (64, 136, 384),                          # the smallest tiles
    (50, 16400, 128),                                       # 64x256 tiles (many channels)
    (65, 264, 512), (130, 300, 256),                        # N % 8 != 0 -> 2-byte stores
    (257, 1000, 640), (300, 520, 1024),
    (1100, 6200, 256),                                      # many 128x256 tiles, ragged both ways
])
def test_linear_matches_oracle(mq, T, N, K):
    rng = np.random.default_rng(T * 7 + N)
    wq, sc = make_weight(rng, N, K)
    x = (rng.standard_normal((T, K)) * 1.5).astype(np.float16)
    ref, mag = orc.w4g128_linear(x, wq, sc)
    wp = mq.w4g128_prepack(dev(pack_int4(wq)), dev(sc))
    say(f"T={T} N={N} K={K}")
    y = mq.w4g128_gemm(dev(x), wp, N).cpu().numpy()
    check(y, ref, mag, f"w4g128 {(T, N, K)}")


def test_strided_rows_and_untouched_padding(mq):
    rng = np.random.default_rng(41)
    T, N, K = 150, 264, 256
    wq, sc = make_weight(rng, N, K)
    xb = (rng.standard_normal((T, K + 24)) * 1.5).astype(np.float16)
    ref, mag = orc.w4g128_linear(np.ascontiguousarray(xb[:, :K]), wq, sc)
    wp = mq.w4g128_prepack(dev(pack_int4(wq)), dev(sc))
    for pad in (8, 3):                                      # wide stores, then 2-byte stores
        yb = torch.full((T, N + pad), 7.0, dtype=torch.float16, device="cuda")
        say(f"strided ldx={K + 24} ldy={N + pad}")
        mq.w4g128_gemm(dev(xb)[:, :K], wp, N, out=yb[:, :N])
        got = yb.cpu().numpy()
        check(got[:, :N], ref, mag, f"strided pad={pad}")
        assert (got[:, N:] == 7.0).all()


@pytest.mark.parametrize("T,N,K,name", [
    (1280, 37888, 3584, "gate_up 7B"), (1280, 3584, 18944, "down 7B"), (1, 4608, 3584, "qkv decode")])
def test_full_size_sampled(mq, T, N, K, name):
    """The shapes of the 7B model's projections in the launch configuration the benchmark times;
    the oracle computes sampled rows and columns."""
    rng = np.random.default_rng(len(name) + T)
    wq = rng.integers(-8, 8, size=(N, K), dtype=np.int8)
    sc = rng.uniform(0.002, 0.01, size=(N, K // 128)).astype(np.float16)
    x = (rng.standard_normal((T, K)) * 1.5).astype(np.float16)
    wp = mq.w4g128_prepack(dev(pack_int4(wq)), dev(sc))
    say(f"full size {name}: T={T} N={N} K={K}")
    y = mq.w4g128_gemm(dev(x), wp, N).cpu().numpy()
    rows = np.unique(np.concatenate([[0, T - 1], rng.integers(0, T, 24)]))
    cols = np.unique(np.concatenate([[0, N - 1, N - 33], rng.integers(0, N, 160)]))
    ref, mag = orc.w4g128_linear(x[rows], wq[cols], sc[cols])
    check(y[np.ix_(rows, cols)], ref, mag, f"full size {name}")
    assert np.isfinite(y.astype(np.float32)).all()


def test_argument_errors_and_empty_inputs(mq):
    b = mq
    wq = np.zeros((32, 256), dtype=np.int8)
    sc = np.ones((32, 2), dtype=np.float16)
    wp = b.w4g128_prepack(dev(pack_int4(wq)), dev(sc))
    x = torch.zeros((4, 256), dtype=torch.float16, device="cuda")
    assert b.w4g128_gemm(x[:0], wp, 32).shape == (0, 32)
    assert (b.w4g128_gemm(x, wp, 32).cpu().numpy() == 0).all()
    assert b.lib.mquant_w4g128_prepacked_bytes(32, 192) == b.ERR_UNSUPPORTED
    assert b.lib.mquant_w4g128_prepacked_bytes(-1, 128) == b.ERR_BAD_SHAPE
    assert b.w4g128_prepacked_bytes(33, 256) == 2 * 4 * 1024 + 2 * 64 * 2
    y = torch.zeros((4, 32), dtype=torch.float16, device="cuda")
    lib = b.lib
    assert lib.mquant_w4g128_gemm(x.data_ptr(), 192, wp.data_ptr(), y.data_ptr(), 32, 4, 32, 256, None) == b.ERR_BAD_SHAPE
    assert lib.mquant_w4g128_gemm(x.data_ptr(), 256, wp.data_ptr(), y.data_ptr(), 16, 4, 32, 256, None) == b.ERR_BAD_SHAPE
    assert lib.mquant_w4g128_gemm(x.data_ptr(), 260, wp.data_ptr(), y.data_ptr(), 32, 4, 32, 256, None) == b.ERR_ALIGNMENT
    assert lib.mquant_w4g128_gemm(x.data_ptr() + 2, 256, wp.data_ptr(), y.data_ptr(), 32, 3, 32, 256, None) == b.ERR_ALIGNMENT
    assert lib.mquant_w4g128_gemm(x.data_ptr(), 256, wp.data_ptr(), y.data_ptr(), 32, 4, 32, 64, None) == b.ERR_UNSUPPORTED
    assert lib.mquant_w4g128_gemm(None, 256, wp.data_ptr(), y.data_ptr(), 32, 4, 32, 256, None) == b.ERR_NULL
    torch.cuda.synchronize()


@pytest.mark.parametrize("tile", [0, 1])
def test_both_gemm_tiles_on_ragged_shapes(mq, tile):
    """The two tiles that G128_TILE names (256x256 and 96x128), forced, on ragged shapes."""
    mq.tune_set(mq.TUNE_G128_TILE, tile)
    try:
        rng = np.random.default_rng(70 + tile)
        for T, N, K in [(65, 264, 128), (200, 300, 384), (410, 1000, 640)]:
            wq, sc = make_weight(rng, N, K)
            x = (rng.standard_normal((T, K)) * 1.5).astype(np.float16)
            ref, mag = orc.w4g128_linear(x, wq, sc)
            wp = mq.w4g128_prepack(dev(pack_int4(wq)), dev(sc))
            say(f"tile {tile} T={T} N={N} K={K}")
            y = mq.w4g128_gemm(dev(x), wp, N).cpu().numpy()
            check(y, ref, mag, f"w4g128 tile {tile} {(T, N, K)}")
    finally:
        mq.tune_set(mq.TUNE_G128_TILE, -1)


@pytest.mark.parametrize("T,N,K,waves", [
    (1, 17, 1152, 16), (4, 17, 4224, 16), (1, 200, 18944, 16),      # 16 waves: idle, uneven and full K ranges
    (4, 64, 18944, 16), (1, 40, 76672, 16),                         # ... and the largest rows in LDS
    (1, 200, 640, 8), (3, 200, 2176, 8), (2, 4100, 2176, 8), (4, 4100, 4224, 8), (4, 6408, 8192, 8),
    (2, 40, 256, 4), (1, 8200, 384, 4), (1, 16392, 2176, 4), (3, 18950, 4224, 4),
    (1, 16, 128, 0), (1, 16400, 256, 0), (4, 16392, 1152, 0), (3, 16385, 640, 0),   # whole tiles; 2-byte rows
    (4, 40, 19200, 0),                                              # rows that no longer fit LDS
])
def test_few_rows_in_half_tiles(mq, T, N, K, waves):
    """One to four rows: every work-group size of the half-tile form (0: whole tiles), K ranges that
    do not divide over the waves, the last half tile, strided x and y with untouched padding."""
    rng = np.random.default_rng(T * 11 + N + K)
    wq, sc = make_weight(rng, N, K)
    xb = (rng.standard_normal((T, K + 8)) * 1.5).astype(np.float16)
    ref, mag = orc.w4g128_linear(np.ascontiguousarray(xb[:, :K]), wq, sc)
    wp = mq.w4g128_prepack(dev(pack_int4(wq)), dev(sc))
    x = dev(xb)[:, :K]
    yb = torch.full((T, N + 3), 7.0, dtype=torch.float16, device="cuda")
    say(f"few rows T={T} N={N} K={K}")
    names = traced(lambda: mq.w4g128_gemm(x, wp, N, out=yb[:, :N]))
    got = yb.cpu().numpy()
    check(got[:, :N], ref, mag, f"few rows {(T, N, K)}")
    assert (got[:, N:] == 7.0).all()
    form = f"w4g128_gemv_half_kernel<{waves}," if waves else "w4g128_gemv_kernel<"
    assert names is None or (len(names) == 1 and names[0].startswith(form)), names


@pytest.mark.parametrize("T,N,K", [
    (5, 12299, 3584), (16, 20500, 3584),              # three units per work-group and four; the most rows
    (2, 28700, 3584), (9, 36900, 2048),               # shares that cross units, short K
    (12, 10250, 5120), (4, 16400, 5120),              # the fewest units; the last of half a tile
    (2, 20500, 8192), (3, 20500, 11008),              # long K: the scales in more than one round
])
def test_walk_of_several_rows(mq, T, N, K):
    """A work-group per compute unit: strided x and y with untouched padding, and the same bits again."""
    rng = np.random.default_rng(T * 17 + N + K)
    wq, sc = make_weight(rng, N, K)
    xb = (rng.standard_normal((T, K + 8)) * 1.5).astype(np.float16)
    ref, mag = orc.w4g128_linear(np.ascontiguousarray(xb[:, :K]), wq, sc)
    wp, x = mq.w4g128_prepack(dev(pack_int4(wq)), dev(sc)), dev(xb)[:, :K]
    yb = torch.full((T, N + 3), 7.0, dtype=torch.float16, device="cuda")
    say(f"walk T={T} N={N} K={K}")
    names = traced(lambda: mq.w4g128_gemm(x, wp, N, out=yb[:, :N]))
    got = yb.cpu().numpy()
    check(got[:, :N], ref, mag, f"walk {(T, N, K)}")
    assert (got[:, N:] == 7.0).all() and torch.equal(mq.w4g128_gemm(x, wp, N), yb[:, :N])
    assert names is None or (len(names) == 1 and names[0].startswith("w4g128_walk_kernel<")), names


@pytest.mark.parametrize("T,N,K,name", [
    (13, 1003, 128, "w4g128_gemv_kernel<16, 2>"), (20, 1003, 128, "w4g128_gemv_kernel<16, 2>"),
    (17, 18951, 256, "w4g128_gemv_kernel<8, 1>"), (25, 18951, 256, "w4g128_gemv_kernel<8, 1>"),
    (32, 16392, 512, "w4g128_gemv_kernel<8, 1>"), (13, 200, 2176, "w4g128_gemm_kernel<1, 1, 3>"),
    (10, 40, 10368, "w4g128_gemv_kernel<16, 2>"), (11, 40, 10240, "w4g128_gemv_kernel<16, 2>"),     # one conversion
    (11, 40, 10368, "w4g128_gemv_kernel<16, 2>"), (12, 72, 18944, "w4g128_gemv_kernel<16, 2>"),     # the other
])
def test_rows_between_gemv_and_gemm(mq, T, N, K, name):
    """13 to 32 rows on both GEMV forms, every result register that can hold a row, and on the GEMM; both sides of
    the line from which on the GEMV unpacks long K the other way."""
    rng = np.random.default_rng(T * 13 + N + K)
    wq, sc = make_weight(rng, N, K)
    x = (rng.standard_normal((T, K)) * 1.5).astype(np.float16)
    ref, mag = orc.w4g128_linear(x, wq, sc)
    wp, xd = mq.w4g128_prepack(dev(pack_int4(wq)), dev(sc)), dev(x)
    say(f"rows T={T} N={N} K={K}")
    y = torch.full((T, N), float("nan"), dtype=torch.float16, device="cuda")
    names = traced(lambda: mq.w4g128_gemm(xd, wp, N, out=y))
    check(y.cpu().numpy(), ref, mag, f"rows {(T, N, K)}")
    assert names in (None, [name]), names


@pytest.mark.parametrize("shape", range(14))
def test_every_gemm_tile_on_ragged_shapes(mq, shape):
    """Each compiled tile forced on: one stage of K or fewer (K = 128 with up to eight K slices),
    slices that end a stage early (K / 64 not a multiple of the slice count), the pipeline's two
    and three stages, rows and columns that end inside a tile, 2-byte stores, one row."""
    mq.tune_set(mq.TUNE_G128_SHAPE, shape)
    try:
        rng = np.random.default_rng(90 + shape)
        for T, N, K in [(1, 32, 128), (9, 40, 256), (33, 300, 384), (70, 264, 1152), (257, 552, 640), (300, 130, 1920)]:
            wq, sc = make_weight(rng, N, K)
            x = (rng.standard_normal((T, K)) * 1.5).astype(np.float16)
            ref, mag = orc.w4g128_linear(x, wq, sc)
            wp = mq.w4g128_prepack(dev(pack_int4(wq)), dev(sc))
            say(f"tile shape {shape} T={T} N={N} K={K}")
            y = torch.full((T, N), float("nan"), dtype=torch.float16, device="cuda")
            mq.w4g128_gemm(dev(x), wp, N, out=y)
            check(y.cpu().numpy(), ref, mag, f"w4g128 tile shape {shape} {(T, N, K)}")
    finally:
        mq.tune_set(mq.TUNE_G128_SHAPE, -1)


def test_output_beyond_2_31_elements(mq):
    """T x N > 2^31 outputs: 64-bit addressing of y, on sampled rows (K = one group)."""
    T, N, K = 70000, 37888, 128
    rng = np.random.default_rng(77)
    say(f"w4g128 T={T} N={N} K={K}")
    wq = rng.integers(-8, 8, size=(N, K), dtype=np.int8)
    sc = rng.uniform(0.002, 0.01, size=(N, 1)).astype(np.float16)
    x = torch.randn((T, K), device="cuda", generator=torch.Generator(device="cuda").manual_seed(3)).half()
    wp = mq.w4g128_prepack(dev(pack_int4(wq)), dev(sc))
    y = torch.full((T, N), 9.0, dtype=torch.float16, device="cuda")
    mq.w4g128_gemm(x, wp, N, out=y)
    torch.cuda.synchronize()
    mark = 2 ** 31 // N
    rows = torch.tensor([0, 127, 128, mark - 1, mark, mark + 1, T - 129, T - 1], device="cuda")
    ref, mag = orc.w4g128_linear(x[rows].cpu().numpy(), wq, sc)
    check(y[rows].cpu().numpy(), ref, mag, "w4g128 beyond 2^31")
    assert not bool((y == 9.0).all(dim=1).any().item())
    del y
    torch.cuda.empty_cache()
