"""The K-sliced W4A8 GEMM (w4a8_sliced.hip), every compiled tile forced in turn, against the
oracle: int32 accumulators and fp16 bits on the static and per-token epilogues, the split
epilogue within the tolerance of its order of summation, groups of linears in one launch."""
import sys

import numpy as np
import pytest

from oracle import mquant_oracle as orc

torch = pytest.importorskip("torch")
from kernel_trace import traced

pytestmark = pytest.mark.gpu

TILES = 11


@pytest.fixture(scope="module")
def mq():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2502_00425_amd import binding
    return binding


@pytest.fixture
def forced(mq):
    def force(tile):
        mq.tune_set(mq.TUNE_GEMM_SHAPE, tile)
    yield force
    mq.tune_set(mq.TUNE_GEMM_SHAPE, -1)


def say(msg):
    print(f"[parity-sliced] {msg}", flush=True)
    sys.stdout.flush()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def bits(t):
    return t.cpu().numpy().view(np.uint16)


# one k-block (fewer than the K slices), slices that end a stage early, the pipeline's two and
# three stages, rows and columns that end inside a tile, 2-byte stores (N % 8 != 0), one row
SHAPES = [(1, 32, 128), (17, 40, 256), (33, 300, 384), (70, 264, 1152), (257, 552, 640), (300, 130, 1920)]


@pytest.mark.parametrize("tile", range(TILES))
def test_static_and_row_scale_bits(mq, forced, tile):
    forced(tile)
    rng = np.random.default_rng(500 + tile)
    for T, N, K in SHAPES:
        say(f"tile {tile} T={T} N={N} K={K}")
        xq = rng.integers(-128, 128, size=(T, K), dtype=np.int8)
        packed = rng.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
        w_scale = rng.uniform(0.005, 0.02, size=N).astype(np.float16)
        V = T // 3
        acc_want = orc.gemm_i8_i4_i32(xq, orc.unpack_w4(packed))
        _, want = orc.dequant(acc_want, V, 0.07, 0.009, w_scale)
        wp, ws = mq.w4_prepack(dev(packed)), dev(w_scale)
        acc = torch.full((T, N), -7, dtype=torch.int32, device="cuda")
        nan = lambda: torch.full((T, N), float("nan"), dtype=torch.float16, device="cuda")
        y = mq.w4a8_gemm(dev(xq), wp, ws, N, V, 0.07, 0.009, out=nan(), acc_out=acc)
        assert (acc.cpu().numpy() == acc_want).all(), (tile, T, N, K)
        y2 = mq.w4a8_gemm(dev(xq), wp, ws, N, V, 0.07, 0.009, out=nan())
        assert (bits(y) == want.view(np.uint16)).all() and (bits(y2) == want.view(np.uint16)).all(), (tile, T, N, K)
        rows = rng.uniform(0.004, 0.1, size=T).astype(np.float32)
        _, want_r = orc.dequant_rows(acc_want, rows, w_scale)
        y3 = mq.w4a8_gemm_rowscale(dev(xq), wp, ws, dev(rows), N, out=nan())
        assert (bits(y3) == want_r.view(np.uint16)).all(), (tile, T, N, K)


@pytest.mark.parametrize("tile", range(TILES))
def test_split_epilogue(mq, forced, tile):
    """1e-3 of the magnitude of the added terms, as for the other kernels of this entry point."""
    forced(tile)
    rng = np.random.default_rng(600 + tile)
    for T, N, K, n_split in [(19, 96, 256, 1), (75, 300, 1024, 64), (200, 264, 640, 5)]:
        say(f"split tile {tile} T={T} N={N} K={K} n={n_split}")
        xq = rng.integers(-128, 128, size=(T, K), dtype=np.int8)
        wq = rng.integers(-8, 8, size=(N, K), dtype=np.int8)
        idx = np.sort(rng.choice(K, n_split, replace=False)).astype(np.int32)
        wq[:, idx] = 0
        wsplit = rng.integers(-8, 8, size=(n_split, N), dtype=np.int8)
        ssplit = rng.uniform(0.02, 0.3, n_split).astype(np.float32)
        w_scale = rng.uniform(0.005, 0.02, size=N).astype(np.float16)
        u = (wq.astype(np.int16) & 0xF).astype(np.uint8)
        wp = mq.w4_prepack(dev((u[:, 0::2] | (u[:, 1::2] << 4)).astype(np.uint8)))
        V = T // 3
        acc = orc.gemm_i8_i4_i32(xq, wq)
        ref, _ = orc.dequant_rms(acc, xq, V, 0.11, 0.004, w_scale, idx, wsplit, ssplit)
        main, _ = orc.dequant(acc, V, 0.11, 0.004, w_scale)
        mag = np.abs(main) + np.abs(ref - main)
        y = mq.w4a8_gemm_rms(dev(xq), wp, dev(w_scale), N, V, 0.11, 0.004, idx, dev(wsplit), ssplit)
        bad = np.abs(y.cpu().numpy().astype(np.float32) - ref) > 1e-3 * np.maximum(mag, 2.0 ** -14)
        assert not bad.any(), (tile, T, N, K, n_split, int(bad.sum()))


@pytest.mark.parametrize("tile", range(TILES, TILES + 5))
def test_tiles_that_fill_lds(mq, forced, tile):
    """The tiles that take a compute unit's LDS for themselves (three and four stages; 256 x 384), the shapes above."""
    assert mq.lib.mquant_tune_set(mq.TUNE_GEMM_SHAPE, TILES + 5) == mq.ERR_BAD_SHAPE
    test_static_and_row_scale_bits(mq, forced, tile)
    test_split_epilogue(mq, forced, tile)


@pytest.mark.parametrize("T,N,K", [(642, 23944, 1024), (642, 23944, 1152), (1154, 19578, 1024)])
def test_wide_tiles_by_choice(mq, T, N, K):
    """Few rows and short K that the library itself sends to 256 x 384 tiles (16-byte and 2-byte stores; eight and nine
    stages, the last rows and columns inside a tile), static and per-token scales, padding untouched."""
    rng = np.random.default_rng(T + N + K)
    xq = rng.integers(-128, 128, size=(T, K), dtype=np.int8)
    packed = rng.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
    w_scale = rng.uniform(0.005, 0.02, size=N).astype(np.float16)
    acc = orc.gemm_i8_i4_i32(xq, orc.unpack_w4(packed))
    _, want = orc.dequant(acc, T // 3, 0.07, 0.009, w_scale)
    rows = rng.uniform(0.004, 0.1, size=T).astype(np.float32)
    _, want_r = orc.dequant_rows(acc, rows, w_scale)
    wp, ws, xd, rd = mq.w4_prepack(dev(packed)), dev(w_scale), dev(xq), dev(rows)
    buf = torch.full((T, N + 8), 3.0, dtype=torch.float16, device="cuda")
    say(f"wide T={T} N={N} K={K}")
    for call, w in ((lambda: mq.w4a8_gemm(xd, wp, ws, N, T // 3, 0.07, 0.009, out=buf[:, :N]), want),
                    (lambda: mq.w4a8_gemm_rowscale(xd, wp, ws, rd, N, out=buf[:, :N]), want_r)):
        names = traced(call)
        assert names is None or (len(names) == 1 and names[0].startswith("w4a8_wide_kernel<")), names
        assert (bits(buf[:, :N].contiguous()) == w.view(np.uint16)).all()
        assert bool((buf[:, N:] == 3.0).all())


@pytest.mark.parametrize("T,N,K,tile", [(1150, 7676, 1024, "<3, 2,"), (1150, 7672, 1152, "<3, 2,"),
                                        (1010, 10236, 1024, "<2, 3,"), (1010, 10232, 1152, "<2, 3,"),
                                        (526, 10900, 1152, "<2, 2,"), (527, 10912, 1024, "<2, 2,")])
def test_smaller_wide_tiles_by_choice(mq, T, N, K, tile):
    """192 x 256, 128 x 384 and 128 x 256, each with 2-byte and with 16-byte stores, as above."""
    test_wide_tiles_by_choice(mq, T, N, K)
    xq = torch.zeros((T, K), dtype=torch.int8, device="cuda")
    wp = torch.zeros(mq.w4_prepacked_bytes(N, K), dtype=torch.uint8, device="cuda")
    ws = torch.ones(N, dtype=torch.float16, device="cuda")
    names = traced(lambda: mq.w4a8_gemm(xq, wp, ws, N, T // 3, 0.07, 0.009))
    assert names is None or (len(names) == 1 and names[0].startswith("w4a8_wide_kernel" + tile)), names


@pytest.mark.parametrize("T,N,K,tile", [(1150, 7672, 1024, "<3, 2,"), (1010, 10232, 1024, "<2, 3,"), (526, 10904, 1152, "<2, 2,")])
def test_accumulators_of_the_smaller_wide_tiles(mq, T, N, K, tile):
    rng = np.random.default_rng(T + N)
    xq = rng.integers(-128, 128, size=(T, K), dtype=np.int8)
    packed = rng.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
    w_scale = rng.uniform(0.005, 0.02, size=N).astype(np.float16)
    want = orc.gemm_i8_i4_i32(xq, orc.unpack_w4(packed))
    xd, wp, ws = dev(xq), mq.w4_prepack(dev(packed)), dev(w_scale)
    acc = torch.full((T, N), -7, dtype=torch.int32, device="cuda")
    y = torch.empty((T, N), dtype=torch.float16, device="cuda")
    say(f"wide accumulators T={T} N={N} K={K}")
    names = traced(lambda: mq.w4a8_gemm(xd, wp, ws, N, T // 3, 0.07, 0.009, out=y, acc_out=acc))
    assert names is None or (len(names) == 1 and names[0].startswith("w4a8_wide_kernel" + tile)), names
    assert (acc.cpu().numpy() == want).all()
    assert (bits(y) == orc.dequant(want, T // 3, 0.07, 0.009, w_scale)[1].view(np.uint16)).all()


@pytest.mark.parametrize("T", [5, 17, 25, 32])
@pytest.mark.parametrize("K", [128, 3584])
def test_group_of_linears(mq, T, K):
    """The grouped entry: four linears of different widths in one launch, every tile (a forced one takes
    any number of rows) and the library's own choice, against separate calls on the oracle."""
    rng = np.random.default_rng(T + K)
    xq = rng.integers(-128, 128, size=(T, K), dtype=np.int8)
    lin, want = [], []
    for N in (40, 1024, 36, 520):
        packed = rng.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
        w_scale = rng.uniform(0.005, 0.02, size=N).astype(np.float16)
        want.append(orc.dequant(orc.gemm_i8_i4_i32(xq, orc.unpack_w4(packed)), T // 3, 0.07, 0.009, w_scale)[1])
        lin.append((mq.w4_prepack(dev(packed)), dev(w_scale), N, torch.empty((T, N), dtype=torch.float16, device="cuda")))
    try:
        for tile in range(-1, TILES + 5):                # the last, 256 x 384, leaves a group to the one before
            say(f"group T={T} K={K} tile {tile}")
            mq.tune_set(mq.TUNE_GEMM_SHAPE, tile)
            for l in lin:
                l[3].fill_(float("nan"))
            x = dev(xq)
            names = traced(lambda: mq.w4a8_gemv_grouped(x, lin, T // 3, 0.07, 0.009))
            assert names is None or (len(names) == 1 and (tile < 0 or names[0].startswith("w4a8_sliced_kernel<"))), (tile, names)
            for l, w in zip(lin, want):
                assert (bits(l[3]) == w.view(np.uint16)).all(), (tile, l[2])
    finally:
        mq.tune_set(mq.TUNE_GEMM_SHAPE, -1)
