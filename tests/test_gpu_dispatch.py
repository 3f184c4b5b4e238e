"""Which kernel a shape is sent to: the lines between the forms of a linear, at shapes where the
wrong side of a line was measured clearly slower.  Names come from a trace of the call."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
from kernel_trace import kernels

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mq():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2502_00425_amd import binding
    return binding


def say(msg):
    print(f"[dispatch] {msg}", flush=True)
    sys.stdout.flush()


def weight_only(mq, T, N, K):
    say(f"weight-only T={T} N={N} K={K}")
    x = torch.zeros((T, K), dtype=torch.float16, device="cuda")
    wp = torch.zeros(mq.w4g128_prepacked_bytes(N, K), dtype=torch.uint8, device="cuda")
    y = torch.empty((T, N), dtype=torch.float16, device="cuda")
    return kernels(lambda: mq.w4g128_gemm(x, wp, N, out=y))


@pytest.mark.parametrize("T,N,K,name", [
    (1, 37888, 128, "w4g128_gemv_kernel"), (4, 37888, 128, "w4g128_gemv_kernel"),     # 4.2 / 4.6 and 4.3 / 6.0 us
    (4, 18944, 256, "w4g128_gemv_kernel"), (2, 4096, 128, "w4g128_gemv_kernel"),      # 3.2 / 4.1, 2.7 / 3.0
    (3, 6144, 1536, "w4g128_gemv_kernel"),                                            # 4.2 / 5.4
    (1, 3584, 18944, "w4g128_gemv_half_kernel"), (4, 3584, 18944, "w4g128_gemv_half_kernel"),   # 22.5 / 11.3, 23.3 / 12.4
    (1, 37888, 3584, "w4g128_gemv_half_kernel"), (4, 1024, 1024, "w4g128_gemv_half_kernel"),    # 23.6 / 18.9, 4.2 / 3.3
    (4, 8192, 29568, "w4g128_gemv_kernel"),                                           # rows beyond LDS
])
def test_weight_only_few_rows(mq, T, N, K, name):
    """Whole tiles against half tiles at one to four rows (microseconds whole / half)."""
    got = weight_only(mq, T, N, K)
    assert len(got) == 1 and got[0].startswith(name + "<"), got


@pytest.mark.parametrize("T,N,K,names", [
    (13, 37888, 128, ["w4g128_gemv_kernel"]), (13, 16384, 512, ["w4g128_gemv_kernel"]),          # 4.9 us (15.3 on 64x32 tiles), 3.9 (6.9)
    (16, 1024, 128, ["w4g128_gemv_kernel"]),                                                     # 2.6 (3.0)
    (12, 3584, 18944, ["w4g128_gemv_kernel"]), (13, 3584, 18944, ["w4g128_gemm_kernel<1, 1, 3>"]),
    (32, 18944, 3584, ["w4g128_gemm_kernel<1, 2, 3>"]),                                          # 17.9 (GEMV 27.9)
    (33, 37888, 128, ["w4g128_gemm_kernel<2, 8, 3>"]),                                           # 4.7 (64x32: 16.0)
    (128, 37888, 128, ["w4g128_gemm_kernel<2, 8, 3>", "w4g128_gemm_kernel<4, 8, 2>"]),           # 7.2 and 6.9 (64x32: 31.6)
    (512, 4096, 128, ["w4g128_gemm_kernel<2, 8, 3>", "w4g128_gemm_kernel<2, 4, 3>"]),            # 4.6 and 4.5 (64x32: 13.1)
    (384, 18944, 256, ["w4g128_gemm_kernel<4, 8, 2>"]),                                          # 9.2 (96x128: 17.1)
    (1280, 37888, 3584, ["w4g128_gemm_kernel<8, 8, 3>"]), (1280, 3584, 18944, ["w4g128_gemm_kernel<5, 4, 3>"]),
])
def test_weight_only_rows_and_tiles(mq, T, N, K, names):
    """GEMV against GEMM from 13 rows on, and tiles whose start cost suits the length of K
    (microseconds measured, in brackets the kernel on the other side)."""
    got = weight_only(mq, T, N, K)
    assert len(got) == 1 and any(got[0].startswith(n) for n in names), got


def w4a8(mq, T, N, K):
    say(f"W4A8 T={T} N={N} K={K}")
    xq = torch.zeros((T, K), dtype=torch.int8, device="cuda")
    wp = torch.zeros(mq.w4_prepacked_bytes(N, K), dtype=torch.uint8, device="cuda")
    ws = torch.ones(N, dtype=torch.float16, device="cuda")
    y = torch.empty((T, N), dtype=torch.float16, device="cuda")
    wk = torch.empty(max(mq.w4a8_workspace_bytes(T, N, K), 256), dtype=torch.uint8, device="cuda")
    return kernels(lambda: mq.w4a8_gemm(xq, wp, ws, N, 0, 1.0, 1.0, out=y, workspace=wk))


@pytest.mark.parametrize("T,N,K,name", [
    (48, 18944, 384, "w4a8_gemm_kernel<64, 128,"), (48, 37888, 3584, "w4a8_gemm_kernel<64, 256,"),    # 5.0 (6.9), 21.0 (23.8)
    (64, 18944, 3584, "w4a8_gemm_kernel<64, 128,"), (128, 12288, 1024, "w4a8_gemm_kernel<64, 128,"),  # 16.5 (18.4), 7.5 (8.7)
    (1280, 37888, 128, "w4a8_gemm_kernel<"),                                                          # 25.8 (33.7)
    (48, 3584, 3584, "w4a8_sliced_kernel<"), (128, 3584, 18944, "w4a8_sliced_kernel<"),
    (512, 4608, 3584, "w4a8_sliced_kernel<"), (64, 12288, 4096, "w4a8_sliced_kernel<"),
])
def test_w4a8_prompts(mq, T, N, K, name):
    """Sliced tiles for few output channels, the large-tile kernel where the channels fill the chip
    (microseconds measured, in brackets the sliced tile)."""
    got = w4a8(mq, T, N, K)
    assert len(got) == 1 and got[0].startswith(name), got


@pytest.mark.parametrize("T,N,K,name", [
    (17, 3584, 3584, "w4a8_gemv_kernel"), (24, 4608, 3584, "w4a8_gemv_kernel"),         # 5.3 us (6.6), 5.6 (6.8)
    (32, 3584, 3584, "w4a8_gemv_kernel"), (24, 8192, 8192, "w4a8_gemv_kernel"),         # 5.7 (6.9), 9.6 (11.0)
    (20, 37888, 3584, "w4a8_walk_kernel"), (24, 64, 16384, "w4a8_gemv_kernel"),         # 16.5 (tile GEMV 19.3, GEMM 21.3), 10.4 (12.1)
    (17, 1024, 128, "w4a8_gemv_kernel"),                                                # 2.8 (3.2)
    (24, 3584, 18944, "w4a8_sliced_kernel"), (32, 10240, 8192, "w4a8_sliced_kernel"),   # 17.4 (GEMV 18.2), 14.6 (16.0)
    (32, 59136, 8192, "w4a8_sliced_kernel"), (24, 18944, 384, "w4a8_sliced_kernel"),    # 50.8 (57.4), 4.8 (6.7)
    (32, 32437, 4608, "w4a8_sliced_kernel"),                                            # 18.6 (walking kernel in two rounds 21.4)
])
def test_w4a8_decode_rows_above_sixteen(mq, T, N, K, name):
    """GEMV, a work-group per tile or one per compute unit that walks, against sliced GEMM from 17 to 32 rows (microseconds
    measured, in brackets the other side), in the single and in the grouped entry."""
    got = w4a8(mq, T, N, K)
    assert len(got) == 1 and got[0].startswith(name + "<"), got
    xq = torch.zeros((T, K), dtype=torch.int8, device="cuda")
    wp = torch.zeros(mq.w4_prepacked_bytes(N, K), dtype=torch.uint8, device="cuda")
    lin = [(wp, torch.ones(N, dtype=torch.float16, device="cuda"), N, torch.empty((T, N), dtype=torch.float16, device="cuda"))]
    assert kernels(lambda: mq.w4a8_gemv_grouped(xq, lin, 0, 1.0, 1.0)) == got


@pytest.mark.parametrize("T,N,K", [(3000, 3584, 18944), (646, 5683, 1152), (266, 32142, 1664)])
def test_sliced_gemm_keeps_narrow_margins(mq, T, N, K):
    """Shapes that a margin of 14.5 % instead of 12 would send to large tiles, whose epilogues cost more than the estimates
    know (646 x 1152 -> 5683: static 1.02, per-row scales 1.34, three flagged channels 2.57 of the sliced GEMM's time)."""
    say(f"narrow margin T={T} N={N} K={K}")
    xq = torch.zeros((T, K), dtype=torch.int8, device="cuda")
    wp = torch.zeros(mq.w4_prepacked_bytes(N, K), dtype=torch.uint8, device="cuda")
    ws, rs = torch.ones(N, dtype=torch.float16, device="cuda"), torch.ones(T, device="cuda")
    y = torch.empty((T, N), dtype=torch.float16, device="cuda")
    wk = torch.empty(max(mq.w4a8_workspace_bytes(T, N, K), 256), dtype=torch.uint8, device="cuda")
    split = np.arange(4, dtype=np.int32), torch.zeros((4, N), dtype=torch.int8, device="cuda"), np.ones(4, dtype=np.float32)
    for call in (lambda: mq.w4a8_gemm(xq, wp, ws, N, 0, 1.0, 1.0, out=y, workspace=wk),
                 lambda: mq.w4a8_gemm_rowscale(xq, wp, ws, rs, N, out=y, workspace=wk),
                 lambda: mq.w4a8_gemm_rms(xq, wp, ws, N, 0, 1.0, 1.0, *split, out=y, workspace=wk)):
        got = kernels(call)
        assert len(got) == 1 and got[0].startswith("w4a8_sliced_kernel<"), got


def w4a8_as(mq, epi, T, N, K):
    """Kernels of one linear with static scales, per-row scales or that many flagged channels."""
    say(f"W4A8 {epi} T={T} N={N} K={K}")
    xq = torch.zeros((T, K), dtype=torch.int8, device="cuda")
    wp = torch.zeros(mq.w4_prepacked_bytes(N, K), dtype=torch.uint8, device="cuda")
    ws, rs = torch.ones(N, dtype=torch.float16, device="cuda"), torch.ones(T, device="cuda")
    y = torch.empty((T, N), dtype=torch.float16, device="cuda")
    wk = torch.empty(max(mq.w4a8_workspace_bytes(T, N, K), 256), dtype=torch.uint8, device="cuda")
    if epi == "static":
        return kernels(lambda: mq.w4a8_gemm(xq, wp, ws, N, 0, 1.0, 1.0, out=y, workspace=wk))
    if epi == "row":
        return kernels(lambda: mq.w4a8_gemm_rowscale(xq, wp, ws, rs, N, out=y, workspace=wk))
    split = np.arange(epi, dtype=np.int32), torch.zeros((epi, N), dtype=torch.int8, device="cuda"), np.ones(epi, dtype=np.float32)
    return kernels(lambda: mq.w4a8_gemm_rms(xq, wp, ws, N, 0, 1.0, 1.0, *split, out=y, workspace=wk))


@pytest.mark.parametrize("epi,T,N,K,name", [
    ("static", 65, 16448, 1152, "w4a8_gemm_kernel<64, 128,"), ("static", 2863, 3072, 10624, "w4a8_sliced_kernel<3, 4, 2,"),   # 1.24, 1.19
    ("row", 7763, 1425, 12288, "w4a8_sliced_kernel<3, 4, 2,"), ("static", 495, 11712, 27264, "w4a8_gemm_kernel<256, 256,"),   # 1.19, 1.15
    (1, 985, 6016, 28672, "w4a8_gemm_kernel<256, 256,"), ("row", 1217, 3792, 5760, "w4a8_sliced_kernel<5, 4, 2,"),            # 1.14, 1.10
    (1, 329, 11904, 12416, "w4a8_sliced_kernel<3, 8, 3,"), ("row", 40, 23936, 5120, "w4a8_sliced_kernel<2, 4, 4,"),           # 0.64, 0.75
    ("static", 763, 2285, 18944, "w4a8_sliced_kernel<2, 4, 4,"), ("static", 144, 12480, 11776, "w4a8_sliced_kernel<3, 4, 4,"),  # 0.76, 0.80
    ("row", 662, 3584, 18944, "w4a8_sliced_kernel<3, 4, 4,"), ("static", 457, 13856, 5120, "w4a8_sliced_kernel<4, 8, 3,"),      # 0.96, 0.95
])
def test_tiles_that_have_a_compute_unit_alone(mq, epi, T, N, K, name):
    """The sliced tiles with three and four stages against all others (their time over the other side's: over 1 they are not
    taken)."""
    got = w4a8_as(mq, epi, T, N, K)
    assert got[0].startswith(name) and (len(got) == 1 or got[1].startswith("splitk_reduce_kernel")), got


@pytest.mark.parametrize("epi,T,N,K,name", [
    ("row", 948, 17105, 1024, "w4a8_sliced_kernel<"), ("static", 772, 18764, 1152, "w4a8_sliced_kernel<"),    # 1.62, 1.35
    ("row", 3487, 24077, 1152, "w4a8_wide_kernel<2, 2,"), ("static", 7730, 13814, 1536, "w4a8_wide_kernel<2, 2,"),   # 1.36, 1.27
    ("row", 4523, 3861, 1152, "w4a8_gemm_kernel<192, 128,"), ("row", 5691, 14208, 1792, "w4a8_wide_kernel<2, 2,"),   # 1.10, 1.14
    ("static", 1280, 37888, 3584, "w4a8_wide_kernel<4, 3,"), ("row", 1280, 37888, 3584, "w4a8_wide_kernel<4, 3,"),   # 0.94, 0.96
    ("static", 4096, 4608, 3584, "w4a8_wide_kernel<4, 3,"), ("row", 2048, 10240, 8192, "w4a8_wide_kernel<4, 3,"),    # 0.90, 0.90
    ("static", 4096, 37888, 3584, "w4a8_wide_kernel<4, 3,"),                                                  # 0.96
])
def test_largest_tile(mq, epi, T, N, K, name):
    """256 x 384 against the sliced GEMM and the tiles of one and two work-groups to a compute unit (its time over the other
    side's: over 1 it is not taken)."""
    got = w4a8_as(mq, epi, T, N, K)
    assert len(got) == 1 and got[0].startswith(name), got


@pytest.mark.parametrize("epi,T,N,K,name", [
    ("row", 1329, 52928, 3968, "w4a8_wide_kernel<2, 2,"), ("static", 1289, 16796, 3584, "w4a8_wide_kernel<2, 2,"),   # 1.09, 1.06
    ("row", 1795, 18020, 3072, "w4a8_wide_kernel<2, 2,"), ("row", 6579, 4992, 3456, "w4a8_wide_kernel<2, 2,"),       # 1.07, 1.07
    ("static", 900, 10240, 8192, "w4a8_wide_kernel<3, 2,"), ("static", 2048, 4608, 3584, "w4a8_wide_kernel<2, 3,"),  # 0.82, 0.85
])
def test_smaller_large_tiles(mq, epi, T, N, K, name):
    """192 x 256 and 128 x 384 against 128 x 256 (their time over the other side's: over 1 they are not taken)."""
    got = w4a8_as(mq, epi, T, N, K)
    assert len(got) == 1 and got[0].startswith(name), got
