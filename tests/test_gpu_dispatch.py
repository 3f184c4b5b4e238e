"""Which kernel a shape is sent to: the lines between the forms of a linear, at shapes where the
wrong side of a line was measured clearly slower.  Names come from a trace of the call."""
import sys

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
