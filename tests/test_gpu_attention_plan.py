"""Attention whose work plan lengthens the workgroups' ranges to a divisor of a
query tile's key tiles (every part then starts and ends with a workgroup), and
its neighbours whose ranges still cross tiles, against the oracle; 1e-2 as the
other attention tests."""
import numpy as np
import pytest

from tests.test_gpu_kernels import _attention_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,heads,d,n_q,n_kv,fb,nf", [
    (2, 16, 72, 384, 4096, 1920, 384),    # 12 -> 16 of 64 key tiles
    (2, 16, 72, 300, 1024, 8, 296),       # 3 -> 4 of 16, a ragged query tile
    (1, 16, 72, 384, 4096, 0, 384),       # 6 -> 8
    (2, 16, 72, 640, 4096, 64, 640),      # 20, not 32: ranges cross tiles
    (1, 6, 64, 1024, 4096, 0, 1024),      # 64 channels
    (1, 10, 64, 880, 6400, 0, 880),       # 14, not 20 of 100
    (2, 16, 72, 96, 64 * 61, 8, 96),      # 61 key tiles: no divisor near
])
def test_attention_plan(orch_lib, B, heads, d, n_q, n_kv, fb, nf):
    rows = np.r_[np.arange(0, n_q, 29), n_q - 1]
    err = _attention_case(orch_lib, "bf16", B, heads, d, n_q, n_kv, fb, nf, seed=n_q + n_kv, sample_rows=rows)
    assert err <= 1e-2, err
