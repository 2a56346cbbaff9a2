"""The phased 256 x 256 projection GEMM (taken past one round of 256 tiles): two,
four and six k-tiles (its prologue and tail alone, then with its loop), a ragged
last tile of rows, against the oracle on sampled rows and bit for bit against
the 128 x 128 tile, which adds k in the same order; and a shape of one round."""
import numpy as np
import pytest
import torch

from oracle import dit
from tests._gpu_util import empty, rel_l2, rounded, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [(8200, 128, 2048), (4100, 256, 4096), (8450, 384, 2048), (2047, 256, 768)])
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_phased_tile(orch_lib, monkeypatch, M, K, N, epi):
    rng = np.random.default_rng(M + K + N + epi)
    A, W, bias = (rng.standard_normal(s, dtype=np.float32) * f for s, f in (((M, K), 1), ((N, K), 0.02), ((N,), 0.02)))
    gate, h0 = rng.standard_normal((2, N)) * 0.5, rng.standard_normal((M, N), dtype=np.float32)
    rpb = (M + 1) // 2
    Ad, Wd, bd = to_dev(A, "bf16"), to_dev(W, "bf16"), to_dev(bias)
    outs = []
    for tile in ("0", "2"):
        monkeypatch.setenv("ORCH_GEMM_TILE", tile)
        out = to_dev(h0) if epi == 2 else empty((M, N), "bf16")
        orch_lib.linear(Ad, M, K, Wd, N, bd, epi, to_dev(gate) if epi == 2 else None, N, rpb, out, 1)
        outs.append(out)
    assert torch.equal(outs[0], outs[1])
    rows = np.r_[np.arange(0, M, 61), M - 1]
    y = dit.linear(rounded(A[rows], "bf16"), rounded(W, "bf16"), rounded(bias, "f32"))
    got = to_host(outs[0])[rows]
    if epi == 2:
        got, ref = got - rounded(h0[rows], "f32"), rounded(gate, "f32")[rows // rpb] * y
    else:
        ref = dit.gelu_tanh(y) if epi == 1 else y
    assert rel_l2(got, ref) <= (2e-5 if epi == 2 else 5e-3)     # as test_linear
