"""The projection GEMM for few output tiles: every configuration (forced) at one
row and ragged rows, at k-tile counts that leave key groups short or without a
stage, every epilogue, against the oracle; bit for bit against the 128 x 128 tile
where a single group adds all of k; and the choice it is left to at small steps."""
import numpy as np
import pytest
import torch

from oracle import dit
from tests._gpu_util import empty, rel_l2, rounded, to_dev, to_host
from tests.test_gpu_kernels import test_linear, test_qkv_scatter

pytestmark = pytest.mark.gpu

SMALL = range(4, 9)     # ORCH_GEMM_TILE indices of the small configurations
ONE_GROUP = (7, 8)


@pytest.mark.parametrize("tile", SMALL)
@pytest.mark.parametrize("M,K,N", [(1, 128, 64), (95, 384, 192), (130, 640, 128)])
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_small_tiles(orch_lib, monkeypatch, tile, M, K, N, epi):
    monkeypatch.setenv("ORCH_GEMM_TILE", str(tile))
    test_linear(orch_lib, "bf16", M, K, N, epi)


@pytest.mark.parametrize("tile", SMALL)
@pytest.mark.parametrize("H,heads,n_tok,kv_tokens,off", [(384, 6, 40, 256, 16), (1152, 16, 100, 256, 44)])
def test_small_tiles_qkv(orch_lib, monkeypatch, tile, H, heads, n_tok, kv_tokens, off):
    """Branch boundaries inside a block of rows; token offsets off 16 bytes."""
    monkeypatch.setenv("ORCH_GEMM_TILE", str(tile))
    test_qkv_scatter(orch_lib, "bf16", H, heads, n_tok, kv_tokens, off)


@pytest.mark.parametrize("tile", ONE_GROUP)
def test_small_one_group_same_bits(orch_lib, monkeypatch, tile):
    rng = np.random.default_rng(tile)
    M, K, N = 200, 1152, 384
    A, W, b = to_dev(rng.standard_normal((M, K)), "bf16"), to_dev(rng.standard_normal((N, K)) * 0.02, "bf16"), to_dev(rng.standard_normal(N))
    outs = []
    for t in (tile, 2):
        monkeypatch.setenv("ORCH_GEMM_TILE", str(t))
        out = empty((M, N), "bf16")
        orch_lib.linear(A, M, K, W, N, b, 1, None, 0, 1, out, 1)
        outs.append(out)
    assert torch.equal(*outs)


@pytest.mark.parametrize("M,K,N", [(96, 384, 1152), (96, 1536, 384), (384, 1152, 1152), (768, 1152, 1152), (96, 64, 64)])
@pytest.mark.parametrize("ws", [False, True])
def test_small_choice(orch_lib, M, K, N, ws):
    """Shapes of short bands as the launcher chooses, with the workspace the
    library asks for and without."""
    rng = np.random.default_rng(M + K)
    A, W, b = rng.standard_normal((M, K)), rng.standard_normal((N, K)) * 0.02, rng.standard_normal(N)
    need = orch_lib.linear_workspace_bytes(M, N, K, 1)
    out = empty((M, N), "bf16")
    w = torch.empty(need, dtype=torch.uint8, device=out.device) if ws and need else None
    orch_lib.linear(to_dev(A, "bf16"), M, K, to_dev(W, "bf16"), N, to_dev(b), 0, None, 0, 1, out, 1, workspace=w)
    ref = dit.linear(rounded(A, "bf16"), rounded(W, "bf16"), rounded(b, "f32"))
    assert rel_l2(to_host(out), ref) <= 5e-3
