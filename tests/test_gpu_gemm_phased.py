"""The phased 256 x 256 projection GEMM (taken past one round of 256 tiles): two,
four and six k-tiles (its prologue and tail alone, then with its loop), a ragged
last tile of rows, against the oracle on sampled rows and bit for bit against
the 128 x 128 tile, which adds k in the same order; the same for its QKV scatter;
and a shape of one round."""
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


@pytest.mark.parametrize("H,heads,n_tok,kv_tokens,off", [(1024, 16, 4201, 4352, 77), (768, 12, 5504, 5504, 0)])
def test_phased_qkv(orch_lib, monkeypatch, H, heads, n_tok, kv_tokens, off):
    """Past one round of 256 x 256 tiles; the branches meet inside a tile (an odd token
    count and offset: V^T stores off 16 bytes)."""
    B, d, stride = 2, H // heads, 2 * kv_tokens * H + 64
    assert -(-B * n_tok // 256) * (3 * H // 256) > 256
    rng = np.random.default_rng(H)
    A, W, bias = (rng.standard_normal(s, dtype=np.float32) * f for s, f in (((B * n_tok, H), 1), ((3 * H, H), 0.02), ((3 * H,), 0.02)))
    Ad, Wd, bd = to_dev(A, "bf16"), to_dev(W, "bf16"), to_dev(bias)
    outs = []
    for tile in ("0", "2"):
        monkeypatch.setenv("ORCH_GEMM_TILE", tile)
        q, kv = empty((B, heads, n_tok, d), "bf16"), torch.full((B, stride), 7.0, dtype=torch.bfloat16, device=Ad.device)
        orch_lib.qkv_projection(Ad, B, n_tok, H, Wd, bd, H, heads, q, kv, stride, kv_tokens, off, 1)
        outs.append((q, kv))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    q, kv = (to_host(t) for t in outs[0])
    toks = np.r_[np.arange(0, n_tok, 97), n_tok - 1]
    band = slice(off, off + n_tok)
    for b in range(B):
        y = dit.linear(rounded(A[b * n_tok + toks], "bf16"), rounded(W, "bf16"), rounded(bias, "f32"))
        K = kv[b, :kv_tokens * H].reshape(heads, kv_tokens, d)
        V = kv[b, kv_tokens * H:2 * kv_tokens * H].reshape(heads, d, kv_tokens)
        got = (q[b][:, toks].transpose(1, 0, 2), K[:, off + toks].transpose(1, 0, 2), V[:, :, off + toks].transpose(2, 0, 1))
        for g, ref in zip(got, np.split(y, 3, axis=1)):
            assert rel_l2(g.reshape(len(toks), H), ref) <= 5e-3     # as test_qkv_scatter
        # every other token, and what lies past the buffer, is untouched
        assert (np.delete(K, np.r_[band], 1) == 7).all() and (np.delete(V, np.r_[band], 2) == 7).all()
        assert (kv[b, 2 * kv_tokens * H:] == 7).all()
