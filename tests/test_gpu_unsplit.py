"""Without a workspace the kernel-level entry points run unsplit: the order of an
output's sums is fixed by its own operands, so a row of a call has the same
bits however many rows the call has.  (bf16; fp32 in the fp32 kernels' tests.)"""
import numpy as np
import pytest
import torch

from tests._gpu_util import empty, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,N", [(64, 128), (384, 1536), (1536, 384), (1152, 1152)])
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_linear_row(orch_lib, K, N, epi):
    """Few rows (where waves would share K) to several rounds of tiles."""
    M, rng = 9000, np.random.default_rng(K + N)
    A, W = to_dev(rng.standard_normal((M, K)), "bf16"), to_dev(rng.standard_normal((N, K)) * 0.02, "bf16")
    b, gate, h = (to_dev(rng.standard_normal(s)) for s in ((N,), (1, N), (M, N)))
    outs = []
    for m in (1, 40, 96, 700, M):
        out = h[:m].clone() if epi == 2 else empty((m, N), "bf16")
        orch_lib.linear(A, m, K, W, N, b, epi, gate if epi == 2 else None, N, m, out, 1)
        outs.append(out)
    for out in outs[:-1]:
        assert torch.equal(out, outs[-1][:out.shape[0]]), out.shape


@pytest.mark.parametrize("H,heads", [(384, 6), (1152, 16)])
def test_qkv_row(orch_lib, H, heads):
    n, d, rng = 2304, H // heads, np.random.default_rng(H)
    A, W = to_dev(rng.standard_normal((n, H)), "bf16"), to_dev(rng.standard_normal((3 * H, H)) * 0.02, "bf16")
    b = to_dev(rng.standard_normal(3 * H))
    outs = []
    for m in (8, 96, n):
        q, kv = empty((heads, m, d), "bf16"), torch.zeros(2 * n * H, dtype=torch.bfloat16, device=A.device)
        orch_lib.qkv_projection(A, 1, m, H, W, b, H, heads, q, kv, 2 * n * H, n, 0, 1)
        outs.append((q, kv[:n * H].reshape(heads, n, d)[:, :m], kv[n * H:].reshape(H, n)[:, :m]))
    for m, out in zip((8, 96), outs):
        q, k, v = outs[-1]
        assert torch.equal(out[0], q[:, :m]) and torch.equal(out[1], k[:, :m]) and torch.equal(out[2], v[:, :m]), m


@pytest.mark.parametrize("M,N,K", [(96, 1536, 384), (96, 384, 1536), (200, 768, 768)])
def test_linear_workspace_is_the_leave(orch_lib, M, N, K):
    """Where waves would share K the entry point asks for a workspace, and less of it
    than asked for is none."""
    need = orch_lib.linear_workspace_bytes(M, N, K, 1)
    assert need > 0
    rng = np.random.default_rng(M + N)
    A, W = to_dev(rng.standard_normal((M, K)), "bf16"), to_dev(rng.standard_normal((N, K)) * 0.02, "bf16")
    b, outs = to_dev(rng.standard_normal(N)), []
    for bytes_ in (0, 8, need):
        out = empty((M, N), "bf16")
        w = torch.empty(bytes_, dtype=torch.uint8, device=A.device) if bytes_ else None
        orch_lib.linear(A, M, K, W, N, b, 0, None, 0, 1, out, 1, workspace=w)
        outs.append(out.float())
    assert torch.equal(outs[0], outs[1])
    # two roundings to bf16 of the same sums
    assert float((outs[0] - outs[2]).norm() / outs[0].norm()) <= 2 * 2.0 ** -9


@pytest.mark.parametrize("d", [32, 64, 72, 80, 96, 128])
@pytest.mark.parametrize("n_kv,fb,nf", [(64, 0, 0), (576, 64, 64), (1024, 0, 0)])
def test_attention_query(orch_lib, d, n_kv, fb, nf):
    """Few queries (where waves would share their keys) to many."""
    heads, n_q, rng = 6, 3000, np.random.default_rng(d + n_kv)
    H = heads * d
    q, stale, fresh = (to_dev(rng.standard_normal(s) * 0.7, "bf16")
                       for s in ((heads, n_q, d), (2 * n_kv * H,), (2 * max(nf, 1) * H,)))
    outs = []
    for n in (1, 96, 700, n_q):
        out = empty((n, H), "bf16")
        orch_lib.attention(q[:, :n].contiguous(), stale, 2 * n_kv * H, fresh, 2 * max(nf, 1) * H, fb, nf, 1, heads, n,
                           n_kv, d, out, 1)
        outs.append(out)
    for out in outs[:-1]:
        assert torch.equal(out, outs[-1][:out.shape[0]]), out.shape


@pytest.mark.parametrize("d", [32, 64, 80, 128])
def test_attention_workspace_is_the_leave(orch_lib, d):
    heads, n_q, n_kv, rng = 6, 96, 256, np.random.default_rng(d)
    H, need = heads * d, orch_lib.attention_workspace_bytes(1, heads, n_q, n_kv, d, 1)
    assert need > 0
    q, stale = (to_dev(rng.standard_normal(s) * 0.7, "bf16") for s in ((heads, n_q, d), (2 * n_kv * H,)))
    outs = []
    for bytes_ in (0, 8, need):
        out = empty((n_q, H), "bf16")
        w = torch.empty(bytes_, dtype=torch.uint8, device=q.device) if bytes_ else None
        orch_lib.attention(q, stale, 2 * n_kv * H, None, 0, 0, 0, 1, heads, n_q, n_kv, d, out, 1, workspace=w)
        outs.append(out.float())
    assert torch.equal(outs[0], outs[1])
    # 1e-2 as between the attention kernels and the oracle
    assert float((outs[0] - outs[2]).norm() / outs[0].norm()) <= 1e-2
