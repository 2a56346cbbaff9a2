"""The fp32 projection GEMM against the oracle at the edges of its tiles and of
its choice of tiles (up to 512 blocks of 32 x 32 outputs, up to 8192, more), with
k-tile counts that leave a group short, for every epilogue, and at shapes that
keep the scalar kernel.  Tolerance as test_linear: fp32 sums of at most 1536
products, 1e-5 (2e-5 where the residual is subtracted again)."""
import numpy as np
import pytest
import torch

from oracle import dit
from tests._gpu_util import DEV, empty, rel_l2, rounded, to_dev, to_host
from tests.test_gpu_kernels import test_linear, test_qkv_scatter

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("epi", [0, 1, 2])
@pytest.mark.parametrize("M,K,N", [(1, 32, 32), (33, 96, 100), (31, 160, 512),    # one, two, many blocks; short groups
                                   (512, 384, 1024), (513, 384, 1024), (999, 96, 608),  # 512 blocks, 544, 608
                                   (4096, 64, 2048), (4100, 64, 2050),                  # 8192 blocks, 8385
                                   (40, 36, 64)])                                       # K % 32: scalar kernel
def test_linear_f32_edges(orch_lib, M, K, N, epi):
    test_linear(orch_lib, "f32", M, K, N, epi)


def test_linear_f32_unaligned(orch_lib):
    """Operands not on 16 bytes take the scalar kernel."""
    rng = np.random.default_rng(5)
    M, K, N = 40, 64, 96
    A, W, b = rng.standard_normal((M, K)), rng.standard_normal((N, K)) * 0.02, rng.standard_normal(N)
    Ad = torch.zeros(M * K + 1, device=DEV)
    Ad[1:] = to_dev(A).reshape(-1)
    out = empty((M, N))
    orch_lib.linear(Ad[1:], M, K, to_dev(W), N, to_dev(b), 0, None, 0, 1, out, 0)
    assert rel_l2(to_host(out), dit.linear(rounded(A, "f32"), rounded(W, "f32"), rounded(b, "f32"))) <= 1e-5


@pytest.mark.parametrize("H,heads,n_tok,kv_tokens,off", [(128, 4, 37, 64, 5), (384, 6, 300, 576, 100)])
def test_qkv_scatter_f32_ragged(orch_lib, H, heads, n_tok, kv_tokens, off):
    """Branch boundaries inside a block of rows, an odd token offset."""
    test_qkv_scatter(orch_lib, "f32", H, heads, n_tok, kv_tokens, off)


@pytest.mark.parametrize("split", [False, True])
def test_fixed_order_stitches_fp32(orch_lib, split):
    """Bands of an fp32 model stitch to the all-rows step bit for bit, whatever
    tiles their heights choose, with the work split off or on."""
    from seeded_inputs import configs, generate
    cfg = configs.scaled(configs.TINY, name="tiny32", latent=32, hidden=256, heads=4, mlp_hidden=1024)
    ctx = orch_lib.DiTStep(cfg, generate.make_weight_blob(cfg, 0))
    x, labels = to_dev(generate.make_latent(cfg, 0)), generate.make_labels(cfg, 0)
    kv = torch.zeros(ctx.stale_kv_bytes() // 4, device=DEV)
    ctx.set_work_split(split)
    full = empty((4, cfg.latent, cfg.latent))
    ctx.step(x, 0, cfg.R, 500, 250, labels, 1.5, kv, 1, full)
    for rb, re in [(0, 1), (1, 6), (6, 16)]:
        out = empty((4, 2 * (re - rb), cfg.latent))
        ctx.step(x, rb, re, 500, 250, labels, 1.5, kv, 0, out)
        assert torch.equal(out, full[:, 2 * rb:2 * re]), (rb, re)
    ctx.close()


@pytest.mark.parametrize("K,N", [(32, 64), (96, 100), (384, 1152), (1184, 384)])     # one, three, twelve, 37 k-tiles
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_row_does_not_depend_on_row_count(orch_lib, K, N, epi):
    """The order of a row's sums is fixed by K: the same bits in calls of one row
    and of some thousands, whatever tile and key groups they take."""
    M = 8300 * 1024 // N + 37     # past 8192 blocks of 32 x 32
    rng = np.random.default_rng(K)
    A, W, b = to_dev(rng.standard_normal((M, K))), to_dev(rng.standard_normal((N, K)) * 0.02), to_dev(rng.standard_normal(N))
    gate, h = to_dev(rng.standard_normal((1, N))), to_dev(rng.standard_normal((M, N)))
    outs = []
    for m in (1, 33, 500, 600 * 1024 // N, M):
        out = h[:m].clone() if epi == 2 else empty((m, N))
        orch_lib.linear(A, m, K, W, N, b, epi, gate if epi == 2 else None, N, m, out, 0)
        outs.append(out)
    for out in outs[:-1]:
        assert torch.equal(out, outs[-1][:out.shape[0]]), out.shape
