"""The kernels before and after a step's blocks at the edges of their tiles,
against the oracle: a single row of eight tokens (half a tile of the final
linear), odd branch boundaries inside a tile, a patch-embedding output on four
bytes, and sinusoids of two, 1024 and more channels.  Tolerances as in the
kernel tests (fp32 results 1e-6 to 1e-5; the bf16 final layer 1e-2)."""
import numpy as np
import pytest
import torch

from oracle import blob as oblob
from oracle import dit
from seeded_inputs import configs, generate
from tests._gpu_util import DEV, empty, rel_l2, rounded, to_dev, to_host

pytestmark = pytest.mark.gpu


def _model(orch_lib, **kw):
    cfg = configs.scaled(configs.TINY, name="edge", **kw)
    blob = generate.make_weight_blob(cfg, 0)
    hdr, params = oblob.read_blob(blob)
    return cfg, orch_lib.DiTStep(cfg, blob), hdr, params


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("hidden,B,rb,re", [(128, 1, 7, 8), (128, 2, 0, 1), (640, 2, 2, 5), (1152, 1, 0, 8)])
def test_final_layer_edges(orch_lib, dtype, hidden, B, rb, re):
    cfg, ctx, hdr, params = _model(orch_lib, dtype=dtype, hidden=hidden, heads=hidden // 64 if hidden < 1152 else 16,
                                   cfg_batch=B, mlp_hidden=128)
    n_tok, H, L = (re - rb) * cfg.R, hidden, cfg.n_blocks
    rng = np.random.default_rng(hidden + rb)
    h, mod = rng.standard_normal((B, n_tok, H)), rng.standard_normal((B, 6 * H * L + 2 * H)) * 0.1
    out = empty((B, 4, 2 * (re - rb), cfg.latent))
    ctx.final_layer(to_dev(h), rb, re, to_dev(mod), out)
    hr, mr = rounded(h, "f32"), rounded(mod, "f32")
    for b in range(B):
        y = dit.final_layer(hdr, params, hr[b], mr[b, -2 * H:-H], mr[b, -H:])
        err = rel_l2(to_host(out)[b], dit.unpatchify_rows(hdr, y, re - rb))
        assert err <= (1e-6 if dtype == "f32" else 1e-2), (b, err)


@pytest.mark.parametrize("hidden,B,rb,re,shift", [(128, 1, 7, 8, 0), (640, 2, 2, 5, 1), (1152, 2, 0, 8, 3)])
def test_patch_embed_edges(orch_lib, hidden, B, rb, re, shift):
    cfg, ctx, hdr, params = _model(orch_lib, hidden=hidden, heads=hidden // 64 if hidden < 1152 else 16, cfg_batch=B,
                                   mlp_hidden=128)
    x = generate.make_latent(cfg, 0)
    n = (re - rb) * cfg.R
    buf = torch.full((B * n * hidden + 8,), float("nan"), device=DEV)
    ctx.patch_embed(to_dev(x), rb, re, buf[shift:])
    ref = dit.patch_embed(hdr, params, x.astype(np.float64), rb, re)
    got = to_host(buf)
    assert np.isnan(got[:shift]).all() and np.isnan(got[shift + B * n * hidden:]).all()
    for b, g in enumerate(got[shift:shift + B * n * hidden].reshape(B, n, hidden)):
        assert rel_l2(g, ref) <= 1e-6, b


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("freq_dim,hidden,heads,B", [(2, 128, 4, 1), (1024, 128, 4, 2), (1030, 640, 10, 2),
                                                     (256, 2048, 16, 2)])
def test_conditioning_edges(orch_lib, dtype, freq_dim, hidden, heads, B):
    cfg, ctx, hdr, params = _model(orch_lib, dtype=dtype, freq_dim=freq_dim, hidden=hidden, heads=heads, cfg_batch=B,
                                   mlp_hidden=128)
    labels, H, L = generate.make_labels(cfg, 0), hidden, cfg.n_blocks
    out = empty((B, 6 * H * L + 2 * H))
    ctx.conditioning(777, labels, out)
    blocks, fin = dit.adaln_vectors(hdr, params, dit.conditioning(hdr, params, 777, labels))
    ref = np.concatenate([np.concatenate(blk, axis=1) for blk in blocks] + list(fin), axis=1)
    assert rel_l2(to_host(out), ref) <= 1e-5
