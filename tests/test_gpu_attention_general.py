"""Attention over fresh + stale K/V for the head sizes and types of the
general matrix-core kernel, against the oracle: every head size, one, two and
four key groups per workgroup (few, some and many queries; fp32 one or two), key counts that
leave a key group without a tile, bands that start and end inside a 32-key
tile, and shapes that keep the scalar kernel (key counts and bands that do not
allow 16-byte loads).

Tolerances: fp32 1e-5 as for the scalar kernel.  bf16 2.2e-3: the result is
rounded once to 8 significant bits (2-norm at most 2^-9 / sqrt(3) x 1.5 =
1.7e-3 over the mantissa's range); the probabilities keep 16 bits.
"""
import numpy as np
import pytest
import torch

from tests._gpu_util import empty, to_dev
from tests.test_gpu_kernels import _attention_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 32), ("bf16", 64), ("bf16", 80), ("bf16", 96), ("bf16", 128), ("f32", 32),
                                     ("f32", 64), ("f32", 72), ("f32", 80), ("f32", 96), ("f32", 128)])
@pytest.mark.parametrize("heads,n_q,n_kv,fb,nf", [
    (4, 1, 64, 0, 0),          # one query, two key tiles
    (2, 33, 1024, 40, 936),    # four key groups; band edges inside key tiles
    (16, 521, 224, 24, 8),     # two key groups, seven key tiles
    (16, 1100, 256, 0, 256),   # one key group, every key fresh
    (2, 40, 104, 8, 40),       # n_kv not a multiple of 32: scalar kernel
    (2, 40, 128, 3, 41),       # band not on 16 bytes: scalar kernel
])
def test_attention_general(orch_lib, dtype, d, heads, n_q, n_kv, fb, nf):
    print(f"\n[{dtype} d {d} heads {heads} n_q {n_q} n_kv {n_kv} band {fb}+{nf}]", flush=True)
    err = _attention_case(orch_lib, dtype, 2, heads, d, n_q, n_kv, fb, nf, seed=n_q + n_kv + d)
    print(f"  rel-L2 {err:.2e}", flush=True)
    # (64 channels, 1100 queries: past the general kernel's range, probabilities rounded)
    assert err <= (1e-5 if dtype == "f32" else 1e-2 if d == 64 and n_q > 1000 else 2.2e-3), err


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 72)])
@pytest.mark.parametrize("k_ramp,shift", [(12.0, 0.0), (0.0, 48.0)])
def test_attention_general_running_max(orch_lib, dtype, d, k_ramp, shift):
    """Scores that grow along the keys (the running max is raised again and
    again) and scores with a large common offset."""
    err = _attention_case(orch_lib, dtype, 2, 4, d, 96, 1024, 256, 96, seed=d, k_ramp=k_ramp, shift=shift)
    # fp32 and the offset: every score passes 48^2 = 2304 at its first channel,
    # and each of the other 71 products rounds it by up to 2^-13 (2-norm 2^-13 /
    # sqrt(3)): sqrt(71 / 3) 2^-13 / sqrt(72) = 7e-5 in the exponent of every
    # probability; twice that.  Else 1e-5 as above, doubled for scores 13 times
    # as large at the ramp's end.
    tol = 2.2e-3 if dtype == "bf16" else 1.4e-4 if shift else 2e-5
    print(f"  rel-L2 {err:.2e}", flush=True)
    assert err <= tol, err


@pytest.mark.parametrize("d", [32, 64, 72, 80, 96, 128])
@pytest.mark.parametrize("n_kv,fb,nf", [(32, 0, 0), (96, 8, 40), (160, 0, 0), (224, 4, 4), (256, 64, 64)])     # 1, 3, 5, 7, 8 key tiles
def test_fp32_query_does_not_depend_on_query_count(orch_lib, d, n_kv, fb, nf):
    """The same bits for a query alone, among few and among thousands."""
    heads, n_q, rng = 4, 9000, np.random.default_rng(d + n_kv)
    H = heads * d
    q, stale, fresh = (to_dev(rng.standard_normal(s) * 0.7) for s in ((heads, n_q, d), (2 * n_kv * H,), (2 * max(nf, 1) * H,)))
    outs = []
    for n in (1, 40, 600, n_q):
        out = empty((n, H))
        orch_lib.attention(q[:, :n].contiguous(), stale, 2 * n_kv * H, fresh, 2 * max(nf, 1) * H, fb, nf, 1, heads, n,
                           n_kv, d, out, 0)
        outs.append(out)
    for out in outs[:-1]:
        assert torch.equal(out, outs[-1][:out.shape[0]]), out.shape
