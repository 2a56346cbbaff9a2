"""Infinities in K and V of the general attention kernel, against the oracle: an
infinite value makes its channel infinite (not a NaN) in every query and leaves
the others alone, and keys whose scores are -infinity or the lowest finite number
take no part, also where they fill a key group's first tile.  Tolerances as in the general kernel's tests."""
import numpy as np
import pytest
import torch

from oracle import dit
from tests._gpu_util import DEV, code, empty, rel_l2, rounded, to_dev, to_host

pytestmark = pytest.mark.gpu

INF = float("inf")


def _attend(orch_lib, dtype, heads, d, n_q, n_kv, q, K, V, split=True):
    """One branch through the entry point, every key stale, with the workspace the
    library asks for or without; the result and the oracle's."""
    H = heads * d
    hdr = {"hidden": H, "heads": heads, "grid": 1}
    need = orch_lib.attention_workspace_bytes(1, heads, n_q, n_kv, d, code(dtype)) if split else 0
    ws = torch.empty(need, dtype=torch.uint8, device=DEV) if need else None
    out = empty((1, n_q, H), dtype)
    orch_lib.attention(to_dev(q.reshape(n_q, heads, d).transpose(1, 0, 2), dtype),
                       to_dev(dit.kv_to_buffer_layout(hdr, K, V), dtype), 2 * n_kv * H, None, 0, 0, 0, 1, heads, n_q,
                       n_kv, d, out, code(dtype), workspace=ws)
    return to_host(out)[0], dit.attention(rounded(q, dtype), rounded(K, dtype), rounded(V, dtype), heads)


def _check(got, ref, dtype):
    finite = np.isfinite(ref)
    assert not np.isnan(ref).any()
    np.testing.assert_array_equal(got[~finite], ref[~finite])
    assert rel_l2(got[finite], ref[finite]) <= (1e-5 if dtype == "f32" else 2.2e-3)


# (64 channels without a workspace is the other kernel's)
@pytest.mark.parametrize("dtype,d,split", [("bf16", 32, True), ("bf16", 64, True), ("bf16", 128, True), ("f32", 72, True),
                                           ("bf16", 32, False), ("bf16", 128, False), ("f32", 72, False)])
def test_infinite_values(orch_lib, dtype, d, split):
    """Both signs, one key each; what the first bf16 of a probability leaves is
    zero, positive or negative as the query has it."""
    heads, n_q, n_kv, rng = 8, 70, 256, np.random.default_rng(d)
    q, K, V = (rng.standard_normal((n, heads * d)) * s for n, s in ((n_q, 0.7), (n_kv, 0.7), (n_kv, 1.0)))
    V[17, 3], V[100, d + 7], V[255, heads * d - 1] = INF, -INF, INF
    got, ref = _attend(orch_lib, dtype, heads, d, n_q, n_kv, q, K, V, split)
    assert (~np.isfinite(ref)).sum() == 3 * n_q
    _check(got, ref, dtype)


@pytest.mark.parametrize("dtype,d,n_kv,key", [("f32", 72, 96, 40),     # two groups, three tiles
                                              ("bf16", 80, 160, 130),  # four groups, five tiles: in the full group
                                              ("bf16", 80, 160, 70)])  # and in one that is a tile short
def test_infinite_value_in_short_group(orch_lib, dtype, d, n_kv, key):
    heads, n_q, rng = 4, 33, np.random.default_rng(n_kv)
    q, K, V = (rng.standard_normal((n, heads * d)) * s for n, s in ((n_q, 0.7), (n_kv, 0.7), (n_kv, 1.0)))
    V[key, 5] = INF
    got, ref = _attend(orch_lib, dtype, heads, d, n_q, n_kv, q, K, V)
    _check(got, ref, dtype)


@pytest.mark.parametrize("dtype,d,split", [("bf16", 64, True), ("bf16", 80, True), ("bf16", 128, True), ("f32", 32, True),
                                           ("f32", 72, True), ("bf16", 80, False), ("bf16", 128, False)])
# key ranges (32 keys a tile); the whole range only where a finite score is left
@pytest.mark.parametrize("masked,value", [((32, 64), -INF), ((1, 224), -INF), ((32, 64), -2.9e25), ((1, 224), -3.0e38),
                                          ((224, 256), -1.7e38), ((0, 256), -3.0e38)])
def test_masked_keys(orch_lib, dtype, d, split, masked, value):
    """Keys masked through a channel of their own (1 in Q): scores of -infinity, or
    the lowest ones (every key masked: all alike)."""
    heads, n_q, n_kv, rng = 4, 33, 256, np.random.default_rng(d)
    q, K, V = (rng.standard_normal((n, heads * d)) * s for n, s in ((n_q, 0.7), (n_kv, 0.7), (n_kv, 1.0)))
    q[:, ::d], K[:, ::d] = 1.0, 0.0
    K[masked[0]:masked[1], ::d] = value
    got, ref = _attend(orch_lib, dtype, heads, d, n_q, n_kv, q, K, V, split)
    assert np.isfinite(ref).all()
    _check(got, ref, dtype)
