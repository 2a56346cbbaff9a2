"""The U-Net band block at the edges of its kernels, against the oracle: slabs of
channel groups in the row sums (one, several, groups that do not split evenly or
hold two or three channels) and, in each of the convolution's three tiles, splits of as many
k-tiles as the ring has stages (four; the 64-channel tile's three never), one more and both at
once, and partial pixel tiles, one and several.  The split is read off the workspace; which tile a shape takes follows from
the launch plan's estimate.  Bounds as in the parity tests."""
import numpy as np
import pytest
import torch

from oracle import unet
from oracle.blob import bf16_to_float
from seeded_inputs import configs, generate
from tests._gpu_util import DEV, rel_l2, to_host

pytestmark = pytest.mark.gpu


def _al256(b):
    return (b + 255) // 256 * 256


@pytest.mark.parametrize("side,C,G,Co,rb,re,splits", [
    # 64-channel tiles (three stages)
    (16, 64, 32, 64, 3, 10, 2),      # splits of four and five k-tiles; two channels a group
    (10, 192, 64, 64, 0, 10, 6),     # three channels a group, one slab
    (8, 64, 1, 320, 0, 8, 2),        # one group
    (12, 640, 32, 320, 2, 3, 16),    # four slabs, one row
    (9, 1152, 6, 128, 1, 8, 16),     # six slabs of one group, 192 channels
    (24, 128, 8, 384, 5, 20, 3),     # splits of six; three pixel tiles, the last partial
    # 128-channel tiles (four stages)
    (16, 256, 32, 2304, 0, 2, 9),    # splits of four k-tiles: the drain alone
    (8, 512, 32, 1280, 2, 3, 16),    # four and five
    (12, 320, 32, 1280, 0, 12, 9),   # five; two pixel tiles, the last partial
    # 160-channel tiles (four stages)
    (8, 512, 32, 1600, 3, 4, 16),    # four and five
    (12, 320, 32, 1600, 1, 12, 9),   # five; two pixel tiles, the last partial
])
@pytest.mark.parametrize("refresh", [0, 1])
def test_unet_edges(orch_lib, side, C, G, Co, rb, re, splits, refresh):
    cfg = configs.UNetConvConfig("edge", side, side, C, G, Co)
    pr = generate.make_unet_params(cfg, 0)
    params = {k: v.astype(np.float64) for k, v in pr.items() if k != "weight_bits"}
    params["weight"] = bf16_to_float(pr["weight_bits"]).astype(np.float64)
    x, old = generate.make_unet_input(cfg, 0), generate.make_unet_input(cfg, 1)
    act = generate.f32_to_bf16_bits(unet.full_step(params, old.astype(np.float64), G)["act"].astype(np.float32))
    sums = unet.row_group_sums(old, G).astype(np.float32)
    shape = orch_lib.unet_shape(cfg, 1e-5)
    dev = {k: torch.from_numpy(v).to(DEV) for k, v in pr.items() if k != "weight_bits"}

    def bits(b):
        return torch.from_numpy(np.ascontiguousarray(b).view(np.int16)).to(DEV).view(torch.bfloat16)
    act_d, sums_d = bits(act), torch.from_numpy(sums).to(DEV)
    r, need = re - rb, orch_lib.unet_conv_workspace_bytes(shape, re - rb)
    assert need == (_al256(r * G * 8) + _al256((r + 2) * (side + 2) * C * 2)
                    + (_al256(splits * r * side * Co * 4) if splits > 1 else 0))
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    out = torch.full((re - rb, side, Co), float("nan"), device=DEV)
    orch_lib.unet_conv_band(shape, rb, re, torch.from_numpy(x[rb:re].copy()).to(DEV), dev["gamma"], dev["beta"],
                            bits(pr["weight_bits"]), dev["bias"], act_d, sums_d, refresh, out, ws)
    ref = unet.band_step(params, x[rb:re].astype(np.float64), side, rb, re, G, bf16_to_float(act).astype(np.float64),
                         sums.astype(np.float64), 1e-5)
    assert rel_l2(to_host(out), ref["out"]) <= 1e-2
    if refresh:
        assert rel_l2(to_host(sums_d)[rb:re], ref["sums"]) <= 1e-5
        assert rel_l2(to_host(act_d)[rb:re], ref["act"]) <= 1e-2
