"""The U-Net band block at the edges of its kernels, against the oracle: slabs of
channel groups in the row sums (one, several, groups that do not split evenly or
hold two or three channels), convolutions of exactly as many k-tiles as their
ring has stages, one more and odd and even counts, and split plans; bounds as in
the parity tests."""
import numpy as np
import pytest
import torch

from oracle import unet
from oracle.blob import bf16_to_float
from seeded_inputs import configs, generate
from tests._gpu_util import DEV, rel_l2, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,C,G,Co,rb,re", [
    (16, 64, 32, 64, 3, 10),       # nine k-tiles, two channels a group
    (10, 192, 64, 64, 0, 10),      # three channels a group: slabs of 96 not cut at 16 lanes
    (8, 64, 1, 320, 0, 8),         # one group
    (12, 640, 32, 320, 2, 3),      # four slabs; one row, split plan
    (9, 1152, 6, 128, 1, 8),       # six groups of 192: slabs of one or more groups
    (24, 128, 8, 384, 5, 20),      # 128-channel tile, eighteen k-tiles
])
@pytest.mark.parametrize("refresh", [0, 1])
def test_unet_edges(orch_lib, side, C, G, Co, rb, re, refresh):
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
    ws = torch.empty(orch_lib.unet_conv_workspace_bytes(shape, re - rb), dtype=torch.uint8, device=DEV)
    out = torch.full((re - rb, side, Co), float("nan"), device=DEV)
    orch_lib.unet_conv_band(shape, rb, re, torch.from_numpy(x[rb:re].copy()).to(DEV), dev["gamma"], dev["beta"],
                            bits(pr["weight_bits"]), dev["bias"], act_d, sums_d, refresh, out, ws)
    ref = unet.band_step(params, x[rb:re].astype(np.float64), side, rb, re, G, bf16_to_float(act).astype(np.float64),
                         sums.astype(np.float64), 1e-5)
    assert rel_l2(to_host(out), ref["out"]) <= 1e-2
    if refresh:
        assert rel_l2(to_host(sums_d)[rb:re], ref["sums"]) <= 1e-5
        assert rel_l2(to_host(act_d)[rb:re], ref["act"]) <= 1e-2
