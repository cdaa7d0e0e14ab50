"""Tiles whose K steps two groups of waves share, on either side of the line past which one row tile reads its weights all of a step at once
(tile_rules.hpp: reads_weights_past_l2): one row tile and two, weights below and above it, every kind of output of the operators."""
import numpy as np
import pytest
import torch

from oracle import eet_oracle as orc
from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, gate, host, kernels_of

pytestmark = pytest.mark.gpu

OP_MAX, OP_MEAN = 6e-3, 6e-4       # as tests/test_gpu_ops.py: fp16 outputs of order one, fp32 sums

AT_ONCE, SPREAD = 0, 2


@pytest.mark.parametrize("M,K,N,tile,schedule", [
    (64, 1280, 14016, "64, 64", AT_ONCE),            # 34 MiB
    (21, 1408, 14144, "64, 64", AT_ONCE),
    (64, 1280, 13504, "64, 64", SPREAD),             # 33 MiB less 12 KiB
    (65, 3712, 6592, "64, 64", SPREAD),              # 47 MiB, two row tiles
    (128, 1536, 14080, "128, 64", AT_ONCE),
    (69, 1152, 16256, "128, 64", AT_ONCE),
    (128, 1280, 13504, "128, 64", SPREAD),
    (200, 2816, 6400, "128, 64", SPREAD),            # 34 MiB, two row tiles
])
def test_linear(M, K, N, tile, schedule):
    from paper_2104_12470_amd import eet
    x, w = wl.normal(401, M, (M, K)), wl.normal(402, N, (N, K), 1.0 / np.sqrt(K))
    b, r = wl.normal(403, N, (N,), 0.5), wl.normal(404, M, (M, N))
    xd, wd, bd, rd = dev(x), dev(w), dev(b), dev(r)
    y = torch.full((M + 1, N), float("nan"), dtype=torch.float16, device="cuda:0")
    lin = orc.linear(x, w, b)
    for act, res, want in ((0, None, lin), (1, None, orc.gelu_tanh(lin)), (0, rd, lin + r.astype(np.float64))):
        y.fill_(float("nan"))
        names = kernels_of(lambda: eet.eet_op_linear(xd, wd, bd, y[:M], residual=res, act=act))
        mine = [n for n in names if f"gemm_mfma_dma64<{tile}," in n]
        assert mine and all(n.split("<")[1].split(", ")[6:8] == ["2", str(schedule)] for n in mine), names
        gate(host(y[:M]), want, f"{M}x{K}x{N} act {act}", OP_MAX, OP_MEAN)
        assert torch.isnan(y[M]).all()
