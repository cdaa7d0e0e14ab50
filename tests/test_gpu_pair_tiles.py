"""Tiles of which two workgroups share a CU (192 x 128 and 128 x 128 with two LDS stages): a bias alone or with a residual goes out through
LDS, GELU and a prompt's cache rows straight.  Every kind of output at the smallest K and at a larger one, with ragged rows and a half column tile: a bias alone, a residual, rows with strides,
and a prompt's cache rows in both layouts.  Which tile a shape takes is asked of the rules that the library compiles."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from oracle import eet_oracle as orc
from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, gate, host

OP_MAX, OP_MEAN = 6e-3, 6e-4       # as tests/test_gpu_ops.py: fp16 outputs of order one, fp32 sums
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHAPES = [(801, 64, 12352, "192x128 x2"), (3339, 320, 5056, "192x128 x2"), (1753, 448, 11904, "192x128 x2"),
          (301, 64, 12352, "128x128 x2, shared schedule"), (1480, 320, 3136, "128x128 x2, shared schedule"), (2319, 384, 3264, "128x128 x2, shared schedule"),
          (615, 512, 9856, "128x128 x2"), (3019, 576, 2432, "128x128 x2"), (1012, 2304, 6208, "128x128 x2")]
# (heads, sequences, padded length, tile of the QKV projection)
PROMPTS = [(5, 84, 64, "128x128 x2, shared schedule"), (7, 112, 64, "192x128 x2")]


def prompt_workload(heads, batch, S):
    return wl.Workload(f"pair{heads}", 47, heads * 64, heads, 64, 1, batch, S, S - 9, S, 1, S + 2)


def test_shapes_take_the_tile_they_are_there_for(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = tmp_path / "tile_rules_audit"
    subprocess.run([cxx, "-std=c++17", "-O1", os.path.join(ROOT, "tests", "tile_rules_audit.cpp"), "-o", str(exe)], check=True)
    ask = [("route", M, N, K, t) for M, K, N, t in SHAPES]
    for heads, batch, S, t in PROMPTS:
        ask.append(("mapped", int(sum(wl.lengths(prompt_workload(heads, batch, S)))), 3 * heads * 64, heads * 64, t))
    out = subprocess.run([str(exe)], input="".join("%s %d %d %d\n" % q[:4] for q in ask), capture_output=True, text=True, check=True)
    assert out.stdout.splitlines() == [q[4] for q in ask]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [s[:3] for s in SHAPES])
def test_linear(M, K, N):
    from paper_2104_12470_amd import eet
    x, w = wl.normal(395, M, (M, K)), wl.normal(396, N, (N, K), 1.0 / np.sqrt(K))
    b, r = wl.normal(397, N, (N,), 0.5), wl.normal(398, M, (M, N))
    lin = orc.linear(x, w, b)
    xd, wd, bd, rd = dev(x), dev(w), dev(b), dev(r)
    y = torch.full((M + 1, N), float("nan"), dtype=torch.float16, device="cuda:0")
    for res, want in ((None, lin), (rd, lin + r.astype(np.float64))):
        y.fill_(float("nan"))
        eet.eet_op_linear(xd, wd, bd, y[:M], residual=res)
        torch.cuda.synchronize()
        gate(host(y[:M]), want, f"{M}x{K}x{N}", OP_MAX, OP_MEAN)
        assert torch.isnan(y[M]).all()
    xs = torch.full((M, K + 64), float("nan"), dtype=torch.float16, device="cuda:0")
    ys = torch.full((M, N + 8), float("nan"), dtype=torch.float16, device="cuda:0")
    xs[:, :K] = xd
    eet.eet_op_linear_strided(xs[:, :K], wd, bd, ys[:, :N], residual=rd)
    torch.cuda.synchronize()
    gate(host(ys[:, :N]), lin + r.astype(np.float64), f"strided {M}x{K}x{N}", OP_MAX, OP_MEAN)
    assert torch.isnan(ys[:, N:]).all()


@pytest.mark.gpu
@pytest.mark.parametrize("heads,batch,S", [p[:3] for p in PROMPTS])
def test_cache_rows(heads, batch, S):
    from paper_2104_12470_amd import eet
    from tests.test_gpu_layer import full_parity, make_gpu_layer
    w = prompt_workload(heads, batch, S)
    full_parity(eet, w)
    W, x, lens = wl.layer_weights(w, 0, True), wl.prompt_embeddings(w), [int(v) for v in wl.lengths(w)]
    xl = np.full_like(x, np.nan)                       # the same prompts with the pads in front: the same bits
    for b, n in enumerate(lens):
        xl[b, S - n:] = x[b, :n]
    left, right = make_gpu_layer(eet, w, W), make_gpu_layer(eet, w, W)
    out_l, out_r = left.prefill_left_padded(dev(xl), lens), right.prefill(dev(x), lens)
    torch.cuda.synchronize()
    for b, n in enumerate(lens):
        assert torch.equal(out_l[b, S - n:], out_r[b, :n]), b
    assert torch.equal(left.kv_cache, right.kv_cache)
    left.close()
    right.close()
