"""Projections of layer widths through the tiles that tile_rules.hpp's full_tile chooses: every height at its smallest K, with ragged rows, a ragged half tile of
columns, one round and several; and the K/V cache rows of a prompt out of one of them.  Which tile a shape takes is asked of the header that the library compiles."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from oracle import eet_oracle as orc
from paper_2104_12470_amd import workloads as wl
from tests import tile_shapes
from tests.gpu_util import dev, gate, host, kernels_of

OP_MAX, OP_MEAN = 6e-3, 6e-4       # as tests/test_gpu_ops.py: fp16 outputs of order one, fp32 sums

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# (M, K, N, tile)
SHAPES = [(2743, 768, 4992, "256x256"), (2549, 832, 4992, "224x256"), (2161, 768, 4992, "192x256"), (1773, 896, 4992, "160x256"), (1385, 768, 4992, "128x256"),
          (1093, 768, 4224, "192x128"), (1289, 1088, 2944, "128x128"), (1153, 832, 2176, "96x128"), (5377, 1216, 6016, "rounds")]      # (up to K = 1152 these rounds are the pairs')

ASK = r"""
#include <cstdio>
#include "%s/paper_2104_12470_amd/csrc/tile_rules.hpp"
int main() {
    int M, N, K;
    while (std::scanf("%%d %%d %%d", &M, &N, &K) == 3) {
        const char* full[] = {"none", "256x256", "224x256", "192x256", "160x256", "128x256", "192x128", "128x128", "96x128"};
        const char* old[] = {"64x64", "64x64", "128x64", "128x64", "128x128", "128x128", "192x128", "96x128", "128x128", "192x128", "128x256", "256x256"};
        std::printf("%%d %%s %%s\n", eet::rows_in_whole_rounds(M, N), full[eet::full_tile(M, N, K)], old[eet::tile_for(M, N, K)]);
    }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("full")
    (d / "ask.cpp").write_text(ASK % ROOT)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", str(d / "ask.cpp"), "-o", str(d / "ask")], check=True)

    def run(sizes):
        out = subprocess.run([str(d / "ask")], input="".join(f"{M} {N} {K}\n" for M, N, K in sizes), capture_output=True, text=True, check=True)
        return [line.split() for line in out.stdout.splitlines()]
    return run


def test_shapes_take_the_tile_they_are_there_for(ask):
    got = ask([(M, N, K) for M, K, N, _ in SHAPES])
    for (M, K, N, tile), (cut, full, _) in zip(SHAPES, got):
        assert cut == "0" and (full == tile or tile == "rounds" and full != "none"), (M, K, N, cut, full)
    assert {f for _, f, _ in got} >= {"256x256", "224x256", "192x256", "160x256", "128x256", "192x128", "128x128", "96x128"}


def test_shapes_that_other_tests_hold_to_a_tile_keep_it(ask):
    """Where full_tile has a say it agrees with the tile that tests/tile_shapes.py names."""
    sizes = [(M, N, K) for M, K, N, _ in tile_shapes.LARGE_TILES] + [(s[0], s[2], s[1]) for s in tile_shapes.STRIDED]
    for w, routes in tile_shapes.LAYERS:
        T, H, F = int(sum(wl.lengths(w))), w.hidden, w.ffn
        sizes += [{"qkv": (T, 3 * H, H), "o": (T, H, H), "ffn1": (T, F, H), "ffn2": (T, H, F)}[r] for r in routes]
    answers = ask(sizes)
    assert all(full in ("none", old) or cut != "0" for cut, full, old in answers), [(s, a) for s, a in zip(sizes, answers) if a[1] not in ("none", a[2])]


def test_pairs_that_nearly_fill_a_round_are_not_taken_apart(ask):
    """Sizes of 420 to 512 tiles of which two share a CU, measured 5 to 17 % slower as two rounds of one tile per CU, and below K = 1024 5 to 9 % slower on taller ones;
    a few tiles more or less on either side, and the tall tiles stay where they are ahead."""
    pairs = [((1031, 10880, 1152), "192x128"), ((4290, 1920, 1408), "128x128"), ((3302, 2432, 832), "128x128"), ((5545, 1408, 1728), "128x128"),
             ((8223, 896, 1856), "128x128"), ((2275, 10880, 896), "192x128"), ((4802, 2432, 832), "192x128"), ((8799, 1408, 960), "192x128"),
             ((5377, 6016, 768), "128x128"), ((6000, 3072, 768), "192x128"), ((5060, 6528, 832), "128x128"), ((5414, 2944, 1024), "128x128"), ((2109, 7680, 1152), "128x128")]
    assert [(full, old) for _, full, old in ask([s for s, _ in pairs])] == [("none", t) for _, t in pairs]
    tall = [((5377, 6016, 1216), "192x256"), ((2140, 4096, 4096), "160x256"), ((1137, 15360, 7232), "160x256"), ((3054, 3072, 12288), "160x256"), ((6758, 2048, 2048), "224x256"), ((1153, 2176, 832), "96x128")]
    assert [full for _, full, _ in ask([s for s, _ in tall])] == [t for _, t in tall]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,tile", SHAPES)
def test_linear_full_tiles(M, K, N, tile):
    from paper_2104_12470_amd import eet
    x, w = wl.normal(390, M, (M, K)), wl.normal(391, N, (N, K), 1.0 / np.sqrt(K))
    b, r = wl.normal(392, N, (N,), 0.5), wl.normal(393, M, (M, N))
    xd, wd, bd, rd = dev(x), dev(w), dev(b), dev(r)
    y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda:0")
    names = kernels_of(lambda: eet.eet_op_linear(xd, wd, bd, y, act=1))
    if tile != "rounds":
        assert any(f"gemm_mfma_dma64<{tile.replace('x', ', ')}," in n for n in names), names
    lin = orc.linear(x, w, b)
    gate(host(y), orc.gelu_tanh(lin), f"full tile linear+gelu {M}x{K}x{N}", OP_MAX, OP_MEAN)
    y.fill_(float("nan"))
    eet.eet_op_linear(xd, wd, bd, y, residual=rd)
    torch.cuda.synchronize()
    gate(host(y), lin + r.astype(np.float64), f"full tile linear+res {M}x{K}x{N}", OP_MAX, OP_MEAN)


@pytest.mark.gpu
def test_prompts_through_full_tiles(ask):
    """Cache rows (QKV) and mapped rows (output and second feed-forward projection) out of tall tiles, against the oracle."""
    from paper_2104_12470_amd import eet
    from tests.test_gpu_layer import full_parity
    w = wl.Workload("full1024", 43, 1024, 8, 4096, 1, 6, 500, 430, 500, 1, 502)
    T = int(sum(wl.lengths(w)))
    full = [f for _, f, _ in ask([(T, 3072, 1024), (T, 4096, 1024), (T, 1024, 4096)])]
    assert full[0].endswith("x256") and full[1].endswith("x256") and full[2] == "96x128", (T, full)
    full_parity(eet, w, random_affine=False)
