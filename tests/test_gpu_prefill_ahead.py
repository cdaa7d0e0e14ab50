"""Which prefill attentions touch weights on the side: those of stacks whose weights no longer are in the memory-side cache when their turn comes, by the rule in
tile_rules.hpp, never an operator's.  Touching changes no bit: a stack that does it is the chain of its layers, which on their own do not."""
import os
import shutil
import subprocess

import pytest
import torch

from oracle import eet_oracle as orc
from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, gate, host, kernels_of

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHAPES = [(4, 64, [43] * 5, "attn_prefill16<64, true"),        # short prompts
          (2, 128, [100, 1, 300], "attn_prefill16<128, true"),
          (3, 64, [300, 20], "attn_prefill<true"),
          (2, 128, [600, 513], "attn_prefill_wide<128, true")]


def test_rule(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "ask.cpp").write_text(r"""
#include <cstdio>
#include "%s/paper_2104_12470_amd/csrc/tile_rules.hpp"
int main() {
    long rows, H, F, layers;
    while (std::scanf("%%ld %%ld %%ld %%ld", &rows, &H, &F, &layers) == 4)
        std::printf("%%d\n", eet::prefill_touches_weights(rows, 2 * (H * H + H * F), layers * 2 * (4 * H * H + 2 * H * F), layers * 4 * H * rows));
}
""" % ROOT)
    subprocess.run([cxx, "-std=c++17", "-O1", str(tmp_path / "ask.cpp"), "-o", str(tmp_path / "ask")], check=True)
    cached = [(177, 768, 3072, 1), (3150, 1024, 4096, 1), (120, 320, 1280, 7), (48, 704, 2816, 2), (55, 768, 3072, 2), (1192, 1408, 5632, 3)]     # 1 to 4 % slower with it
    gone = [(37, 1024, 4096, 24), (3150, 1024, 4096, 24), (3072, 768, 3072, 12), (3072, 512, 2048, 24), (900, 1536, 6144, 5)]
    other = [(9, 1024, 4096, 24), (12000, 1024, 4096, 12), (500, 4096, 16384, 2)]
    out = subprocess.run([str(tmp_path / "ask")], input="".join("%d %d %d %d\n" % q for q in cached + gone + other), capture_output=True, text=True, check=True)
    assert out.stdout.split() == ["0"] * len(cached) + ["1"] * len(gone) + ["0"] * len(other)


@pytest.mark.gpu
@pytest.mark.parametrize("heads,d,lens,kernel", SHAPES)
def test_stack_that_touches_weights_is_the_chain_of_its_layers(heads, d, lens, kernel):
    from paper_2104_12470_amd import eet
    H, B, S, F, layers = heads * d, len(lens), max(lens), 24576, 12          # 230 to 308 MB of weights, 9.5 to 12.7 of a layer touched
    w = wl.Workload("ahead", 89, H, heads, F, 1, B, S, 1, S, 0, S)
    W = {k: torch.from_numpy(v).to("cuda:0") for k, v in wl.layer_weights(w, 0, random_affine=True).items()}
    cfg = eet.make_config(H, heads, F, B, S, S, w.ln_eps)
    layer, stack = eet.DecoderLayer(cfg, W), eet.DecoderStack(cfg, [W] * layers)
    x = dev(wl.prompt_embeddings(w))
    out = torch.empty_like(x)
    names = kernels_of(lambda: stack.prefill(x, lens, out))
    assert any(kernel in n and "true>" in n for n in names), names
    for k in range(layers):
        then = torch.empty_like(x)
        names = kernels_of(lambda: layer.prefill(x, lens, then))
        assert any(kernel in n and "false>" in n for n in names), names
        kv = stack.kv_cache.view(layers, 2, B, heads, S, d)[k]
        for b, n in enumerate(lens):
            assert torch.equal(kv[:, b, :, :n], layer.kv_cache.view(2, B, heads, S, d)[:, b, :, :n]), (k, b)
        x = then
    assert torch.equal(out, x)
    layer.close()
    stack.close()


@pytest.mark.gpu
@pytest.mark.parametrize("heads,d,lens,kernel", SHAPES)
def test_operator_touches_none(heads, d, lens, kernel):
    from paper_2104_12470_amd import eet
    B, S = len(lens), max(lens)
    q, k, v = (wl.normal(89, t, (B, S, heads, d)) for t in (1, 2, 3))
    want = orc.attention_prefill(q, k, v, lens)
    ctx = torch.empty((B, S, heads * d), dtype=torch.float16, device="cuda:0")
    qd, kd, vd = dev(q.reshape(B, S, -1)), dev(k.transpose(0, 2, 1, 3)), dev(v.transpose(0, 2, 1, 3))
    names = kernels_of(lambda: eet.eet_op_attention_prefill(qd, kd, vd, ctx, lens, heads))
    assert any(kernel in n and "false>" in n for n in names), names
    for b, n in enumerate(lens):
        gate(host(ctx)[b, :n].reshape(n, heads, d), want[b, :n], f"sequence {b}", 6e-3, 6e-4)
