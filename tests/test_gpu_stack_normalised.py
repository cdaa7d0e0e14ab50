"""Stacks whose second feed-forward projection is cut along K: the launch that adds up the ranges also does the next layer's first LayerNorm.  The same bits
as the layers one by one, in prompts, encoder passes and decode steps."""
import numpy as np
import pytest
import torch

from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, host, kernels_of

pytestmark = pytest.mark.gpu


def same(a, b):
    return np.array_equal(host(a).view(np.uint16), host(b).view(np.uint16))


def build(hidden, heads, ffn, batch, S, cap, n_layers):
    from paper_2104_12470_amd import eet
    w = wl.Workload(f"norm{hidden}x{ffn}", 79, hidden, heads, ffn, n_layers, batch, S, 1, S, 2, cap)
    Ws = [{k: torch.from_numpy(v) for k, v in wl.layer_weights(w, l, random_affine=True).items()} for l in range(n_layers)]
    cfg = eet.make_config(hidden, heads, ffn, batch, S, cap, w.ln_eps)
    return w, eet.DecoderStack(cfg, Ws, use_graph=False), [eet.DecoderLayer(cfg, W) for W in Ws]


def launches(names):
    return sum("layernorm" in n for n in names)


# rows below and from 64 on (two orders of additions), widths on both sides of 2048, with and without pad rows, a feed-forward part narrower than the layer
@pytest.mark.parametrize("hidden,heads,ffn,lens,S", [(1024, 16, 8192, [37], 37), (512, 8, 5120, [20, 20], 20), (768, 6, 3072, [160], 160), (1024, 8, 4096, [100, 50], 100),
                                                     (2048, 16, 8192, [60], 60), (2048, 32, 8192, [100, 100], 100), (2560, 20, 6784, [48], 48),
                                                     (2560, 20, 6784, [80, 60], 80), (1280, 10, 512, [30], 30)])
def test_prompts_and_encoder_passes(hidden, heads, ffn, lens, S):
    B, n = len(lens), 4
    w, stack, layers = build(hidden, heads, ffn, B, S, S + 4, n)
    x = dev(wl.prompt_embeddings(w))
    for encode in (False, True):
        got = stack.encode(x, lens) if encode else stack.prefill(x, lens)
        h = x
        for layer in layers:
            h = layer.encode(h, lens) if encode else layer.prefill(h, lens)
        torch.cuda.synchronize()
        assert np.all(np.isfinite(host(got))) and same(got, h)
    # the point of it: three LayerNorm launches less than one by one; with pad rows layers 1 and 3 have a set-up launch, and normalise there
    alone = sum(launches(kernels_of(lambda: layer.prefill(x, lens))) for layer in layers)
    assert alone - launches(kernels_of(lambda: stack.prefill(x, lens))) == (0 if ffn < hidden else 1 if min(lens) < S else 3)
    stack.close()
    for layer in layers:
        layer.close()


@pytest.mark.parametrize("hidden,heads,ffn,batch", [(2048, 16, 8192, 40), (2048, 32, 8192, 64), (2560, 20, 6784, 100), (4096, 32, 10880, 33)])
def test_decode_steps(hidden, heads, ffn, batch):
    n, cap = 3, 12
    w, stack, layers = build(hidden, heads, ffn, batch, 2, cap, n)
    x, lens = dev(wl.prompt_embeddings(w)), [1 + b % 2 for b in range(batch)]
    h = x
    stack.prefill(x, lens)
    for layer in layers:
        h = layer.prefill(h, lens)
    for k in range(2):
        tok = dev(wl.decode_embeddings(w, k))
        got = stack.decode_step(tok)
        h = tok
        for layer in layers:
            h = layer.decode_step(h)
        torch.cuda.synchronize()
        assert np.all(np.isfinite(host(got))) and same(got, h), k
    alone = sum(launches(kernels_of(lambda: layer.decode_step(tok))) for layer in layers)
    assert alone - launches(kernels_of(lambda: stack.decode_step(tok))) == n - 1
    stack.close()
    for layer in layers:
        layer.close()
