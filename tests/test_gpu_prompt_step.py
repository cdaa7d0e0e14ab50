"""Short prompts and encoder passes in one launch (csrc/prompt_step.hip): one and many row tiles, sequences that share tiles and that span them, two blocks of
queries, both head sizes, K of one to sixteen units, even and uneven ranges of the feed-forward part, pad rows on either side, more layers than a launch
takes, a recorded prefill, and the sizes just past what it takes."""
import numpy as np
import pytest
import torch

from oracle import eet_oracle as orc
from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, gate, host, kernels_of

pytestmark = pytest.mark.gpu


def build(hidden, heads, ffn, lens, layers=1, extra=3):
    from paper_2104_12470_amd import eet
    B, S = len(lens), max(lens) + 2
    w = wl.Workload(f"prompt{hidden}x{ffn}x{sum(lens)}", 97, hidden, heads, ffn, layers, B, S, 1, S, 2, S + extra)
    Ws = [wl.layer_weights(w, l, random_affine=True) for l in range(layers)]
    return eet, w, Ws, eet.make_config(hidden, heads, ffn, B, S, S + extra, w.ln_eps)


def on_device(W):
    return {k: torch.from_numpy(v) for k, v in W.items()}


@pytest.mark.parametrize("hidden,heads,ffn,lens,one", [
    (64, 1, 64, [1], True),
    (256, 2, 1024, [16], True),                          # a tile exactly; heads of 128
    (192, 3, 320, [17], True),                           # three and five units
    (576, 9, 1344, [5, 1, 20, 7], True),                 # two ranges of 11 and 10 units
    (1024, 16, 4096, [37], True),                        # four ranges
    (1024, 8, 2688, [60, 36], True),                     # three ranges of 14
    (512, 8, 2048, [200], True),                         # two blocks of queries
    (256, 4, 640, [1 + b % 6 for b in range(60)], True),  # many sequences to a tile
    (256, 4, 1024, [129, 128, 200], True),               # 457 rows
    (768, 12, 3072, [90, 60], False),                    # more items than are taken
    (768, 12, 3072, [30, 60, 64, 23], False),
    (512, 8, 2048, [100, 150, 80], False),
    (1024, 8, 4096, [100], False),
    (384, 6, 1536, [130, 190], True),                    # 1224 items
    (384, 6, 1536, [130, 200], False),                   # 1284, 24 of them attention
    (256, 4, 1024, [300, 220], False),                   # more rows than are taken
    (1024, 16, 4096, [16], False),                       # rows of the small-layer kernel
    (1024, 16, 4160, [20], False),                       # feed-forward part too wide
])
@pytest.mark.parametrize("left", [False, True])
def test_prompt(hidden, heads, ffn, lens, one, left):
    eet, w, Ws, cfg = build(hidden, heads, ffn, lens)
    layer, S = eet.DecoderLayer(cfg, on_device(Ws[0])), w.padded_len
    oracle = orc.DecoderLayerOracle(Ws[0], heads, len(lens), w.max_seq, w.ln_eps)
    x = wl.prompt_embeddings(w)
    want = oracle.prefill(x, lens)
    given = np.full_like(x, np.nan)                      # pad rows are never read
    for b, n in enumerate(lens):
        given[b, S - n if left else 0:][:n] = x[b, :n]
    run = lambda: (layer.prefill_left_padded if left else layer.prefill)(dev(given), lens)     # noqa: E731
    got = host(run())
    for b, n in enumerate(lens):
        valid, pads = (got[b, S - n:], got[b, :S - n]) if left else (got[b, :n], got[b, n:])
        gate(valid, want[b, :n], f"sequence {b}")
        assert np.all(pads == 0)
    kc, vc = layer.cache_views()
    for b, n in enumerate(lens):
        gate(host(kc[b, :, :n]), oracle.k_cache[b, :, :n], f"K cache b={b}", 1.5e-2, 1.5e-3)
        gate(host(vc[b, :, :n]), oracle.v_cache[b, :, :n], f"V cache b={b}", 1.5e-2, 1.5e-3)
    xs = wl.decode_embeddings(w, 0)
    gate(host(layer.decode_step(dev(xs))), oracle.decode_step(xs), "the step that follows")
    assert layer.cache_lens(len(lens)) == [n + 1 for n in lens]
    assert any("prompt_layers" in n for n in kernels_of(run)) == one
    layer.close()


@pytest.mark.parametrize("hidden,heads,ffn,lens", [(256, 2, 1024, [40, 3, 30]), (576, 9, 1344, [150]), (320, 5, 1280, [1 + b % 5 for b in range(50)])])
def test_encoder(hidden, heads, ffn, lens):
    eet, w, Ws, cfg = build(hidden, heads, ffn, lens, layers=4)
    stack = eet.DecoderStack(cfg, [on_device(W) for W in Ws])
    x = wl.prompt_embeddings(w)
    want = x.astype(np.float64)
    for rep in range(3):                                 # the layers' keys and values share one region
        got = host(stack.encode(dev(x), lens))
        if rep == 0:
            first = got
            h = dev(x)
            for W in Ws:
                layer = eet.DecoderLayer(cfg, on_device(W))
                h = layer.encode(h, lens)
                torch.cuda.synchronize()
                layer.close()
                want = orc.DecoderLayerOracle(W, heads, len(lens), w.max_seq, w.ln_eps).encode(want, lens)
            assert np.array_equal(got.view(np.uint16), host(h).view(np.uint16))
            for b, n in enumerate(lens):
                gate(got[b, :n], want[b, :n], f"sequence {b}", 5e-2, 5e-3)      # four layers, each fed the GPU's own rounding
        assert np.array_equal(got.view(np.uint16), first.view(np.uint16))
    stack.close()


def test_stack_is_the_chain_of_its_layers():
    lens = [9, 30, 1]
    eet, w, Ws, cfg = build(128, 2, 320, lens, layers=35)
    stack = eet.DecoderStack(cfg, [on_device(W) for W in Ws])
    x = dev(wl.prompt_embeddings(w))
    got, h = stack.prefill(x, lens), x
    kv = stack.kv_cache.view(35, 2, 3, 2, w.max_seq, 64)
    for l, W in enumerate(Ws):
        layer = eet.DecoderLayer(cfg, on_device(W))
        h = layer.prefill(h, lens)
        for b, n in enumerate(lens):
            assert torch.equal(kv[l][:, b, :, :n], layer.kv_cache.view(2, 3, 2, w.max_seq, 64)[:, b, :, :n]), (l, b)
        layer.close()
    assert torch.equal(got, h)
    stack.close()


def test_weights_read_once():
    """One row tile through a stack whose weights no cache keeps until the next call: they are loaded with the hint, and the bits are those of the single
    layers, whose weights are kept."""
    lens, layers = [6, 4], 15
    eet, w, Ws, cfg = build(1024, 16, 2688, lens)
    W = {k: v.to("cuda:0") for k, v in on_device(Ws[0]).items()}
    stack, layer = eet.DecoderStack(cfg, [W] * layers), eet.DecoderLayer(cfg, W)
    h = x = dev(wl.prompt_embeddings(w))
    kinds = lambda names: [n.split("prompt_layers<")[1].split(">")[0] for n in names if "prompt_layers<" in n]     # noqa: E731
    assert kinds(kernels_of(lambda: stack.prefill(x, lens))) == ["true"] and kinds(kernels_of(lambda: layer.prefill(x, lens))) == ["false"]
    got = stack.prefill(x, lens)
    for l in range(layers):
        h = layer.prefill(h, lens)
        torch.cuda.synchronize()
        a, b = (kv.view(2, 2, 16, w.max_seq, 64) for kv in (stack.kv_cache.view(layers, -1)[l], layer.kv_cache))
        assert all(torch.equal(a[:, s, :, :n], b[:, s, :, :n]) for s, n in enumerate(lens)), l
    assert bool(torch.isfinite(got[0, :6]).all()) and torch.equal(got, h)
    stack.close()
    layer.close()


def test_recorded_prefill():
    """A prefill that the caller records and replays, with eager work and other prompts on the same handle in between."""
    lens = [20, 3, 14]
    eet, w, Ws, cfg = build(256, 4, 1024, lens, layers=3)
    stack = eet.DecoderStack(cfg, [on_device(W) for W in Ws])
    x, side = dev(wl.prompt_embeddings(w)), torch.cuda.Stream()
    out, g = torch.empty_like(x), torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        want = stack.prefill(x, lens).clone()
        side.synchronize()
        with torch.cuda.graph(g, stream=side):
            stack.prefill(x, lens, out)
        for _ in range(4):
            out.zero_()
            stack.prefill(x[:2].contiguous(), [7, 21])
            g.replay()
            side.synchronize()
            assert torch.equal(out, want)
            torch.randn(64, 64, device="cuda:0").sum()
    stack.close()
