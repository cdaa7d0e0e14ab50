"""Prompts of up to 256 rows whose output and second feed-forward projection are cut along K (tile_rules.hpp: prompt_k_ranges), on either
side of its row limits and weight floors, with uneven ranges and pad rows in both layouts."""
import numpy as np
import pytest
import torch

from oracle import eet_oracle as orc
from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, gate, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,heads,ffn,lens", [
    (512, 8, 1152, [17]),                    # 4 uneven ranges of 9 steps: the 64-row tile, K is no multiple of 256
    (512, 4, 2048, [20, 12]),                # 32 rows: K groups of 256 in ranges of 256
    (512, 8, 1408, [33]),
    (768, 12, 3072, [40, 1, 23]),            # 64 rows
    (768, 6, 3072, [64, 1]),                 # 65: the output projection below the floor
    (1024, 16, 2688, [100, 28]),             # 128
    (1024, 16, 4096, [129]),                 # two row tiles
    (1536, 12, 2048, [200, 56]),             # 256
    (768, 12, 3072, [200, 57]),              # 257: as before
])
@pytest.mark.parametrize("left", [False, True])
def test_prompt(hidden, heads, ffn, lens, left):
    from paper_2104_12470_amd import eet
    S, B = max(lens) + 3, len(lens)
    w = wl.Workload(f"cut{hidden}x{ffn}", 43, hidden, heads, ffn, 1, B, S, 1, S, 1, S + 2)
    W = wl.layer_weights(w, 0, random_affine=True)
    cfg = eet.make_config(hidden, heads, ffn, B, S, S + 2, w.ln_eps)
    layer, oracle = eet.DecoderLayer(cfg, {k: torch.from_numpy(v) for k, v in W.items()}), orc.DecoderLayerOracle(W, heads, B, S + 2, w.ln_eps)
    x = wl.prompt_embeddings(w)
    want = oracle.prefill(x, lens)
    given = x
    if left:
        given = np.zeros_like(x)
        for b, n in enumerate(lens):
            given[b, S - n:] = x[b, :n]
    got = host((layer.prefill_left_padded if left else layer.prefill)(dev(given), lens))
    for b, n in enumerate(lens):
        valid, pads = (got[b, S - n:], got[b, :S - n]) if left else (got[b, :n], got[b, n:])
        gate(valid, want[b, :n], f"sequence {b}")
        assert np.all(pads == 0)
    xs = wl.decode_embeddings(w, 0)
    gate(host(layer.decode_step(dev(xs))), oracle.decode_step(xs), "the step that follows")
    layer.close()
