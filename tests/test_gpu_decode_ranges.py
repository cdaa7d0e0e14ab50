"""Decode attention whose key ranges are merged by the last workgroup of each (sequence, head) pair to finish: layers too large for a step in one launch
and for the small-layer output projection.  Fewer than 128 pairs, 128 and more (one range); an empty last range; step after step on the same counters, and in a stack's recorded step."""
import numpy as np
import pytest
import torch

from oracle import eet_oracle as orc
from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, gate, host, kernels_of

pytestmark = pytest.mark.gpu


def setup(heads, d, lens, max_seq):
    from paper_2104_12470_amd import eet
    B, H = len(lens), heads * d
    w = wl.Workload(f"ranges{heads}x{d}x{B}", 71, H, heads, 128, 1, B, 1, 1, 1, 2, max_seq)
    W = wl.layer_weights(w, 0, random_affine=True)
    cfg = eet.make_config(H, heads, w.ffn, B, 1, max_seq, w.ln_eps)
    rows = wl.normal(71, 9, (2, B, heads, max_seq, d))
    for b, n in enumerate(lens):
        rows[:, b, :, n:] = np.nan                   # slots that hold no key yet are never read
    oracle = orc.DecoderLayerOracle(W, heads, B, max_seq, w.ln_eps)
    oracle.batch, oracle.lens[:], oracle.k_cache[:], oracle.v_cache[:] = B, lens, rows[0], rows[1]
    return eet, w, {k: torch.from_numpy(v) for k, v in W.items()}, cfg, rows, oracle


@pytest.mark.parametrize("heads,d,lens,max_seq", [
    (17, 128, [300], 320),                           # two ranges
    (17, 128, [17], 2100),                           # sixteen, most of them empty
    (18, 128, [700, 1, 350], 720),                   # 54 pairs
    (36, 64, [500, 600], 640),                       # heads of 64
    (64, 64, [766, 767], 800),                       # 128 pairs: one range
    (32, 128, [767, 900, 30, 1279], 1300),
    (32, 128, [767, 900, 30, 200, 500], 920),        # 160: one range
])
def test_steps_against_the_oracle(heads, d, lens, max_seq):
    eet, w, W, cfg, rows, oracle = setup(heads, d, lens, max_seq)
    layer = eet.DecoderLayer(cfg, W)
    layer.kv_cache.copy_(dev(rows).view(-1))
    eet.eet_restore(layer.handle, lens)
    for k in range(3):
        xs = wl.decode_embeddings(w, k % 2)
        tok = dev(xs)
        got = torch.empty_like(tok)
        names = kernels_of(lambda: layer.decode_step(tok, got))
        assert any("attn_decode<" in n for n in names) and not any("combine" in n for n in names), names
        gate(host(got), oracle.decode_step(xs), f"step {k}")
    layer.close()


@pytest.mark.parametrize("heads,d,lens,max_seq", [(18, 128, [500, 690], 720), (32, 128, [767, 900, 30, 1279], 1300)])
def test_recorded_step(heads, d, lens, max_seq):
    """Two layers of a stack on one set of counters and partials (and 128 pairs, which have none), directly and recorded, against two oracle layers."""
    eet, w, W, cfg, rows, oracle = setup(heads, d, lens, max_seq)
    second = setup(heads, d, lens, max_seq)[-1]      # the stack's second layer: the same weights and cache
    direct, graph = eet.DecoderStack(cfg, [W, W], use_graph=False), eet.DecoderStack(cfg, [W, W])
    x = wl.decode_embeddings(w, 0)
    tok = dev(x)
    out = [torch.empty_like(tok) for _ in range(2)]
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for st in (direct, graph):
            st.kv_cache.copy_(torch.cat([dev(rows).view(-1)] * 2))
            eet.eet_stack_restore(st.handle, lens)
        for k in range(6):
            direct.decode_step(tok, out[0])
            graph.decode_step(tok, out[1])
            stream.synchronize()
            assert np.array_equal(host(out[0]).view(np.uint16), host(out[1]).view(np.uint16)), k
            between = oracle.decode_step(x).astype(np.float16)           # the first layer's output as the second one reads it
            gate(host(out[0]), second.decode_step(between), f"step {k}")
    direct.close()
    graph.close()
