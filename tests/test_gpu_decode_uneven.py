"""Decode attention of uneven and even sequences on more (sequence, head) pairs than CUs, in a layer's step and in a stack's recorded one.  All of it
against the oracle."""
import numpy as np
import pytest
import torch

from oracle import eet_oracle as orc
from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, gate, host

pytestmark = pytest.mark.gpu


def uneven(batch, lo, hi):
    lens = [lo + (hi - lo) * (b * 7 % batch) // batch for b in range(batch)]
    lens[batch // 2] = hi
    return lens


def build(heads, d, lens, max_seq, rows):
    H, B = heads * d, len(lens)
    w = wl.Workload(f"uneven{heads}x{d}x{B}", 67, H, heads, 128, 1, B, 1, 1, 1, 2, max_seq)
    W = wl.layer_weights(w, 0, random_affine=True)
    cfg = eet_module().make_config(H, heads, w.ffn, B, 1, max_seq, w.ln_eps)
    oracle = orc.DecoderLayerOracle(W, heads, B, max_seq, w.ln_eps)
    return w, {k: torch.from_numpy(v) for k, v in W.items()}, cfg, oracle


def eet_module():
    from paper_2104_12470_amd import eet
    return eet


def set_oracle(oracle, lens, rows):
    oracle.batch, oracle.lens[:len(lens)] = len(lens), lens
    oracle.k_cache[:], oracle.v_cache[:] = rows[0], rows[1]


@pytest.mark.parametrize("heads,d,lens", [
    (4, 128, uneven(65, 1, 699)),                    # 260 pairs
    (4, 128, uneven(64, 1, 720)),                    # 256
    (4, 128, [720] * 65),                            # even
    (5, 64, uneven(52, 1, 800)),
    (8, 64, uneven(64, 1, 800)),                     # 512
    (5, 64, uneven(52, 500, 800)),
])
def test_step_against_the_oracle(heads, d, lens):
    eet, max_seq = eet_module(), max(lens) + 8
    rows = wl.normal(67, 9, (2, len(lens), heads, max_seq, d))
    for b, n in enumerate(lens):
        rows[:, b, :, n:] = np.nan                   # slots that hold no key yet are never read
    w, W, cfg, oracle = build(heads, d, lens, max_seq, rows)
    layer = eet.DecoderLayer(cfg, W)
    layer.kv_cache.copy_(dev(rows).view(-1))
    eet.eet_restore(layer.handle, lens)
    set_oracle(oracle, lens, rows)
    for k in range(2):
        xs = wl.decode_embeddings(w, k)
        tok = dev(xs)
        got = torch.empty_like(tok)
        layer.decode_step(tok, got)
        gate(host(got), oracle.decode_step(xs), f"step {k}")
    layer.close()


def test_recorded_steps_at_other_lengths():
    """A stack's recorded steps: uneven, then even sequences after a restore, then uneven ones again, each as the direct steps bit for bit."""
    eet, heads, d, batch, max_seq = eet_module(), 4, 128, 65, 760
    rows = wl.normal(67, 9, (2, batch, heads, max_seq, d))
    w, W, cfg, oracle = build(heads, d, [1] * batch, max_seq, rows)
    direct, graph = eet.DecoderStack(cfg, [W], use_graph=False), eet.DecoderStack(cfg, [W])
    tok = dev(wl.decode_embeddings(w, 0))
    out = [torch.empty_like(tok) for _ in range(2)]
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for lens in (uneven(batch, 1, 720), [700] * batch, uneven(batch, 1, 730)):
            for st in (direct, graph):
                st.kv_cache.copy_(dev(rows).view(-1))
                eet.eet_stack_restore(st.handle, lens)
            set_oracle(oracle, lens, rows)
            for k in range(2):
                direct.decode_step(tok, out[0])
                graph.decode_step(tok, out[1])
                stream.synchronize()
                gate(host(out[0]), oracle.decode_step(wl.decode_embeddings(w, 0)), f"{lens[:3]}, step {k}")
                assert np.array_equal(host(out[0]).view(np.uint16), host(out[1]).view(np.uint16))
    direct.close()
    graph.close()
