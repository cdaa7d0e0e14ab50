"""A layer's decode step attends as the operator does, bit for bit.

The step and eet_op_attention_decode run one kernel on one cut of the keys, whoever merges the key ranges, and that cut depends on the
numbers of sequences and heads and on the capacity alone: a sequence's result is the same whatever the lengths of its neighbours and
whether its step was recorded at other lengths.  The layer here hands the attention through: the projection of Q is its
bias, the output projection the identity, and the feed-forward part adds nothing to an input of zeros."""
import numpy as np
import pytest
import torch

from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu


def uneven(batch, lo, hi):
    lens = [lo + (hi - lo) * (b * 7 % batch) // batch for b in range(batch)]
    lens[batch // 2] = hi
    return lens


def layer_that_hands_on(heads, d, batch, max_seq):
    from paper_2104_12470_amd import eet
    H = heads * d
    W = wl.layer_weights(wl.Workload("handson", 83, H, heads, 128, 1, batch, 1, 1, 1, 2, max_seq), 0, random_affine=True)
    W["w_qkv"][:H] = 0
    W["b_qkv"][:H] = wl.normal(83, 3, (H,))
    W["w_o"] = np.eye(H, dtype=np.float16)
    for name in ("b_o", "w_fc2", "b_fc2"):
        W[name] = np.zeros_like(W[name])
    cfg = eet.make_config(H, heads, 128, batch, 1, max_seq, 1e-5)
    layer = eet.DecoderLayer(cfg, {k: torch.from_numpy(v) for k, v in W.items()})
    q = dev(W["b_qkv"][:H].astype(np.float16)).repeat(batch, 1).view(batch, heads, d)
    return eet, layer, q


def operator(eet, q, kv, lens, max_seq):
    batch, heads, d = q.shape
    kv = kv.view(2, batch, heads, max_seq, d)
    ctx = torch.empty_like(q)
    scratch = torch.empty(max(1, eet.eet_op_attention_decode_scratch_bytes(batch, heads, d, max_seq)), dtype=torch.uint8, device="cuda:0")
    eet.eet_op_attention_decode(q, kv[0].contiguous(), kv[1].contiguous(), ctx, torch.tensor(lens, dtype=torch.int32, device="cuda:0"), scratch)
    return ctx


@pytest.mark.parametrize("heads,d,lens,max_seq", [
    (17, 128, [300], 320),                           # two ranges
    (17, 128, [17], 2100),                           # sixteen, most of them empty
    (18, 128, [700, 1, 350], 720),                   # 54 pairs, four ranges
    (36, 64, [500, 600], 640),                       # heads of 64
    (31, 128, [767, 900, 30, 1279], 1300),           # 124, four ranges
    (64, 64, [766, 767], 800),                       # 128 pairs and more: one range
    (32, 128, [767, 900, 30, 1279], 1300),
    (32, 128, uneven(5, 1, 900), 910),
    (4, 128, uneven(65, 1, 720), 730),               # 260, uneven
    (5, 64, uneven(52, 1, 800), 810),
    (4, 128, [720] * 65, 730),                       # even
])
def test_step_attends_as_the_operator(heads, d, lens, max_seq):
    eet, layer, q = layer_that_hands_on(heads, d, len(lens), max_seq)
    layer.kv_cache.copy_(dev(wl.normal(83, 9, (2, len(lens), heads, max_seq, d))).view(-1))
    eet.eet_restore(layer.handle, lens)
    tok = torch.zeros((len(lens), heads * d), dtype=torch.float16, device="cuda:0")
    out = torch.empty_like(tok)
    for k in range(2):
        layer.decode_step(tok, out)
        want = operator(eet, q, layer.kv_cache, [n + k + 1 for n in lens], max_seq)
        assert np.array_equal(host(out), host(want).reshape(len(lens), -1)), f"step {k}"
    assert np.abs(host(out)).max() > 0.05
    layer.close()


def test_a_recorded_step_serves_other_lengths():
    """A step that the caller records, replayed at lengths of another spread: as direct steps and as the operator."""
    heads, d, batch, max_seq = 4, 128, 65, 760
    eet, layer, q = layer_that_hands_on(heads, d, batch, max_seq)
    rows = dev(wl.normal(83, 9, (2, batch, heads, max_seq, d))).view(-1)
    tok = torch.zeros((batch, heads * d), dtype=torch.float16, device="cuda:0")
    out = torch.empty_like(tok)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        layer.kv_cache.copy_(rows)
        eet.eet_restore(layer.handle, [700] * batch, stream=stream)
        layer.decode_step(tok, out, stream=stream)
        stream.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            layer.decode_step(tok, out, stream=stream)
        for lens in (uneven(batch, 1, 720), [700] * batch, uneven(batch, 1, 740)):
            for replay in (True, False):
                layer.kv_cache.copy_(rows)
                eet.eet_restore(layer.handle, lens, stream=stream)
                for k in range(2):
                    graph.replay() if replay else layer.decode_step(tok, out, stream=stream)
                    stream.synchronize()
                    want = operator(eet, q, layer.kv_cache, [n + k + 1 for n in lens], max_seq)
                    stream.synchronize()
                    assert np.array_equal(host(out), host(want).reshape(batch, -1)), f"{'replayed' if replay else 'direct'}, step {k}"
    layer.close()
