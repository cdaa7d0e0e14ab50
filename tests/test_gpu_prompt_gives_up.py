"""Prompts in one launch (csrc/prompt_step.hip) whose waits come to their bound: what they leave is NaN, and the lengths come back with an error.  The waits
are ones that no item can end: the launch is recorded with its set-up in front, the set-up is taken out of the recording, and the numbers that the
items take start at 1 instead of 0, so that the first item never runs."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import eet_oracle as orc
from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, gate, host

pytestmark = pytest.mark.gpu

LENS, H, HEADS, F = [5, 3, 6], 128, 2, 256


def build(layers):
    from paper_2104_12470_amd import eet
    w = wl.Workload(f"late{layers}", 97, H, HEADS, F, layers, 3, 6, 3, 6, 4, 24)
    Ws = [wl.layer_weights(w, l, random_affine=True) for l in range(layers)]
    cfg = eet.make_config(H, HEADS, F, 3, 6, 24, w.ln_eps)
    tw = [{k: torch.from_numpy(v) for k, v in W.items()} for W in Ws]
    return eet, w, Ws, (eet.DecoderLayer(cfg, tw[0]) if layers == 1 else eet.DecoderStack(cfg, tw, use_graph=False))


def recorded(run, launches, first):
    """A recording of `run`, which is that many launches behind one another, without the first ones."""
    hip = ctypes.CDLL("libamdhip64.so")
    g = torch.cuda.CUDAGraph(keep_graph=True)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        run()
    graph = ctypes.c_void_p(g.raw_cuda_graph())
    for k in range(first):
        n = ctypes.c_size_t(0)
        assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0 and n.value == launches - k
        n, root = ctypes.c_size_t(1), ctypes.c_void_p()
        assert hip.hipGraphGetRootNodes(graph, ctypes.byref(root), ctypes.byref(n)) == 0 and n.value == 1
        assert hip.hipGraphDestroyNode(root) == 0
    g.instantiate()
    return g


def counters(words):
    """Where the item number and the counters of one row tile and one layer lie, a line of 32 words each, found as a finished prompt leaves them."""
    now = words.cpu().numpy()
    items = 3 * H // 64 + HEADS * len(LENS) + H // 64 + F // 64 + H // 64
    left = {0: items, 32: 0, 64: 3 * H // 64, 96: HEADS * sum(LENS), 128: H // 64, 160: F // 64}
    at = [i for i in range(0, len(now) - 256, 64) if all(now[i + k] == v and not now[i + k + 1:i + k + 32].any() for k, v in left.items())]
    assert len(at) == 1
    return words[at[0]:at[0] + 32 * (1 + 5 + H // 64)]


def test_a_wait_given_up_is_not_taken_for_a_result():
    eet, w, Ws, layer = build(1)
    oracle = orc.DecoderLayerOracle(Ws[0], HEADS, 3, 24, w.ln_eps)
    x = wl.prompt_embeddings(w)
    tokens, out = dev(x), torch.empty(x.shape, dtype=torch.float16, device="cuda:0")
    g = recorded(lambda: layer.prefill(tokens, LENS, out), 2, 1)

    def whole():
        layer.prefill(tokens, LENS, out)
        want = oracle.prefill(x, LENS)
        torch.cuda.synchronize()
        for b, n in enumerate(LENS):
            gate(host(out)[b, :n], want[b, :n], f"sequence {b}")
        assert layer.cache_lens(3) == LENS

    whole()
    control = counters(layer.workspace.view(torch.int32))
    control.zero_()
    control[0] = 1
    torch.cuda.synchronize()
    g.replay()
    torch.cuda.synchronize()
    for b, n in enumerate(LENS):
        assert np.all(np.isnan(host(out)[b, :n])) and not host(out)[b, n:].any()
    for k in range(2):
        with pytest.raises(eet.EETError) as e:
            layer.cache_lens(3)
        assert e.value.code == eet.EET_ERR_HIP
        got = layer.decode_step(dev(wl.decode_embeddings(w, k)))
        torch.cuda.synchronize()
        assert np.all(np.isnan(host(got))), k
    whole()
    for k in range(2):
        xs = wl.decode_embeddings(w, k)
        got = layer.decode_step(dev(xs))
        torch.cuda.synchronize()
        gate(host(got), oracle.decode_step(xs), f"step {k}")
    layer.close()


def test_what_the_first_layers_said_stays_said():
    """More layers than a launch takes: the set-up in front of the second launch leaves alone what the first may have said."""
    eet, w, Ws, stack = build(33)
    tokens = dev(wl.prompt_embeddings(w))
    out = torch.empty_like(tokens)
    g = recorded(lambda: stack.prefill(tokens, LENS, out), 4, 2)
    stack.prefill(tokens, LENS, out)
    torch.cuda.synchronize()
    assert stack.cache_lens(3) == LENS
    words = stack.workspace.view(torch.int64)
    now = words.cpu().numpy()
    at = [i for i in range(0, len(now) - 256, 32) if not now[i:i + 32].any() and np.all(now[i + 32:i + 256] == -1)]
    assert len(at) == 1
    words[at[0]] = 1 << 31                                     # as a wait given up in the first launch leaves it
    torch.cuda.synchronize()
    g.replay()
    torch.cuda.synchronize()
    with pytest.raises(eet.EETError) as e:
        stack.cache_lens(3)
    assert e.value.code == eet.EET_ERR_HIP
    stack.prefill(tokens, LENS, out)
    torch.cuda.synchronize()
    assert stack.cache_lens(3) == LENS
    stack.close()
