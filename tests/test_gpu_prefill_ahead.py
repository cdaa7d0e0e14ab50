"""Which prefill attentions touch weights on the side: a layer's, by its rule, and never an operator's, whose kernels have nothing of it.  One launch of each of
the three kernels, with one chunk of pairs; the numbers are those of the oracle either way."""
import numpy as np
import pytest
import torch

from oracle import eet_oracle as orc
from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, gate, host, kernels_of

pytestmark = pytest.mark.gpu

SHAPES = [(4, 64, [43] * 5, "attn_prefill16<64, true"),        # short prompts
          (2, 128, [100, 1, 300], "attn_prefill16<128, true"),
          (3, 64, [300, 20], "attn_prefill<true"),
          (2, 128, [600, 513], "attn_prefill_wide<128, true")]


@pytest.mark.parametrize("heads,d,lens,kernel", SHAPES)
def test_layer_touches_weights(heads, d, lens, kernel):
    from paper_2104_12470_amd import eet
    H, B, S = heads * d, len(lens), max(lens)
    w = wl.Workload("ahead", 89, H, heads, 4 * H, 1, B, S, 1, S, 0, S)
    W = wl.layer_weights(w, 0, random_affine=True)
    layer = eet.DecoderLayer(eet.make_config(H, heads, 4 * H, B, S, S, w.ln_eps), {k: torch.from_numpy(v) for k, v in W.items()})
    x = wl.prompt_embeddings(w)
    tok = dev(x)
    out = torch.empty_like(tok)
    names = kernels_of(lambda: layer.prefill(tok, lens, out))
    assert any(kernel in n and "true>" in n for n in names), names
    oracle = orc.DecoderLayerOracle(W, heads, B, S, w.ln_eps)
    want = oracle.prefill(x, lens)
    for b, n in enumerate(lens):
        gate(host(out)[b, :n], want[b, :n], f"sequence {b}")
    layer.close()


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
