"""Decode steps in one launch of more sequences than one group of rows holds: groups of equal and unequal size, up to all of them, both head sizes, more
layers than a launch takes, ragged lengths, and steps of other numbers of sequences in between."""
import numpy as np
import pytest
import torch

from oracle import eet_oracle as orc
from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, gate, host, kernels_of

pytestmark = pytest.mark.gpu


def build(hidden, heads, ffn, batch, layers, S, cap):
    from paper_2104_12470_amd import eet
    w = wl.Workload(f"groups{hidden}x{batch}", 89, hidden, heads, ffn, layers, batch, S, 1, S, 4, cap)
    Ws = [wl.layer_weights(w, l, random_affine=True) for l in range(layers)]
    cfg = eet.make_config(hidden, heads, ffn, batch, S, cap, w.ln_eps)
    return eet, w, Ws, cfg


@pytest.mark.parametrize("hidden,heads,ffn,batch,S,cap", [
    (64, 1, 64, 128, 9, 14),            # eight groups of 16
    (256, 2, 1024, 17, 40, 50),         # heads of 128; 9 and 8
    (320, 5, 1280, 33, 12, 520),        # three of 11
    (1024, 16, 4096, 40, 6, 10),        # 14, 14, 12
    (768, 6, 3072, 50, 5, 9),           # 13, 13, 13, 11
    (256, 4, 640, 64, 30, 511),         # 256 pairs
    (448, 7, 1792, 48, 8, 511),         # 336 pairs: the last capacity that more of them take
])
def test_steps_against_the_oracle(hidden, heads, ffn, batch, S, cap):
    eet, w, Ws, cfg = build(hidden, heads, ffn, batch, 1, S, cap)
    layer = eet.DecoderLayer(cfg, {k: torch.from_numpy(v) for k, v in Ws[0].items()})
    oracle = orc.DecoderLayerOracle(Ws[0], heads, batch, cap, w.ln_eps)
    lens, x = [1 + b * 5 % S for b in range(batch)], wl.prompt_embeddings(w)
    layer.prefill(dev(x), lens)
    oracle.prefill(x, lens)
    for k in range(4):
        xs = wl.decode_embeddings(w, k)
        got = layer.decode_step(dev(xs))
        torch.cuda.synchronize()
        gate(host(got), oracle.decode_step(xs), f"step {k}")
    assert layer.cache_lens(batch) == oracle.lens[:batch].tolist()
    tok = dev(wl.decode_embeddings(w, 0))
    if max(lens) + 5 <= cap:
        assert [n for n in kernels_of(lambda: layer.decode_step(tok)) if "eet" in n and "decode_layers" not in n] == []
    layer.close()


@pytest.mark.parametrize("hidden,heads,ffn,batch,alone", [
    (1024, 16, 4096, 28, True), (1024, 16, 4096, 29, False),    # pairs times hidden: 448 and 464 K
    (1024, 16, 4096, 40, False),
    (768, 12, 3072, 48, True),
    (512, 4, 2048, 128, True), (512, 8, 2048, 88, False),       # 1280 and 1296 items
])
def test_a_layer_on_its_own_stops_earlier(hidden, heads, ffn, batch, alone):
    """Steps in one launch of a layer, up to where its launches are ahead, and of two layers, beyond it: which kernels run, and the oracle."""
    S, cap = 6, 24
    eet, w, Ws, cfg = build(hidden, heads, ffn, batch, 2, S, cap)
    tw = [{k: torch.from_numpy(v) for k, v in W.items()} for W in Ws]
    layer, stack = eet.DecoderLayer(cfg, tw[0]), eet.DecoderStack(cfg, tw, use_graph=False)
    oracles = [orc.DecoderLayerOracle(W, heads, batch, cap, w.ln_eps) for W in Ws]
    lens, x = [1 + b * 5 % S for b in range(batch)], wl.prompt_embeddings(w)
    layer.prefill(dev(x), lens)
    stack.prefill(dev(x), lens)
    oracles[1].prefill(oracles[0].prefill(x, lens).astype(np.float16), lens)
    for k in range(2):
        xs = wl.decode_embeddings(w, k)
        got, both = layer.decode_step(dev(xs)), stack.decode_step(dev(xs))
        torch.cuda.synchronize()
        want = oracles[0].decode_step(xs)
        gate(host(got), want, f"layer, step {k}")
        gate(host(both), oracles[1].decode_step(want.astype(np.float16)), f"stack, step {k}", 5e-2, 5e-3)
    assert layer.cache_lens(batch) == stack.cache_lens(batch) == oracles[0].lens[:batch].tolist()
    tok = dev(wl.decode_embeddings(w, 0))
    for st, one in ((layer, alone), (stack, True)):
        names = kernels_of(lambda: st.decode_step(tok))
        assert (any("decode_layers" in n for n in names), any("attn_decode" in n for n in names)) == (one, not one), names
    layer.close()
    stack.close()


@pytest.mark.parametrize("layers", [2, 35])
def test_other_numbers_of_sequences_in_between(layers):
    """Prompts of 40, 5, 21 and 40 sequences on one handle, steps after each, a recorded step of 40 replayed in between: every sequence as on a handle of
    its own number, bit for bit."""
    eet, w, Ws, cfg = build(128, 2, 320, 40, layers, 6, 24)
    tw = [{k: torch.from_numpy(v) for k, v in W.items()} for W in Ws]
    stack = eet.DecoderStack(cfg, tw, use_graph=False)
    x, lens = wl.prompt_embeddings(w), [1 + b % 6 for b in range(40)]
    stack.prefill(dev(x), lens)
    tok, g = dev(wl.decode_embeddings(w, 3)), torch.cuda.CUDAGraph()
    out = torch.empty_like(tok)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        stack.decode_step(tok, out)
    for B in (40, 5, 21, 40):
        alone = eet.DecoderStack(eet.make_config(128, 2, 320, B, 6, 24, w.ln_eps), tw, use_graph=False)
        for st in (stack, alone):
            st.prefill(dev(x[:B]), lens[:B])
        for k in range(3):
            xs = dev(wl.decode_embeddings(w, k)[:B])
            got, want = stack.decode_step(xs), alone.decode_step(xs)
            torch.cuda.synchronize()
            assert np.all(np.isfinite(host(want))) and np.array_equal(host(got).view(np.uint16), host(want).view(np.uint16)), (B, k)
            if k == 1:                                         # 40 rows over what the handle holds now
                g.replay()
                want = alone.decode_step(tok[:B].contiguous())
                torch.cuda.synchronize()
                assert np.array_equal(host(out)[:B].view(np.uint16), host(want).view(np.uint16)), B
        alone.close()
    stack.close()


@pytest.mark.parametrize("how", ["said before", "a wait that ends by itself"])
def test_a_wait_given_up_in_one_group(how):
    """A step of two groups where the second has given up a wait before, or gives up now: its count of emptied parts starts far below what its items wait for,
    so each of them runs into its own bound.  Its sequences are NaN, the first group's are not, and the lengths come back with an error."""
    eet, w, Ws, cfg = build(128, 2, 256, 20, 1, 6, 24)
    layer = eet.DecoderLayer(cfg, {k: torch.from_numpy(v) for k, v in Ws[0].items()})
    layer.prefill(dev(wl.prompt_embeddings(w)), [3] * 20)
    torch.cuda.synchronize()
    words = layer.workspace.view(torch.int64)
    now = words.cpu().numpy()
    at = [i for i in range(0, len(now) - 256, 16) if not now[i:i + 32].any() and np.all(now[i + 32:i + 256] == -1)]
    assert len(at) == 2
    if how == "said before":
        words[at[1]] = 1 << 31
    else:
        words[at[1] + 16] = 0xfff00000
    torch.cuda.synchronize()
    got = host(layer.decode_step(dev(wl.decode_embeddings(w, 0))))
    torch.cuda.synchronize()
    assert np.all(np.isfinite(got[:10])) and np.all(np.isnan(got[10:]))
    with pytest.raises(eet.EETError) as e:
        layer.cache_lens(20)
    assert e.value.code == eet.EET_ERR_HIP
    layer.close()
