"""Decode steps that run as one launch (csrc/decode_step.hip), at the edges of what it takes: waves without a unit of K and
with unequal numbers of them, 1 to 16 rows and the rows just past each variant, both head sizes, key ranges that are merged,
empty or end at the new token, the widest layer, one that is just past the narrow variant, and stacks of more layers than a launch takes."""
import numpy as np
import pytest
import torch

from oracle import eet_oracle as orc
from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, gate, host, kernels_of

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eet():
    from paper_2104_12470_amd import eet as binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


def layer_and_oracle(eet, w, layer=0):
    W = wl.layer_weights(w, layer, random_affine=True)
    cfg = eet.make_config(w.hidden, w.heads, w.ffn, w.batch, w.padded_len, w.max_seq, w.ln_eps)
    return eet.DecoderLayer(cfg, {k: torch.from_numpy(v) for k, v in W.items()}), orc.DecoderLayerOracle(W, w.heads, w.batch, w.max_seq, w.ln_eps)


@pytest.mark.parametrize("hidden,heads,ffn,batch,len_hi,max_seq", [
    (64, 1, 64, 1, 9, 16),             # one unit of K: seven waves idle
    (192, 3, 320, 3, 20, 32),          # three and five units
    (576, 9, 1536, 9, 12, 24),         # nine units; the variant of 16 rows
    (1024, 16, 4096, 16, 8, 16),       # the narrow variant full
    (1088, 17, 4352, 8, 8, 16),        # just past it
    (1024, 8, 4160, 5, 8, 16),         # past it by the feed-forward width alone
    (2048, 16, 8192, 2, 8, 16),        # the widest
    (256, 2, 704, 2, 300, 1040),       # four key ranges per pair, the last ones empty
    (256, 4, 640, 4, 144, 528),        # four ranges; key 144 is the first of its range when it is the new token
    (128, 2, 256, 8, 70, 74),          # the variant of 8 rows; up to the capacity
])
def test_steps_against_the_oracle(eet, hidden, heads, ffn, batch, len_hi, max_seq):
    steps = 4
    w = wl.Workload(f"step{hidden}x{ffn}", 31, hidden, heads, ffn, 1, batch, len_hi, max(1, len_hi - 7), len_hi, steps, max_seq)
    layer, oracle = layer_and_oracle(eet, w)
    lens, x = wl.lengths(w), wl.prompt_embeddings(w)
    layer.prefill(dev(x), lens)
    oracle.prefill(x, lens)
    for k in range(steps):
        xs = wl.decode_embeddings(w, k)
        got = layer.decode_step(dev(xs))
        torch.cuda.synchronize()
        gate(host(got), oracle.decode_step(xs), f"step {k}")
    assert layer.cache_lens(batch) == oracle.lens[:batch].tolist()
    kc, vc = layer.cache_views()
    for b in range(batch):
        n = int(lens[b]) + steps
        gate(host(kc[b, :, :n]), oracle.k_cache[b, :, :n], f"K cache b={b}", 1.5e-2, 1.5e-3)
        gate(host(vc[b, :, :n]), oracle.v_cache[b, :, :n], f"V cache b={b}", 1.5e-2, 1.5e-3)
    layer.close()


@pytest.mark.parametrize("d,lens", [(64, [1, 1022, 1023, 1024, 1025, 1055, 1056, 1100, 1535, 2046, 2047, 2048, 2100]),
                                    (128, [1, 510, 511, 512, 513, 527, 528, 600, 767, 1022, 1023, 1024, 1100])])
def test_more_keys_than_an_item_holds(eet, d, lens):
    """65 pairs are not split, and an attention item requests 1024 keys (512 of heads of 128) before its query arrives and the rest as it
    goes: caches that end on either side of one and of two such loads, and of a wave's blocks behind them."""
    heads, batch, max_seq = 5, len(lens), max(lens) + 4
    w = wl.Workload(f"refill{d}", 67, heads * d, heads, 448, 1, batch, 1, 1, 1, 2, max_seq)
    layer, oracle = layer_and_oracle(eet, w)
    rows = wl.normal(w.seed, 9, (2, batch, heads, max_seq, d))
    for b, n in enumerate(lens):
        rows[:, b, :, n:] = np.nan                             # slots that hold no key yet are never read
    layer.kv_cache.copy_(dev(rows).view(-1))
    eet.eet_restore(layer.handle, lens)
    oracle.batch, oracle.lens[:], oracle.k_cache[:], oracle.v_cache[:] = batch, lens, rows[0], rows[1]
    for k in range(2):
        xs = wl.decode_embeddings(w, k)
        got = torch.empty_like(dev(xs))
        names = kernels_of(lambda: layer.decode_step(dev(xs), got))
        assert any("decode_layers" in n for n in names), names
        gate(host(got), oracle.decode_step(xs), f"step {k}")
    layer.close()


@pytest.mark.parametrize("n_layers", [2, 3, 33])
def test_stack_equals_the_layer_chain(eet, n_layers):
    """Layers of one launch exchange their rows on the device; one after the other they go through memory.  The same bits, also after a
    second prefill with another number of sequences (another layout of the exchange area) and where a step takes two launches (33 layers)."""
    w = wl.Workload(f"chain{n_layers}", 37, 192, 3, 448, n_layers, 3, 24, 3, 24, 6, 32)
    cfg = eet.make_config(w.hidden, w.heads, w.ffn, w.batch, w.padded_len, w.max_seq, w.ln_eps)
    Ws = [{k: torch.from_numpy(v) for k, v in wl.layer_weights(w, li, random_affine=True).items()} for li in range(n_layers)]
    stack = eet.DecoderStack(cfg, Ws)
    layers = [eet.DecoderLayer(cfg, W) for W in Ws]
    lens, x = wl.lengths(w), wl.prompt_embeddings(w)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for B in (3, 1, 2):
            h = dev(x[:B])
            stack.prefill(h, lens[:B])
            for layer in layers:
                h = layer.prefill(h, lens[:B])
            for k in range(5):
                h = dev(wl.decode_embeddings(w, k)[:B])
                got = stack.decode_step(h)
                for layer in layers:
                    h = layer.decode_step(h)
                stream.synchronize()
                assert np.array_equal(host(got).view(np.uint16), host(h).view(np.uint16)), (B, k)
    stack.close()
    for layer in layers:
        layer.close()


def test_two_streams_at_once(eet):
    """Two stacks whose steps run side by side on two streams, more items each than the device holds: both finish, with the
    bits that each gives on its own."""
    w = wl.Workload("twostreams", 41, 512, 8, 2048, 12, 4, 16, 16, 16, 6, 32)
    cfg = eet.make_config(w.hidden, w.heads, w.ffn, w.batch, w.padded_len, w.max_seq, w.ln_eps)
    Ws = [{k: torch.from_numpy(v) for k, v in wl.layer_weights(w, li, random_affine=True).items()} for li in range(12)]
    lens, x = wl.lengths(w), wl.prompt_embeddings(w)
    xs = [dev(wl.decode_embeddings(w, k)) for k in range(6)]
    stacks, streams = [eet.DecoderStack(cfg, Ws) for _ in range(3)], [torch.cuda.Stream() for _ in range(3)]
    outs = [[torch.empty_like(xs[0]) for _ in xs] for _ in stacks]
    torch.cuda.synchronize()
    for i in range(3):
        with torch.cuda.stream(streams[i]):
            stacks[i].prefill(dev(x), lens)
    torch.cuda.synchronize()
    for k in range(6):                                         # stack 0 alone, then 1 and 2 together
        with torch.cuda.stream(streams[0]):
            stacks[0].decode_step(xs[k], outs[0][k])
    torch.cuda.synchronize()
    for k in range(6):
        for i in (1, 2):
            with torch.cuda.stream(streams[i]):
                stacks[i].decode_step(xs[k], outs[i][k])
    torch.cuda.synchronize()
    for i in (1, 2):
        for k in range(6):
            assert np.array_equal(host(outs[i][k]).view(np.uint16), host(outs[0][k]).view(np.uint16)), (i, k)
    for st in stacks:
        st.close()


@pytest.mark.parametrize("max_batch,latest", [(5, 2), (18, 2), (18, 18)])
def test_recorded_steps_of_other_numbers_of_sequences(eet, max_batch, latest):
    """Steps that a caller recorded for 5 sequences and for 1 are replayed in turn after a prefill of `latest` sequences, between eager steps
    of that many (18: launch by launch, through the attention partials).  Each is another layout of the exchange area; the sequences that a
    step shares with the latest prefill get what the oracle gives, and the others disturb nothing."""
    w = wl.Workload(f"recorded{max_batch}x{latest}", 47, 256, 2, 704, 1, max_batch, 40, 9, 40, 8, 1040)
    W = wl.layer_weights(w, 0, random_affine=True)
    cfg = eet.make_config(w.hidden, w.heads, w.ffn, max_batch, w.padded_len, w.max_seq, w.ln_eps)
    layer = eet.DecoderLayer(cfg, {k: torch.from_numpy(v) for k, v in W.items()})
    lens, x, xs = wl.lengths(w), wl.prompt_embeddings(w), wl.decode_embeddings(w, 0)
    recorded = {}
    for B in (5, 1):
        layer.prefill(dev(x[:B]), lens[:B])
        tok, g = dev(xs[:B]), torch.cuda.CUDAGraph()
        out = torch.empty_like(tok)
        torch.cuda.synchronize()
        with torch.cuda.graph(g):
            layer.decode_step(tok, out)
        recorded[B] = (g, tok, out)
    layer.prefill(dev(x[:latest]), lens[:latest])
    oracles = [orc.DecoderLayerOracle(W, w.heads, 1, w.max_seq, w.ln_eps) for _ in range(2)]
    for b, o in enumerate(oracles):
        o.prefill(x[b:b + 1], lens[b:b + 1])
    for k, B in enumerate((5, latest, 1, 5, 5, latest, latest, 1, 1, latest, 5)):
        if B == latest:
            got = layer.decode_step(dev(xs[:B]))
        else:
            recorded[B][0].replay()
            got = recorded[B][2]
        torch.cuda.synchronize()
        for b in range(min(B, 2)):
            gate(host(got)[b:b + 1], oracles[b].decode_step(xs[b:b + 1]), f"step {k} of {B}, sequence {b}")
    assert layer.cache_lens(latest)[:2] == [int(o.lens[0]) for o in oracles]
    layer.close()


def step_control(layer):
    """The words that the items of a decode step share (kernels.hpp: kStepCtlWords), found as what the set-up of the exchange area leaves: 32
    words of zeros, then sets of all ones."""
    words = layer.workspace.view(torch.int64)
    now = words.cpu().numpy()
    at = [i for i in range(0, len(now) - 256, 32) if not now[i:i + 32].any() and np.all(now[i + 32:i + 256] == -1)]
    assert len(at) == 1
    return words[at[0]:at[0] + 32]


@pytest.mark.parametrize("how", ["said before", "a wait that ends by itself"])
def test_a_wait_given_up_is_not_taken_for_a_result(eet, how):
    """Once a wait inside a step has given up, the step and all that follow leave NaN, count as steps, and the lengths come back with an
    error; a prefill or a restore makes the handle whole.  The wait is one that no item can end: the count of emptied parts starts far
    below what they wait for, so each of them runs into its own bound."""
    w = wl.Workload("gaveup", 53, 128, 2, 256, 1, 3, 9, 2, 9, 4, 32)
    layer, oracle = layer_and_oracle(eet, w)
    lens, x = wl.lengths(w), wl.prompt_embeddings(w)
    layer.prefill(dev(x), lens)
    oracle.prefill(x, lens)
    torch.cuda.synchronize()
    control = step_control(layer)
    if how == "said before":
        control[0] = 1 << 31
    else:
        control[16] = 0xfff00000
    for k in range(2):
        got = layer.decode_step(dev(wl.decode_embeddings(w, k)))
        torch.cuda.synchronize()
        assert np.all(np.isnan(host(got))), k
        with pytest.raises(eet.EETError) as e:
            layer.cache_lens(3)
        assert e.value.code == eet.EET_ERR_HIP
    eet.eet_restore(layer.handle, lens)
    for k in range(2):
        xs = wl.decode_embeddings(w, k)
        got = layer.decode_step(dev(xs))
        torch.cuda.synchronize()
        gate(host(got), oracle.decode_step(xs), f"step {k}")
    assert layer.cache_lens(3) == oracle.lens[:3].tolist()
    layer.close()


def test_a_stack_counts_the_keys_its_sequences_hold(eet):
    """Weights and K/V rows of a step that moves more than the memory-side cache (256 MiB) holds are loaded as read once, and what a step moves
    grows with the sequences: two layers of hidden 1024 (50 MB of weights) pass the line at 25000 keys.  A stack created with use_graph
    launches such steps directly too and gives the same bits on both sides, back and forth (recorded steps: test_gpu_stack_recorded.py)."""
    layers, H, line = 2, 1024, (256 << 20) - 2 * 2 * 12 * 1024 * 1024
    keys = line // (layers * 4 * H)                            # visible keys of both sequences together, the new tokens' among them: the last that fit
    w = wl.Workload("held", 59, H, 16, 4 * H, layers, 2, 1, 1, 1, 4, keys // 2 + 8)
    cfg = eet.make_config(w.hidden, w.heads, w.ffn, w.batch, w.padded_len, w.max_seq, w.ln_eps)
    Ws = [{k: torch.from_numpy(v) for k, v in wl.layer_weights(w, li).items()} for li in range(layers)]
    direct, graph = eet.DecoderStack(cfg, Ws, use_graph=False), eet.DecoderStack(cfg, Ws)
    direct.kv_cache.copy_(torch.randn(direct.kv_cache.shape, dtype=torch.float16, device="cuda:0"))
    graph.kv_cache.copy_(direct.kv_cache)
    below = [keys // 2 - 1, keys - keys // 2 - 1]
    tok, stream = dev(wl.decode_embeddings(w, 0)), torch.cuda.Stream()
    out = [torch.empty_like(tok) for _ in range(2)]
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for _ in range(2):
            for st in (direct, graph):
                eet.eet_stack_restore(st.handle, below)
            for once in ("false", "true", "true"):
                names = [n for n in kernels_of(lambda: direct.decode_step(tok, out[0])) if "decode_layers" in n]
                assert len(names) == 1 and names[0].split("decode_layers<")[1].split(">")[0].endswith(once), names
                graph.decode_step(tok, out[1])
                stream.synchronize()
                assert np.array_equal(host(out[0]).view(np.uint16), host(out[1]).view(np.uint16))
    direct.close()
    graph.close()


@pytest.mark.parametrize("heads,batch,kernel", [(5, 13, "attn_decode"), (4, 16, "decode_layers"), (8, 14, "attn_decode"), (8, 15, "decode_layers")])
def test_steps_that_outgrow_one_launch(eet, heads, batch, kernel):
    """From 8192 keys per sequence on, 65 to 112 pairs of heads of 128 go launch by launch (64 and 113 and more, up to 223, never).  The sequences
    cross the line between two steps, direct and recorded, and a restore takes them back; the oracle follows all of it."""
    H, first = 128 * heads, 8190
    w = wl.Workload(f"outgrow{heads}x{batch}", 61, H, heads, 256, 1, batch, 1, 1, 1, 4, 8208)
    W = wl.layer_weights(w, 0, random_affine=True)
    cfg = eet.make_config(H, heads, w.ffn, batch, 1, w.max_seq, w.ln_eps)
    Ws = [{k: torch.from_numpy(v) for k, v in W.items()}]
    direct, graph = eet.DecoderStack(cfg, Ws, use_graph=False), eet.DecoderStack(cfg, Ws)
    oracle = orc.DecoderLayerOracle(W, heads, batch, w.max_seq, w.ln_eps)
    rows = wl.normal(w.seed, 9, (2, batch, heads, w.max_seq, 128))
    direct.kv_cache.copy_(dev(rows).view(-1))
    graph.kv_cache.copy_(direct.kv_cache)
    xs = wl.decode_embeddings(w, 0)
    lens, stream, tok = [first] * batch, torch.cuda.Stream(), dev(xs)
    out = [torch.empty_like(tok) for _ in range(2)]
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for _ in range(2):
            for st in (direct, graph):
                eet.eet_stack_restore(st.handle, lens)
            oracle.batch, oracle.lens[:batch] = batch, lens
            oracle.k_cache[:batch], oracle.v_cache[:batch] = rows[0], rows[1]
            for k in range(4):
                names = kernels_of(lambda: direct.decode_step(tok, out[0]))
                assert any(("decode_layers" if first + k + 1 <= 8192 else kernel) in n for n in names), (k, names)
                graph.decode_step(tok, out[1])
                stream.synchronize()
                gate(host(out[0]), oracle.decode_step(xs), f"step {k}")
                assert np.array_equal(host(out[0]).view(np.uint16), host(out[1]).view(np.uint16)), k
    direct.close()
    graph.close()
