"""A stack whose decode steps are several launches replays them from its recorded graph (one whose steps are one launch is launched directly): the same
bits as direct launches, step after step, also after a prefill of another batch size."""
import numpy as np
import pytest
import torch

from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, host, kernels_of

pytestmark = pytest.mark.gpu


def test_replayed_steps_match_direct_launches():
    from paper_2104_12470_amd import eet
    H, heads, F, B, S = 128, 2, 8256, 4, 20                  # more feed-forward columns than a step in one launch takes
    w = wl.Workload("recorded", 71, H, heads, F, 2, B, S, 1, S, 4, S + 8)
    Ws = [{k: torch.from_numpy(v) for k, v in wl.layer_weights(w, l, random_affine=True).items()} for l in range(2)]
    cfg = eet.make_config(H, heads, F, B, S, S + 8, w.ln_eps)
    direct, graphed = eet.DecoderStack(cfg, Ws, use_graph=False), eet.DecoderStack(cfg, Ws, use_graph=True)
    side = torch.cuda.Stream()
    x = dev(wl.prompt_embeddings(w))
    tok = torch.empty((B, H), dtype=torch.float16, device="cuda:0")
    out = torch.empty_like(tok)
    torch.cuda.synchronize()
    for lens in ([3, 20, 7, 1], [5, 19]):
        n = len(lens)
        with torch.cuda.stream(side):
            for st in (direct, graphed):
                st.prefill(x[:n], lens)
            for k in range(4):
                xs = dev(wl.decode_embeddings(w, k)[:n])
                tok[:n].copy_(xs)
                want = direct.decode_step(xs)
                graphed.decode_step(tok[:n], out[:n])
                side.synchronize()
                assert np.all(np.isfinite(host(want)))
                assert np.array_equal(host(out[:n]).view(np.uint16), host(want).view(np.uint16)), (n, k)
                assert graphed.cache_lens(n) == direct.cache_lens(n) == [v + k + 1 for v in lens]
                torch.randn(64, 64, device="cuda:0").sum()   # eager work in between
    direct.close()
    graphed.close()


def test_recordings_on_either_side_of_the_memory_side_cache():
    """Weights and K/V rows of a step that moves more than the memory-side cache (256 MiB) holds are loaded as read once, so a stack keeps a recording for either
    side and takes the one that its sequences call for, back and forth by way of a restore: direct and replayed launches load as they should, either
    recording is made once, and the bits are the same."""
    from paper_2104_12470_amd import eet
    layers, H, F = 2, 1024, 8256                             # more feed-forward columns than a step in one launch takes
    keys = ((256 << 20) - layers * 2 * (4 * H * H + 2 * H * F)) // (layers * 4 * H)      # visible keys of both sequences together: the last that fit
    w = wl.Workload("sides", 73, H, 16, F, layers, 2, 1, 1, 1, 4, keys // 2 + 8)
    cfg = eet.make_config(w.hidden, w.heads, w.ffn, w.batch, w.padded_len, w.max_seq, w.ln_eps)
    Ws = [{k: torch.from_numpy(v) for k, v in wl.layer_weights(w, li).items()} for li in range(layers)]
    direct, graphed = eet.DecoderStack(cfg, Ws, use_graph=False), eet.DecoderStack(cfg, Ws)
    direct.kv_cache.copy_(torch.randn(direct.kv_cache.shape, dtype=torch.float16, device="cuda:0"))
    graphed.kv_cache.copy_(direct.kv_cache)
    below = [keys // 2 - 1, keys - keys // 2 - 1]
    tok, stream = dev(wl.decode_embeddings(w, 0)), torch.cuda.Stream()
    out = [torch.empty_like(tok) for _ in range(2)]
    recorded = set()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for _ in range(3):
            for st in (direct, graphed):
                eet.eet_stack_restore(st.handle, below)
            for once in ("false", "true", "true"):
                for st, o in ((direct, out[0]), (graphed, out[1])):
                    names = kernels_of(lambda: st.decode_step(tok, o))
                    loads = [n.split("attn_decode<")[1].split(">")[0] for n in names if "attn_decode<" in n]
                    assert len(loads) == layers and all(n.endswith(once) for n in loads), names
                    launched, made = "hipGraphLaunch" in names, "hipGraphInstantiate" in names
                    assert (launched, made) == ((True, once not in recorded) if st is graphed else (False, False)), names
                recorded.add(once)
                stream.synchronize()
                assert bool(torch.isfinite(out[0]).all()) and torch.equal(out[0], out[1])
                assert graphed.cache_lens(2) == direct.cache_lens(2)
    direct.close()
    graphed.close()
