"""A stack whose decode steps are several launches replays them from its recorded graph (one whose steps are one launch is launched directly): the same
bits as direct launches, step after step, also after a prefill of another batch size."""
import numpy as np
import pytest
import torch

from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, host

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
