"""Prefill attention of prompts of up to 512 tokens, 256 with heads of 64 (attn_prefill16): both workgroup sizes (fewer than 160 or
320 tiles of 128 rows, and more), both head sizes, both windows, lengths on either side of the 16-row waves, the 64-key tiles and
the 64- and 128-row query tiles, and the last length before the kernels for longer prompts."""
import numpy as np
import pytest
import torch

from oracle import eet_oracle as orc
from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, gate, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,lens", [
    (2, [1, 15, 16, 17, 63, 64, 65, 127, 128, 129]),          # 64-row workgroups
    (1, [200, 255, 256]),
    (1, [257, 511, 512]),                                     # heads of 64: the kernel for longer prompts
    (1, [513]),                                               # the kernels for longer prompts
    (80, [1, 48, 64, 65]),                                    # 320 tiles: 128-row workgroups
    (27, [16, 17, 33, 112, 113, 127, 128, 129, 130, 2, 64]),  # 351
])
def test_against_the_oracle(d, heads, lens, causal):
    from paper_2104_12470_amd import eet
    B, S, cap, H = len(lens), max(lens) + 1, max(lens) + 3, heads * d
    q, k, v = (wl.normal(500 + d, t, (B, S, heads, d)) for t in (1, 2, 3))
    want = orc.attention_prefill(q, k, v, lens, causal=causal)
    kc, vc = (np.full((B, heads, cap, d), np.nan, np.float16) for _ in range(2))       # slots and rows past a sequence are never read
    qp = q.copy()
    for b, n in enumerate(lens):
        kc[b, :, :n] = k[b, :n].transpose(1, 0, 2)
        vc[b, :, :n] = v[b, :n].transpose(1, 0, 2)
        qp[b, n:] = np.nan
    ctx = torch.full((B, S, H), 7.0, dtype=torch.float16, device="cuda:0")
    op = eet.eet_op_attention_prefill if causal else eet.eet_op_attention_encoder
    op(dev(qp.reshape(B, S, H)), dev(kc), dev(vc), ctx, lens, heads)
    torch.cuda.synchronize()
    got = host(ctx).reshape(B, S, heads, d)
    for b, n in enumerate(lens):
        gate(got[b, :n], want[b, :n], f"sequence {b} of {n}", 6e-3, 6e-4)
        assert np.all(got[b, n:] == 7.0)
