"""Prefill attention of more than 512 tokens with heads of 128 (attn_prefill_wide): on either side of the rule that gives a launch of few tiles to the
form whose two groups of waves take half of every key tile each, with lengths around the 32-key halves, the 64-key tiles and the 128- and 256-row
query tiles; a prompt of one key, which the upper group never sees."""
import numpy as np
import pytest
import torch

from oracle import eet_oracle as orc
from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, gate, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("heads,lens", [
    (1, [513]),
    (2, [1, 31, 32, 33, 64, 96, 97, 544, 545, 576, 577, 639, 640, 641]),      # few tiles: halves
    (1, [1023, 1025]),
    (1, [2049]),
    (52, [513]),                                                             # 260 tiles of 128 rows: whole keys
    (44, [1024]),                                                            # 352: halves with a sequence mask, whole without
    (44, [1025]),                                                            # 396: whole
])
def test_against_the_oracle(heads, lens, causal):
    from paper_2104_12470_amd import eet
    d, B, S, cap = 128, len(lens), max(lens) + 1, max(lens) + 3
    H = heads * d
    q, k, v = (wl.normal(700, t, (B, S, heads, d)) for t in (1, 2, 3))
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


def test_a_group_whose_first_keys_score_minus_infinity():
    """Keys 32 to 63 of -inf, all that the upper group sees in its first tile, have weight zero and leave the others' as they are."""
    from paper_2104_12470_amd import eet
    d, n = 128, 600
    q, k, v = (wl.normal(701, t, (1, n, 1, d)) for t in (1, 2, 3))
    q = np.abs(q) + np.float16(0.01)
    k[:, 32:64] = -np.inf
    want = orc.attention_prefill(q, k, v, [n], causal=True)
    assert np.isfinite(want[0, :32]).all() and np.isfinite(want[0, 64:]).all()
    ctx = torch.zeros((1, n, d), dtype=torch.float16, device="cuda:0")
    eet.eet_op_attention_prefill(dev(q.reshape(1, n, d)), dev(k.transpose(0, 2, 1, 3).copy()), dev(v.transpose(0, 2, 1, 3).copy()), ctx, [n], 1)
    torch.cuda.synchronize()
    gate(host(ctx).reshape(n, 1, d), want[0], "with keys of -inf", 6e-3, 6e-4)
