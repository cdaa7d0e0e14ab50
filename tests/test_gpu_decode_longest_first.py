"""Decode attention of more pairs than CUs over 512 slots and more: its workgroups take the sequences longest first, up to as many as a wave counts (128).
Whatever the lengths and however many, every sequence is somebody's, with a scratch buffer and without, against a plain reference in float32."""
import math
import random

import pytest
import torch

pytestmark = pytest.mark.gpu


def lengths(kind, batch, capacity):
    r = random.Random(batch * capacity)
    if kind == "mixed":
        out = [r.randint(1, capacity) for _ in range(batch)]
        out[0], out[-1] = 1, capacity
        return out
    if kind == "equal":
        return [capacity // 2] * batch
    return [(capacity, 1, capacity // 2)[b % 3] for b in range(batch)]               # three lengths, many ties


@pytest.mark.parametrize("kind", ["mixed", "equal", "ties"])
@pytest.mark.parametrize("batch,heads,d,capacity", [(2, 129, 64, 512), (33, 8, 128, 513), (64, 5, 64, 1000), (65, 4, 128, 600), (128, 3, 64, 777),
                                                     (129, 2, 64, 512), (129, 5, 128, 600), (200, 8, 64, 1024), (300, 1, 128, 513), (300, 4, 64, 700)])
def test_every_sequence_is_served(kind, batch, heads, d, capacity):
    from paper_2104_12470_amd import eet
    g = torch.Generator(device="cuda:0")
    g.manual_seed(5)
    q = torch.randn((batch, heads * d), generator=g, device="cuda:0").half()
    k, v = (torch.randn((batch, heads, capacity, d), generator=g, device="cuda:0").half() for _ in range(2))
    lens = lengths(kind, batch, capacity)
    n = torch.tensor(lens, dtype=torch.int32, device="cuda:0")
    ctx = torch.full_like(q, float("nan"))
    scratch = torch.empty(max(1, eet.eet_op_attention_decode_scratch_bytes(batch, heads, d, capacity)), dtype=torch.uint8, device="cuda:0")
    eet.eet_op_attention_decode(q, k, v, ctx, n, scratch)
    alone = torch.full_like(q, float("nan"))
    eet.eet_op_attention_decode_static(q, k, v, alone, n)
    assert torch.equal(ctx.view(torch.int16), alone.view(torch.int16))
    seen = torch.arange(capacity, device="cuda:0")[None, None] < n[:, None, None]
    s = (k.float() * q.view(batch, heads, 1, d).float()).sum(-1) / math.sqrt(d)
    p = torch.softmax(s.masked_fill(~seen, -math.inf), -1)
    want = (p[..., None] * v.float()).sum(2).view(batch, heads * d)
    err = (ctx.float() - want).abs()
    # sums in float32 on both sides, one rounding to fp16 of values below 4: half an ulp of them, 2^-10
    assert float(err.max()) <= 1.1 * 2.0 ** -10, float(err.max())
