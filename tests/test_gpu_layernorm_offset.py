"""The LayerNorm inside the one-launch prompts (csrc/prompt_step.hip) and steps (csrc/decode_step.hip) on rows whose mean is 1250 and some 10000 of their
deviations.  The K part of w_qkv is the identity, so the layer's K cache holds the normalised rows themselves, rounded once."""
import numpy as np
import pytest
import torch

from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, host, kernels_of

pytestmark = pytest.mark.gpu


def rows_far_from_zero(rows, hidden, seed):
    """5000, and 4 more or less in half of the columns each (even rows) or in one of 64 in turn (odd rows): exact in fp16, their mean exactly 5000 (no power
    of two: products with the mean are rounded)."""
    x = np.full((rows, hidden), 5000.0, np.float32)
    for r in range(rows):
        at = np.random.default_rng(seed + r).permutation(hidden)
        n = hidden // 2 if r % 2 == 0 else hidden // 128 + 1
        x[r, at[:n]] += 4
        x[r, at[n:2 * n]] -= 4
    return x.astype(np.float16)


@pytest.mark.parametrize("hidden,heads,ffn,rows,step", [
    (256, 4, 1024, 40, False), (576, 9, 1344, 20, False), (768, 6, 3072, 33, False), (1024, 16, 4096, 48, False),
    (64, 1, 64, 1, True), (768, 12, 3072, 2, True), (1024, 8, 4096, 4, True), (576, 9, 1344, 7, True), (832, 13, 2048, 16, True), (256, 2, 1024, 40, True),
    (1152, 18, 4608, 1, True), (1984, 31, 7936, 3, True), (2048, 16, 8192, 8, True)])
def test_rows_far_from_zero(hidden, heads, ffn, rows, step):
    from paper_2104_12470_amd import eet
    B, S = (rows, 1) if step else (1, rows)
    w = wl.Workload(f"offset{hidden}x{rows}", 61, hidden, heads, ffn, 1, B, S, 1, S, 2, S + 4)
    W = wl.layer_weights(w, 0, random_affine=True)
    W["w_qkv"][hidden:2 * hidden], W["b_qkv"][hidden:2 * hidden] = np.eye(hidden, dtype=np.float16), 0
    layer = eet.DecoderLayer(eet.make_config(hidden, heads, ffn, B, S, S + 4, w.ln_eps), {k: torch.from_numpy(v) for k, v in W.items()})
    x = rows_far_from_zero(rows, hidden, hidden)
    if step:
        layer.prefill(dev(wl.prompt_embeddings(w)), [1] * B)
        call = lambda: layer.decode_step(dev(x))                       # noqa: E731
    else:
        call = lambda: layer.prefill(dev(x)[None], [rows])             # noqa: E731
    assert any(("decode_layers" if step else "prompt_layers") in n for n in kernels_of(call))
    k = host(layer.cache_views()[0]).astype(np.float64)                # [batch, heads, slots, d]
    got = k[:, :, 1].reshape(rows, hidden) if step else k[0, :, :rows].transpose(1, 0, 2).reshape(rows, hidden)
    x64, g, b = x.astype(np.float64), W["ln1_g"].astype(np.float64), W["ln1_b"].astype(np.float64)
    t = (x64 - x64.mean(1, keepdims=True)) / np.sqrt(x64.var(1, keepdims=True) + w.ln_eps) * g
    # rounded to fp16 once (2^-11, or 2^-25 of the smallest); the mean and the differences are exact, the deviation and the products a few 2^-24 off
    bound = 2.0 ** -11 * np.abs(t + b) + 2.0 ** -25 + 2.0 ** -20 * (np.abs(t) + np.abs(b))
    assert np.all(np.abs(got - (t + b)) <= bound), np.max(np.abs(got - (t + b)) / bound)
    layer.close()
