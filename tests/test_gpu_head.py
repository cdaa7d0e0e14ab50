"""Final LayerNorm, output projection and greedy choice in one launch (up to 16 rows of up to 1792): against float64 over the hidden states that the
model leaves, at every number of row blocks, K in one and two pieces, tables that fill the chip and that do not."""
import numpy as np
import pytest
import torch

from paper_2104_12470_amd import workloads as wl
from tests.gpu_util import dev, host, kernels_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,rows,vocab", [(64, 1, 5), (192, 3, 1000), (704, 16, 777), (960, 2, 33000), (1024, 1, 50257), (1024, 9, 2049),
                                               (1152, 5, 4000), (1536, 16, 20011), (1792, 4, 129)])
def test_logits_and_choice(hidden, rows, vocab):
    from paper_2104_12470_amd import eet
    S, cap = 3, 8
    w = wl.Workload(f"head{hidden}x{rows}", 73, hidden, hidden // 64, 896, 1, rows, S, 1, S, 2, cap)
    head = wl.model_head(w, vocab, cap)
    head["lnf_g"] = (1 + 0.1 * wl.normal(73, 11, (hidden,))).astype(np.float16)
    head["lnf_b"] = (0.1 * wl.normal(73, 12, (hidden,))).astype(np.float16)
    tie = vocab // 2                                              # equal columns: the first of them is chosen
    head["wte"][tie:] = head["wte"][:vocab - tie][:len(head["wte"][tie:])]
    cfg = eet.make_config(hidden, hidden // 64, 896, rows, S, cap, w.ln_eps)
    W = {k: torch.from_numpy(v) for k, v in wl.layer_weights(w, 0, random_affine=True).items()}
    model = eet.DecoderModel(cfg, [W], {k: torch.from_numpy(v) for k, v in head.items()}, vocab)
    ids = dev(wl.uniform_int(73, 13, rows * S, 0, vocab - 1).reshape(rows, S).astype(np.int32))
    lens = [1 + b % S for b in range(rows)]
    wte = head["wte"][:vocab].astype(np.float64)

    def check(logits, chosen, x):
        x = host(x).astype(np.float64)
        x = (x - x.mean(1, keepdims=True)) / np.sqrt(x.var(1, keepdims=True) + w.ln_eps) * head["lnf_g"].astype(np.float64) + head["lnf_b"].astype(np.float64)
        want, got = x @ wte.T, host(logits).astype(np.float64)
        assert np.all(np.isfinite(got))
        # each normalised value and the result are rounded to fp16 once, 2^-11 of it; float32 sums are far below that
        bound = 2.0 ** -11 * (np.abs(want) + np.sqrt((x ** 2) @ (wte.T ** 2)) * 4) + 1e-4
        assert np.all(np.abs(got[:, :vocab] - want) <= bound), np.max(np.abs(got[:, :vocab] - want) / bound)
        assert np.all(got[:, vocab:] == 0)
        assert host(chosen).tolist() == np.argmax(host(logits)[:, :vocab], axis=1).tolist()

    logits, chosen = model.prefill(ids, lens)
    torch.cuda.synchronize()
    xn = model.hidden_states(False)[1]
    check(logits, chosen, torch.stack([xn[b, lens[b] - 1] for b in range(rows)]))
    for _ in range(3):                                            # the counter of the launch is zero again every time
        logits, chosen = model.decode_step(chosen)
        torch.cuda.synchronize()
        check(logits, chosen, model.hidden_states(True)[1])
    assert any("head_rows" in k for k in kernels_of(lambda: model.decode_step(chosen)))
    model.close()
