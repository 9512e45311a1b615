"""fp32 attention with scores that are not finite: a row whose exponentials do
not sum to a positive number (all scores -inf, any of them +inf or NaN) has
probabilities of zero, and a single key at -inf is left out, for score rows on
chip (up to 512 tokens) and in memory alike."""
import numpy as np
import pytest

import synth
from _parity import IDX, to_torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seq", [5, 40, 130, 513])
@pytest.mark.parametrize("kind", ["all -inf", "all +inf", "all nan", "one -inf", "one +inf"])
def test_scores_not_finite(kind, seq):
    import torch
    from paper_2202_11836_amd import Stage
    print(f"case fp32 scores {kind} S {seq}", flush=True)
    h, batch = 64, 2
    cfg = synth.StageConfig("inf", 1, h, 1, 128, batch, seq, seq, seq, "f32", 3)
    st = Stage(1, h, 1, 128, seed=2, dtype="f32")
    x = to_torch(synth.make_inputs(cfg)["x"], "f32", "cpu")
    g = torch.Generator().manual_seed(4)
    # score of key t: (b_q[0] * k_t + a finite part) / 8, k_t = b_k[0] or 100 x_t[0]
    w, b = torch.randn(3 * h, h, generator=g) * 0.1, torch.zeros(3 * h)
    w[[0, h]] = 0.0
    value = float(kind.split()[1])
    if kind.startswith("all"):
        b[0], b[h] = 1.0, value
    else:
        b[0] = np.sign(value)
        w[h, 0] = 100.0
        w[1:h, 0] = w[h + 1:, 0] = 0.0
        x[:, seq // 2, 0] = 1e37  # times 100: past the largest fp32
    st.set_param(0, IDX["W_qkv"], w)
    st.set_param(0, IDX["b_qkv"], b)
    st.forward(x.cuda())
    ctx = st.saved(0, 2, batch * seq).cpu().reshape(batch, seq, h)
    st.close()
    q, k, v = (x @ w.T + b).chunk(3, -1)
    s = (q.double() @ k.double().transpose(1, 2)) / 8.0
    e = torch.exp(s - s.amax(-1, keepdim=True))
    total = e.sum(-1, keepdim=True)
    p = torch.where(total > 0, e / total, torch.zeros_like(e))
    ref = p @ v.double()
    if kind != "one -inf":
        assert float(ref.abs().max()) == 0.0 and float(ctx.abs().max()) == 0.0
    else:
        # two contractions in fp32 (as in test_gpu_f32.py) and scores of up to
        # about 40 in the exponent, 40 x 6e-8 each
        assert float((ctx - ref).norm() / ref.norm()) <= 1e-5
