"""fp32 stages at the sizes where their contraction kernels change path:
one token; a sequence length that is not a multiple of 4 (score rows that
are not 16-byte aligned, 4-byte loads); tile and k-tile remainders; outputs
with at least 256 tiles of 64 x 64 (the larger work-group) including the
unaligned score matrix; weight gradients split over tokens; more than 4096
tokens (db_1 from a pass of its own).  Every output against the float64
oracle: relative L2 <= 1e-5, i.e. fp32 rounding (6e-8) times the square root
of the longest sum (about 6000 terms) times two, for the two contractions a
value goes through."""
import pytest

import synth
from _parity import rel_l2, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,ffn,batch,seq,lo", [
    (64, 64, 1, 1, 1), (128, 320, 3, 37, 1), (192, 256, 2, 65, 20), (64, 192, 5, 132, 60),
    (320, 1280, 8, 140, 30), (768, 128, 9, 131, 100), (64, 128, 41, 104, 50)])
def test_f32_stage(hidden, ffn, batch, seq, lo):
    print(f"case f32 h {hidden} f {ffn} B {batch} S {seq}", flush=True)
    cfg = synth.StageConfig("f32", 1, hidden, hidden // 64, ffn, batch, seq, lo, seq, "f32", 6)
    inp, params = synth.make_inputs(cfg), synth.make_params(cfg, perturb=True)
    got, ref = run_gpu(cfg, inp, params), run_oracle(cfg, inp, params)
    pairs = {"y": (got["y"], ref["y"]), "dx": (got["dx"], ref["dx"])}
    for n in synth.PARAM_NAMES:
        # one token has one key: no query or key gradient
        if not (seq == 1 and n in ("W_qkv", "b_qkv")):
            pairs[n] = (got["grads"][0][n], ref["grads"][0][n])
    bad = {n: rel_l2(a, b) for n, (a, b) in pairs.items() if not rel_l2(a, b) <= 1e-5}
    assert not bad, bad
