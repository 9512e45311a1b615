"""The bf16 GEMMs of gemm_mid.hip (tiles of 128 x 128, 128 x 64 and 64 x 64,
k split over wavefronts and over work-groups) and the rows of a LayerNorm
backward block that goes with small token counts.

On the CPU: its hand-issued transposing LDS reads are waited for (the check of
test_lds_tr_reads.py on this source).  On the GPU: one layer against the
oracle at sizes whose products take every tile and split (2, 4 and 6 partials,
ragged last tiles in both directions, one k-tile, odd token counts, weight
gradients by 64 x 64 and 128 x 128 tiles), with the bf16 tolerance of the
gradients (relative L2 1e-2; the key-bias block of b_qkv, analytically zero,
left out), on a stage that has run a larger batch before (buffers sized for
another plan)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_2202_11836_amd.build as B
import synth
from _parity import make_stage, rel_l2, run_gpu, run_oracle
from test_lds_tr_reads import check_asm


def test_transposing_reads_are_waited_for(tmp_path):
    if shutil.which(B.HIPCC) is None and not os.path.exists(B.HIPCC):
        pytest.skip("hipcc not found")
    out = tmp_path / "gemm_mid.s"
    flags = [f for f in B.COMMON_FLAGS if f != "-fPIC"]
    r = subprocess.run([B.HIPCC] + flags + ["--cuda-device-only", "-S",
                                            os.path.join(B.CSRC, "gemm_mid.hip"), "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    problems, nreads = check_asm(out.read_text())
    assert nreads > 0
    assert not problems, "\n".join(problems[:20])


@pytest.mark.gpu
@pytest.mark.parametrize("hidden,ffn,batch,seq", [
    (64, 192, 1, 7), (128, 512, 1, 64), (320, 896, 3, 100), (768, 3072, 3, 77), (768, 1536, 11, 75),
    (512, 2048, 8, 128), (768, 3072, 7, 363), (1024, 4096, 2, 512), (2048, 8192, 3, 77)])
def test_one_layer(hidden, ffn, batch, seq):
    print(f"case mid gemm h {hidden} f {ffn} B {batch} S {seq}", flush=True)
    cfg = synth.StageConfig("mid", 1, hidden, hidden // 64, ffn, batch, seq, max(1, seq // 3), seq,
                            "bf16", 8)
    params = synth.make_params(cfg, perturb=True)
    st = make_stage(cfg, params)
    big = cfg.with_(batch=batch + 2, seq=seq + 9, len_hi=seq + 9)
    run_gpu(big, synth.make_inputs(big), params, stage=st)
    inp = synth.make_inputs(cfg, seed=9)
    got, ref = run_gpu(cfg, inp, params, stage=st), run_oracle(cfg, inp, params)
    pairs = {"y": (got["y"], ref["y"]), "dx": (got["dx"], ref["dx"])}
    for n in synth.PARAM_NAMES:
        a, b = got["grads"][0][n], ref["grads"][0][n]
        if n == "b_qkv":
            a, b = (np.concatenate([t[:hidden], t[2 * hidden:]]) for t in (a, b))
        pairs[n] = (a, b)
    bad = {n: rel_l2(a, b) for n, (a, b) in pairs.items() if not rel_l2(a, b) <= 1e-2}
    st.close()
    assert not bad, bad
