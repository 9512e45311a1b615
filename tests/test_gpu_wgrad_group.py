"""The stream-K group of bf16 weight gradients (taken above 8192 tokens) where it
is ragged: a token count that is not a multiple of its k-tiles of 64, partly
filled 256 x 256 tiles in both directions (320, 896, 960 rows), four gradients
and the two of either half layer, a partial buffer that has to grow for a smaller
batch, and partials in the no-alloc backward's scratch (fp32 splits too).  Every
test asserts that partials are in use, so that another choice of the dispatch
cannot leave it testing something else."""
import numpy as np
import pytest

import synth
from _parity import IDX, make_stage, rel_l2, run_gpu, run_oracle, to_torch
from test_gpu_units import ATTN_PARAMS, chain_grads, make_unit_stage, run_chain

pytestmark = pytest.mark.gpu

H, F, BATCH, SEQ = 320, 896, 41, 200  # 8200 tokens
REDUCED = ["wgrad_group_gemm", "wgrad_group_splitk_reduce"]


def _cfg(batch=BATCH, seq=SEQ):
    return synth.StageConfig("group", 1, H, H // 64, F, batch, seq, seq // 2, seq, "bf16", 12)


def _inputs(cfg, seed=3):
    import torch
    inp = synth.make_inputs(cfg, seed=seed)
    mask = torch.from_numpy(np.ascontiguousarray(inp["mask"], dtype=np.uint8)).cuda()
    return inp, to_torch(inp["x"], cfg.dtype), mask, to_torch(inp["dy"], cfg.dtype)


def _bad(grads, ref, names):
    """Relative L2 of the bf16 gradient tolerance (1e-2); the key block of b_qkv is
    analytically zero."""
    errs = {}
    for n in names:
        a, b = grads[n], ref[n]
        if n == "b_qkv":
            a, b = (np.concatenate([t[:H], t[2 * H:]]) for t in (a, b))
        errs[n] = rel_l2(a, b)
    return {n: e for n, e in errs.items() if not e <= 1e-2}


def test_ragged_layer_and_its_halves():
    print(f"case stream-K group h {H} f {F} T {BATCH * SEQ}", flush=True)
    cfg = _cfg()
    inp, x, mask, dy = _inputs(cfg)
    params = synth.make_params(cfg, perturb=True)
    ref = run_oracle(cfg, inp, params)["grads"][0]
    whole = make_stage(cfg, params)
    halves = [make_unit_stage(cfg, params, u, 1) for u in (0, 1)]
    for st in [whole] + halves:
        st.trace(REDUCED)
    whole.forward(x, mask)
    whole.backward(dy)
    run_chain(halves, x, mask, dy)
    for st in [whole] + halves:
        assert st.trace_read()[0] == 2  # a group with partials, and their reduction
    got = {n: whole.grad(0, IDX[n]).double().cpu().numpy() for n in synth.PARAM_NAMES}
    assert not _bad(got, ref, synth.PARAM_NAMES)
    g = chain_grads(halves, [(0, 1), (1, 1)], 1)[0]
    got = {n: t.double().cpu().numpy() for n, t in g.items()}
    assert set(got) == set(synth.PARAM_NAMES) and ATTN_PARAMS < set(got)
    assert not _bad(got, ref, synth.PARAM_NAMES)
    for st in [whole] + halves:
        st.close()


def test_smaller_batch_needs_more_partials():
    """16384 tokens (39.3 MB of partials), then 8200 (47.2 MB) in fewer sequences."""
    import torch
    print("case stream-K partials grow for a smaller batch", flush=True)
    big, cfg = _cfg(32, 512), _cfg(20, 410)
    params = synth.make_params(cfg, perturb=True)
    st, fresh = make_stage(cfg, params), make_stage(cfg, params)
    run_gpu(big, synth.make_inputs(big), params, stage=st)
    held = st.device_bytes()
    _, x, mask, dy = _inputs(cfg)
    st.trace(REDUCED)
    y, dx = st.forward(x, mask), st.backward(dy)
    assert st.trace_read()[0] == 2
    assert st.device_bytes() > held
    assert torch.equal(y, fresh.forward(x, mask)) and torch.equal(dx, fresh.backward(dy))
    for i in range(12):
        assert torch.equal(st.grad(0, i), fresh.grad(0, i)), i
    # and back: nothing is allocated again
    held = st.device_bytes()
    run_gpu(big, synth.make_inputs(big), params, stage=st)
    assert st.device_bytes() == held
    for s in (st, fresh):
        s.close()


@pytest.mark.parametrize("dtype,hidden,ffn,batch,seq", [
    ("bf16", H, F, BATCH, SEQ), ("f32", 128, 320, 8, 81), ("f32", 64, 64, 41, 104)])
def test_noalloc_with_partials(dtype, hidden, ffn, batch, seq):
    """Partials of the weight gradients in the static scratch: bitwise the
    backward's results."""
    import torch
    print(f"case no-alloc with partials {dtype} h {hidden} f {ffn} T {batch * seq}", flush=True)
    cfg = synth.StageConfig("noalloc", 2, hidden, hidden // 64, ffn, batch, seq, seq // 2, seq, dtype, 5)
    params = synth.make_params(cfg, perturb=True)
    _, x, mask, dy = _inputs(cfg)
    ref, na = make_stage(cfg, params), make_stage(cfg, params)
    ref.trace(["w2_wgrad_splitk_reduce"] if dtype == "f32" else REDUCED)
    ref.forward(x, mask)
    dx = ref.backward(dy)
    assert ref.trace_read()[0] == (2 if dtype == "f32" else 4)  # in both layers
    na.forward(x, mask)
    assert torch.equal(dx, na.backward_noalloc(dy, torch.empty_like(dy)))
    for l in range(2):
        for i in range(12):
            assert torch.equal(ref.grad(l, i), na.grad(l, i)), (l, i)
    for s in (ref, na):
        s.close()
