"""Work that shares a launch with a GEMM or an attention product, at the sizes
where its kernels change path.

fp32 attention with its score rows on chip: one key, edges of the 32-row and
32-key blocks and of the four score-row lengths (64, 128, 256, 512), and the
first lengths that keep the score matrix in memory (513: rows that are not
16-byte aligned, 516: rows that are).  Tolerance as in test_gpu_f32.py: relative
L2 1e-5 against the float64 oracle.

The start of a bf16 forward pass beside its first GEMM: the same outputs, bit
for bit, from an input that is not 16-byte aligned (copied by the runtime
first), for whole layers and a feed-forward half, with masks of more than one
512-byte step, odd token counts, and with no mask against a mask of ones.

The rest of the backward (column sums, dx) beside weight gradients of every tile
is held to the oracle by test_gpu_mid_gemm.py; here a feed-forward half, whose dx
comes from the other half of the code, against the same half in a whole layer."""
import numpy as np
import pytest

import synth
from _parity import IDX, rel_l2, run_gpu, run_oracle, to_torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,batch,seq", [
    (64, 3, 1), (128, 2, 31), (64, 3, 33), (192, 2, 64), (64, 2, 65), (128, 1, 128), (64, 3, 129),
    (64, 2, 256), (64, 1, 257), (64, 1, 512), (64, 2, 513), (64, 1, 516)])
def test_f32_attention(hidden, batch, seq):
    print(f"case f32 attention h {hidden} B {batch} S {seq}", flush=True)
    cfg = synth.StageConfig("attn", 1, hidden, hidden // 64, 128, batch, seq, max(1, seq // 3), seq,
                            "f32", 11)
    inp, params = synth.make_inputs(cfg), synth.make_params(cfg, perturb=True)
    got, ref = run_gpu(cfg, inp, params), run_oracle(cfg, inp, params)
    pairs = {"y": (got["y"], ref["y"]), "dx": (got["dx"], ref["dx"])}
    for n in synth.PARAM_NAMES:
        if not (seq == 1 and n in ("W_qkv", "b_qkv")):  # one key: no query or key gradient
            pairs[n] = (got["grads"][0][n], ref["grads"][0][n])
    got["stage"].close()
    bad = {n: rel_l2(a, b) for n, (a, b) in pairs.items() if not rel_l2(a, b) <= 1e-5}
    assert not bad, bad


@pytest.mark.parametrize("hidden,ffn,batch,seq,first_unit", [
    (64, 128, 1, 1, 0), (128, 320, 3, 77, 0), (192, 768, 2, 600, 0), (768, 3072, 2, 128, 0),
    (64, 192, 1, 5, 1), (320, 1280, 3, 131, 1), (1024, 4096, 2, 512, 1)])
def test_start_of_forward(hidden, ffn, batch, seq, first_unit):
    import torch
    from paper_2202_11836_amd import Stage
    print(f"case start h {hidden} f {ffn} B {batch} S {seq} unit {first_unit}", flush=True)
    cfg = synth.StageConfig("start", 1, hidden, hidden // 64, ffn, batch, seq, max(1, seq // 2), seq,
                            "bf16", 3)
    st = Stage(None, hidden, hidden // 64, ffn, seed=5, dtype="bf16", first_unit=first_unit,
               n_units=2 - first_unit)
    inp = synth.make_inputs(cfg)
    x, dy = to_torch(inp["x"], "bf16"), to_torch(inp["dy"], "bf16")
    mask = torch.from_numpy(np.ascontiguousarray(inp["mask"], dtype=np.uint8)).cuda()
    room = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")
    odd = room[1:].view_as(x)
    odd.copy_(x)
    names = [n for n in synth.PARAM_NAMES if not first_unit or IDX[n] >= IDX["W_1"]]

    def run(x, mask):
        y = st.forward(x, mask)
        dx = st.backward(dy)
        torch.cuda.synchronize()
        return [y.clone(), dx.clone()] + [st.grad(0, IDX[n]).clone() for n in names]

    masked = run(x, mask)
    for a, b in zip(masked, run(odd, mask)):
        assert torch.equal(a, b)
    for a, b in zip(run(x, None), run(x, torch.ones_like(mask))):
        assert torch.equal(a, b)
    st.close()


@pytest.mark.parametrize("hidden,ffn,batch,seq", [(64, 192, 1, 7), (320, 896, 3, 100), (768, 3072, 3, 77)])
def test_ffn_half_dx(hidden, ffn, batch, seq):
    import torch
    from paper_2202_11836_amd import Stage
    print(f"case ffn half dx h {hidden} f {ffn} B {batch} S {seq}", flush=True)
    cfg = synth.StageConfig("half", 1, hidden, hidden // 64, ffn, batch, seq, seq, seq, "bf16", 4)
    whole = Stage(1, hidden, hidden // 64, ffn, seed=5, dtype="bf16")
    attn = Stage(None, hidden, hidden // 64, ffn, seed=5, dtype="bf16", first_unit=0, n_units=1)
    half = Stage(None, hidden, hidden // 64, ffn, seed=5, dtype="bf16", first_unit=1, n_units=1)
    inp = synth.make_inputs(cfg)
    x, dy = to_torch(inp["x"], "bf16"), to_torch(inp["dy"], "bf16")
    whole.forward(x)
    dx = whole.backward(dy)
    half.forward(attn.forward(x))
    dx2 = attn.backward(half.backward(dy))
    torch.cuda.synchronize()
    # H1 and its gradient pass between the halves in bf16: two roundings of
    # 2^-9 each relative to the values that the whole layer keeps.
    assert rel_l2(dx2.double().cpu().numpy(), dx.double().cpu().numpy()) <= 1e-2
    for s in (whole, attn, half):
        s.close()


@pytest.mark.parametrize("pinned", [False, True])
@pytest.mark.parametrize("dtype,hidden,batch,seq", [("bf16", 128, 3, 77), ("bf16", 1024, 32, 384),
                                                    ("f32", 128, 2, 40)])
def test_forward_from_host_memory(dtype, hidden, batch, seq, pinned):
    """x and the key mask in host memory: copied by the runtime, not read by the
    kernels (a first GEMM that reads x itself, one that does not, fp32)."""
    import torch
    from paper_2202_11836_amd import Stage, stage_forward
    print(f"case host input {dtype} h {hidden} B {batch} S {seq} pinned {pinned}", flush=True)
    cfg = synth.StageConfig("host", 1, hidden, hidden // 64, 256, batch, seq, max(1, seq // 2), seq,
                            dtype, 3)
    inp = synth.make_inputs(cfg)
    x = to_torch(inp["x"], dtype, "cpu")
    mask = torch.from_numpy(np.ascontiguousarray(inp["mask"], dtype=np.uint8))
    dy = to_torch(inp["dy"], dtype)
    if pinned:
        x, mask = (torch.empty_like(t, pin_memory=True).copy_(t) for t in (x, mask))
    st = Stage(1, hidden, hidden // 64, 256, seed=5, dtype=dtype)

    def run(x, mask):
        y = torch.empty(batch, seq, hidden, dtype=dy.dtype, device="cuda")
        st._sync_stream()
        stage_forward(st.handle, x, mask, batch, seq, y)
        dx = st.backward(dy)
        torch.cuda.synchronize()
        return [y, dx.clone()] + [st.grad(0, i) for i in range(12)]

    ref = run(x.cuda(), mask.cuda())
    for a in (run(x.cuda(), mask), run(x, mask.cuda()), run(x, mask)):
        for t, r in zip(a, ref):
            assert torch.equal(t, r)
    st.close()


@pytest.mark.parametrize("dtype,hidden,batch,seq", [("bf16", 128, 3, 77), ("f32", 128, 2, 40)])
def test_step_in_a_captured_graph(dtype, hidden, batch, seq):
    """A forward and a backward_noalloc recorded in a graph: every replay, on new
    inputs and with eager passes between them, gives the eager result."""
    import torch
    from paper_2202_11836_amd import Stage
    print(f"case graph {dtype} h {hidden} B {batch} S {seq}", flush=True)
    cfg = synth.StageConfig("graph", 2, hidden, hidden // 64, 256, batch, seq, max(1, seq // 2), seq,
                            dtype, 3)
    st = Stage(2, hidden, hidden // 64, 256, seed=5, dtype=dtype)
    inps = [synth.make_inputs(cfg, seed=s) for s in (1, 2, 3)]
    x, dy = to_torch(inps[0]["x"], dtype), to_torch(inps[0]["dy"], dtype)
    mask = torch.from_numpy(np.ascontiguousarray(inps[0]["mask"], dtype=np.uint8)).cuda()
    y, dx = torch.empty_like(x), torch.empty_like(x)

    def step():
        st.forward(x, mask, out=y)
        st.backward_noalloc(dy, dx)

    def results():
        torch.cuda.synchronize()
        return [y.clone(), dx.clone()] + [st.grad(l, i) for l in range(2) for i in range(12)]

    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for inp in inps:
        x.copy_(to_torch(inp["x"], dtype))
        dy.copy_(to_torch(inp["dy"], dtype))
        mask.copy_(torch.from_numpy(np.ascontiguousarray(inp["mask"], dtype=np.uint8)))
        step()
        eager = results()
        y.zero_(), dx.zero_()
        graph.replay()
        for a, b in zip(results(), eager):
            assert torch.equal(a, b)
    st.close()
