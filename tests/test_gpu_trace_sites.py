"""Trace sites (stage_trace_site): work that shares a launch is reported under
each of its sites, and a launch of several traced sites is recorded once."""
import pytest

pytestmark = pytest.mark.gpu

FORWARD = ["qkv_gemm_fwd", "out_gemm_fwd", "add_ln1_fwd", "ffn1_gelu_gemm_fwd", "ffn2_gemm_fwd",
           "add_ln2_fwd"]
BACKWARD = ["ln2_bwd", "ffn2_dgrad_dgelu_gemm", "ffn1_dgrad_resid_gemm", "ln1_bwd", "out_dgrad_gemm",
            "qkv_dgrad_resid_gemm"]
F32 = ["scores_gemm_fwd", "softmax_fwd", "context_gemm_fwd", "ln2_bwd_colreduce", "w2_wgrad_gemm",
       "b1_colsum", "b1_colreduce", "w1_wgrad_gemm", "ln1_bwd_colreduce", "wo_wgrad_gemm", "dp_gemm_bwd",
       "softmax_bwd", "dv_gemm_bwd", "dq_gemm_bwd", "dk_gemm_bwd", "bqkv_colsum", "bqkv_colreduce",
       "wqkv_wgrad_gemm"]
F32_SPLIT = ["w2_wgrad_splitk_reduce", "w1_wgrad_splitk_reduce", "wo_wgrad_splitk_reduce",
             "wqkv_wgrad_splitk_reduce"]
BF16 = ["key_extent", "attn_fwd", "attn_bwd_dq", "attn_bwd_dkdv", "wgrad_group_gemm",
        "wgrad_group_splitk_reduce"]


# fp32: score rows on chip, with and without splits of the weight gradients, and
# in memory; bf16: the copies and the attention halves in shared launches, and
# (16384 tokens) in launches of their own.
@pytest.mark.parametrize("dtype,hidden,batch,seq,sites", [
    ("f32", 128, 2, 40, F32), ("f32", 128, 8, 80, F32 + F32_SPLIT), ("f32", 64, 1, 520, F32 + F32_SPLIT),
    ("bf16", 128, 2, 40, BF16), ("bf16", 1024, 32, 512, BF16)])
def test_every_site_is_reported(dtype, hidden, batch, seq, sites):
    import torch
    from paper_2202_11836_amd import Stage, stage_site_count, stage_site_name
    print(f"case trace sites {dtype} h {hidden} B {batch} S {seq}", flush=True)
    st = Stage(1, hidden, hidden // 64, 4 * hidden, seed=1, dtype=dtype)
    x = torch.randn(batch, seq, hidden, device="cuda").to(st.torch_dtype)

    def launches(names):
        st.trace(names)
        st.forward(x)
        st.backward(x)
        n, ms = st.trace_read()
        assert n == 0 or ms > 0.0
        return n

    counts = {n: launches(n) for n in FORWARD + BACKWARD + sites}
    assert all(counts.values()), [n for n, c in counts.items() if not c]
    shared = ["w2_wgrad_gemm", "w1_wgrad_gemm"] if dtype == "f32" else ["attn_bwd_dq", "attn_bwd"]
    assert launches(shared) == 1
    every = launches([stage_site_name(i) for i in range(stage_site_count())])
    assert len(FORWARD + BACKWARD) < every <= sum(launches(stage_site_name(i))
                                                  for i in range(stage_site_count()))
    st.close()
