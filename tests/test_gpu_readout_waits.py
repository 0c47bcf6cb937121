"""GPU: the readout's loads into LDS are waited for before other waves use the
bytes.  Without lambda no other load stands between the first requests and the
barrier that publishes them, so a call without lambda must equal, bit for bit,
the same call with lambda = 1, and itself when run again."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,H,T,C", [
    ("bf16", 8, 16, 2100, 24),   # ragged last chunk, pipelined
    ("bf16", 2, 5, 515, 3),      # a last chunk of 3 tokens, few states
    ("bf16", 32, 16, 1024, 9),
    ("f32", 4, 16, 1031, 16),
])
def test_no_lambda_equals_unit_lambda(dtype, B, H, T, C):
    import torch
    from paper_2606_10650_amd import dla
    from paper_2606_10650_amd.workloads import WORKLOADS, make_prefix_torch
    w = WORKLOADS["cfg2"].replace(B=B, H=H, T=T, C=C, dtype=dtype, mean_len=20.0, seed=11)
    q, k, v, g = make_prefix_torch(w, "cuda", with_q=True)
    ones = torch.ones((B, H, T, C), dtype=k.dtype, device="cuda")

    def run(lam):
        cache = dla.cache_alloc(B, H, C, w.dk, w.dv, device="cuda")
        return dla.prefill(cache, q, k, v, g, lam, tau=w.tau)[0]

    want = run(ones)
    for _ in range(3):
        assert torch.equal(run(None), want)
