"""GPU: the delta form's prefill over the inputs that its 64-token chunks must
not lose precision on, against the float64 oracle."""
import numpy as np
import pytest

from oracle import oracle_forward
from tests import harness as H
from paper_2606_10650_amd.workloads import WORKLOADS, make_beta, make_inputs, store, to_f64

pytestmark = pytest.mark.gpu


def _check(w, x, beta, bo=None, mo=None, what="", max_frac=None):
    """Decisions bit for bit (near ties pinned), scores to 1e-5 (relative above
    1), outputs and states to the parity tolerances.  (The readout forms its
    in-chunk decays from float32 offsets, a relative error of up to 2^-23 times
    a chunk's summed gates in an output.)"""
    import torch
    from paper_2606_10650_amd import dla
    xf = H.f64(x, w)
    ref = oracle_forward(xf["k"], xf["v"], xf["g"], w.C, w.tau, q=xf["q"], lam=xf["lam"],
                         beta=beta.astype(np.float64), b_override=bo, m_override=mo)
    bo, mo, _, _ = H.near_tie_overrides(ref, bo, mo, what=what, max_frac=max_frac)
    n = w.B * w.H
    q, k, v, g, lam = H.inputs_to_device(w, x, w.B, w.H)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).reshape(w.B, w.H, w.T).cuda()  # noqa: E731
    cache = dla.cache_alloc(w.B, w.H, w.C, w.dk, w.dv, device="cuda")
    out, b, m, s = (a.cpu() for a in dla.prefill_delta(
        cache, q, k, v, g, dev(beta), lam, tau=w.tau, boundary_override=dev(bo),
        merge_override=dev(mo)))
    s = s.numpy().reshape(n, w.T)
    err = np.abs(s - ref["score"]) / np.maximum(ref["score"], 1.0)
    print(f"[scores] {what}: largest error {np.nanmax(err):.2e}, {int(np.isnan(s).sum())} NaN", flush=True)
    assert err.max() < 1e-5
    H.assert_decisions(b.numpy(), m.numpy(), ref, what)
    H.assert_outputs(out.float().numpy().reshape(n, w.T, w.dv), ref["out"],
                     H.TOL[w.dtype] + 2.0 ** -23 * np.abs(x["g"]).sum(1).max(), what)
    H.assert_cache(dla.cache_export(cache), ref["cache"], H.STATE_TOL[False], what=what)


@pytest.mark.parametrize("dtype,dk,dv", [("bf16", 128, 128), ("f32", 128, 64), ("f32", 64, 128)])
@pytest.mark.parametrize("gate", [-50.0, -1e3, -1e6])
@pytest.mark.parametrize("expanding", [False, True])
def test_steep_gates(dtype, dk, dv, gate, expanding):
    """Reset gates between ordinary ones, at a chunk's first and last token and
    inside; with one token of beta |k|^2 > 2 beside one of them, which takes its
    chunk token by token."""
    T, C = 300, 12
    w = WORKLOADS["cfg2"].replace(B=1, H=2, T=T, C=C, dk=dk, dv=dv, dtype=dtype, mean_len=25.0,
                                  seed=int(-gate) % 1000 + dk)
    x = make_inputs(w)
    x["g"][:, [5, 63, 64, 140, 170, 191, 230]] = gate
    if expanding:
        x["k"][:, 150] = store(to_f64(x["k"][:, 150], dtype) * 1.6, dtype)
    beta = make_beta(w)
    if expanding:
        beta[:, 150] = 1.0
    _check(w, x, beta, what=f"gate {gate} {dtype} {expanding}", max_frac=0.02)
