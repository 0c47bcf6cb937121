"""GPU: the gated scan's dense-boundary path (row tables of all waves) and its
register-held states, at the edges: runs of boundaries that start and end
anywhere in a 64-token chunk, capacities around the register limits (64, 256),
and a ragged last chunk.  Decisions, scores and the final cache against the
float64 oracle."""
import numpy as np
import pytest

from tests import harness as H
from paper_2606_10650_amd.workloads import WORKLOADS, make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C", [2, 3, 63, 64, 65, 128, 200, 256, 257])
@pytest.mark.parametrize("dtype,dk,dv", [("bf16", 64, 64), ("f32", 64, 128)])
def test_dense_runs(C, dtype, dk, dv):
    from paper_2606_10650_amd import dla
    T = 64 * 9 + 37
    w = WORKLOADS["cfg2"].replace(B=1, H=2, T=T, C=C, dk=dk, dv=dv, dtype=dtype, mean_len=30.0,
                                  seed=100 + C)
    x = make_inputs(w)
    # forced runs: dense from the first token on, alone at a chunk's last token,
    # across a chunk edge, every second token, and to the end of the call
    bo = np.full((2, T), -1, np.int8)
    mo = np.full((2, T), -1, np.int32)
    rng = np.random.default_rng(C)
    for a, b, step in ((0, 70, 1), (127, 128, 1), (180, 200, 1), (256, 330, 2), (T - 50, T, 1)):
        bo[:, a:b:step] = 1
    bo[:, 400:440] = 0
    mo[:, ::3] = rng.integers(0, max(C - 1, 1), size=mo[:, ::3].shape)   # every third merge forced
    ref = H.run_oracle(w, x, b_override=bo, m_override=mo)
    bo2, mo2, _, _ = H.near_tie_overrides(ref, bo, mo, f"dense runs C={C} {dtype}", max_frac=0.02)
    q, k, v, g, lam = H.inputs_to_device(w, x, 1, 2)
    import torch
    dev = lambda a: torch.from_numpy(a).reshape(1, 2, T).cuda()  # noqa: E731
    cache = dla.cache_alloc(1, 2, C, dk, dv, device="cuda")
    out, b, m, s = dla.prefill(cache, q, k, v, g, lam, tau=w.tau, boundary_override=dev(bo2),
                               merge_override=dev(mo2))
    H.assert_decisions(b.cpu().numpy(), m.cpu().numpy(), ref)
    assert np.abs(s.cpu().numpy().reshape(2, T) - ref["score"]).max() < 1e-5
    H.assert_outputs(out.float().cpu().numpy(), ref["out"], H.TOL[dtype])
    H.assert_cache(dla.cache_export(cache), ref["cache"], H.STATE_TOL[False])
