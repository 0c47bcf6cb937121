"""GPU: the scans' dense-boundary path (row tables of all waves) and their
register-held states, at the edges: runs of boundaries that start and end
anywhere in a 64-token chunk, capacities around the register limits (64, 256),
and a ragged last chunk, for the gated and the delta form.  Decisions, scores
and the final cache against the float64 oracle.  And the delta scan's token by
token path, which takes the chunks that hold a non-finite input."""
import numpy as np
import pytest

from oracle import oracle_forward
from tests import harness as H
from paper_2606_10650_amd.workloads import WORKLOADS, make_beta, make_inputs, store, to_f64

pytestmark = pytest.mark.gpu


def _oracle(w, x, beta, bo=None, mo=None):
    xf = H.f64(x, w)
    return oracle_forward(xf["k"], xf["v"], xf["g"], w.C, w.tau, q=xf["q"], lam=xf["lam"],
                          beta=None if beta is None else beta.astype(np.float64), b_override=bo,
                          m_override=mo)


def _run(w, x, beta, bo, mo):
    import torch
    from paper_2606_10650_amd import dla
    q, k, v, g, lam = H.inputs_to_device(w, x, w.B, w.H)
    dev = lambda a: torch.from_numpy(a).reshape(w.B, w.H, w.T).cuda()  # noqa: E731
    cache = dla.cache_alloc(w.B, w.H, w.C, w.dk, w.dv, device="cuda")
    kw = dict(tau=w.tau, boundary_override=dev(bo), merge_override=dev(mo))
    if beta is None:
        r = dla.prefill(cache, q, k, v, g, lam, **kw)
    else:
        r = dla.prefill_delta(cache, q, k, v, g, dev(beta), lam, **kw)
    out, b, m, s = (a.float().cpu().numpy() if a.is_floating_point() else a.cpu().numpy() for a in r)
    n = w.B * w.H
    return (out.reshape(n, w.T, w.dv), b.reshape(n, w.T), m.reshape(n, w.T), s.reshape(n, w.T),
            dla.cache_export(cache))


@pytest.mark.parametrize("C", [2, 3, 63, 64, 65, 128, 200, 256, 257])
@pytest.mark.parametrize("form,dtype,dk,dv", [
    ("gated", "bf16", 64, 64), ("gated", "f32", 64, 128),
    ("delta", "bf16", 128, 128), ("delta", "f32", 128, 64), ("delta", "bf16", 64, 128)])
def test_dense_runs(form, dtype, dk, dv, C):
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
    beta = make_beta(w) if form == "delta" else None
    ref = _oracle(w, x, beta, bo, mo)
    bo2, mo2, _, _ = H.near_tie_overrides(ref, bo, mo, f"dense runs {form} C={C} {dtype}",
                                          max_frac=0.02)
    out, b, m, s, exp = _run(w, x, beta, bo2, mo2)
    H.assert_decisions(b, m, ref)
    assert np.abs(s - ref["score"]).max() < 1e-5
    H.assert_outputs(out, ref["out"], H.TOL[dtype])
    H.assert_cache(exp, ref["cache"], H.STATE_TOL[False])


@pytest.mark.parametrize("C", [64, 65, 200])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_dense_runs_of_the_largest_states(dtype, C):
    """128 x 128 states, whose bookkeeping leaves the registers past 64 states."""
    test_dense_runs("gated", dtype, 128, 128, C)


@pytest.mark.parametrize("form", ["gated", "delta"])
def test_long_runs_of_boundaries(form):
    """Runs of dense chunks, which from the third on go by the row tables at once,
    between chunks with 7, 8 and 9 boundaries on either side of the tables' first
    use, and sparse ones."""
    T, C = 64 * 14 + 5, 33
    w = WORKLOADS["cfg2"].replace(B=1, H=2, T=T, C=C, dk=64, dv=64, mean_len=30.0, seed=77)
    x = make_inputs(w)
    bo = np.zeros((2, T), np.int8)
    mo = np.full((2, T), -1, np.int32)
    for chunk, step in enumerate((9, 8, 7, 1, 2, 1, 3, 64, 7, 8, 1, 1, 64, 1)):
        bo[:, 64 * chunk:64 * chunk + 64:step] = 1
    mo[:, ::5] = np.random.default_rng(1).integers(0, C - 1, size=mo[:, ::5].shape)
    beta = make_beta(w) if form == "delta" else None
    ref = _oracle(w, x, beta, bo, mo)
    bo2, mo2, _, _ = H.near_tie_overrides(ref, bo, mo, f"long runs {form}", max_frac=0.02)
    out, b, m, s, exp = _run(w, x, beta, bo2, mo2)
    H.assert_decisions(b, m, ref)
    assert np.abs(s - ref["score"]).max() < 1e-5
    H.assert_outputs(out, ref["out"], H.TOL["bf16"])
    H.assert_cache(exp, ref["cache"], H.STATE_TOL[False])


@pytest.mark.parametrize("dtype,dk,dv", [("bf16", 128, 128), ("f32", 64, 64), ("bf16", 128, 64)])
@pytest.mark.parametrize("where", ["k", "v", "beta"])
@pytest.mark.parametrize("t0", [0, 63, 64, 100, 210])
def test_delta_non_finite_input(dtype, dk, dv, where, t0):
    """A NaN at token t0 of head 0: no decision or score before it and no other
    head changes; from it on the scores are NaN and no state opens (NaN >= tau is
    false).  Outputs are compared up to t0's block of 32 tokens, whose values the
    readout multiplies by zero weights for the tokens before."""
    T, C = 230, 6
    w = WORKLOADS["cfg2"].replace(B=1, H=2, T=T, C=C, dk=dk, dv=dv, dtype=dtype, mean_len=20.0,
                                  seed=300 + t0)
    x = make_inputs(w)
    beta = make_beta(w)
    ref = _oracle(w, x, beta)
    bo, mo, _, _ = H.near_tie_overrides(ref, what=f"non-finite {where} {t0}")
    if where == "beta":
        beta[0, t0] = np.nan
    elif dtype == "f32":
        x[where][0, t0, 5] = np.nan
    else:
        x[where][0, t0, 5] = 0x7FC0
    out, b, m, s, exp = _run(w, x, beta, bo, mo)
    for h, n in ((0, t0), (1, T)):
        sub = {key: ref[key][h:h + 1, :n] for key in ("b", "merge")}
        H.assert_decisions(b[h:h + 1, :n], m[h:h + 1, :n], sub)
        assert n == 0 or np.abs(s[h, :n] - ref["score"][h, :n]).max() < 1e-5
        n -= 0 if h else t0 % 32
        if n:
            H.assert_outputs(out[h:h + 1, :n], ref["out"][h:h + 1, :n], H.TOL[dtype])
    # from t0 (beta, or an empty cache: from the next token) to the next forced
    # boundary, which starts a state without the NaN
    forced = np.flatnonzero(bo[0, t0 + 1:] == 1)
    later = slice(t0 + (where == "beta" or t0 == 0), t0 + 1 + forced[0] + 1 if len(forced) else T)
    free = bo[0, later] == -1
    assert np.isnan(s[0, later]).all() and (b[0, later][free] == 0).all()


@pytest.mark.parametrize("dtype,tau", [("bf16", 0.5), ("f32", 0.5), ("bf16", 1.2)])
def test_delta_keys_that_are_not_normalised(dtype, tau):
    """Keys of norm about 11: a delta step with beta |k|^2 > 2 expands, and only
    the boundaries (every token here, or most) keep the states bounded."""
    w = WORKLOADS["cfg1_iid"].replace(T=200, dk=128, dv=64, C=7, tau=tau, dtype=dtype, seed=9)
    x = make_inputs(w)
    scale = np.sqrt(128.0)
    x["k"] = store(to_f64(x["k"], dtype) * scale, dtype)
    beta = make_beta(w)
    ref = _oracle(w, x, beta)
    bo, mo, _, _ = H.near_tie_overrides(ref, what=f"unnormalised keys {dtype}", max_frac=0.02)
    out, b, m, s, exp = _run(w, x, beta, bo, mo)
    H.assert_decisions(b, m, ref)
    assert np.abs(s - ref["score"]).max() < 1e-5
    H.assert_outputs(out, ref["out"], H.TOL[dtype])
    H.assert_cache(exp, ref["cache"], H.STATE_TOL[False])
