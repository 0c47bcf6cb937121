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


@pytest.mark.parametrize("dtype,dk,dv", [("f32", 128, 128), ("f32", 64, 64), ("bf16", 128, 64)])
@pytest.mark.parametrize("lo,hi", [(0.05, 1.0), (1.8, 2.0)])
def test_float32_precision(dtype, dk, dv, lo, hi):
    """Scores and the newest state to float32 rounding.  A token by token scan
    in float32 is off by up to 5.5e-7 in the score (2^-24 of the three terms of
    the difference, each near D, over twice a score of about 0.1) and 3.8e-7 in
    the state; twice that is allowed."""
    import torch
    from paper_2606_10650_amd import dla
    T, n = 330, 8
    w = WORKLOADS["cfg2"].replace(B=1, H=n, T=T, C=40, dk=dk, dv=dv, dtype=dtype, mean_len=30.0,
                                  seed=17 + dk)
    x = make_inputs(w)
    beta = np.random.default_rng(dk).uniform(lo, hi, (n, T)).astype(np.float32)
    xf = H.f64(x, w)
    bo = np.full((n, T), 0, np.int8)              # forced: the states are the oracle's
    bo[:, 25::31] = 1
    ref = oracle_forward(xf["k"], xf["v"], xf["g"], w.C, w.tau, q=xf["q"], lam=xf["lam"],
                         beta=beta.astype(np.float64), b_override=bo)
    _, k, v, g, _ = H.inputs_to_device(w, x, 1, n)
    cache = dla.cache_alloc(1, n, w.C, dk, dv, device="cuda")
    dev = lambda a: torch.from_numpy(a).reshape(1, n, T).cuda()  # noqa: E731
    s = dla.prefill_delta(cache, None, k, v, g, dev(beta), None, tau=w.tau, skip_readout=True,
                          boundary_override=dev(bo))[3].cpu().numpy().reshape(n, T)
    err = np.abs(s - ref["score"]) / np.maximum(ref["score"], 1.0)
    S = H.true_states(dla.cache_export(cache))
    worst = 0.0
    for h in range(n):
        m = int(ref["cache"].m[h])
        Sr = ref["cache"].S[h, m - 1]
        worst = max(worst, np.linalg.norm(S[h, m - 1] - Sr) / np.linalg.norm(Sr))
    print(f"[precision] {dtype} {dk}x{dv} beta {lo}..{hi}: score {err.max():.2e} state {worst:.2e}",
          flush=True)
    assert err.max() < 1.1e-6
    assert worst < 8e-7


def _forced(w, x, beta, bo):
    """Scores and newest states of a prefill with every boundary forced, and the
    oracle's; the cache is large enough that nothing merges."""
    import torch
    from paper_2606_10650_amd import dla
    xf = H.f64(x, w)
    ref = oracle_forward(xf["k"], xf["v"], xf["g"], w.C, w.tau, q=xf["q"], lam=xf["lam"],
                         beta=beta.astype(np.float64), b_override=bo)
    n = w.B * w.H
    q, k, v, g, _ = H.inputs_to_device(w, x, w.B, w.H)
    cache = dla.cache_alloc(w.B, w.H, w.C, w.dk, w.dv, device="cuda")
    dev = lambda a: torch.from_numpy(a).reshape(w.B, w.H, w.T).cuda()  # noqa: E731
    out, _, _, s = dla.prefill_delta(cache, q, k, v, g, dev(beta), None, tau=w.tau,
                                     boundary_override=dev(bo))
    return s.cpu().numpy().reshape(n, w.T), ref, dla.cache_export(cache)


@pytest.mark.parametrize("dtype,dk,dv", [("f32", 128, 128), ("f32", 64, 64), ("bf16", 64, 128)])
@pytest.mark.parametrize("scale", [0.0, 1e-4, 1e-3, 1e-2, 0.3])
def test_steps_that_erase_the_state(dtype, dk, dv, scale):
    """beta = 1 and a repeated key replace a state's value by one `scale` times as
    large, so that |S|^2 is a small rest of large terms: at a chunk's first and
    last tokens, across two chunks, against states from before the chunk, from
    inside it and in a run of boundaries; afterwards ordinary tokens.  A float32
    state keeps the new value to 2^-24 of the old one, hence the scores."""
    T, n = 270, 3
    w = WORKLOADS["cfg2"].replace(B=1, H=n, T=T, C=80, dk=dk, dv=dv, dtype=dtype, mean_len=40.0,
                                  seed=5)
    x = make_inputs(w)
    beta = make_beta(w)
    rng = np.random.default_rng(3)
    bo = np.zeros((n, T), np.int8)
    pairs = [1, 12, 30, 62, 64, 100, 126, 128, 131] + list(range(194, 226, 2))
    k = to_f64(x["k"], dtype)
    v = to_f64(x["v"], dtype)
    for t in pairs + [63, 127]:                                # (63, 64), (127, 128): next chunk
        bo[:, t] = 1
        bo[:, t + 1] = 0
        for h in range(n):
            e = np.zeros(dk)                                   # |k| = 1 exactly
            e[rng.choice(dk, 4, replace=False)] = 0.5
            k[h, t] = k[h, t + 1] = e
        v[:, t + 1] = scale * rng.standard_normal((n, dv))
        beta[:, t:t + 2] = 1.0
    x["k"], x["v"] = store(k, dtype), store(v, dtype)
    s, ref, exp = _forced(w, x, beta, bo)
    err = np.abs(s - ref["score"]) / np.maximum(ref["score"], 1.0)
    tol = 1e-5 + (4.0 * 2.0 ** -24 / scale if scale else 0.0)
    print(f"[erase] {dtype} {dk}x{dv} {scale}: largest score error {np.nanmax(err):.2e} of {tol:.1e}, "
          f"{int(np.isnan(s).sum())} NaN", flush=True)
    assert err.max() < tol
    S = H.true_states(exp)
    for h in range(n):
        m = int(ref["cache"].m[h])
        assert exp["m"][h] == m and (exp["n"][h, :m] == ref["cache"].n[h, :m]).all()
        assert np.allclose(exp["ibar"][h, :m], ref["cache"].ibar[h, :m], rtol=tol, atol=tol)
        Sr = ref["cache"].S[h, m - 1]
        assert np.linalg.norm(S[h, m - 1] - Sr) < 1e-5 * np.linalg.norm(Sr)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_values_whose_square_overflows(dtype):
    """Two values of size 1e25 (their squares are past float32) in a chunk: no
    token before them, and no state that begins after them, changes."""
    T, n = 200, 2
    w = WORKLOADS["cfg2"].replace(B=1, H=n, T=T, C=40, dk=64, dv=64, dtype=dtype, mean_len=20.0,
                                  seed=8)
    x = make_inputs(w)
    beta = make_beta(w)
    bo = np.zeros((n, T), np.int8)
    bo[:, [20, 90, 110, 150]] = 1
    v = to_f64(x["v"], dtype)
    v[:, 100:102] *= 1e25
    x["v"] = store(v, dtype)
    s, ref, exp = _forced(w, x, beta, bo)
    ok = np.r_[0:100, 111:T]
    assert np.abs(s - ref["score"])[:, ok].max() < 1e-5
    S = H.true_states(exp)
    for h in range(n):
        m = int(ref["cache"].m[h])
        Sr = ref["cache"].S[h, m - 1]
        assert np.linalg.norm(S[h, m - 1] - Sr) < 1e-5 * np.linalg.norm(Sr)


@pytest.mark.parametrize("dtype,T", [("bf16", 2600), ("f32", 1100)])
def test_token_by_token_chunks_pipelined_matches_serial(dtype, T):
    """Chunks that go token by token from the start, from a token that erases the
    state, or because the chunk before had one: the pipelined call, whose scan
    runs in segments, equals the serial one bit for bit."""
    import torch
    from paper_2606_10650_amd import dla
    n = 3
    w = WORKLOADS["cfg2"].replace(B=1, H=n, T=T, C=90, dk=64, dv=128, dtype=dtype, mean_len=40.0,
                                  seed=21)
    x = make_inputs(w)
    beta = make_beta(w)
    k, v = to_f64(x["k"], dtype), to_f64(x["v"], dtype)
    for t in list(range(70, T - 1, 97)) + list(range(T // 2, T // 2 + 300, 2)):
        k[:, t + 1] = k[:, t]
        v[:, t + 1] *= 0.01
        beta[:, t:t + 2] = 1.0
    k[:, 900] *= 1.7                              # beta |k|^2 > 2
    beta[:, 900] = 1.0
    x["k"], x["v"] = store(k, dtype), store(v, dtype)
    q, kd, vd, g, lam = H.inputs_to_device(w, x, 1, n)
    bt = torch.from_numpy(beta).reshape(1, n, T).cuda()
    got = []
    for serial in (False, True):
        cache = dla.cache_alloc(1, n, w.C, w.dk, w.dv, device="cuda")
        r = dla.prefill_delta(cache, q, kd, vd, g, bt, lam, tau=w.tau, serial=serial)
        got.append([a.view(torch.int16) if a.dtype == torch.bfloat16 else a for a in r] +
                   [torch.from_numpy(np.ascontiguousarray(a)) for a in dla.cache_export(cache).values()
                    if isinstance(a, np.ndarray)])
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_largest_capacity(dtype):
    """1024 states of 128 x 128, the scan's largest working set in LDS, with
    merges once the cache is full."""
    T, C = 1100, 1024
    w = WORKLOADS["cfg2"].replace(B=1, H=1, T=T, C=C, dtype=dtype, mean_len=2.0, seed=4)
    x = make_inputs(w)
    bo = np.ones((1, T), np.int8)
    bo[:, 1050::3] = 0
    _check(w, x, make_beta(w), bo=bo, what=f"capacity 1024 {dtype}", max_frac=0.2)
