"""A decode step split over several workgroups per head against the same heads in
a batch large enough to go unsplit: equal decisions and states, outputs within
the reordering of float32 sums.  Forced merges visit every pair, so that pairs
lie inside a workgroup's range, across two, and at the newest state."""
import numpy as np
import pytest
import torch

from paper_2606_10650_amd import dla, policies

pytestmark = pytest.mark.gpu

UNSPLIT = 1024   # heads from which a step is not split


def _fill(c, k, v, g, bo, mo, fill):
    dla.prefill(c, None, k[:, :, :fill].contiguous(), v[:, :, :fill].contiguous(),
                g[:, :, :fill].contiguous(), tau=0.5, skip_readout=True, want_exports=False,
                boundary_override=bo, merge_override=mo)


@pytest.mark.parametrize("heads,C,dk,dv,states,full", [
    (3, 4, 64, 64, "f32", True),        # too few states for a split
    (3, 24, 128, 128, "bf16", True),    # the smallest ranges: two states each
    (300, 64, 64, 64, "bf16", True),    # more workgroups than the chip holds at once
    (5, 33, 64, 128, "bf16", True),     # 16 ranges, the last one short
    (32, 17, 128, 128, "f32", True),    # about one workgroup per compute unit
    (33, 40, 128, 64, "f32", False),    # room left: no merge, the newest state in mid-cache
    (65, 9, 128, 128, "bf16", True),
    (300, 64, 64, 64, "f32", True),
    (2, 12, 128, 128, "f32", False),
])
@pytest.mark.parametrize("delta", [False, True])
def test_split_matches_unsplit(heads, C, dk, dv, states, full, delta):
    n = C if full else C // 2                     # states before the step
    fill, steps = 3 * n, min(C - 1, 6)
    gen = torch.Generator(device="cuda").manual_seed(C * 1000 + heads)
    T = fill + steps
    rnd = lambda *s: torch.randn((1, heads, *s), generator=gen, device="cuda")  # noqa: E731
    q, k, v = rnd(T, dk), rnd(T, dk) / dk ** 0.5, rnd(T, dv)
    g = -0.05 * torch.rand((1, heads, T), generator=gen, device="cuda")
    lam = rnd(T, C)
    beta = torch.rand((1, heads, T), generator=gen, device="cuda")
    _, b, m = policies.every_k(fill, 3, C)
    bo, mo = (torch.from_numpy(a).cuda().expand(1, heads, fill).contiguous() for a in (b, m))
    # the steps: every head joins or opens in turn, merging another pair each time
    h, t = np.arange(heads)[:, None], np.arange(steps)[None]
    sb = torch.from_numpy(((h + t) % 3 != 0).astype(np.int8)).cuda()[None]
    sm = torch.from_numpy(((h * 5 + t * 7 + C - 2) % (C - 1)).astype(np.int32)).cuda()[None]
    got = []
    for rep in (1, -(-UNSPLIT // heads)):
        r = lambda x: x.repeat(rep, *([1] * (x.dim() - 1)))  # noqa: E731
        cache = dla.cache_alloc(rep, heads, C, dk, dv, device="cuda",
                                state_dtype=dla.DLA_BF16 if states == "bf16" else dla.DLA_F32)
        L = dla.cache_layout(rep, heads, C, dk, dv, cache.state_dtype)
        cache.buf[L.states_offset:].zero_()       # slots that no state takes compare equal
        _fill(cache, r(k), r(v), r(g), r(bo), r(mo), fill)
        res = []
        for i in range(steps):
            at = lambda x: r(x[:, :, fill + i].contiguous())  # noqa: E731
            kw = dict(tau=0.5, boundary_override=r(sb[:, :, i].contiguous()),
                      merge_override=r(sm[:, :, i].contiguous()))
            if delta:
                res.append(dla.decode_step_delta(cache, at(q), at(k), at(v), at(g), at(beta), at(lam), **kw))
            else:
                res.append(dla.decode_step(cache, at(q), at(k), at(v), at(g), at(lam), **kw))
        torch.cuda.synchronize()
        es = 2 if states == "bf16" else 4
        st = cache.buf[L.states_offset:L.states_offset + heads * C * dk * dv * es].clone()
        meta = cache.buf[L.meta_offset:L.meta_offset + heads * L.meta_stride]
        meta = meta.view(heads, L.meta_stride)[:, :32 + 24 * C].clone()
        got.append((res, st, meta))
    (a, sta, ma), (u, stu, mu) = got
    assert torch.equal(ma, mu), "metadata"
    assert torch.equal(sta, stu), "states"
    for x, y in zip(a, u):
        for i in (1, 2, 3):
            assert torch.equal(x[i][0], y[i][0])
        ox, oy = x[0][0].double(), y[0][0].double()
        # C dk products summed in float32, in two orders
        assert (ox - oy).norm() <= 1e-5 * oy.norm()
        assert (ox - oy).abs().max() <= 1e-4 * oy.abs().max()
