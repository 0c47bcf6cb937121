"""A readout whose token tiles are shared by two workgroups (few heads) against
the same heads in a batch that fills the chip, where one workgroup serves all
tiles: every tile is computed by the same instructions, so outputs are equal
bit for bit.  Lengths at the edges of tiles, of chunks and of a part's tiles,
with and without states before the call."""
import pytest
import torch

from paper_2606_10650_amd import dla

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T", [1, 32, 129, 255, 513, 1090])
@pytest.mark.parametrize("dk,dv,lam", [(64, 64, True), (128, 128, True), (128, 64, False)])
def test_parts_match_whole(dtype, T, dk, dv, lam):
    H, C, rep = 3, 20, 48      # 48 x 3 heads: more than 128 workgroups for one chunk
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(T + dk)
    rnd = lambda *s: torch.randn((1, H, *s), generator=gen, device="cuda")  # noqa: E731
    calls = []
    for n in (70, T):          # the first call leaves states that the second reads
        q, k, v = rnd(n, dk).to(dt), (rnd(n, dk) / dk ** 0.5).to(dt), rnd(n, dv).to(dt)
        g = -0.05 * torch.rand((1, H, n), generator=gen, device="cuda")
        bo = (torch.rand((1, H, n), generator=gen, device="cuda") < 0.05).to(torch.int8)
        calls.append((q, k, v, g, rnd(n, C).to(dt) if lam else None, bo))
    got = []
    for r in (1, rep):
        cache = dla.cache_alloc(r, H, C, dk, dv, device="cuda")
        out = []
        for call in calls:
            q, k, v, g, lm, bo = (None if a is None else a.repeat(r, *([1] * (a.dim() - 1)))
                                  for a in call)
            out.append(dla.prefill(cache, q, k, v, g, lm, tau=0.5, boundary_override=bo)[0][0])
        got.append(out)
    torch.cuda.synchronize()
    for a, b in zip(*got):
        assert torch.equal(a, b)
