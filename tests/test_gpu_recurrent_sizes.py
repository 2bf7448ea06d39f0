"""The decode step where its launch changes form: 32 / 64 state columns per workgroup, states past the caches or not."""
import math

import pytest

from paper_2605_05838_amd import binding


# 64 columns from BH * d / 64 = 4 workgroups per CU on; states past the caches above 352 MiB (2 816 pairs of 128, 11 264 of 64)
@pytest.mark.gpu
@pytest.mark.parametrize("BH,d,T,dtype,eta", [((73, 7), 128, 2, "bf16", True), ((32, 16), 128, 3, "f32", False),
                                              ((33, 31), 64, 2, "f32", True), ((64, 16), 64, 3, "bf16", False),
                                              ((256, 11), 128, 1, "bf16", False), ((939, 3), 128, 2, "f32", True),
                                              ((313, 9), 128, 2, "bf16", True), ((1610, 7), 64, 2, "bf16", False),
                                              ((1610, 7), 64, 1, "f32", True)])
def test_recurrent_step_on_both_sides_of_every_size_rule(BH, d, T, dtype, eta):
    """o, S and M of every (batch, head) pair against the recurrence in float64.  Bounds: fp32 sums of d terms 1e-5; a
    16-bit o is rounded once more, 2^-8 / sqrt(3) = 2.3e-3 of its value at most in the root mean square."""
    import torch
    B, H = BH
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    n = lambda *s: torch.randn(s, device="cuda", generator=g)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k = ((x / x.norm(dim=-1, keepdim=True)).to(dt) for x in (n(B, T, H, d), n(B, T, H, d)))
    v = n(B, T, H, d).to(dt)
    al, be, mu = torch.sigmoid(n(B, T, H) + 3), torch.sigmoid(n(B, T, H)), torch.sigmoid(n(B, T, H) + 2)
    et = torch.sigmoid(n(B, T, H)) * 2 if eta else None
    S, M = 0.3 * n(B, H, d, d), 0.1 * n(B, H, d, d)
    rS, rM, ro = S.double(), M.double(), []
    for t in range(T):
        col = lambda x: x[:, t].double()[..., None, None]
        kt = k[:, t].double()[..., None]
        e = v[:, t].double()[..., None, :] - (col(al) * kt * rS).sum(-2, keepdim=True)
        rM = col(mu) * rM - (col(et) if eta else 1.0) * kt * e
        rS = col(al) * rS - col(be) * rM
        ro.append(d ** -0.5 * (q[:, t].double()[..., None] * rS).sum(-2))
    o = binding.mdn_recurrent_step(q, k, v, be, al, mu, S, M, eta=et, scale=d ** -0.5)
    rel = lambda x, ref: float((x.double() - ref).norm() / ref.norm())
    assert rel(S, rS) < 1e-5 and rel(M, rM) < 1e-5
    assert rel(o, torch.stack(ro, 1)) < (3e-3 if dtype == "bf16" else 1e-5)
    assert math.isfinite(float(S.abs().max()))
