"""16-bit scans whose storing waves bring later chunks' operands into the L2 (calls of more than twice the last-level cache, 16 columns
per workgroup) against calls of two of the same heads, which do not: the same sums in the same order, bit for bit."""
import pytest
import torch

from paper_2605_05838_amd import binding

pytestmark = pytest.mark.gpu


# bytes a call moves at least, see touch_pays: the smaller T of a pair passes the line in the forward with kept states alone
@pytest.mark.parametrize("T,H,d", [(64 * 205, 16, 128), (64 * 226 + 37, 16, 128), (64 * 445, 16, 64), (64 * 480 + 1, 16, 64)])
def test_touched_calls_give_the_results_of_untouched_ones(T, H, d):
    g = torch.Generator(device="cuda").manual_seed(T)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")
    unit = lambda: torch.nn.functional.normalize(rand(1, T, H, d), dim=-1).bfloat16()
    gate = lambda lo, hi: torch.rand((1, T, H), generator=g, device="cuda") * (hi - lo) + lo
    x = [unit(), unit(), rand(1, T, H, d).bfloat16(), gate(0.1, 0.9), gate(0.9, 1.0), gate(0.5, 0.95)]  # q k v beta alpha mu
    dO = rand(1, T, H, d).bfloat16()
    outs = []
    old = binding.set_segments(1)
    try:
        for heads in (slice(None), slice(H - 2, H)):
            y = [t[:, :, heads].contiguous() for t in x]
            f = binding.mdn_chunk_fwd(*y, scale=d ** -0.5, save_vt=True, save_states=True, save_operands=True)
            b = binding.mdn_chunk_bwd(*y, f["vt"], dO[:, :, heads].contiguous(), states=f["states"], operands=f["operands"], scale=d ** -0.5)
            outs.append({**{n: f[n] for n in ("o", "vt")}, **{n: b[n] for n in ("dq", "dk", "dv", "dbeta", "dalpha", "dmu")},
                         "S": f["S"], "M": f["M"]})
    finally:
        binding.set_segments(old)
    for n, few in outs[1].items():
        many = outs[0][n][:, H - 2:] if n in "SM" else outs[0][n][:, :, H - 2:]
        assert torch.isfinite(few).all() and torch.equal(many, few), n
