"""16-bit scans whose storing waves bring later chunks' operands into the L2 (16 columns per workgroup and more to move than touch_pays asks
for) against calls of two of the same heads, which do not: the same sums in the same order, bit for bit."""
import pytest
import torch

from paper_2605_05838_amd import binding

pytestmark = pytest.mark.gpu


def inputs(B, T, H, d):
    g = torch.Generator(device="cuda").manual_seed(T)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")
    unit = lambda: torch.nn.functional.normalize(rand(B, T, H, d), dim=-1).bfloat16()
    gate = lambda lo, hi: torch.rand((B, T, H), generator=g, device="cuda") * (hi - lo) + lo
    x = [unit(), unit(), rand(B, T, H, d).bfloat16(), gate(0.1, 0.9), gate(0.9, 1.0), gate(0.5, 0.95)]  # q k v beta alpha mu
    return x, rand(B, T, H, d).bfloat16()


def same(many, few, H, names, states=()):
    for n in names:
        assert torch.isfinite(few[n]).all() and torch.equal(many[n][:, :, H - 2:], few[n]), n
    for n in states:
        assert torch.isfinite(few[n]).all() and torch.equal(many[n][:, H - 2:], few[n]), n


# (about the first sizes beyond the lines: of the forward and the reverse scan of B T H / 64 chunk blocks)
@pytest.mark.parametrize("B,T,H,d", [(1, 64 * 205, 16, 128), (1, 64 * 226 + 37, 16, 128), (1, 64 * 450, 16, 64), (1, 64 * 480 + 1, 16, 64),
                                     (2, 64 * 102 + 50, 16, 128)])
def test_kept_states(B, T, H, d):
    x, dO = inputs(B, T, H, d)
    outs = []
    old = binding.set_segments(1)
    try:
        for heads in (slice(None), slice(H - 2, H)):
            y = [t[:, :, heads].contiguous() for t in x]
            f = binding.mdn_chunk_fwd(*y, scale=d ** -0.5, save_vt=True, save_states=True, save_operands=True)
            b = binding.mdn_chunk_bwd(*y, f["vt"], dO[:, :, heads].contiguous(), states=f["states"], operands=f["operands"], scale=d ** -0.5)
            kept = f["states"].view(torch.bfloat16).view(B, -1, f["states"].numel() * f["states"].element_size() // 2 // B // y[0].shape[2])
            outs.append({**{n: f[n] for n in ("o", "vt", "S", "M")}, "kept": kept, **b})
    finally:
        binding.set_segments(old)
    same(*outs, H, ("o", "vt", "dq", "dk", "dv", "dbeta", "dalpha", "dmu"), ("S", "M", "kept"))


@pytest.mark.parametrize("save_vt", [False, True])
@pytest.mark.parametrize("T,H,d", [(64 * 401 + 5, 16, 128), (64 * 657, 16, 64)])
def test_nothing_or_rows_alone_kept(T, H, d, save_vt):
    x, _ = inputs(1, T, H, d)
    many, few = (binding.mdn_chunk_fwd(*(t[:, :, h].contiguous() for t in x), scale=d ** -0.5, save_vt=save_vt) for h in (slice(None), slice(H - 2, H)))
    same(many, few, H, ("o",) + ("vt",) * save_vt, ("S", "M"))


@pytest.mark.parametrize("segments", [0, 3])
def test_split_reverse_scan(segments):
    """The automatic number of segments and another one: every launch begins and ends its touches at its own segment."""
    T, H, d = 64 * 330 + 17, 16, 128
    x, dO = inputs(1, T, H, d)
    outs = []
    old = binding.set_segments(segments)
    try:
        for heads, k in ((slice(None), segments), (slice(H - 2, H), 1)):
            binding.set_segments(k)
            y = [t[:, :, heads].contiguous() for t in x]
            f = binding.mdn_chunk_fwd(*y, scale=d ** -0.5, save_vt=True, save_states=True, save_operands=True)
            outs.append(binding.mdn_chunk_bwd(*y, f["vt"], dO[:, :, heads].contiguous(), states=f["states"], operands=f["operands"], scale=d ** -0.5))
            outs[-1]["o"] = f["o"]
    finally:
        binding.set_segments(old)
    same(*outs, H, ("o", "dq", "dk", "dv", "dbeta", "dalpha", "dmu"))


def test_packed_batch():
    """Two long sequences and their ends inside a chunk: rows and chunk blocks come from the tables (the backward takes each by itself)."""
    H, d, cu = 16, 128, (0, 64 * 170 + 7, 64 * 170 + 7 + 64 * 205 + 33)
    x, dO = inputs(1, cu[-1], H, d)
    g = torch.Generator(device="cuda").manual_seed(1)
    S0, M0 = (0.1 * torch.randn((2, H, d, d), device="cuda", generator=g) for _ in range(2))
    outs = []
    for heads in (slice(None), slice(H - 2, H)):
        y = [t[:, :, heads].contiguous() for t in x]
        s = {"S0": S0[:, heads].contiguous(), "M0": M0[:, heads].contiguous()}
        f = binding.mdn_chunk_fwd_varlen(*y, cu, scale=d ** -0.5, save_vt=True, **s)
        b = binding.mdn_chunk_bwd_varlen(*y, f["vt"], dO[:, :, heads].contiguous(), cu, scale=d ** -0.5, **s)
        outs.append({**{n: f[n] for n in ("o", "vt", "S", "M")}, **b})
    same(*outs, H, ("o", "vt", "dq", "dk", "dv", "dbeta", "dalpha", "dmu"), ("S", "M", "dS0", "dM0"))
