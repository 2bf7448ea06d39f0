"""The operand rings of the 16-bit forward scan at their ends: sequences of fewer chunks than a ring holds up to a few more, whole and
with a partial last chunk, in the instances whose q rows are a tile and in those that hold them in registers (see q_tile_pays)."""
import pytest
import torch

from gpu_util import gather_pairs, host, select_pairs, to_dev, worst_err
from oracle import mdn_oracle as orc
from paper_2605_05838_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,d", [(1, 3, 128), (1, 2, 64), (5, 8, 128), (5, 16, 64)])  # 16 columns, 16, 32, 32
@pytest.mark.parametrize("T", [64, 128, 192, 256, 320, 1, 65, 150, 203, 300])
def test_forward_ring_ends(B, H, d, T):
    w = synth.custom(B=B, T=T, H=H, dk=d, dv=d, dtype="bf16", seed=T + d + B, s0_std=0.05)
    t = to_dev(w)
    x = (t["q"], t["k"], t["v"], t["beta"], t["alpha"], t["mu"])
    plain = binding.mdn_chunk_fwd(*x, S0=t["S0"], scale=w.scale)
    kept = binding.mdn_chunk_fwd(*x, S0=t["S0"], scale=w.scale, save_vt=True, save_states=True, save_operands=True)
    for n in ("o", "S", "M"):  # the same sums in the same order
        assert torch.equal(plain[n], kept[n]), n
    pairs = [(0, 0), (B - 1, H - 1)]
    z = select_pairs(w, pairs)
    ref = orc.forward(z["q"], z["k"], z["v"], z["alpha"], z["beta"], z["mu"], S0=z["S0"], scale=w.scale)
    for n in ("o", "S", "M"):
        err = worst_err(gather_pairs(host(kept[n]), pairs, is_state=n != "o"), ref[n])
        assert err <= 2e-2, (n, err)


@pytest.mark.parametrize("B,T,H,d", [(1, 64 * 11, 2, 128), (1, 64 * 12 + 5, 3, 128), (2, 64 * 9 + 63, 5, 128), (1, 64 * 10, 3, 64), (1, 64 * 11 + 1, 1, 64),  # 16 columns
                                     (5, 64 * 9, 8, 128), (5, 64 * 9 + 1, 8, 128)])  # 32
def test_q_in_registers_gives_what_a_tile_gives(B, T, H, d):
    g = torch.Generator(device="cuda").manual_seed(T)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")
    unit = lambda: torch.nn.functional.normalize(rand(B, T, H, d), dim=-1).bfloat16()
    gate = lambda lo, hi: torch.rand((B, T, H), generator=g, device="cuda") * (hi - lo) + lo
    x = [unit(), unit(), rand(B, T, H, d).bfloat16(), gate(0.1, 0.9), gate(0.9, 1.0), gate(0.5, 0.95)]  # q k v beta alpha mu
    plain = binding.mdn_chunk_fwd(*x, scale=d ** -0.5)
    kept = binding.mdn_chunk_fwd(*x, scale=d ** -0.5, save_vt=True, save_states=True, save_operands=True)
    for n in ("o", "S", "M"):
        assert torch.isfinite(plain[n]).all() and torch.equal(plain[n], kept[n]), n


@pytest.mark.parametrize("d,lens", [(128, (1, 64, 65, 150, 1700, 128, 203, 1500)), (64, (1, 64, 1500))])
def test_short_sequences_among_long_ones(d, lens):
    """More chunks on average than a tile of q is taken for: sequences of one chunk up to four with q in registers, against calls of
    their own, with a tile."""
    H, T = d // 64, sum(lens)
    w = synth.custom(B=1, T=T, H=H, dk=d, dv=d, dtype="bf16", seed=d)
    t = to_dev(w)
    x = [t[n] for n in ("q", "k", "v", "beta", "alpha", "mu")]
    cu = [sum(lens[:i]) for i in range(len(lens) + 1)]
    S0, M0 = (0.1 * torch.randn(len(lens), H, d, d, device="cuda", generator=torch.Generator(device="cuda").manual_seed(i)) for i in (1, 2))
    f = binding.mdn_chunk_fwd_varlen(*x, cu, S0=S0, M0=M0, scale=w.scale)
    for i, (a, b) in enumerate(zip(cu, cu[1:])):
        one = binding.mdn_chunk_fwd(*(y[:, a:b].clone() for y in x), S0=S0[i:i + 1], M0=M0[i:i + 1], scale=w.scale)
        assert torch.equal(f["o"][:, a:b], one["o"]), lens[i]
        assert torch.equal(f["S"][i], one["S"][0]) and torch.equal(f["M"][i], one["M"][0]), lens[i]
