"""The operand rings of the 16-bit forward scan at their ends: sequences of fewer chunks than a ring holds up to a few more, whole and
with a partial last chunk, in the instances whose q rows are a tile (16 columns; 32 with kept states) and whose are not (32 without)."""
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
