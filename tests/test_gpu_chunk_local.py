"""The chunk-local operands where a token's products overflow, and where every block of A = (P K~^T) .* Gamma^- counts: keys with a common part, so that no product of two
of them is small, slow gates, and lengths that end inside each of the 16-token blocks the triangular inverse is built from."""
import numpy as np
import pytest
import torch

from gpu_util import host, rel_err, rms_rel_err, to_dev
from oracle import mdn_oracle as orc
from paper_2605_05838_amd import binding, synth

pytestmark = pytest.mark.gpu

# 16-bit storage: the bound of the other parity tests.  32-bit: sums of up to 64 + 128 terms that partly cancel, 2^-24 sqrt(192) times
# a growth of ten for T's entries.
TOL = {"f32": 8e-6, "bf16": 2e-2}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,T", [(64, 15), (64, 64), (128, 31), (128, 33), (64, 49), (128, 128), (64, 113)])
def test_correlated_keys(dtype, d, T):
    w = synth.custom(B=1, T=T, H=2, dk=d, dv=d, dtype=dtype, seed=100 * d + T, backward=True, alpha_logit_mean=3.0, mu_logit_mean=2.0)
    rng = np.random.default_rng(T)
    k = w.arrays["k"].astype(np.float64) + rng.standard_normal((1, 1, 1, d)) * d ** -0.5
    k = (k / np.linalg.norm(k, axis=-1, keepdims=True)).astype(np.float32)
    w.arrays["k"] = synth.bf16_round(k) if dtype == "bf16" else k
    t = to_dev(w)
    x = (t["q"], t["k"], t["v"], t["beta"], t["alpha"], t["mu"])
    f = binding.mdn_chunk_fwd(*x, scale=w.scale, save_vt=True, save_states=True, save_operands=True)
    g = binding.mdn_chunk_bwd(*x, f["vt"], t["dO"], states=f["states"], operands=f["operands"], scale=w.scale)
    a = {n: None if v is None else v.astype(np.float64) for n, v in w.arrays.items()}
    z = (a["q"], a["k"], a["v"], a["alpha"], a["beta"], a["mu"])
    rf, rb = orc.forward(*z, scale=w.scale), orc.backward(*z, a["dO"], scale=w.scale)
    pairs = [(n, f[n], rf[n]) for n in ("o", "S", "M")] + [(n, g[n], rb[n]) for n in ("dq", "dk", "dv", "dbeta", "dalpha", "dmu")]
    errs = {n: max(rel_err(host(y), ref), rms_rel_err(host(y), ref)) for n, y, ref in pairs}
    assert max(errs.values()) <= TOL[dtype], errs


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,t", [(128, 3), (128, 12), (64, 20), (64, 27), (128, 40), (64, 63)])
def test_a_token_that_overflows_leaves_the_tokens_before_it_alone(dtype, d, t):
    """A key of 1e25 in every element: finite, and so are its products with ordinary keys, but not the later rows of T.  What the tokens
    before it give, V~ and dq, is that of a call without it, bit for bit."""
    w = synth.custom(B=1, T=64, H=2, dk=d, dv=d, dtype=dtype, seed=t, backward=True)
    x = to_dev(w)

    def run():
        a = (x["q"], x["k"], x["v"], x["beta"], x["alpha"], x["mu"])
        f = binding.mdn_chunk_fwd(*a, scale=w.scale, save_vt=True)
        return f["vt"][:, :t], binding.mdn_chunk_bwd(*a, f["vt"], x["dO"], scale=w.scale)["dq"][:, :t]

    plain = [y.clone() for y in run()]
    x["k"][0, t] = 1e25
    for n, y, ref in zip(("vt", "dq"), run(), plain):
        assert torch.isfinite(ref).all() and torch.equal(y, ref), n
