"""GPU parity of the layer's elementwise front end and back end (mdn_frontend_*, mdn_epilogue_*) against the fp64
oracle, through the C ABI."""
import numpy as np
import pytest
import torch

from oracle import layer_ops_oracle as lo
from paper_2605_05838_amd import binding

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}     # fp32: elementwise arithmetic and 64-lane sums; bf16: rounding of inputs and outputs


def rel(x, ref):
    return float(np.abs(x.astype(np.float64) - ref).max() / max(np.abs(ref).max(), 1e-30))


def _t(a, dtype):
    t = torch.from_numpy(a.astype(np.float32)).cuda()
    return t.to(torch.bfloat16) if dtype == "bf16" else t


def _h(t):
    return t.float().cpu().numpy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
def test_frontend_and_epilogue_match_the_oracle(dtype, d):
    check(dtype, d, 2, 203, 5)


# Rows enough for several trips of the largest launches, not a multiple of what a workgroup takes, heads that divide the step
# from trip to trip and heads that do not: the adjoints (256 workgroups of 16 waves of 512 / d rows, half as many in 32-bit
# storage), the forwards (32 workgroups of 4 waves per CU).  And a single row.
@pytest.mark.parametrize("dtype,d,B,T,H", [("bf16", 64, 1, 14003, 5), ("bf16", 128, 1, 2311, 16), ("f32", 64, 1, 7021, 5),
                                           ("f32", 128, 1, 1151, 16), ("f32", 64, 3, 8747, 5), ("f32", 128, 1, 16385, 4),
                                           ("bf16", 64, 1, 1, 1), ("f32", 128, 1, 1, 1)])
def test_many_rows_and_one_match_the_oracle(dtype, d, B, T, H):
    check(dtype, d, B, T, H)


def check(dtype, d, B, T, H):
    rng = np.random.default_rng(61)
    xq, xk, xv, dq, dk, dv, o, g, dy = (rng.standard_normal((B, T, H, d)) for _ in range(9))
    dh = rng.uniform(-0.5, 0.5, H).astype(np.float32)
    w = rng.uniform(0.5, 1.5, d).astype(np.float32)
    dev = [_t(a, dtype) for a in (xq, xk, xv, dq, dk, dv, o, g, dy)]
    # the oracle sees exactly the values the kernels see (after rounding to the storage type)
    xq, xk, xv, dq, dk, dv, o, g, dy = (_h(t).astype(np.float64) for t in dev)
    dht, wt = torch.from_numpy(dh).cuda(), torch.from_numpy(w).cuda()
    f = binding.mdn_frontend_fwd(dev[0], dev[1], dev[2], dht)
    b = binding.mdn_frontend_bwd(dev[0], dev[1], dev[2], dht, dev[3], dev[4], dev[5])
    y = binding.mdn_epilogue_fwd(dev[6], dev[7], wt)
    e = binding.mdn_epilogue_bwd(dev[6], dev[7], wt, dev[8])
    torch.cuda.synchronize()
    rf = lo.frontend_forward(xq, xk, xv, dh)
    rb = lo.frontend_backward(xq, xk, xv, dh, dq, dk, dv)
    tol = TOL[dtype]
    for k in ("q", "k", "v"):
        assert rel(_h(f[k]), rf[k]) <= tol, k
    for k in ("dx_q", "dx_k", "dx_v"):
        assert rel(_h(b[k]), rb[k]) <= tol, k
    # sums over B T (d) terms of either sign in 32 bits, whatever the storage: against the sum of their sizes, which is at
    # most sqrt(rows) of the result here, a few times 2^-24
    assert rel(_h(b["dd"]), rb["dd"]) <= 1e-4
    assert rel(_h(y), lo.epilogue_forward(o, g, w)) <= tol
    re_ = lo.epilogue_backward(o, g, w, dy)
    assert rel(_h(e["do"]), re_["do"]) <= tol and rel(_h(e["dg"]), re_["dg"]) <= tol
    assert rel(_h(e["dw"]), re_["dw"]) <= 1e-4


@pytest.mark.parametrize("d", [64, 128])
def test_parameter_gradients_of_16_bit_tensors_are_computed_in_32_bits(d):
    """One row with |o| = 1 (no sum depends on its order): dw = dy sigmoid(g) o / sqrt(1 + eps) of 16-bit tensors is bit for
    bit that of the same values in 32-bit tensors."""
    gen = torch.Generator(device="cuda").manual_seed(62)
    for _ in range(8):
        o, g, dy = (3.0 * torch.randn((1, 1, 1, d), device="cuda", generator=gen) for _ in range(3))
        w = 0.5 + torch.rand(d, device="cuda", generator=gen)
        dw = [binding.mdn_epilogue_bwd(*(t.bfloat16().to(dt) for t in (o.sign(), g)), w, dy.bfloat16().to(dt))["dw"]
              for dt in (torch.bfloat16, torch.float32)]
        assert torch.equal(*dw)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tensors_at_any_element_offset(dtype):
    """Contiguous views that start at an odd element of their buffer give the results of aligned copies, bit for bit (one
    row: no sum depends on the order of the workgroups)."""
    d, gen = 128, torch.Generator(device="cuda").manual_seed(63)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    flat = torch.randn(10 * (d + 1), device="cuda", generator=gen).to(dt)
    par = torch.rand(2 * d, device="cuda", generator=gen)
    odd = [flat[1 + i * (d + 1):][:d].view(1, 1, 1, d) for i in range(9)]
    got = []
    for x, w, dh in ((odd, par[1:1 + d], par[:1]), ([t.clone() for t in odd], par[1:1 + d].clone(), par[:1].clone())):
        got.append([*binding.mdn_frontend_fwd(*x[:3], dh).values(), *binding.mdn_frontend_bwd(*x[:3], dh, *x[3:6]).values(),
                    binding.mdn_epilogue_fwd(*x[6:8], w), *binding.mdn_epilogue_bwd(*x[6:8], w, x[8]).values()])
    assert any(t.data_ptr() % 16 for t in odd) and all(torch.equal(a, b) for a, b in zip(*got))
