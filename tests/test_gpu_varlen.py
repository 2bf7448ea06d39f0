"""GPU parity of the packed variable-length entry points against the oracle run sequence by sequence."""
import numpy as np
import pytest
import torch

from gpu_util import host, to_dev, worst_err
from oracle import mdn_oracle as orc
from paper_2605_05838_amd import binding, synth

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-4, "bf16": 2e-2}


@pytest.mark.parametrize("dtype,d,lens", [("f32", 64, (70, 128, 5, 191)), ("bf16", 128, (256, 33, 200))])
def test_packed_sequences_forward_and_backward(dtype, d, lens):
    T, H = sum(lens), 3
    w = synth.custom(B=1, T=T, H=H, dk=d, dv=d, dtype=dtype, seed=71, with_eta=True, backward=True)
    t = to_dev(w)
    n = len(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).tolist()
    rng = np.random.default_rng(3)
    S0 = (rng.standard_normal((n, H, d, d)) * 0.2).astype(np.float32)
    M0 = (rng.standard_normal((n, H, d, d)) * 0.1).astype(np.float32)
    dSf = rng.standard_normal((n, H, d, d)).astype(np.float32)
    dMf = rng.standard_normal((n, H, d, d)).astype(np.float32)
    dev = lambda a: torch.from_numpy(a).cuda()
    f = binding.mdn_chunk_fwd_varlen(t["q"], t["k"], t["v"], t["beta"], t["alpha"], t["mu"], cu, eta=t["eta"], S0=dev(S0),
                                     M0=dev(M0), scale=w.scale, save_vt=True)
    g = binding.mdn_chunk_bwd_varlen(t["q"], t["k"], t["v"], t["beta"], t["alpha"], t["mu"], f["vt"], t["dO"], cu,
                                     eta=t["eta"], S0=dev(S0), M0=dev(M0), dS_final=dev(dSf), dM_final=dev(dMf),
                                     scale=w.scale, want_deta=True)
    torch.cuda.synchronize()
    a = {k: (None if v is None else v.astype(np.float64)) for k, v in w.arrays.items()}
    tol = TOL[dtype]
    for i in range(n):
        sl = slice(cu[i], cu[i + 1])
        seq = {k: a[k][:, sl] for k in ("q", "k", "v", "alpha", "beta", "mu", "eta", "dO")}
        s0, m0 = S0[i:i + 1].astype(np.float64), M0[i:i + 1].astype(np.float64)
        rf = orc.forward(seq["q"], seq["k"], seq["v"], seq["alpha"], seq["beta"], seq["mu"], eta=seq["eta"], S0=s0, M0=m0,
                         scale=w.scale)
        assert worst_err(host(f["o"])[:, sl], rf["o"]) <= tol, (i, "o")
        assert worst_err(host(f["S"])[i:i + 1], rf["S"]) <= tol and worst_err(host(f["M"])[i:i + 1], rf["M"]) <= tol, (i, "S/M")
        rb = orc.backward(seq["q"], seq["k"], seq["v"], seq["alpha"], seq["beta"], seq["mu"], seq["dO"], eta=seq["eta"],
                          S0=s0, M0=m0, dS_T=dSf[i:i + 1].astype(np.float64), dM_T=dMf[i:i + 1].astype(np.float64),
                          scale=w.scale)
        for name in ("dq", "dk", "dv", "dalpha", "dbeta", "dmu", "deta"):
            assert worst_err(host(g[name])[:, sl], rb[name]) <= tol, (i, name)
        for name in ("dS0", "dM0"):
            assert worst_err(host(g[name])[i:i + 1], rb[name]) <= tol, (i, name)


@pytest.mark.parametrize("dtype,d,lens", [("f32", 64, (70, 128, 5, 191, 1, 64)), ("bf16", 128, (256, 33, 200, 1, 63, 65)),
                                          ("bf16", 64, (40,) * 9), ("f32", 128, (300,)),
                                          ("f32", 64, (700, 333, 64, 1, 900, 250)), ("bf16", 128, (1030, 1100))])
def test_packed_sequences_as_one_stream_of_tokens(dtype, d, lens):
    """No per-sequence states in or out: the library may merge neighbours, with alpha = mu = 0 at the sequence starts.  Every
    sequence must come out as the oracle computes it by itself from zero states (sequence starts inside chunks, on chunk
    boundaries, sequences of one token), and the caller's alpha, mu must be left as they were."""
    T, H = sum(lens), 3
    w = synth.custom(B=1, T=T, H=H, dk=d, dv=d, dtype=dtype, seed=72, with_eta=True, backward=True)
    t = to_dev(w)
    n = len(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).tolist()
    al0, mu0 = t["alpha"].clone(), t["mu"].clone()
    f = binding.mdn_chunk_fwd_varlen(t["q"], t["k"], t["v"], t["beta"], t["alpha"], t["mu"], cu, eta=t["eta"],
                                     scale=w.scale, save_vt=True, want_states=False)
    g = binding.mdn_chunk_bwd_varlen(t["q"], t["k"], t["v"], t["beta"], t["alpha"], t["mu"], f["vt"], t["dO"], cu,
                                     eta=t["eta"], scale=w.scale, want_deta=True, want_state_grads=False)
    torch.cuda.synchronize()
    assert f["S"] is None and g["dS0"] is None
    assert torch.equal(al0, t["alpha"]) and torch.equal(mu0, t["mu"])
    a = {k: (None if v is None else v.astype(np.float64)) for k, v in w.arrays.items()}
    tol = TOL[dtype]
    for i in range(n):
        sl = slice(cu[i], cu[i + 1])
        seq = {k: a[k][:, sl] for k in ("q", "k", "v", "alpha", "beta", "mu", "eta", "dO")}
        rf = orc.forward(seq["q"], seq["k"], seq["v"], seq["alpha"], seq["beta"], seq["mu"], eta=seq["eta"], scale=w.scale)
        assert worst_err(host(f["o"])[:, sl], rf["o"]) <= tol, (i, "o")
        assert worst_err(host(f["vt"])[:, sl], rf["vt"]) <= tol, (i, "vt")
        rb = orc.backward(seq["q"], seq["k"], seq["v"], seq["alpha"], seq["beta"], seq["mu"], seq["dO"], eta=seq["eta"],
                          scale=w.scale)
        for name in ("dq", "dk", "dv", "dalpha", "dbeta", "dmu", "deta"):
            assert worst_err(host(g[name])[:, sl], rb[name]) <= tol, (i, name)
        # the first token's alpha, mu multiply zero states: their gradients are exactly zero
        assert float(host(g["dalpha"])[:, cu[i]].max()) == 0.0 and float(host(g["dmu"])[:, cu[i]].min()) == 0.0, i


@pytest.mark.parametrize("dtype,d,lens", [("f32", 64, (70, 128, 5, 191, 1, 64, 3, 2)), ("bf16", 128, (256, 33, 200, 1, 63, 65)),
                                          ("bf16", 64, (40,) * 9), ("f32", 128, (300,)), ("f32", 64, (7, 9)),
                                          ("f32", 64, (700, 333, 64, 1, 900, 250)), ("bf16", 128, (1030, 1100))])
def test_packed_prompts_with_final_states_of_every_sequence(dtype, d, lens):
    """Zero initial states, final states wanted (prefill of a batch of prompts): o and every sequence's S, M against the oracle
    (sequences that end inside a chunk, on a chunk boundary, sequences shorter than a chunk, a total length below one
    chunk, lengths far apart)."""
    T, H = sum(lens), 2
    w = synth.custom(B=1, T=T, H=H, dk=d, dv=d, dtype=dtype, seed=73, with_eta=True)
    t = to_dev(w)
    n = len(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).tolist()
    f = binding.mdn_chunk_fwd_varlen(t["q"], t["k"], t["v"], t["beta"], t["alpha"], t["mu"], cu, eta=t["eta"],
                                     scale=w.scale)
    torch.cuda.synchronize()
    a = {k: (None if v is None else v.astype(np.float64)) for k, v in w.arrays.items()}
    tol = TOL[dtype]
    for i in range(n):
        sl = slice(cu[i], cu[i + 1])
        seq = {k: a[k][:, sl] for k in ("q", "k", "v", "alpha", "beta", "mu", "eta")}
        rf = orc.forward(seq["q"], seq["k"], seq["v"], seq["alpha"], seq["beta"], seq["mu"], eta=seq["eta"], scale=w.scale)
        assert worst_err(host(f["o"])[:, sl], rf["o"]) <= tol, (i, "o")
        assert worst_err(host(f["S"])[i:i + 1], rf["S"]) <= tol, (i, "S")
        assert worst_err(host(f["M"])[i:i + 1], rf["M"]) <= tol, (i, "M")


@pytest.mark.parametrize("dtype,n", [("f32", 229), ("bf16", 3)])
def test_packed_states_in_and_out_of_many_short_and_of_uneven_sequences(dtype, n):
    """More sequences than one launch's list of entries holds (lengths 1 to 4), and three sequences whose order of
    dispatch (longest first) is not the caller's: states and their adjoints have to come back in the caller's order."""
    d, H = 64, 1
    lens = [1 + i % 4 for i in range(n)] if n > 3 else [65, 1, 130]
    T = sum(lens)
    w = synth.custom(B=1, T=T, H=H, dk=d, dv=d, dtype=dtype, seed=74, with_eta=True, backward=True)
    t = to_dev(w)
    cu = np.concatenate([[0], np.cumsum(lens)]).tolist()
    rng = np.random.default_rng(4)
    S0, M0, dSf = ((rng.standard_normal((n, H, d, d)) * 0.2).astype(np.float32) for _ in range(3))
    dev = lambda a: torch.from_numpy(a).cuda()
    x = tuple(t[k] for k in ("q", "k", "v", "beta", "alpha", "mu"))
    f = binding.mdn_chunk_fwd_varlen(*x, cu, eta=t["eta"], S0=dev(S0), M0=dev(M0), scale=w.scale, save_vt=True)
    g = binding.mdn_chunk_bwd_varlen(*x, f["vt"], t["dO"], cu, eta=t["eta"], S0=dev(S0), M0=dev(M0), dS_final=dev(dSf),
                                     scale=w.scale, want_deta=True)
    torch.cuda.synchronize()
    a = {k: (None if v is None else v.astype(np.float64)) for k, v in w.arrays.items()}
    ref = {k: [] for k in ("o", "S", "M", "dq", "dk", "dv", "dalpha", "dbeta", "dmu", "deta", "dS0", "dM0")}
    for i in range(n):
        q = [a[k][:, cu[i]:cu[i + 1]] for k in ("q", "k", "v", "alpha", "beta", "mu")]
        kw = dict(eta=a["eta"][:, cu[i]:cu[i + 1]], S0=S0[i:i + 1].astype(np.float64), M0=M0[i:i + 1].astype(np.float64),
                  scale=w.scale)
        rf = orc.forward(*q, **kw)
        rb = orc.backward(*q, a["dO"][:, cu[i]:cu[i + 1]], dS_T=dSf[i:i + 1].astype(np.float64), **kw)
        for k in ref:
            ref[k].append((rf if k in rf else rb)[k])
    for k, parts in ref.items():
        x = np.concatenate(parts, axis=0 if k in ("S", "M", "dS0", "dM0") else 1)
        assert worst_err(host((f if k in f else g)[k]), x) <= TOL[dtype], k


def test_packed_batch_of_very_short_sequences_runs_group_by_group():
    """16 heads x 5 000 sequences of 1 .. 7 tokens need 80 000 chunk blocks, more than one group takes: outputs, states and
    gradients are bit for bit those of the same sequences in two calls (whose groups are others)."""
    H, d, n = 16, 64, 5000
    lens = [1 + (5 * i + i // 7) % 7 for i in range(n)]
    cu = np.concatenate([[0], np.cumsum(lens)]).tolist()
    w = synth.custom(B=1, T=cu[-1], H=H, dk=d, dv=d, dtype="bf16", seed=74, with_eta=True, backward=True)
    t = to_dev(w)
    gen = torch.Generator(device="cuda").manual_seed(5)
    S0, M0, dS, dM = (0.2 * torch.randn((n, H, d, d), device="cuda", generator=gen) for _ in range(4))

    def run(a, b):
        x = [t[k][:, cu[a]:cu[b]].contiguous() for k in ("q", "k", "v", "beta", "alpha", "mu")]
        eta, dO = (t[k][:, cu[a]:cu[b]].contiguous() for k in ("eta", "dO"))
        c = [v - cu[a] for v in cu[a:b + 1]]
        s0, m0, ds, dm = (z[a:b].contiguous() for z in (S0, M0, dS, dM))
        f = binding.mdn_chunk_fwd_varlen(*x, c, eta=eta, S0=s0, M0=m0, scale=w.scale, save_vt=True)
        g = binding.mdn_chunk_bwd_varlen(*x, f["vt"], dO, c, eta=eta, S0=s0, M0=m0, dS_final=ds, dM_final=dm, scale=w.scale,
                                         want_deta=True)
        return {k: v for k, v in {**f, **g}.items() if torch.is_tensor(v) and k != "workspace"}

    whole, left, right = run(0, n), run(0, n // 2), run(n // 2, n)
    for k in whole:
        dim = 0 if k in ("S", "M", "dS0", "dM0") else 1
        assert torch.equal(whole[k], torch.cat((left[k], right[k]), dim=dim)), k


@pytest.mark.parametrize("dtype,d,lens", [("f32", 64, (3, 17, 1, 40, 64, 2, 130, 9, 9, 9, 300, 5)),
                                          ("bf16", 128, (3, 17, 1, 40, 64, 2, 130, 9, 9, 9, 300, 5)),
                                          ("bf16", 64, (7, 9)), ("f32", 128, (20, 30, 14)),
                                          ("bf16", 64, (1, 2, 3) * 400)])
def test_short_sequences_merged_into_pieces(dtype, d, lens):
    """Calls without states that save an eighth of their chunks by merging neighbours (one piece for everything, starts on
    and off chunk boundaries, more starts than one launch takes), every sequence against the oracle by itself."""
    test_packed_sequences_as_one_stream_of_tokens(dtype, d, lens)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 64), ("f32", 128), ("bf16", 128)])
def test_packed_sequences_of_whole_chunks_equal_the_fixed_length_batch(dtype, d):
    """The kernels' instances for whole chunks against the general ones: a batch of two sequences and the same sequences packed
    (with states: one set of launches, nothing merged) go through the same arithmetic, so every output agrees bit for bit."""
    B, T, H = 2, 192, 3
    w = synth.custom(B=B, T=T, H=H, dk=d, dv=d, dtype=dtype, seed=75, with_eta=True, s0_std=0.2, backward=True)
    t = to_dev(w)
    gen = torch.Generator(device="cuda").manual_seed(6)
    M0, dS, dM = (0.2 * torch.randn((B, H, d, d), device="cuda", generator=gen) for _ in range(3))
    row = lambda x: x.reshape(1, B * T, *x.shape[2:])
    x = [t[k] for k in ("q", "k", "v", "beta", "alpha", "mu")]
    for adjoints in ({}, dict(dS_final=dS, dM_final=dM)):
        kw = dict(S0=t["S0"], M0=M0, scale=w.scale)
        f = binding.mdn_chunk_fwd(*x, eta=t["eta"], save_vt=True, **kw)
        g = binding.mdn_chunk_bwd(*x, f["vt"], t["dO"], eta=t["eta"], want_deta=True, **adjoints, **kw)
        p, cu = [row(a) for a in x], [0, T, 2 * T]
        pf = binding.mdn_chunk_fwd_varlen(*p, cu, eta=row(t["eta"]), save_vt=True, **kw)
        pg = binding.mdn_chunk_bwd_varlen(*p, pf["vt"], row(t["dO"]), cu, eta=row(t["eta"]), want_deta=True, **adjoints, **kw)
        for k, v in {**pf, **pg}.items():
            ref = f[k] if k in f else g[k]
            assert torch.equal(v.reshape(ref.shape), ref), k


def _by_sequence(t, cu, scale, states=None, adjoints=None):
    """The gradients of a packed batch from one call per sequence (and the forward's outputs): states S0, M0, adjoints dS, dM of
    all sequences, or None."""
    parts = {}
    for i in range(len(cu) - 1):
        sl = slice(cu[i], cu[i + 1])
        x = [t[k][:, sl].clone() for k in ("q", "k", "v", "beta", "alpha", "mu")]
        kw = dict(scale=scale, eta=t["eta"][:, sl].clone())
        if states:
            kw.update(S0=states[0][i:i + 1], M0=states[1][i:i + 1])
        f = binding.mdn_chunk_fwd(*x, save_vt=True, **kw)
        if adjoints:
            kw.update(dS_final=adjoints[0][i:i + 1], dM_final=adjoints[1][i:i + 1])
        g = binding.mdn_chunk_bwd(*x, f["vt"], t["dO"][:, sl].clone(), want_deta=True, **kw)
        for k, v in {**f, **g}.items():
            if torch.is_tensor(v) and k != "workspace":
                parts.setdefault(k, []).append(v)
    return {k: torch.cat(v, dim=0 if k in ("S", "M", "dS0", "dM0") else 1) for k, v in parts.items()}


def test_sequences_that_are_groups_of_their_own_equal_calls_on_each():
    """Adjoints of the final states come in and each of the two sequences needs more than half of a group's limit: they run one
    after the other, as batches of one (17 heads: the second one's gates are not 16-byte aligned)."""
    H, d, cu = 17, 128, [0, 3845, 7685]
    w = synth.custom(B=1, T=cu[-1], H=H, dk=d, dv=d, dtype="bf16", seed=76, with_eta=True, backward=True)
    t = to_dev(w)
    gen = torch.Generator(device="cuda").manual_seed(7)
    S0, M0, dS, dM = (0.2 * torch.randn((2, H, d, d), device="cuda", generator=gen) for _ in range(4))
    ref = _by_sequence(t, cu, w.scale, (S0, M0), (dS, dM))
    x = [t[k] for k in ("q", "k", "v", "beta", "alpha", "mu")]
    kw = dict(eta=t["eta"], S0=S0, M0=M0, scale=w.scale)
    f = binding.mdn_chunk_fwd_varlen(*x, cu, save_vt=True, **kw)
    g = binding.mdn_chunk_bwd_varlen(*x, f["vt"], t["dO"], cu, dS_final=dS, dM_final=dM, want_deta=True, **kw)
    for k, v in {**f, **g}.items():
        assert torch.equal(v, ref[k]), k


@pytest.mark.parametrize("states", [False, True], ids=["without_states", "with_states"])
def test_a_long_sequence_among_short_ones(states):
    """One sequence that is nearly the whole batch: the scans take it for what the launch lasts (16 columns per workgroup, a CU
    for each), and the backward runs it by itself, split into two
    segments.  Every output agrees bit for bit with the calls on each sequence."""
    H, d, cu = 8, 128, [0, 100, 20137, 20200]
    w = synth.custom(B=1, T=cu[-1], H=H, dk=d, dv=d, dtype="bf16", seed=77, with_eta=True, backward=True)
    t = to_dev(w)
    gen = torch.Generator(device="cuda").manual_seed(8)
    S0, M0 = (0.2 * torch.randn((3, H, d, d), device="cuda", generator=gen) for _ in range(2))
    ref = _by_sequence(t, cu, w.scale, (S0, M0) if states else None)
    x = [t[k] for k in ("q", "k", "v", "beta", "alpha", "mu")]
    kw = dict(eta=t["eta"], scale=w.scale, **(dict(S0=S0, M0=M0) if states else {}))
    f = binding.mdn_chunk_fwd_varlen(*x, cu, save_vt=True, want_states=states, **kw)
    binding.profile_begin()
    g = binding.mdn_chunk_bwd_varlen(*x, f["vt"], t["dO"], cu, want_deta=True, want_state_grads=states, **kw)
    launches = binding.profile_end(with_launch_counts=True)
    assert launches["grad"][2] == launches["scan_bwd"][2] == 4 and launches["rebuild"][2] == 3
    for k, v in {**f, **g}.items():
        if v is not None:
            assert torch.equal(v, ref[k]), k


@pytest.mark.parametrize("d", [64, 128])
def test_more_workgroups_of_a_packed_batch_than_cus(d):
    """40 sequences of 1 to 300 tokens of 8 heads: two workgroups per CU where they fit, sequences looked up in the device table.
    Every output agrees bit for bit with the calls on each sequence, which leave most CUs idle."""
    rng = np.random.default_rng(79)
    lens = [1, 2, 63, 64, 65, 127, 128, 129, 192, 300] + rng.integers(1, 300, 30).tolist()
    H, n, cu = 8, len(lens), np.concatenate([[0], np.cumsum(lens)]).tolist()
    w = synth.custom(B=1, T=cu[-1], H=H, dk=d, dv=d, dtype="bf16", seed=79, with_eta=True, backward=True)
    t = to_dev(w)
    gen = torch.Generator(device="cuda").manual_seed(9)
    S0, M0, dS, dM = (0.2 * torch.randn((n, H, d, d), device="cuda", generator=gen) for _ in range(4))
    x = [t[k] for k in ("q", "k", "v", "beta", "alpha", "mu")]
    kw = dict(eta=t["eta"], S0=S0, M0=M0, scale=w.scale)
    f = binding.mdn_chunk_fwd_varlen(*x, cu, save_vt=True, **kw)
    for adjoints in (None, (dS, dM)):
        ref = _by_sequence(t, cu, w.scale, (S0, M0), adjoints)
        a = adjoints or (None, None)
        g = binding.mdn_chunk_bwd_varlen(*x, f["vt"], t["dO"], cu, dS_final=a[0], dM_final=a[1], want_deta=True, **kw)
        for k, v in {**f, **g}.items():
            assert torch.equal(v, ref[k]), (k, adjoints is not None)
