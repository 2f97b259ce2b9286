"""GPU parity of the delta-rule forward and backward (DeltaNet and Gated DeltaNet rows of Table 1) against the fp64
token-by-token oracle, element by element, through the C ABI.  Tolerance: max|x - ref| / RMS(ref) <= 2e-2 for the bf16 output (its
own container rounding discounted, as for the other kinds), 2e-2 for the fp32 final state too: the pseudo-values
u_t pass through one bf16 rounding inside the path, so the state carries rounding of the size of a bf16 input."""
import numpy as np
import pytest

import lsm_workloads as wl
from lsm_testlib import BF16_HALF_ULP, host, rel_err

pytestmark = pytest.mark.gpu

TOL = 2e-2


def dev(x, layout=0):
    import torch
    d = torch.device("cuda:0")
    def mv(a, dt, per_token):
        if a is None:
            return None
        t = torch.from_numpy(np.ascontiguousarray(a)).to(d).to(dt)
        if layout == 1 and per_token:
            t = t.transpose(1, 2)
        return t.contiguous()
    t = {n: mv(x[n], torch.bfloat16, True) for n in ("q", "k", "v")}
    t.update({n: mv(x[n], torch.float32, True) for n in ("log_alpha", "beta", "b")})
    t["m0"] = mv(x["m0"], torch.float32, False)
    return t


def run_and_check(x, layout=0, report=None):
    import torch
    import paper_2503_05447_amd as pkg
    from oracle import delta_oracle_fwd
    t = dev(x, layout)
    o, mT = pkg.lsm_delta_fwd(t["q"], t["k"], t["v"], t["log_alpha"], t["beta"], t["b"], t["m0"], layout=layout)
    torch.cuda.synchronize()
    if layout == 1:
        o = o.transpose(1, 2)
    o_ref, mT_ref = delta_oracle_fwd(x["q"], x["k"], x["v"], x["log_alpha"], x["beta"], x["b"], x["m0"])
    eo, eraw, em = rel_err(host(o), o_ref, BF16_HALF_ULP), rel_err(host(o), o_ref), rel_err(host(mT), mT_ref)
    if report is not None:
        report.update(o=eo, o_raw=eraw, final_state=em)
    print("delta fwd B=%d H=%d T=%d gated=%s layout=%d: o %.3e (raw %.3e) final_state %.3e"
          % (x["B"], x["H"], x["T"], x["gated"], layout, eo, eraw, em), flush=True)
    assert eo <= TOL and em <= TOL, (eo, em)
    return o, mT


# (B, H, T): one chunk; a ragged chunk; several chunks and a ragged tail; many chunks
SHAPES = [(1, 2, 64), (2, 2, 37), (2, 3, 200), (1, 4, 1300)]


@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_delta_forward_matches_oracle(shape, gated):
    B, H, T = shape
    x = wl.make_delta_inputs(B, H, T, 128, 128, gated, seed=4100 + T + int(gated), init_state=True)
    run_and_check(x)


@pytest.mark.parametrize("gated", [False, True])
def test_delta_forward_separate_strengths_and_no_initial_state(gated):
    x = wl.make_delta_inputs(2, 2, 330, 128, 128, gated, seed=4200 + int(gated), init_state=False, tie_b=False)
    if gated:   # all three per-token parameters at once (the general form both rows are instances of)
        rng = np.random.default_rng(7)
        x["beta"] = (0.2 + 0.7 * rng.random((2, 2, 330))).astype(np.float32)
    run_and_check(x)


@pytest.mark.parametrize("decay", ["weak", "strong4", "harsh"])
def test_gated_delta_decay_strengths(decay):
    x = wl.make_delta_inputs(1, 3, 700, 128, 128, True, seed=4300, decay=decay, init_state=True)
    run_and_check(x)


def test_delta_token_major_layout():
    x = wl.make_delta_inputs(2, 3, 150, 128, 128, True, seed=4400, init_state=True)
    run_and_check(x, layout=1)


def test_delta_correlated_keys():
    """Keys drawn from a handful of directions (plus noise), as trained models produce them: the triangular system of
    a chunk is then far from the identity."""
    x = wl.make_delta_inputs(1, 2, 512, 128, 128, False, seed=4500, init_state=True)
    rng = np.random.default_rng(4501)
    base = rng.standard_normal((6, 128)).astype(np.float32)
    pick = rng.integers(0, 6, size=(1, 2, 512))
    k = base[pick] + 0.3 * rng.standard_normal((1, 2, 512, 128)).astype(np.float32)
    k /= np.sqrt((k * k).sum(-1, keepdims=True))
    x["k"] = wl.bf16_round(k)
    run_and_check(x)


def test_delta_zero_erase_equals_the_scalar_kind_bitwise_inputs():
    """beta = 0: the path must agree with the per-token scalar-decay forward on values b v (same oracle pin, on the GPU)."""
    import torch
    import paper_2503_05447_amd as pkg
    x = wl.make_delta_inputs(1, 2, 300, 128, 128, True, seed=4600, init_state=True)
    x["beta"] = np.zeros((1, 2, 300), np.float32)
    x["b"] = np.ones((1, 2, 300), np.float32)
    o, mT = run_and_check(x)
    t = dev(x)
    o2, mT2 = pkg.lsm_chunk_fwd(t["q"], t["k"], t["v"], t["log_alpha"], pkg.DECAY_SCALAR, 64, t["m0"])
    torch.cuda.synchronize()
    assert rel_err(host(o), host(o2)) <= 2 ** -7      # two bf16 containers of nearly the same fp32 values
    assert rel_err(host(mT), host(mT2)) <= 1e-2


def run_bwd_and_check(x, layout=0):
    import torch
    import paper_2503_05447_amd as pkg
    from oracle import delta_oracle_bwd
    t = dev(x, layout)
    d = torch.device("cuda:0")
    def mv(a, dt, per_token):
        if a is None:
            return None
        z = torch.from_numpy(np.ascontiguousarray(a)).to(d).to(dt)
        return (z.transpose(1, 2) if (layout == 1 and per_token) else z).contiguous()
    d_o, d_mT = mv(x["d_o"], torch.bfloat16, True), mv(x["d_mT"], torch.float32, False)
    r = pkg.lsm_delta_bwd(t["q"], t["k"], t["v"], d_o, t["log_alpha"], t["beta"], t["b"], t["m0"], d_mT, layout=layout)
    torch.cuda.synchronize()
    ref = delta_oracle_bwd(x["q"], x["k"], x["v"], x["d_o"], x["log_alpha"], x["beta"], x["b"], x["m0"], x["d_mT"])
    names = dict(dq="dq", dk="dk", dv="dv", d_log_alpha="d_log_alpha", d_beta="d_beta", d_b="d_b", d_init_state="d_m0")
    rep = {}
    for n_, rn in names.items():
        assert (r[n_] is None) == (ref[rn] is None), n_
        if r[n_] is None:
            continue
        got = r[n_]
        if layout == 1 and n_ != "d_init_state":
            got = got.transpose(1, 2)
        rep[n_] = rel_err(host(got), ref[rn], BF16_HALF_ULP if n_ in ("dq", "dk", "dv") else 0.0)
    print("delta bwd B=%d H=%d T=%d gated=%s layout=%d: %s"
          % (x["B"], x["H"], x["T"], x["gated"], layout, " ".join("%s %.2e" % kv for kv in rep.items())), flush=True)
    for n_, e in rep.items():
        assert e <= TOL, (n_, e)


# (B, H, T): one chunk; a ragged chunk; several chunks; eleven chunks (every chunk a segment of the gradient walker);
# 40 sequences of 24 chunks (segments of two chunks)
BWD_SHAPES = [(1, 2, 64), (2, 2, 37), (2, 3, 200), (1, 3, 700), (5, 8, 1500)]
# every sequence one segment (from 192 sequences on): whole chunks, a ragged tail of one token, one ragged chunk
WHOLE_SHAPES = [(6, 32, 128), (8, 25, 129), (6, 32, 50)]
# the gradient walker's segments shorter than the other walkers': two in each of theirs, and two where those have one
FINER_SHAPES = [(9, 16, 500), (18, 16, 200)]


@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("shape", BWD_SHAPES + WHOLE_SHAPES + FINER_SHAPES)
def test_delta_backward_matches_oracle(shape, gated):
    B, H, T = shape
    x = wl.make_delta_inputs(B, H, T, 128, 128, gated, seed=5100 + T + int(gated), init_state=True, d_final=True)
    run_bwd_and_check(x)


@pytest.mark.parametrize("gated", [False, True])
def test_delta_backward_separate_strengths_no_edge_states(gated):
    x = wl.make_delta_inputs(2, 2, 330, 128, 128, gated, seed=5200 + int(gated), init_state=False, d_final=False, tie_b=False)
    if gated:   # all three per-token parameters at once
        rng = np.random.default_rng(8)
        x["beta"] = (0.2 + 0.7 * rng.random((2, 2, 330))).astype(np.float32)
    run_bwd_and_check(x)


@pytest.mark.parametrize("decay", ["weak", "strong4", "harsh"])
def test_gated_delta_backward_decay_strengths(decay):
    x = wl.make_delta_inputs(1, 3, 500, 128, 128, True, seed=5300, decay=decay, init_state=True, d_final=True)
    run_bwd_and_check(x)


def test_delta_backward_token_major_layout():
    x = wl.make_delta_inputs(2, 3, 150, 128, 128, True, seed=5400, init_state=True, d_final=True)
    run_bwd_and_check(x, layout=1)


def test_delta_backward_correlated_keys():
    x = wl.make_delta_inputs(1, 2, 512, 128, 128, False, seed=5500, init_state=True, d_final=True)
    rng = np.random.default_rng(5501)
    base = rng.standard_normal((6, 128)).astype(np.float32)
    pick = rng.integers(0, 6, size=(1, 2, 512))
    k = base[pick] + 0.3 * rng.standard_normal((1, 2, 512, 128)).astype(np.float32)
    k /= np.sqrt((k * k).sum(-1, keepdims=True))
    x["k"] = wl.bf16_round(k)
    run_bwd_and_check(x)


@pytest.mark.parametrize("gated", [False, True])
def test_delta_backward_with_kept_forward_results_is_bitwise_the_same(gated):
    import torch
    import paper_2503_05447_amd as pkg
    x = wl.make_delta_inputs(2, 3, 330, 128, 128, gated, seed=5600 + int(gated), init_state=True, d_final=True)
    t = dev(x)
    d = torch.device("cuda:0")
    d_o = torch.from_numpy(x["d_o"]).to(d).to(torch.bfloat16)
    d_mT = torch.from_numpy(x["d_mT"]).to(d)
    args = (t["q"], t["k"], t["v"])
    o1, m1 = pkg.lsm_delta_fwd(*args, t["log_alpha"], t["beta"], t["b"], t["m0"])
    r1 = pkg.lsm_delta_bwd(*args, d_o, t["log_alpha"], t["beta"], t["b"], t["m0"], d_mT)
    ws = pkg.lsm_delta_workspace(*args, t["log_alpha"])
    o2, m2 = pkg.lsm_delta_fwd(*args, t["log_alpha"], t["beta"], t["b"], t["m0"], workspace=ws, save_states=True)
    r2 = pkg.lsm_delta_bwd(*args, d_o, t["log_alpha"], t["beta"], t["b"], t["m0"], d_mT, workspace=ws, states_saved=True)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(m1, m2)
    for n_ in r1:
        assert (r1[n_] is None) == (r2[n_] is None)
        if r1[n_] is not None:
            assert torch.equal(r1[n_], r2[n_]), n_


@pytest.mark.parametrize("T", [1, 63, 65, 128])
def test_delta_tiny_and_boundary_lengths(T):
    for gated in (False, True):
        x = wl.make_delta_inputs(1, 1, T, 128, 128, gated, seed=5700 + T, init_state=True, d_final=True)
        run_and_check(x)
        run_bwd_and_check(x)


def test_delta_degenerate_strengths():
    """Erase strength 0 (nothing erased), 1 (full erase, the Gated row's own setting) and a write strength of 0 for
    half of the tokens (those tokens only erase)."""
    rng = np.random.default_rng(5800)
    for beta_val in (0.0, 1.0):
        x = wl.make_delta_inputs(1, 2, 260, 128, 128, False, seed=5801, init_state=True, d_final=True, tie_b=False)
        x["beta"] = np.full((1, 2, 260), beta_val, np.float32)
        x["b"] = (x["b"] * (rng.random((1, 2, 260)) < 0.5)).astype(np.float32)
        run_and_check(x)
        run_bwd_and_check(x)


def test_delta_unit_key_returns_its_value_on_the_gpu():
    """The stored-value property through the kernels: a = b = 1, keys of unit length, the query equal to the key:
    o_t = (k_t . k_t) v_t, i.e. v_t up to the bf16 rounding of the key's length (2^-8) and of o."""
    import torch
    import paper_2503_05447_amd as pkg
    x = wl.make_delta_inputs(1, 2, 200, 128, 128, False, seed=5900, init_state=True)
    x["beta"] = np.ones((1, 2, 200), np.float32)
    x["b"] = np.ones((1, 2, 200), np.float32)
    x["q"] = x["k"].copy()
    t = dev(x)
    o, _ = pkg.lsm_delta_fwd(t["q"], t["k"], t["v"], None, t["beta"], t["b"], t["m0"])
    torch.cuda.synchronize()
    kk = (x["k"].astype(np.float64) ** 2).sum(-1, keepdims=True)
    # k M_t = v_t + (1 - k.k) (k M_{t-1} - v_t): exact only for an exactly unit key; allow the first-order term
    assert rel_err(host(o), x["v"].astype(np.float64), 2.0 ** -8 + 4 * np.abs(1 - kk).max()) <= 1e-2
    run_and_check(x)


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("gated", [False, True])
def test_delta_packed_sequences_equal_separate_calls(gated, keep):
    """Packed variable-length input (lengths with ragged chunks, one shorter than a chunk, one empty): every sequence
    must come out bit for bit as from a call of its own, forward and backward."""
    import torch
    import paper_2503_05447_amd as pkg
    lens = [130, 40, 0, 64, 77]
    T, H, n = sum(lens), 2, len(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    x = wl.make_delta_inputs(1, H, T, 128, 128, gated, seed=6000 + int(gated), tie_b=False)
    rng = np.random.default_rng(6001)
    x["m0"] = (rng.standard_normal((n, H, 128, 128)) * 0.1).astype(np.float32)
    x["d_mT"] = (rng.standard_normal((n, H, 128, 128)) * 0.1).astype(np.float32)
    if gated:
        x["beta"] = (0.2 + 0.7 * rng.random((1, H, T))).astype(np.float32)
    t = dev(x)
    d = torch.device("cuda:0")
    d_o, d_mT = torch.from_numpy(x["d_o"]).to(d).to(torch.bfloat16), torch.from_numpy(x["d_mT"]).to(d)
    cu_d = torch.from_numpy(cu).to(d)
    ws = pkg.lsm_delta_workspace(t["q"], t["k"], t["v"], t["log_alpha"], cu_seqlens=cu_d) if keep else None
    o, mT = pkg.lsm_delta_fwd(t["q"], t["k"], t["v"], t["log_alpha"], t["beta"], t["b"], t["m0"], cu_seqlens=cu_d, workspace=ws,
                              save_states=keep)
    r = pkg.lsm_delta_bwd(t["q"], t["k"], t["v"], d_o, t["log_alpha"], t["beta"], t["b"], t["m0"], d_mT, cu_seqlens=cu_d,
                          workspace=ws, states_saved=keep)
    torch.cuda.synchronize()
    piece = lambda a, lo, hi: None if a is None else a[:, :, lo:hi].contiguous()
    for s_, (lo, hi) in enumerate(zip(cu[:-1], cu[1:])):
        if hi == lo:   # the empty sequence passes its states through
            assert torch.equal(mT[s_], t["m0"][s_]) and torch.equal(r["d_init_state"][s_], d_mT[s_])
            continue
        args = [piece(t[n_], lo, hi) for n_ in ("q", "k", "v")]
        pars = [piece(t[n_], lo, hi) for n_ in ("log_alpha", "beta", "b")]
        o_s, mT_s = pkg.lsm_delta_fwd(*args, *pars, t["m0"][s_:s_ + 1].contiguous())
        r_s = pkg.lsm_delta_bwd(*args, piece(d_o, lo, hi), *pars, t["m0"][s_:s_ + 1].contiguous(), d_mT[s_:s_ + 1].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(o[:, :, lo:hi], o_s) and torch.equal(mT[s_:s_ + 1], mT_s), s_
        for n_ in ("dq", "dk", "dv", "d_log_alpha", "d_beta", "d_b"):
            if r_s[n_] is not None:
                assert torch.equal(r[n_][:, :, lo:hi], r_s[n_]), (n_, s_)
        assert torch.equal(r["d_init_state"][s_:s_ + 1], r_s["d_init_state"]), s_


def half_unit(x):
    """Largest distance of a number of x's binade to its bf16 head and remainder: the head is within 2^(e-8), that rest within half
    a unit of its own eight bits."""
    return 2.0 ** (np.floor(np.log2(np.maximum(np.abs(x), 1e-30))) - 17)


def nearly_orthogonal(seed):
    """One chunk, 16 recurrences: token t's key is feature 64 + t and a bit of feature 0, which couples the tokens by 2^-12."""
    x = wl.make_delta_inputs(2, 8, 64, 128, 128, False, seed=seed, tie_b=False, d_final=True)
    k = np.zeros((2, 8, 64, 128), np.float32)
    k[..., np.arange(64), 64 + np.arange(64)] = 1.0
    k[..., 0] = c = wl.bf16_round(np.float32(0.0157))
    x["k"] = k
    x["d_mT"] = wl.bf16_round(x["d_mT"])
    x["q"], x["d_o"] = np.zeros_like(x["q"]), np.zeros_like(x["d_o"])
    return x, float(c) ** 2


def test_delta_pseudo_values_are_rounded_once():
    """Rows 64 + t of the final state are u_t, which is kept as a bf16 head and remainder: no further from the exact one than that,
    the coupling's share of three such roundings (T, R, remainder times remainder) and 24 of fp32 (two for each matrix product)."""
    import torch
    import paper_2503_05447_amd as pkg
    from oracle import delta_oracle_fwd
    x, coupling = nearly_orthogonal(6100)
    t = dev(x)
    _, mT = pkg.lsm_delta_fwd(t["q"], t["k"], t["v"], None, t["beta"], t["b"])
    torch.cuda.synchronize()
    u = delta_oracle_fwd(x["q"], x["k"], x["v"], None, x["beta"], x["b"], None)[1][:, :, 64:]
    over = np.abs(host(mT)[:, :, 64:] - u) / (half_unit(u) + 64 * coupling * 3 * half_unit(np.abs(u).max()) + 24 * 2.0 ** -24 * np.abs(u))
    print("pseudo-values: %.3f of the bound" % over.max())
    assert over.max() <= 1.0


def test_delta_gradients_of_the_right_hand_side_are_rounded_once():
    """Rows 64 + t of d_init_state are d_mT - beta_t W_t (no queries): beta W is multiplied as a bf16 head and remainder, d_mT is bf16
    already.  Bound as for the pseudo-values."""
    import torch
    import paper_2503_05447_amd as pkg
    from oracle import delta_oracle_bwd
    x, coupling = nearly_orthogonal(6200)
    t = dev(x)
    d_o, d_mT = torch.from_numpy(x["d_o"]).to(t["q"].device).to(torch.bfloat16), torch.from_numpy(x["d_mT"]).to(t["q"].device)
    r = pkg.lsm_delta_bwd(t["q"], t["k"], t["v"], d_o, None, t["beta"], t["b"], None, d_mT)
    torch.cuda.synchronize()
    ref = delta_oracle_bwd(x["q"], x["k"], x["v"], x["d_o"], None, x["beta"], x["b"], None, x["d_mT"])["d_m0"][:, :, 64:]
    w = x["d_mT"][:, :, 64:].astype(np.float64) - ref
    over = np.abs(host(r["d_init_state"])[:, :, 64:] - ref) / (half_unit(w) + 64 * coupling * 3 * half_unit(np.abs(w).max()) +
                                                               24 * 2.0 ** -24 * (np.abs(w) + np.abs(ref)))
    print("gradients of the right-hand side: %.3f of the bound" % over.max())
    assert over.max() <= 1.0


def one_chunk(T):
    z = lambda *s: np.zeros((1, 1, T) + s, np.float32)
    return dict(B=1, H=1, T=T, dk=128, dv=128, q=z(128), k=z(128), v=z(128), d_o=z(128), m0=None, d_mT=None, log_alpha=None,
                beta=None, b=np.ones((1, 1, T), np.float32))


def backward_of(x):
    import torch
    import paper_2503_05447_amd as pkg
    from oracle import delta_oracle_bwd
    t = dev(x)
    d_o = torch.from_numpy(x["d_o"]).to(t["q"].device).to(torch.bfloat16)
    r = pkg.lsm_delta_bwd(t["q"], t["k"], t["v"], d_o, t["log_alpha"], t["beta"], t["b"])
    torch.cuda.synchronize()
    return r, delta_oracle_bwd(x["q"], x["k"], x["v"], x["d_o"], x["log_alpha"], x["beta"], x["b"], None, None)


def test_delta_decay_gradient_keeps_what_is_small_beside_the_diagonal():
    """Token 0's k.dk is 1.5 2^23 from its own query, less 63 erase terms of 2^-6, a quarter of a unit for every 16 tokens.  q.dq has
    the same large number; what is left, a unit, is the decay gradient's.  Bound: one rounding of k.dk, and those of W (2^-17 each)."""
    x = one_chunk(64)
    t = np.arange(1, 64)
    x["log_alpha"] = np.zeros((1, 1, 64), np.float32)
    x["k"][0, 0, 0, 0], x["q"][0, 0, 0, 0], x["d_o"][0, 0, 0, 0], x["v"][0, 0, 0, 0] = 1.0, 2.0 ** 12, 1.5 * 2.0 ** 11, 1.0
    x["k"][0, 0, t, t], x["k"][0, 0, t, 0], x["q"][0, 0, t, t], x["d_o"][0, 0, t, 0] = 1.0, 2.0 ** -6, 1.0, 1.0
    r, ref = backward_of(x)
    err = np.abs(host(r["d_log_alpha"]) - ref["d_log_alpha"]).max()
    print("decay gradient: off by %.3f units of k.dk" % err)
    assert err <= 0.5 + 64 * 2.0 ** -6 * 2.0 ** -17


def test_delta_erase_gradient_has_the_product_of_the_remainders():
    """d beta_1 = -W_1 . u_0, both 1 + 255 2^-16, exact as a bf16 head and remainder: the product of the remainders is 2^-16 of it, and
    nothing else is rounded but fp32 sums."""
    x = one_chunk(2)
    x["beta"] = np.full((1, 1, 2), 0.5, np.float32)
    x["k"][0, 0, :, 0] = 1.0
    x["k"][0, 0, 1, 1] = 1.0
    x["b"][0, 0, 0] = 1.0 + 255 * 2.0 ** -16
    x["v"][0, 0, 0, 0] = x["d_o"][0, 0, 1, 0] = x["q"][0, 0, 1, 0] = 1.0
    x["q"][0, 0, 1, 1] = 255 * 2.0 ** -16
    r, ref = backward_of(x)
    want = float(ref["d_beta"][0, 0, 1])
    assert abs(want + (1.0 + 255 * 2.0 ** -16) ** 2) < 1e-12
    err = abs(float(r["d_beta"][0, 0, 1]) - want)
    print("erase gradient: relative error %.2e" % (err / abs(want)))
    assert err <= 2.0 ** -20 * abs(want)


def test_delta_packed_factors_of_cut_sequences_only():
    """The factors of the segments ([sequence][segment][128][128] fp32, five such planes before the workspace's end) are formed for the
    sequences that are cut, and for none of a single segment."""
    import torch
    import paper_2503_05447_amd as pkg
    lens, H = [1500, 40, 200, 64, 900], 8
    seqs, total = len(lens) * H, sum(lens)
    chunks = -(-total // 64)
    m = -(-chunks // min(-(-256 // seqs), chunks))
    nseg, own = -(-chunks // m), [-(-n // (64 * m)) for n in lens]
    assert sorted(set(own)) == [1, 3, 4]
    x = wl.make_delta_inputs(1, H, total, 128, 128, False, seed=6300)
    t = dev(x)
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device=t["q"].device)
    ws = pkg.lsm_delta_workspace(t["q"], t["k"], t["v"], None, cu_seqlens=cu)
    ws.fill_(0xff)
    pkg.lsm_delta_fwd(t["q"], t["k"], t["v"], None, t["beta"], t["b"], cu_seqlens=cu, workspace=ws, save_states=True)
    torch.cuda.synchronize()
    plane = seqs * nseg * 65536
    factors = ws[ws.numel() - 5 * plane:ws.numel() - 4 * plane].reshape(seqs, nseg, 65536)
    written = (factors != 0xff).any(2).cpu().numpy()
    for s in range(seqs):
        n = own[s // H]
        assert written[s].tolist() == [i < n and n > 1 for i in range(nseg)], (s, n)


@pytest.mark.parametrize("gated", [False, True])
def test_delta_packed_segments_of_several_chunks(gated):
    """Sequences of one segment and of two beside each other, in segments of 13 chunks, the gradient walker's of 2 chunks: against the
    oracle sequence by sequence (calls of their own are cut otherwise)."""
    import torch
    import paper_2503_05447_amd as pkg
    from oracle import delta_oracle_bwd, delta_oracle_fwd
    lens, H = [1500, 40, 0, 700, 64, 130], 16
    T, n = sum(lens), len(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    x = wl.make_delta_inputs(1, H, T, 128, 128, gated, seed=6400 + int(gated), tie_b=False, decay="weak")
    rng = np.random.default_rng(6401)
    x["m0"] = (rng.standard_normal((n, H, 128, 128)) * 0.1).astype(np.float32)
    x["d_mT"] = (rng.standard_normal((n, H, 128, 128)) * 0.1).astype(np.float32)
    t = dev(x)
    d_o, d_mT = torch.from_numpy(x["d_o"]).to(t["q"].device).to(torch.bfloat16), torch.from_numpy(x["d_mT"]).to(t["q"].device)
    cu_d = torch.from_numpy(cu).to(t["q"].device)
    pars = (t["log_alpha"], t["beta"], t["b"], t["m0"])
    o, mT = pkg.lsm_delta_fwd(t["q"], t["k"], t["v"], *pars, cu_seqlens=cu_d)
    r = pkg.lsm_delta_bwd(t["q"], t["k"], t["v"], d_o, *pars, d_mT, cu_seqlens=cu_d)
    torch.cuda.synchronize()
    for s_, (lo, hi) in enumerate(zip(cu[:-1], cu[1:])):
        if hi == lo:
            assert torch.equal(mT[s_], t["m0"][s_]) and torch.equal(r["d_init_state"][s_], d_mT[s_])
            continue
        cut = lambda a: None if a is None else np.ascontiguousarray(a[:, :, lo:hi])
        args = [cut(x[m]) for m in ("q", "k", "v")]
        par = [cut(x[m]) for m in ("log_alpha", "beta", "b")]
        o_ref, mT_ref = delta_oracle_fwd(*args, *par, x["m0"][s_:s_ + 1])
        ref = delta_oracle_bwd(*args, cut(x["d_o"]), *par, x["m0"][s_:s_ + 1], x["d_mT"][s_:s_ + 1])
        errs = dict(o=rel_err(host(o[:, :, lo:hi]), o_ref, BF16_HALF_ULP), final_state=rel_err(host(mT[s_:s_ + 1]), mT_ref),
                    d_init_state=rel_err(host(r["d_init_state"][s_:s_ + 1]), ref["d_m0"]))
        for m in ("dq", "dk", "dv", "d_log_alpha", "d_beta", "d_b"):
            if ref[m] is not None:
                errs[m] = rel_err(host(r[m][:, :, lo:hi]), ref[m], BF16_HALF_ULP if m in ("dq", "dk", "dv") else 0.0)
        print("packed, %d tokens: %s" % (hi - lo, " ".join("%s %.1e" % e for e in errs.items())), flush=True)
        assert max(errs.values()) <= TOL, errs


def test_delta_rejects_what_it_does_not_serve():
    import torch
    import paper_2503_05447_amd as pkg
    d = torch.device("cuda:0")
    q = torch.zeros(1, 1, 64, 64, device=d, dtype=torch.bfloat16)
    with pytest.raises(pkg.LsmError):
        pkg.lsm_delta_fwd(q, q, q)
    q32 = torch.zeros(1, 1, 64, 128, device=d, dtype=torch.float32)
    with pytest.raises(pkg.LsmError):
        pkg.lsm_delta_fwd(q32, q32, q32)
