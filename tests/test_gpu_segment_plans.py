"""The walkers at the sizes where their segment plans change.  fp32 walkers (every shape outside the bf16 family): one
32-token step and its edges, one and several segments, segments of several units.  Both families: packed batches, whose
boundary slots and workgroups are numbered across sequences.  Against the fp64 oracle, tolerances of the parity tests."""
import itertools

import numpy as np
import pytest

import lsm_workloads as wl
from lsm_testlib import check, compare_case, gpu_forward, host, to_device

pytestmark = pytest.mark.gpu

KINDS = [wl.KIND_NONE, wl.KIND_HEAD, wl.KIND_SCALAR, wl.KIND_VECTOR]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("T", [31, 32, 33, 63, 65, 97])
def test_step_and_unit_edges(kind, T):
    for dtype, dk, dv, chunk in (("f32", 64, 128, 64), ("bf16", 64, 64, 16), ("f32", 256, 64, 128), ("f32", 128, 256, 32)):
        x = wl.make_inputs(1, 2, T, dk, dv, kind, dtype=dtype, seed=2000 + T, decay="weak", init_state=True, d_final=True)
        compare_case(x, chunk)


# heads x units of 64 tokens against the plan's 1024 (64-wide values) or 512 workgroups
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("shape", [(1, 300, 300, 64, 64, 64), (2, 600, 70, 64, 64, 64), (1, 70, 1000, 64, 128, 128)])
def test_segments_of_several_units(kind, shape):
    B, H, T, dk, dv, chunk = shape
    x = wl.make_inputs(B, H, T, dk, dv, kind, dtype="f32", seed=2100 + T, decay="weak", init_state=True, d_final=True)
    compare_case(x, chunk)


# the bf16 family's scan over segments: batches of eight, and of 24 (more than 8 sequences in 32 segments), either direction
@pytest.mark.parametrize("kind", [wl.KIND_NONE, wl.KIND_HEAD, wl.KIND_SCALAR])
@pytest.mark.parametrize("H,T", [(9, 2048), (9, 2000), (8, 2048), (9, 1088)])
def test_scan_over_segments_in_batches(kind, H, T):
    x = wl.make_inputs(1, H, T, 128, 128, kind, seed=2600 + T, decay="weak", init_state=True, d_final=True)
    if kind == wl.KIND_HEAD:  # heads of one size, as in test_packed_batch_with_shared_segments
        x["g"] = -np.linspace(0.05, 0.2, H, dtype=np.float32)
    compare_case(x, 64)


@pytest.mark.parametrize("kind", [wl.KIND_SCALAR, wl.KIND_VECTOR])
@pytest.mark.parametrize("chunk", [16, 64])
def test_decay_gradient_error_does_not_grow_with_the_segment(kind, chunk):
    """Four sequences alone are cut into segments of one unit; 256 copies of them (1024 recurrences) into one segment each.
    Either way the decay gradient's sums run back over a chunk (at least 32 tokens), so its error against the oracle is the same but for
    the rounding of the states they start from: a few percent (1.3 allowed).  Sums over the whole segment of 2048 tokens are
    sqrt(2048 / 64) > 5 times as many roundings away."""
    import torch
    import paper_2503_05447_amd as pkg
    from oracle import lsm_oracle_bwd
    x = wl.make_inputs(1, 4, 2048, 64, 64, kind, dtype="f32", seed=2300 + kind, decay="weak", init_state=True, d_final=True)
    want = lsm_oracle_bwd(x["q"], x["k"], x["v"], x["g"], kind, x["d_o"], x["m0"], x["d_mT"])["dg"]
    t = to_device(x)
    err = []
    for copies in (1, 256):
        c = {n: a.repeat(copies, *[1] * (a.dim() - 1)) for n, a in t.items()}
        r = pkg.lsm_chunk_bwd(c["q"], c["k"], c["v"], c["g"], kind, c["d_o"], chunk, c["m0"], c["d_mT"])
        torch.cuda.synchronize()
        err.append(np.linalg.norm(host(r["dg"][-1:]) - want) / np.linalg.norm(want))
        del c, r
    print("dg 2-norm error: alone %.2e, one of 256 copies %.2e" % tuple(err))
    assert err[1] <= 1.3 * err[0]


@pytest.mark.parametrize("T", [32, 33, 64, 512])
@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 128), (256, 64)])
def test_vector_decay_sums_are_rounded_once(T, dk, dv):
    """What a state alone contributes is e^{sum of log-decays} times it: the sum's one rounding to fp32 is the only one of its size.
    The sums here are -64, -(64 + 2^-18) after the first 16 of 32 tokens from either end, and on, exactly representable, -(64 + 2^-17):
    a half sum kept in fp32 comes out 2^-17 = 7.6e-6 off, and with it o, dq and both states.  Bound: expf (1 ulp), the matrix
    products' and the state's roundings, together below 16 x 2^-24 = 9.5e-7."""
    import torch
    import paper_2503_05447_amd as pkg
    H = 2 if T < 512 else 64
    x = wl.make_inputs(1, H, T, dk, dv, wl.KIND_VECTOR, dtype="f32", seed=2800 + T, decay="zero", init_state=True, d_final=True)
    g = x["g"]
    g[:, :, 3:8] = -12.75
    g[:, :, 10] = -(0.25 + 2.0 ** -18)   # sum of the first 16: -(64 + 2^-18)
    if T > 16:
        g[:, :, 16] = -2.0 ** -18
    x["m0"] *= np.float32(2.0 ** 92)
    x["v"][:] = 0
    t = to_device(x)
    o, mT = gpu_forward(x, 64, t)
    dq = pkg.lsm_chunk_bwd(t["q"], t["k"], t["v"], t["g"], x["kind"], t["d_o"], 64, t["m0"], t["d_mT"])["dq"]
    w = np.exp(np.cumsum(g.astype(np.float64), axis=2))
    m0 = x["m0"].astype(np.float64)
    for name, got, want in (("o", host(o), (x["q"].astype(np.float64) * w) @ m0), ("final_state", host(mT), w[:, :, -1, :, None] * m0),
                            ("dq", host(dq), (x["d_o"].astype(np.float64) @ m0.swapaxes(2, 3)) * w)):
        got, want = got[:, :, 20:], want[:, :, 20:]
        if name == "final_state":
            err = np.abs(got / want - 1).max()
        else:
            err = np.linalg.norm(got - want) / np.linalg.norm(want)
        print(name, "%.2e" % err)
        assert err < 16 * 2.0 ** -24, name


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("case", [("f32", 64, 64, 64), ("f32", 128, 64, 64), ("f32", 64, 128, 16), ("bf16", 64, 64, 64), ("f32", 256, 64, 64)])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_non_finite_rows_do_not_reach_the_tokens_before_them(kind, case, value):
    """One element of one token's q, k, v or d_o that is not finite, in the middle of a 32-token step, its first or one of its last two
    tokens, alone in the last step: o and dq of earlier tokens and dk and dv of later ones do not depend on it and come out bit for bit
    as without it; the token's own result is not finite."""
    import torch
    import paper_2503_05447_amd as pkg
    dtype, dk, dv, chunk = case
    T, col = 97, 37
    x = wl.make_inputs(1, 2, T, dk, dv, kind, dtype=dtype, seed=2500, decay="weak", init_state=True, d_final=True)

    def run(t):
        o, _ = pkg.lsm_chunk_fwd(t["q"], t["k"], t["v"], t["g"], kind, chunk, t["m0"])
        r = pkg.lsm_chunk_bwd(t["q"], t["k"], t["v"], t["g"], kind, t["d_o"], chunk, t["m0"], t["d_mT"])
        return dict(r, o=o)
    clean = run(to_device(x))
    for name, s0 in itertools.product(("q", "k", "v", "d_o"), (45, 64, 94, 95, 96)):
        t = to_device(x)
        t[name][:, :, s0, col] = value
        got = run(t)
        for out, keep in (("o", slice(0, s0)), ("dq", slice(0, s0)), ("dk", slice(s0 + 1, T)), ("dv", slice(s0 + 1, T))):
            assert torch.equal(got[out][:, :, keep], clean[out][:, :, keep]), (name, out)
        own = {"q": "o", "k": "o", "v": "o", "d_o": "dq"}[name]
        assert not torch.isfinite(got[own][:, :, s0].float()).all(dim=-1).any(), name
        if name == "v":  # one value column of o
            other = [c for c in range(dv) if c != col]
            assert torch.equal(got["o"][..., other], clean["o"][..., other])
            assert not torch.isfinite(got["o"][:, :, s0:, col].float()).any()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T", [511, 512])
def test_final_state_is_rounded_once(T, d):
    """Under a strong decay the last token makes up nearly all of the final state: one product, rounded once when it is added
    (2-norm 2^-23 / sqrt(12) x 0.74 for mantissas spread evenly over their logarithm, 2.5e-8), last of the sum.  Anything that
    is added after it rounds a second time: sqrt(2) as much, 3.6e-8.  The bound lies between, ragged last step or not."""
    import torch
    from oracle import lsm_oracle_fwd
    x = wl.make_inputs(1, 16, T, d, d, wl.KIND_SCALAR, dtype="f32", seed=2400 + T + d, decay="strong4", init_state=True)
    mT = gpu_forward(x, 64)[1]
    torch.cuda.synchronize()
    want = lsm_oracle_fwd(x["q"], x["k"], x["v"], x["g"], x["kind"], x["m0"])[1]
    err = np.linalg.norm(host(mT) - want) / np.linalg.norm(want)
    print("final state 2-norm error %.2e" % err)
    assert err < 3.0e-8


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("case", [("f32", 100, 64, 64, 64, 1), ("f32", 100, 64, 64, 128, 1), ("bf16", 40, 128, 128, 64, 1),
                                  ("bf16", 40, 128, 256, 64, 1), ("bf16", 3, 128, 128, 64, 1), ("bf16", 4, 128, 128, 64, 10),
                                  ("bf16", 12, 128, 128, 64, 1), ("bf16", 2, 128, 128, 64, 0), ("bf16", 8, 128, 128, 64, 0),
                                  ("bf16", 60, 64, 64, 64, 1), ("f32", 40, 256, 64, 64, 1), ("f32", 20, 128, 256, 64, 1),
                                  ("f32", 20, 64, 128, 16, 1), ("bf16", 30, 64, 128, 128, 1), ("f32", 5, 64, 64, 64, 0)])
def test_packed_batch_with_shared_segments(kind, case):
    """Enough heads that a segment spans several chunks (the case of 3 heads: one chunk each; of 4 heads: several, and the
    reverse scan in segments of them); empty sequences first, inside and last; sequences of one token.  times = 0: the batch
    seven times over, more sequences than a wave has lanes."""
    import torch
    import paper_2503_05447_amd as pkg
    from oracle import lsm_oracle_bwd, lsm_oracle_fwd
    lens = [0, 1, 300, 64, 0, 129, 1, 700, 33, 0]
    dtype, H, dk, dv, chunk, times = case
    lens = [a if a == 1 else a * times for a in lens] if times else lens * 7
    T, n = sum(lens), len(lens)
    x = wl.make_inputs(1, H, T, dk, dv, kind, dtype=dtype, seed=2200 + kind, decay="weak")
    if dtype == "bf16" and kind == wl.KIND_HEAD:
        # bf16 rows of the state gradient put an error of 2^-9 / sqrt(3) = 1.1e-3 of the head's own size on dk and dv.  The
        # drawn decays range from weak to almost none and the heads differ tenfold in size, so the largest of 1.3e7
        # elements (5.5 sigma) of the largest head comes to 2e-2 of the size of all: decays of one size here.
        x["g"] = -np.linspace(0.05, 0.2, H, dtype=np.float32)
    rng = np.random.default_rng(2201)
    x["m0"] = (rng.standard_normal((n, H, dk, dv)) * 0.1).astype(np.float32)
    x["d_mT"] = (rng.standard_normal((n, H, dk, dv)) * 0.1).astype(np.float32)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    t = to_device(x)
    cu_d = torch.from_numpy(cu).to(t["q"].device)
    o, mT = pkg.lsm_chunk_fwd(t["q"], t["k"], t["v"], t["g"], kind, chunk, t["m0"], cu_seqlens=cu_d)
    r = pkg.lsm_chunk_bwd(t["q"], t["k"], t["v"], t["g"], kind, t["d_o"], chunk, t["m0"], t["d_mT"], cu_seqlens=cu_d)
    torch.cuda.synchronize()
    per_tok = kind in (wl.KIND_SCALAR, wl.KIND_VECTOR)
    ref = {m: [] for m in ("o", "dq", "dk", "dv", "dg", "dg_tok")}
    for s, (lo, hi) in enumerate(zip(cu[:-1], cu[1:])):
        m0, dm = x["m0"][s:s + 1], x["d_mT"][s:s + 1]
        if lo == hi:
            assert torch.equal(mT[s], t["m0"][s]) and torch.equal(r["d_init_state"][s], t["d_mT"][s])
            continue
        cut = lambda a: np.ascontiguousarray(a[:, :, lo:hi])
        g = cut(x["g"]) if per_tok else x["g"]
        o_s, mT_s = lsm_oracle_fwd(cut(x["q"]), cut(x["k"]), cut(x["v"]), g, kind, m0)
        r_s = lsm_oracle_bwd(cut(x["q"]), cut(x["k"]), cut(x["v"]), g, kind, cut(x["d_o"]), m0, dm)
        check("final_state", host(mT[s:s + 1]), mT_s, dtype)
        check("d_init_state", host(r["d_init_state"][s:s + 1]), r_s["d_m0"], dtype)
        ref["o"].append(o_s)
        if kind == wl.KIND_HEAD:   # the same recurrence with the head's decay per token
            gt = np.ascontiguousarray(np.broadcast_to(g[None, :, None], (1, H, hi - lo)).astype(np.float32))
            ref["dg_tok"].append(lsm_oracle_bwd(cut(x["q"]), cut(x["k"]), cut(x["v"]), gt, wl.KIND_SCALAR, cut(x["d_o"]), m0, dm)["dg"].ravel())
        for m in ("dq", "dk", "dv", "dg"):
            ref[m].append(r_s[m])
    check("o", host(o), np.concatenate(ref["o"], axis=2), dtype)
    for m in ("dq", "dk", "dv"):
        check(m, host(r[m]), np.concatenate(ref[m], axis=2), dtype)
    if per_tok:
        check("dg", host(r["dg"]), np.concatenate(ref["dg"], axis=2), dtype)
    elif kind == wl.KIND_HEAD:
        # one value per head, summed over all tokens: terms of either sign, each within the tolerance of its own size
        got, want = host(r["dg"]), sum(ref["dg"])
        tok = np.sqrt(np.mean(np.concatenate([np.atleast_1d(a) ** 2 for a in ref["dg_tok"]])))
        lim = {"f32": 1e-4, "bf16": 2e-2}[dtype] * np.maximum(np.abs(want), tok * np.sqrt(T))
        assert (np.abs(got - want) <= lim).all()


@pytest.mark.parametrize("lens", [[2050, 2046], [1, 4095], [63, 65, 6016]])
def test_packed_batch_of_few_long_sequences(lens):
    """Either side of 32 chunks a sequence, where segments of one chunk become segments of two: against one call per sequence."""
    import torch
    import paper_2503_05447_amd as pkg
    H, T, n = 4, sum(lens), len(lens)
    x = wl.make_inputs(1, H, T, 128, 128, wl.KIND_SCALAR, seed=3000 + n, decay="default", init_state=False)
    rng = np.random.default_rng(3001)
    x["m0"] = (rng.standard_normal((n, H, 128, 128)) * 0.1).astype(np.float32)
    x["d_mT"] = (rng.standard_normal((n, H, 128, 128)) * 0.1).astype(np.float32)
    t = to_device(x)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    kw = {"cu_seqlens": torch.from_numpy(cu).to(t["q"].device)}
    o, mT = pkg.lsm_chunk_fwd(t["q"], t["k"], t["v"], t["g"], wl.KIND_SCALAR, 64, t["m0"], **kw)
    r = pkg.lsm_chunk_bwd(t["q"], t["k"], t["v"], t["g"], wl.KIND_SCALAR, t["d_o"], 64, t["m0"], t["d_mT"], **kw)
    for s in range(n):
        c = {m: t[m][:, :, cu[s]:cu[s + 1]].contiguous() for m in ("q", "k", "v", "g", "d_o")}
        m0, dm = t["m0"][s:s + 1].contiguous(), t["d_mT"][s:s + 1].contiguous()
        o1, mT1 = pkg.lsm_chunk_fwd(c["q"], c["k"], c["v"], c["g"], wl.KIND_SCALAR, 64, m0)
        r1 = pkg.lsm_chunk_bwd(c["q"], c["k"], c["v"], c["g"], wl.KIND_SCALAR, c["d_o"], 64, m0, dm)
        check("o", host(o[:, :, cu[s]:cu[s + 1]]), host(o1), "bf16")
        check("final_state", host(mT[s:s + 1]), host(mT1), "bf16")
        for m in ("dq", "dk", "dv", "dg"):
            check(m, host(r[m][:, :, cu[s]:cu[s + 1]]), host(r1[m]), "bf16")
        check("d_init_state", host(r["d_init_state"][s:s + 1]), host(r1["d_init_state"]), "bf16")


@pytest.mark.parametrize("dtype,dk,dv", [("f32", 64, 64), ("f32", 128, 256), ("bf16", 64, 64), ("bf16", 128, 128), ("bf16", 128, 256)])
def test_head_decay_gradient_holds_every_sequence(dtype, dk, dv):
    """The per-head sum over a packed batch misses by less than a quarter of what one of its one-token sequences adds (rms over
    heads; the rounding of 105 bf16 tokens comes to a tenth of that), so none of them, and no boundary, is left out."""
    import torch
    import paper_2503_05447_amd as pkg
    from oracle import lsm_oracle_bwd
    lens, H = [0, 1, 70, 1, 33, 0], 8
    T, n = sum(lens), len(lens)
    x = wl.make_inputs(1, H, T, dk, dv, wl.KIND_HEAD, dtype=dtype, seed=2900, decay="weak")
    rng = np.random.default_rng(2901)
    x["m0"] = (rng.standard_normal((n, H, dk, dv)) * 0.1).astype(np.float32)
    x["d_mT"] = (rng.standard_normal((n, H, dk, dv)) * 0.1).astype(np.float32)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    t = to_device(x)
    got = host(pkg.lsm_chunk_bwd(t["q"], t["k"], t["v"], t["g"], wl.KIND_HEAD, t["d_o"], 64, t["m0"], t["d_mT"],
                                 cu_seqlens=torch.from_numpy(cu).to(t["q"].device))["dg"])
    part = []
    for s, (lo, hi) in enumerate(zip(cu[:-1], cu[1:])):
        if lo < hi:
            cut = lambda a: np.ascontiguousarray(a[:, :, lo:hi])
            part.append(lsm_oracle_bwd(cut(x["q"]), cut(x["k"]), cut(x["v"]), x["g"], wl.KIND_HEAD, cut(x["d_o"]),
                                       x["m0"][s:s + 1], x["d_mT"][s:s + 1])["dg"].ravel())
    err, one = np.abs(got - sum(part)).max(), min(np.sqrt(np.mean(part[i] ** 2)) for i in (0, 2))
    print("error %.2e, one token %.2e" % (err, one))
    assert err < 0.25 * one


@pytest.mark.parametrize("kind", [wl.KIND_NONE, wl.KIND_HEAD, wl.KIND_SCALAR])
@pytest.mark.parametrize("dtype,H,T,dk,dv", [("f32", 1, 1, 64, 64), ("f32", 2, 97, 64, 64), ("f32", 2, 35, 64, 64), ("bf16", 2, 99, 128, 64),
                                             ("f32", 257, 35, 128, 64), ("f32", 3, 65, 128, 64), ("f32", 2, 130, 64, 128),
                                             ("f32", 2, 95, 256, 64), ("f32", 257, 33, 64, 64), ("bf16", 2, 98, 64, 64),
                                             ("bf16", 257, 34, 64, 64), ("f32", 2, 66, 256, 128)])
def test_products_in_three_parts(kind, dtype, H, T, dk, dv):
    """Walks with helper waves (up to 256 workgroups of 64-wide values) and without, last steps of one, two and three tokens, every
    width: forward and backward against the oracle, and fp32 results to 2^-21 in the 2-norm: a handful of roundings of 2^-24 of
    sums whose terms cancel by a small factor."""
    from oracle import lsm_oracle_fwd
    x = wl.make_inputs(1, H, T, dk, dv, kind, dtype=dtype, seed=2600 + T, decay="weak", init_state=True, d_final=True)
    compare_case(x, 64)
    if dtype == "f32":
        o, mT = gpu_forward(x, 64)
        want = lsm_oracle_fwd(x["q"], x["k"], x["v"], x["g"], x["kind"], x["m0"])
        for name, got, ref in (("o", o, want[0]), ("final_state", mT, want[1])):
            err = np.linalg.norm(host(got) - ref) / np.linalg.norm(ref)
            assert err <= 2.0 ** -21, (name, err)


@pytest.mark.parametrize("name", ["q", "k", "v", "m0"])
def test_numbers_above_the_largest_bf16_one(name):
    """fp32 numbers that round to infinity in bf16 have finite results."""
    from oracle import lsm_oracle_fwd
    x = wl.make_inputs(1, 2, 70, 64, 64, wl.KIND_SCALAR, dtype="f32", seed=2700, decay="weak", init_state=True)
    for n in ("q", "k", "v", "m0"):
        x[n] *= np.float32(2.0 ** -4)
    x[name].reshape(-1)[64 * 40 + 5] = 3.4e38
    got = gpu_forward(x, 64)
    want = lsm_oracle_fwd(x["q"], x["k"], x["v"], x["g"], x["kind"], x["m0"])
    for a, b in zip(got, want):
        a = host(a)
        assert np.isfinite(a).all()
        rows = lambda t: t.reshape(-1, t.shape[-1])
        big = np.abs(rows(b)).max(axis=1, keepdims=True)
        assert (np.abs(rows(a) - rows(b)) <= 2.0 ** -18 * big).all()


def two_norm_error(got, want):
    return np.linalg.norm(host(got) - want) / np.linalg.norm(want)


@pytest.mark.parametrize("exponent", [-116, -124])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("name", ["q", "k", "v", "m0", "d_o"])
def test_numbers_below_the_smallest_bf16_parts(name, d, exponent):
    """A bf16 number ends at 2^-133, the three parts of an fp32 number of 2^-110 and less would be cut there.  One operand is scaled
    down, others up, so that all results are normal numbers; the bound is that of test_products_in_three_parts, and the family's
    1e-4 for the decay gradient, whose terms cancel."""
    import torch
    from oracle import lsm_oracle_bwd, lsm_oracle_fwd
    from lsm_testlib import gpu_backward
    x = wl.make_inputs(1, 2, 99, d, d, wl.KIND_SCALAR, dtype="f32", seed=2750 + d, decay="weak", init_state=True, init_std=8.0)
    small, up = 2.0 ** exponent, 2.0 ** 20
    scale = {"q": dict(q=small, v=up, m0=up, d_o=up), "k": dict(k=small, v=up, m0=small, d_o=up),
             "v": dict(v=small, k=up, m0=small * up, d_o=up), "m0": dict(m0=small, v=0.0, q=up, d_o=up),
             "d_o": dict(d_o=small, q=up, k=up, v=up, m0=up)}[name]
    for n, f in scale.items():
        x[n] = (x[n].astype(np.float64) * f).astype(np.float32)
    o, mT = gpu_forward(x, 64)
    r = gpu_backward(x, 64)
    torch.cuda.synchronize()
    o_ref, mT_ref = lsm_oracle_fwd(x["q"], x["k"], x["v"], x["g"], x["kind"], x["m0"])
    ref = lsm_oracle_bwd(x["q"], x["k"], x["v"], x["g"], x["kind"], x["d_o"], x["m0"], None)
    errs = {}
    for n, got, want in [("o", o, o_ref), ("final_state", mT, mT_ref), ("d_init_state", r["d_init_state"], ref["d_m0"])] + \
            [(n, r[n], ref[n]) for n in ("dq", "dk", "dv", "dg")]:
        if want.any():
            errs[n] = two_norm_error(got, want)
    print(" ".join("%s %.1e" % e for e in errs.items()))
    for n, e in errs.items():
        assert e <= (1e-4 if n == "dg" else 2.0 ** -21), (n, e)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("where", ["scores", "values", "state"])
def test_what_a_strong_decay_leaves_keeps_its_bits(where, dtype):
    """Only the first five tokens have values, and one token decays by e^-84 = 2^-121.2: what they leave is the whole result of the
    tokens after it.  scores: those of the pairs across it, values: their weighted rows that enter the state, state: the running
    state of the steps after.  The bound is that of test_products_in_three_parts (bf16 elements: of the state, which is fp32)."""
    from oracle import lsm_oracle_fwd
    T, cut = (32, 6) if where != "state" else (99, 40)
    x = wl.make_inputs(1, 2, T, 64, 64, wl.KIND_SCALAR, dtype=dtype, seed=2760, decay="zero")
    x["g"][:, :, cut] = -84.0
    x["v"][:, :, 5:] = 0
    for n, f in {"scores": dict(v=2.0 ** 20), "values": dict(k=2.0 ** 20), "state": dict(k=8.0, v=8.0, q=2.0 ** 20)}[where].items():
        x[n] *= np.float32(f)
    o, mT = gpu_forward(x, 64)
    o_ref, mT_ref = lsm_oracle_fwd(x["q"], x["k"], x["v"], x["g"], x["kind"], None)
    errs = [two_norm_error(mT, mT_ref)] + ([two_norm_error(o[:, :, cut:], o_ref[:, :, cut:])] if dtype == "f32" else [])
    print(where, " ".join("%.1e" % e for e in errs))
    assert max(errs) <= 2.0 ** -21


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64)])
@pytest.mark.parametrize("where", ["q", "v", "d_o", "scores", "state", "results"])
def test_numbers_that_outgrow_the_factor(where, dtype, d):
    """Operands from 2^104 and results from 2^80 on are infinite once they are 2^24 and 2^48 times as large: they are formed again from
    the numbers themselves (scores: from their bits).  Bounds: fp32 as in test_products_in_three_parts; bf16 results carry their own
    rounding, 2^-9 at most, and that of the scores of the adjoint."""
    import torch
    from lsm_testlib import gpu_backward, oracle_all
    x = wl.make_inputs(1, 2, 99, d, d, wl.KIND_SCALAR, dtype=dtype, seed=2770 + d, decay="weak", init_state=True)
    power = {"q": dict(q=106, k=-20, v=-20, m0=-40), "v": dict(v=106, k=-30, m0=76), "d_o": dict(d_o=106, q=-20, k=-20, v=-20),
             "scores": dict(q=55, k=55, v=-100, m0=-45), "state": dict(m0=110, q=-100), "results": dict(q=50, k=30, v=10, m0=40)}[where]
    for n, p in power.items():
        x[n] *= np.float32(2.0 ** p)
    o, mT = gpu_forward(x, 64)
    r = gpu_backward(x, 64)
    torch.cuda.synchronize()
    o_ref, mT_ref, ref = oracle_all(x)
    errs = {n: two_norm_error(got, want) for n, got, want in
            [("o", o, o_ref), ("final_state", mT, mT_ref), ("d_init_state", r["d_init_state"], ref["d_m0"])] +
            [(n, r[n], ref[n]) for n in ("dq", "dk", "dv", "dg")]}
    print(" ".join("%s %.1e" % e for e in errs.items()))
    for n, e in errs.items():
        assert e <= (1e-4 if n == "dg" else 2.0 ** -8 if dtype == "bf16" and n in ("o", "dq", "dk", "dv") else 2.0 ** -21), (n, e)


@pytest.mark.parametrize("kind", [wl.KIND_NONE, wl.KIND_SCALAR])
@pytest.mark.parametrize("dtype,dk,dv", [("f32", 64, 64), ("f32", 128, 64), ("f32", 64, 128), ("bf16", 64, 64), ("bf16", 128, 64)])
def test_helper_waves_leave_the_same_bits(dtype, dk, dv, kind):
    """20 units of 64 tokens and 16 heads: a packed call has more than 256 workgroups, whose 64-wide walks have no helper waves, each
    of the separate calls has fewer; the segments are of one unit in either, and so are all sums."""
    import torch
    import paper_2503_05447_amd as pkg
    lens, H = [300, 64, 129, 33, 257, 99, 1], 16
    T, n = sum(lens), len(lens)
    x = wl.make_inputs(1, H, T, dk, dv, kind, dtype=dtype, seed=2950, decay="weak")
    rng = np.random.default_rng(2951)
    x["m0"] = (rng.standard_normal((n, H, dk, dv)) * 0.1).astype(np.float32)
    x["d_mT"] = (rng.standard_normal((n, H, dk, dv)) * 0.1).astype(np.float32)
    t = to_device(x)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)

    def run(c, m0, dm, **kw):
        o, mT = pkg.lsm_chunk_fwd(c["q"], c["k"], c["v"], c["g"], kind, 64, m0, **kw)
        return dict(pkg.lsm_chunk_bwd(c["q"], c["k"], c["v"], c["g"], kind, c["d_o"], 64, m0, dm, **kw), o=o, final_state=mT)
    whole = run(t, t["m0"], t["d_mT"], cu_seqlens=torch.from_numpy(cu).to(t["q"].device))
    for s in range(n):
        part = {m: None if t[m] is None else t[m][:, :, cu[s]:cu[s + 1]].contiguous() for m in ("q", "k", "v", "g", "d_o")}
        alone = run(part, t["m0"][s:s + 1].contiguous(), t["d_mT"][s:s + 1].contiguous())
        for m, got in alone.items():
            if got is not None:
                want = whole[m][s:s + 1] if m in ("final_state", "d_init_state") else whole[m][:, :, cu[s]:cu[s + 1]]
                assert torch.equal(got, want), (m, s)


@pytest.mark.parametrize("dk,dv", [(64, 64), (64, 128), (256, 64)])
@pytest.mark.parametrize("T,power", [(1, {}), (2, {}), (34, {}), (99, {}), (99, dict(v=106, k=-30, m0=76)), (99, dict(d_o=106, q=-20, k=-20, v=-20)),
                                     (99, dict(m0=110, q=-100)), (99, dict(v=-112, m0=-116))])
def test_vector_decay_bf16_rows_as_they_came(T, power, dk, dv):
    """bf16 rows enter the gradient walkers' products unsplit, state and weighted rows in three parts of 2^24 times the number: one
    and two tokens (the last two of a step go apart), a ragged step, numbers that outgrow the factor and such as fall below the
    parts of a bf16 number.  Bounds: bf16 results one rounding (2^-9 at most) and the adjoint's, fp32 ones as in
    test_numbers_that_outgrow_the_factor."""
    import torch
    from lsm_testlib import gpu_backward, oracle_all
    x = wl.make_inputs(1, 2, T, dk, dv, wl.KIND_VECTOR, dtype="bf16", seed=2900 + T + dk, decay="weak", init_state=True, d_final=True)
    for n, p in power.items():
        x[n] *= np.float32(2.0 ** p)
    r = gpu_backward(x, 64)
    torch.cuda.synchronize()
    ref = oracle_all(x)[2]
    errs = {n: two_norm_error(r[m], ref[n]) for n, m in [("dq", "dq"), ("dk", "dk"), ("dv", "dv"), ("dg", "dg"), ("d_m0", "d_init_state")]}
    print(" ".join("%s %.1e" % e for e in errs.items()))
    for n, e in errs.items():
        assert e <= (1e-4 if n == "dg" else 2.0 ** -21 if n == "d_m0" else 2.0 ** -8), (n, e)
