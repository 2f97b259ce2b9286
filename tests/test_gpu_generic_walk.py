"""The fp32 walkers (every shape outside the bf16 family) at the sizes where their segment plan and their 32-token steps
change: one step and its edges, one and several segments, segments of several units, packed batches whose boundary slots
are numbered across sequences.  Against the fp64 oracle with the tolerances of the other parity tests."""
import numpy as np
import pytest

import lsm_workloads as wl
from lsm_testlib import check, compare_case, host, to_device

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


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("chunk", [64, 128])
def test_packed_batch_with_shared_segments(kind, chunk):
    """Enough heads that a segment spans several units; empty sequences first, inside and last; sequences of one token."""
    import torch
    import paper_2503_05447_amd as pkg
    from oracle import lsm_oracle_bwd, lsm_oracle_fwd
    lens = [0, 1, 300, 64, 0, 129, 1, 700, 33, 0]
    T, H, n = sum(lens), 100, len(lens)
    x = wl.make_inputs(1, H, T, 64, 64, kind, dtype="f32", seed=2200 + kind, decay="weak")
    rng = np.random.default_rng(2201)
    x["m0"] = (rng.standard_normal((n, H, 64, 64)) * 0.1).astype(np.float32)
    x["d_mT"] = (rng.standard_normal((n, H, 64, 64)) * 0.1).astype(np.float32)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    t = to_device(x)
    cu_d = torch.from_numpy(cu).to(t["q"].device)
    o, mT = pkg.lsm_chunk_fwd(t["q"], t["k"], t["v"], t["g"], kind, chunk, t["m0"], cu_seqlens=cu_d)
    r = pkg.lsm_chunk_bwd(t["q"], t["k"], t["v"], t["g"], kind, t["d_o"], chunk, t["m0"], t["d_mT"], cu_seqlens=cu_d)
    torch.cuda.synchronize()
    per_tok = kind in (wl.KIND_SCALAR, wl.KIND_VECTOR)
    ref = {m: [] for m in ("o", "dq", "dk", "dv", "dg")}
    for s, (lo, hi) in enumerate(zip(cu[:-1], cu[1:])):
        m0, dm = x["m0"][s:s + 1], x["d_mT"][s:s + 1]
        if lo == hi:
            assert torch.equal(mT[s], t["m0"][s]) and torch.equal(r["d_init_state"][s], t["d_mT"][s])
            continue
        cut = lambda a: np.ascontiguousarray(a[:, :, lo:hi])
        g = cut(x["g"]) if per_tok else x["g"]
        o_s, mT_s = lsm_oracle_fwd(cut(x["q"]), cut(x["k"]), cut(x["v"]), g, kind, m0)
        r_s = lsm_oracle_bwd(cut(x["q"]), cut(x["k"]), cut(x["v"]), g, kind, cut(x["d_o"]), m0, dm)
        check("final_state", host(mT[s:s + 1]), mT_s, "f32")
        check("d_init_state", host(r["d_init_state"][s:s + 1]), r_s["d_m0"], "f32")
        ref["o"].append(o_s)
        for m in ("dq", "dk", "dv", "dg"):
            ref[m].append(r_s[m])
    check("o", host(o), np.concatenate(ref["o"], axis=2), "f32")
    for m in ("dq", "dk", "dv"):
        check(m, host(r[m]), np.concatenate(ref[m], axis=2), "f32")
    if per_tok:
        check("dg", host(r["dg"]), np.concatenate(ref["dg"], axis=2), "f32")
    elif kind == wl.KIND_HEAD:
        check("dg", host(r["dg"]), sum(ref["dg"]), "f32")
