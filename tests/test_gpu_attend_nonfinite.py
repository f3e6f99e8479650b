"""NaN and infinities in queries and in stored values: a row whose definition is NaN comes out NaN (output and log-sum-exp),
in every form of the attention call, and no other row is touched by it.  The oracle says which rows those are.  (Not
covered: infinite stored keys.  The oracle turns every key, by 0 too, and infinity times 0 makes all its scores NaN, while
keys that did not move are used as they are here.)"""
import numpy as np
import pytest

import attend_bounds as ab
from paper_2604_03143_amd import workload as wl
from helpers import OracleRun

pytestmark = pytest.mark.gpu

NAN, INF = np.uint16(0x7FC0), np.uint16(0x7F80)

# (sessions, agents, H, n_q, Hq, span, own block orders, stored elsewhere).  Packed rows with 16- and 32-row tiles for the
# listed pages, more lists than compute units (36 agents x 8 KV heads), a wavefront per agent in one chunk and in several; the same
# with own block orders; the pipelined pass (ten sessions), with diffs stored here and elsewhere.
FORMS = [(1, 3, 2, 1, 6, 150, 0, 0), (1, 3, 2, 6, 6, 150, 0, 0), (2, 18, 8, 1, 24, 600, 0, 0), (1, 3, 2, 17, 4, 60, 0, 0),
         (1, 2, 2, 17, 4, 2600, 0, 1), (1, 3, 2, 1, 6, 150, 40, 1), (1, 3, 2, 17, 4, 150, 40, 0), (1, 3, 2, 17, 4, 900, 100, 1),
         (10, 4, 8, 1, 24, 577, 0, 0), (10, 4, 8, 1, 24, 640, 0, 1)]


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("where", ["q nan", "q inf", "k nan", "k nan everywhere", "v nan", "v inf"])
def test_rows_with_nan_scores_are_nan(tdo, form, where):
    import torch
    from paper_2604_03143_amd import tdk
    import gpu_helpers as gh
    sessions, agents, H, n_q, Hq, span, block, moved = form
    blocks = span // block if block else 1
    spec = wl.RoundSpec("nonf", 111, 1, H, 128, 16, 1.0e6, sessions, agents, blocks, span // blocks, 300, 500,
                        1.0 if "everywhere" in where else 0.2)
    rnd = wl.make_round(spec)
    if block:
        rnd = wl.permute_blocks(rnd, seed_tag=3)
    o = OracleRun(tdo, rnd)
    o.rerotate(); o.perturb()
    d = o.encode()
    A, n = rnd.n_agents, int(d.offset[-1])
    g = np.random.default_rng([spec.stream, n_q, Hq, span])
    q = wl.f32_to_bf16_bits(g.standard_normal((A, n_q, Hq, 128)).astype(np.float32))
    hit = 1                                               # the agent that gets the values
    pay = d.payload.reshape(d.payload.shape[0], 2, 16, H, 128)
    lo, hi = int(d.offset[hit]), int(d.offset[hit] + d.count[hit])
    assert hi > lo
    value = NAN if "nan" in where else INF
    if where[0] == "q":
        q[hit, n_q - 1, 1, 7] = value
    elif "everywhere" in where:
        pay[lo:hi, 0, :, 0, 5] = value
    else:
        pay[(lo + hi) // 2, 0 if where[0] == "k" else 1, 3, 0, 5] = value
    seg_diff = [s[:, 1] - 30 * moved for s in rnd.segments] if block else None
    pos_diff = rnd.agent_pos0 - 30 * moved
    scale = 1.0 / np.sqrt(128.0)
    hr = tdo.HostRound(rnd, diff_pos0=pos_diff, segment_diff_pos=seg_diff)
    with np.errstate(all="ignore"):
        want_o, want_l, tol_o, tol_l = ab.expected_and_bounds(tdo, o.g, hr, o.mk, o.mv, d, q, n_q, Hq, scale)
    r = tdk.round_from_workload(rnd, diff_pos0=pos_diff, segment_diff_pos=seg_diff)
    try:
        mk, mv, dq = gh.up(o.mk), gh.up(o.mv), gh.up(q)
        cnt, off = torch.from_numpy(d.count).cuda(), torch.from_numpy(d.offset).cuda()
        idx, dpay = torch.from_numpy(d.idx[:n].copy()).cuda(), gh.up(d.payload[:n].copy())
        ovf = torch.zeros(1, dtype=torch.int32, device="cuda")
        nbytes = tdk.tdk_attend_workspace_bytes(r, n_q, Hq)
        ws = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
        out = torch.full((A, n_q, Hq, 128), 7.0, dtype=torch.float32, device="cuda")
        lse = torch.full((A, n_q, Hq), 7.0, dtype=torch.float32, device="cuda")
        tdk.tdk_attend_shared(r, 0, tdk.layer_io(mk, mv, None, None, 0), tdk.diff(cnt, off, idx, dpay, n, ovf),
                              tdk.attend_io(dq, n_q, Hq, scale, out, lse, ws, nbytes))
        torch.cuda.synchronize()
        got_o, got_l = out.cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)
    finally:
        r.destroy()
    assert np.isnan(want_o).any() or np.isinf(want_o).any()
    assert np.array_equal(np.isnan(got_l), np.isnan(want_l))
    assert np.array_equal(np.isnan(got_o), np.isnan(want_o))
    assert np.array_equal(np.isinf(got_o), np.isinf(want_o))
    fine = np.isfinite(want_o) & np.isfinite(tol_o)       # (a bound over infinite keys is infinite)
    assert fine.any() and np.all(np.abs(got_o - want_o)[fine] <= tol_o[fine])
