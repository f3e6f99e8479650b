"""The attention kernel that gives every wavefront one agent's query rows (more than 32 rows per agent and KV head, per-agent block
orders, and calls with fewer rows that the planner gives it), at the sizes where its tiles end: rows around multiples of 32 and
of a workgroup's 128, spans around multiples of a 64-token step and of a chunk, lists around a 32-token tile.  Then the packed form
in the master's order, plain and with pipelined steps.  Which of them a round with few rows takes, and in which chunks, is pinned by
attend_plan_check.cpp.  Bounds as in test_gpu_attend.py."""
import numpy as np
import pytest

import attend_bounds as ab
from paper_2604_03143_amd import workload as wl
from helpers import OracleRun
from test_gpu_attend import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("span", [1, 63, 64, 65, 128, 129, 200])
@pytest.mark.parametrize("n_q", [33, 64, 65])
def test_rows_and_spans_around_a_tile(tdo, span, n_q):
    """One query head per KV head: 33, 64 and 65 rows per agent (two and three wavefronts), three agents, so that
    workgroups mix agents and the last one has idle wavefronts."""
    spec = wl.RoundSpec("rows1", 81, 1, 1, 128, 16, 1.0e6, 1, 3, 1, span, 3, 200, 0.3)
    _case(tdo, spec, n_q, 1)


@pytest.mark.parametrize("T,style,scale,grow", [(16, 0, -0.2, None), (32, 1, None, None), (16, 1, 1.0, (0, 16, 7, 250, 1)),
                                                (32, 0, None, (5, 0, 33, 64, 1))])
def test_page_sizes_styles_scales_and_moved_mirrors(tdo, T, style, scale, grow):
    spec = wl.RoundSpec("rows2", 82, 1, 2, 128, T, 5.0e5, 1, 5, 3, 111, 3, 300, 0.3)
    _case(tdo, spec, 9, 8, style=style, scale=scale, grow=grow)


@pytest.mark.parametrize("frac,spans", [(0.15, (10, 421)), (1.0, (6, 80))])
def test_span_cut_into_chunks(tdo, frac, spans):
    """Few agents on a large chip: the span is cut into several chunks, whose lists begin inside the agent's list."""
    spec = wl.RoundSpec("rows3", 83, 1, 2, 128, 16, 1.0e6, 1, 2, spans[0], spans[1], 3, 500, frac)
    _case(tdo, spec, 17, 4)


@pytest.mark.parametrize("n_q", [1, 6])
@pytest.mark.parametrize("grow", [None, (0, 16, 7, 250)])
def test_few_rows_with_stored_positions_moved(tdo, n_q, grow):
    """Identity layouts in the shared launch, in chunks of one step, also when the stored diffs have moved (3 and 18 rows per agent
    and KV head: 16-row and 32-row tiles for the listed pages)."""
    for style in (0, 1):
        spec = wl.RoundSpec("rows4", 84, 1, 2, 128, 16, 1.0e6, 1, 4, 3, 75, 3, 300, 0.4)
        _case(tdo, spec, n_q, 6, style=style, grow=grow)


@pytest.mark.parametrize("n_agents,H,n_q,Hq,T,moved,span", [(3, 1, 33, 1, 16, False, 397), (40, 8, 1, 16, 16, False, 5301), (40, 8, 1, 16, 16, True, 5301),
                                                            (40, 8, 1, 16, 16, True, 397), (40, 8, 3, 48, 32, True, 397), (5, 2, 12, 8, 32, True, 397)])
def test_borders_of_blocks_anywhere(tdo, n_agents, H, n_q, Hq, T, moved, span):
    """Agents whose segment borders differ from agent to agent (cuts at random tokens, the segments in random order): steps run
    over the borders, and the scores of the tokens behind one are taken again.  40 agents x 8 KV heads with few rows over
    5301 tokens take the packed form, the others one agent per wavefront."""
    import torch
    from paper_2604_03143_amd import tdk
    import gpu_helpers as gh
    spec = wl.RoundSpec("rows5", 85, 1, H, 128, T, 1.0e6, 1, n_agents, 1, span, 300, 700, 0.25)
    rnd = wl.make_round(spec, perturbed_per_agent=min(spec.span_pages, 12))
    g = np.random.default_rng([85, n_agents, T])
    rnd.segments = []
    for i in range(n_agents):
        cuts = np.unique(np.concatenate([[0], np.sort(g.choice(np.arange(1, span // T), 4, replace=False)) * T + int(g.integers(0, T))]))
        lens = np.diff(np.concatenate([cuts, [span]]))
        order = g.permutation(len(cuts))
        dst = np.empty(len(cuts), np.int64)
        dst[order] = int(rnd.agent_pos0[i]) + np.concatenate([[0], np.cumsum(lens[order])[:-1]])
        rnd.segments.append(np.stack([cuts, dst, lens], 1))
    o = OracleRun(tdo, rnd)
    o.rerotate(); o.perturb()
    d = o.encode()
    seg_diff = [sg[:, 1] - (37 + q) if moved else sg[:, 1] for q, sg in enumerate(rnd.segments)]
    q = wl.f32_to_bf16_bits(g.standard_normal((n_agents, n_q, Hq, 128)).astype(np.float32))
    scale = 1.0 / np.sqrt(128.0)
    hr = tdo.HostRound(rnd, diff_pos0=rnd.agent_pos0, segment_diff_pos=seg_diff)
    want_o, want_l, tol_o, tol_l = ab.expected_and_bounds(tdo, o.g, hr, o.mk, o.mv, d, q, n_q, Hq, scale)
    r = tdk.round_from_workload(rnd, diff_pos0=rnd.agent_pos0, segment_diff_pos=seg_diff)
    try:
        n = int(d.offset[-1])
        mk, mv = gh.up(o.mk), gh.up(o.mv)
        cnt, off = torch.from_numpy(d.count).cuda(), torch.from_numpy(d.offset).cuda()
        idx, pay = torch.from_numpy(d.idx[:n].copy()).cuda(), gh.up(d.payload[:n].copy())
        dd = tdk.diff(cnt, off, idx, pay, n, torch.zeros(1, dtype=torch.int32, device="cuda"))
        nbytes = tdk.tdk_attend_workspace_bytes(r, n_q, Hq)
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        ws.fill_(0xFF)
        out = torch.full((n_agents, n_q, Hq, 128), float("nan"), dtype=torch.float32, device="cuda")
        lse = torch.full((n_agents, n_q, Hq), float("nan"), dtype=torch.float32, device="cuda")
        tdk.tdk_attend_shared(r, 0, tdk.layer_io(mk, mv, None, None, 0), dd,
                              tdk.attend_io(gh.up(q), n_q, Hq, scale, out, lse, ws, nbytes))
        torch.cuda.synchronize()
        ab.assert_within(out.cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64),
                         want_o, want_l, tol_o, tol_l, what=(n_agents, H, n_q, Hq, T, moved, span))
    finally:
        r.destroy()


@pytest.mark.parametrize("n_q,Hq", [(1, 2), (40, 2)])
def test_empty_spans(tdo, n_q, Hq):
    """Rounds whose spans are all empty: out 0, log-sum-exp -inf, from stale memory."""
    import torch
    from paper_2604_03143_amd import tdk
    import gpu_helpers as gh
    spec = wl.RoundSpec("rows6", 86, 1, 2, 128, 16, 1.0e6, 1, 3, 1, 16, 3, 50, 0.2)
    rnd = wl.make_round(spec, spans=[0], agents=[3])
    r = tdk.round_from_workload(rnd)
    try:
        d = gh.DevDiff(3, 1, 2 * 16 * 256)
        d.count.zero_(); d.offset.zero_()
        q = torch.ones((3, n_q, Hq, 128), dtype=torch.bfloat16, device="cuda")
        out = torch.full((3, n_q, Hq, 128), float("nan"), dtype=torch.float32, device="cuda")
        lse = torch.full((3, n_q, Hq), float("nan"), dtype=torch.float32, device="cuda")
        nbytes = tdk.tdk_attend_workspace_bytes(r, n_q, Hq)
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        ws.fill_(0xFF)
        tdk.tdk_attend_shared(r, 0, tdk.layer_io(None, None, None, None, 0), d.c, tdk.attend_io(q, n_q, Hq, 0.1, out, lse, ws, nbytes))
        torch.cuda.synchronize()
        assert (out == 0).all() and torch.isneginf(lse).all()
    finally:
        r.destroy()


@pytest.mark.parametrize("T,style,span,scale,grow", [(16, 0, 63, None, False), (16, 1, 64, 1.0, True), (32, 0, 65, -0.2, False),
                                                     (16, 0, 193, None, True), (32, 1, 700, None, False)])
def test_packed_rows_of_many_lists(tdo, T, style, span, scale, grow):
    """36 agents x 8 KV heads (more lists than compute units) in two sessions, 3 rows per agent and KV head, with listed pages and
    ragged ends: spans of 63 to 65 tokens with a wavefront per agent, 193 and 700 in the packed form in chunks of one and two steps,
    too short for pipelined steps."""
    spec = wl.RoundSpec("rows7", 97, 1, 8, 128, T, 1.0e6, 2, 18, 1, span, 3, 200, 0.25)
    _case(tdo, spec, 1, 24, style=style, scale=scale, grow=np.arange(36) * 5 if grow else None)


# (sessions, agents, KV heads, rows per agent and KV head, span): chunks of 2, 3, 4, 6 and 7 steps, odd and even, the last chunk with a
# ragged step, with one token in it, or (389 tokens) the only one
@pytest.mark.parametrize("T,style,shape,scale,moved", [
    (16, 0, (1, 2, 1, 8, 1100), None, False), (32, 1, (1, 2, 1, 18, 1100), None, True), (16, 1, (10, 2, 2, 16, 900), -0.2, True),
    (32, 0, (1, 25, 1, 32, 900), None, False), (16, 0, (1, 25, 1, 32, 900), 1.0, True), (32, 0, (6, 2, 8, 16, 577), None, True),
    (16, 1, (6, 2, 8, 18, 577), None, False), (32, 1, (6, 2, 8, 18, 577), 1.0, True), (16, 0, (4, 18, 8, 2, 1100), None, True),
    (32, 0, (20, 2, 8, 1, 389), None, False)])
def test_packed_rows_in_chunks_of_several_steps(tdo, T, style, shape, scale, moved):
    """The plain packed form's loop over its steps: tiles replaced while others are read, page masks past the first step, ragged
    ends; 16- and 32-row tiles for the listed pages, stored here or elsewhere."""
    sessions, agents, H, rows, span = shape
    spec = wl.RoundSpec("rows11", 101, 1, H, 128, T, 1.0e6, sessions, agents, 1, span, 3, 200, 0.2)
    _case(tdo, spec, 1, rows * H, style=style, scale=scale, grow=np.arange(sessions * agents) * 5 if moved else None)


# (as above) the same with a wavefront per agent: one chunk of 1, 2, 3 and 4 steps, and several chunks
@pytest.mark.parametrize("T,style,shape,scale,moved", [
    (16, 0, (1, 2, 1, 5, 33), None, False), (32, 0, (20, 2, 8, 1, 65), None, True), (16, 1, (20, 2, 8, 1, 129), 1.0, False),
    (32, 1, (20, 3, 8, 1, 193), None, True), (16, 0, (20, 3, 8, 1, 450), None, True), (32, 0, (20, 3, 1, 1, 2000), None, False),
    (16, 1, (10, 3, 1, 16, 1500), -0.2, True), (32, 1, (1, 2, 8, 20, 2000), None, True)])
def test_few_rows_with_a_wavefront_per_agent(tdo, T, style, shape, scale, moved):
    """1 to 20 rows per agent and KV head: tiles that are mostly empty, one chunk written straight to the result, several merged."""
    sessions, agents, H, rows, span = shape
    spec = wl.RoundSpec("rows12", 102, 1, H, 128, T, 1.0e6, sessions, agents, 1, span, 3, 200, 0.2)
    _case(tdo, spec, 1, rows * H, style=style, scale=scale, grow=np.arange(sessions * agents) * 5 if moved else None)


def test_packed_rows_in_two_blocks_and_several_chunks(tdo):
    """18 rows per agent and KV head: two blocks of 128 rows, the second not full; a span of several chunks."""
    spec = wl.RoundSpec("rows8", 98, 1, 8, 128, 16, 1.0e6, 3, 12, 3, 500, 3, 200, 0.1)
    _case(tdo, spec, 9, 16)


@pytest.mark.parametrize("T,style,span,scale,grow", [(16, 0, 513, None, False), (16, 1, 575, 1.0, True), (32, 0, 577, -0.2, False),
                                                     (32, 1, 640, None, True)])
def test_pipelined_steps_around_their_ends(tdo, T, style, span, scale, grow):
    """Ten sessions of four agents x 8 KV heads, spans of 9 and 10 steps: the master pass with pipelined steps (the planner's
    own test pins that these rounds take it), at odd and even numbers of steps and ragged ends, with listed pages."""
    spec = wl.RoundSpec("rows9", 99, 1, 8, 128, T, 1.0e6, 10, 4, 1, span, 3, 200, 0.2)
    _case(tdo, spec, 1, 24, style=style, scale=scale, grow=np.arange(40) * 5 if grow else None)


def test_pipelined_steps_in_two_blocks_and_several_chunks(tdo):
    """16 rows per agent and KV head: two blocks of 128 rows, the second half full; spans of several chunks."""
    spec = wl.RoundSpec("rows10", 100, 1, 8, 128, 16, 1.0e6, 2, 12, 1, 5301, 3, 200, 0.05)
    _case(tdo, spec, 2, 64)
