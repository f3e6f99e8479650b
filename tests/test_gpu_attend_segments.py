"""Attention over rounds with per-agent segment lists, in the forms that block permutations do not produce: layouts of a
single segment, and segments that moved together or apart.  Bounds as in test_gpu_attend.py."""
import numpy as np
import pytest

import attend_bounds as ab
from paper_2604_03143_amd import workload as wl
from helpers import OracleRun

pytestmark = pytest.mark.gpu


def segment_case(tdo, spec, segments, diff_pos, n_q, Hq, style=0, scale=None, perturbed=None):
    """segments[i]: agent i's rows (first master token, position, tokens); diff_pos[i]: where each of them started when the
    mirrors were stored."""
    import torch
    from paper_2604_03143_amd import tdk
    import gpu_helpers as gh
    rnd = wl.make_round(spec, perturbed_per_agent=perturbed)
    rnd.segments = segments(rnd)
    o = OracleRun(tdo, rnd, style=style)
    o.rerotate(); o.perturb()
    d = o.encode()
    seg_diff = diff_pos(rnd)
    A, n = rnd.n_agents, int(d.offset[-1])
    assert n > 0
    g = np.random.default_rng([spec.stream, n_q, Hq])
    q = wl.f32_to_bf16_bits(g.standard_normal((A, n_q, Hq, 128)).astype(np.float32))
    scale = 1.0 / np.sqrt(128.0) if scale is None else scale
    hr = tdo.HostRound(rnd, diff_pos0=rnd.agent_pos0, segment_diff_pos=seg_diff)
    want_o, want_l, tol_o, tol_l = ab.expected_and_bounds(tdo, o.g, hr, o.mk, o.mv, d, q, n_q, Hq, scale)
    r = tdk.round_from_workload(rnd, style=style, diff_pos0=rnd.agent_pos0, segment_diff_pos=seg_diff)
    try:
        mk, mv, dq = gh.up(o.mk), gh.up(o.mv), gh.up(q)
        cnt, off = torch.from_numpy(d.count).cuda(), torch.from_numpy(d.offset).cuda()
        idx, pay = torch.from_numpy(d.idx[:n].copy()).cuda(), gh.up(d.payload[:n].copy())
        ovf = torch.zeros(1, dtype=torch.int32, device="cuda")
        nbytes = tdk.tdk_attend_workspace_bytes(r, n_q, Hq)
        ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
        out = torch.full((A, n_q, Hq, 128), float("nan"), dtype=torch.float32, device="cuda")
        lse = torch.full((A, n_q, Hq), float("nan"), dtype=torch.float32, device="cuda")
        tdk.tdk_attend_shared(r, 0, tdk.layer_io(mk, mv, None, None, 0), tdk.diff(cnt, off, idx, pay, n, ovf),
                              tdk.attend_io(dq, n_q, Hq, scale, out, lse, ws, nbytes))
        torch.cuda.synchronize()
        return ab.assert_within(out.cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64),
                                want_o, want_l, tol_o, tol_l, what=(spec.name, n_q, Hq, style))
    finally:
        r.destroy()


# rows per agent and KV head: 3 and 16 (16-row tiles for the listed pages), 18 and 40 (32-row tiles); the last round is
# large enough for the form that packs the rows of several agents
@pytest.mark.parametrize("n_agents,H,n_q,Hq,T,style,span", [(4, 2, 1, 6, 16, 0, 250), (5, 1, 4, 4, 32, 1, 97), (4, 2, 6, 6, 16, 1, 250),
                                                            (3, 2, 5, 16, 32, 0, 129), (40, 8, 1, 16, 16, 0, 5301)])
def test_one_segment_per_agent_stored_elsewhere(tdo, n_agents, H, n_q, Hq, T, style, span):
    """Every agent's layout is one segment, stored when it began 37 + 11 i tokens earlier (one agent's did not move): the
    listed pages meet rows turned back by that distance.  Scale 1: near one-hot weights, so that rows that are not turned
    move the results far outside the bound."""
    spec = wl.RoundSpec("one", 101, 1, H, 128, T, 1.0e6, 1, n_agents, 1, span, 600, 900, 0.3)
    segments = lambda rnd: [np.array([[0, int(p), span]], np.int64) for p in rnd.agent_pos0]
    moved = lambda rnd: [s[:, 1] - (0 if i == 1 else 37 + 11 * i) for i, s in enumerate(rnd.segments)]
    segment_case(tdo, spec, segments, moved, n_q, Hq, style=style, scale=1.0 if span < 1000 else None,
                 perturbed=min(spec.span_pages, 12))


def random_segments(rnd, span, T, g):
    """Six segments per agent, cut at random tokens, in random order."""
    out = []
    for p in rnd.agent_pos0:
        cuts = np.unique(np.concatenate([[0], np.sort(g.choice(np.arange(1, span // T), 5, replace=False)) * T + int(g.integers(0, T))]))
        lens = np.diff(np.concatenate([cuts, [span]]))
        order = g.permutation(len(cuts))
        dst = np.empty(len(cuts), np.int64)
        dst[order] = int(p) + np.concatenate([[0], np.cumsum(lens[order])[:-1]])
        out.append(np.stack([cuts, dst, lens], 1))
    return out


def moved_by(rnd, how):
    out = []
    for i, s in enumerate(rnd.segments):
        kind = {"together": 0, "apart": 1, "mixed": i % 3}[how]
        out.append(s[:, 1] - (23 * (i % 7 + 1) if kind == 0 else 11 + 17 * np.arange(len(s)) if kind == 1 else 0))
    return out


# a wavefront per agent: 3, 16, 20 and 40 rows per agent and KV head
@pytest.mark.parametrize("how", ["together", "apart", "mixed"])
@pytest.mark.parametrize("n_q,Hq,T,style", [(1, 6, 16, 0), (4, 8, 32, 1), (5, 8, 32, 0), (10, 8, 16, 1)])
def test_segments_moved_together_and_apart(tdo, how, n_q, Hq, T, style):
    """Lists that run over several segments of an agent.  Together: all of an agent's segments have moved by one distance (one
    turn serves the list); apart: by different ones, so a tile of the list meets rows turned for each; mixed: agents of both
    kinds and one that has not moved, in one round."""
    spec = wl.RoundSpec("seg2", 102, 1, 2, 128, T, 1.0e6, 1, 5, 1, 700, 900, 1200, 0.5)
    g = np.random.default_rng([102, T, n_q])
    segment_case(tdo, spec, lambda rnd: random_segments(rnd, 700, T, g), lambda rnd: moved_by(rnd, how), n_q, Hq, style=style, scale=1.0)


@pytest.mark.parametrize("how", ["apart", "mixed"])
def test_packed_rows_with_half_of_the_pages_listed(tdo, how):
    """The same with 40 agents x 8 KV heads and 3 rows per agent, a round that packs the rows of several agents: the lists go
    to the 16-row pass, with the rows turned for every segment."""
    spec = wl.RoundSpec("seg3", 103, 1, 8, 128, 16, 1.0e6, 1, 40, 1, 900, 900, 1200, 0.5)
    g = np.random.default_rng([103])
    segment_case(tdo, spec, lambda rnd: random_segments(rnd, 900, 16, g), lambda rnd: moved_by(rnd, how), 1, 24, scale=1.0)


@pytest.mark.parametrize("n_q,Hq,T,span,how", [(5, 8, 16, 1400, "together"), (10, 8, 16, 1337, "mixed"), (5, 8, 32, 2600, "apart")])
def test_more_segments_than_a_wavefront_has_lanes(tdo, n_q, Hq, T, span, how):
    """A border in every page, at a random token: up to five segments meet a 64-token step, an agent has more than 64 of them
    and, with nine pages in ten listed, a list of more than 64 pages."""
    spec = wl.RoundSpec("seg4", 104, 1, 2, 128, T, 1.0e6, 1, 3, 1, span, 900, 1200, 0.9)
    g = np.random.default_rng([104, T])

    def segments(rnd):
        out = []
        for p in rnd.agent_pos0:
            cuts = np.concatenate([[0], np.arange(1, span // T) * T + g.integers(0, T, span // T - 1)])
            lens = np.diff(np.concatenate([cuts, [span]]))
            order = g.permutation(len(cuts))
            dst = np.empty(len(cuts), np.int64)
            dst[order] = int(p) + np.concatenate([[0], np.cumsum(lens[order])[:-1]])
            out.append(np.stack([cuts, dst, lens], 1))
        return out

    segment_case(tdo, spec, segments, lambda rnd: [np.maximum(m, 0) for m in moved_by(rnd, how)], n_q, Hq, scale=1.0)
