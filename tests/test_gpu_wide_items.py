"""Launches with eight wavefronts per workgroup (two rows of every 16-token page each): on both sides of the lines that choose them."""
import pytest

from paper_2604_03143_amd import workload as wl

pytestmark = pytest.mark.gpu


# (agents, span): reads while every item has a compute unit (256) to itself; writes from 6 pairs per compute unit (1536) on with items
# of several agents.  16 x 96 pages = 1536 pairs; the last page with one row, fifteen and all sixteen
@pytest.mark.parametrize("agents,span,style", [(4, 33, 0), (6, 15 * 16 + 15, 1), (16, 95 * 16, 0), (16, 95 * 16 + 1, 1), (16, 96 * 16, 0), (20, 1555, 0)])
@pytest.mark.parametrize("heads", [8, 5])
def test_rounds_around_the_lines(tdo, agents, span, style, heads):
    from test_gpu_parity import run_pipeline
    spec = wl.RoundSpec("wide", 94, 1, heads, 128, 16, 1.0e6, 1, agents, 1, span, 3, 900, 0.1)
    run_pipeline(tdo, wl.make_round(spec), style=style)


def test_own_block_orders(tdo):
    from test_gpu_parity import run_pipeline
    spec = wl.RoundSpec("wide_perm", 95, 1, 8, 128, 16, 1.0e6, 1, 18, 20, 70, 3, 900, 0.1)
    run_pipeline(tdo, wl.permute_blocks(wl.make_round(spec), seed_tag=7))


@pytest.mark.parametrize("agents,span", [(4, 33), (5, 200)])
def test_check_layer(tdo, agents, span):
    from test_gpu_check_layer import run_case
    spec = wl.RoundSpec("wide_check", 96, 1, 8, 128, 16, 1.0e6, 1, agents, 1, span, 3, 900, 0.1)
    run_case(tdo, wl.make_round(spec), 0.15, 0.0, noise_everywhere=0.02)


def writes_are_wide(r, agents, span, T=16):
    """The launchers' line for the kernels that write, for one session of a model whose rows fill an access."""
    import torch
    from paper_2604_03143_amd import tdk
    cus, pages, group = torch.cuda.get_device_properties(0).multi_processor_count, -(-span // T), tdk.tdk_round_agents_per_group(r)
    pairs, items = agents * pages, pages * -(-agents // group)
    return T == 16 and 6 * cus <= pairs < 64 * cus and 2 * pairs >= 5 * items


@pytest.mark.parametrize("agents,span,wide", [(6, 15 * 16 + 15, False), (16, 95 * 16, False), (16, 95 * 16 + 1, True), (16, 96 * 16, True), (20, 1555, True)])
def test_the_rounds_above_are_on_their_sides(agents, span, wide):
    from paper_2604_03143_amd import tdk
    r = tdk.round_from_workload(wl.make_round(wl.RoundSpec("wide", 94, 1, 8, 128, 16, 1.0e6, 1, agents, 1, span, 3, 900, 0.1)))
    assert writes_are_wide(r, agents, span) == wide
    r.destroy()


@pytest.mark.parametrize("blocks,block_tokens", [(1, 95 * 16 + 1), (20, 77)])
@pytest.mark.parametrize("style", [0, 1])
@pytest.mark.parametrize("heads", [8, 5])
def test_moved_mirrors_ride_in_a_wide_restore(tdo, heads, style, blocks, block_tokens):
    """Eight wavefronts turn the K rows of the listed pages, two rows each at a time: mirrors stored at other positions, as a whole and, with own
    block orders that change, by segments that moved apart."""
    import numpy as np
    import torch
    import gpu_helpers as gh
    from helpers import OracleRun
    from paper_2604_03143_amd import tdk
    agents, span = 16, blocks * block_tokens
    spec = wl.RoundSpec("wide_moved", 97, 1, heads, 128, 16, 1.0e6, 1, agents, blocks, block_tokens, 3, 900, 0.1)
    order = (lambda rnd, tag: wl.permute_blocks(rnd, seed_tag=tag)) if blocks > 1 else (lambda rnd, tag: rnd)
    old = order(wl.make_round(spec), 4)
    o = OracleRun(tdo, old, style=style)
    o.rerotate(); o.perturb()
    d = o.encode()
    grow = np.array([0, 16, 7, 250, 1, 31, 1000, 64] * 2, np.int64)
    new = order(wl.make_round(spec, hist=old.agent_pos0 + grow), 9)
    where = dict(diff_pos0=old.agent_pos0, segment_diff_pos=[sg[:, 1] for sg in old.segments] if blocks > 1 else None)
    opk, opv = wl.pool_host(new, 0)
    tdo.diff_decode(o.g, tdo.HostRound(new, **where), o.mk, o.mv, opk, opv, d)
    n = int(d.offset[-1])
    g = gh.GpuRun(new, style=style, mk=o.mk, mv=o.mv)
    g.r.destroy()
    g.r = tdk.round_from_workload(new, style=style, **where)
    try:
        assert n > 100 and writes_are_wide(g.r, agents, span)
        cnt, off, idx, pay = (gh.up(a) for a in (d.count, d.offset, d.idx[:n], d.payload[:n]))
        overflow = torch.zeros(1, dtype=torch.int32, device="cuda")
        dd = tdk.diff(cnt, off, idx, pay, n, overflow)
        tdk.tdk_diff_decode(g.r, 0, g.io, dd, g.stream)
        gk, gv = g.pool()
        assert np.array_equal(gk, opk) and np.array_equal(gv, opv)
    finally:
        g.close()
