"""Index lists and payload in one launch (rounds of at most 16384 (agent, page) pairs) at the sizes where its count ends:
pairs around a thread's 16 to 64 flag bytes and around the limit (past it the two launches), more listed pages than
workgroups, more agents than threads, capacities below the lists, nothing listed, every page listed; also through the call
that keeps its flags in static memory, with stale bytes behind the round's own."""
import numpy as np
import pytest

from paper_2604_03143_amd import workload as wl
from helpers import OracleRun
from test_gpu_parity import run_pipeline

pytestmark = pytest.mark.gpu


def _encode_both(tdo, rnd, cap):
    import torch
    from paper_2604_03143_amd import tdk
    import gpu_helpers as gh
    o = OracleRun(tdo, rnd)
    o.rerotate(); o.perturb()
    od = tdo.diff_encode(o.g, o.hr, o.mk, o.mv, o.pk, o.pv, rnd.spec.eps, cap)
    g = gh.GpuRun(rnd, mk=o.mk, mv=o.mv, pk=o.pk, pv=o.pv)
    try:
        for call in (tdk.tdk_diff_encode, tdk.tdk_diff_encode_static):
            gd = gh.DevDiff(rnd.n_agents, cap, 2 * rnd.spec.page_tokens * rnd.spec.row_elems)
            call(g.r, 0, g.io, rnd.spec.eps, gd.c, g.stream)
            torch.cuda.synchronize()
            gh.assert_diff_equal(gd, od, rnd.n_agents)
    finally:
        g.close()
    return od


@pytest.mark.parametrize("agents,pages", [(1, 1), (1, 16), (1, 17), (3, 85), (5, 819), (2, 2048), (2, 2049), (300, 13), (1, 4097),
                                          (1, 12289), (1, 16384), (1, 16385)])
def test_pairs_around_the_count(tdo, agents, pages):
    spec = wl.RoundSpec("lst1", 93, 1, 1, 128, 16, 1.0e6, 1, agents, 1, 16 * pages - 5, 0, 40, 0.0)
    rnd = wl.make_round(spec, perturbed_per_agent=min(pages, max(1, 40 // agents + 1)))
    od = _encode_both(tdo, rnd, rnd.n_agents * pages)
    assert int(od.offset[-1]) == sum(len(p) for p in rnd.perturbed)


@pytest.mark.parametrize("frac", [0.0, 1.0])
def test_nothing_and_everything_listed(tdo, frac):
    """Everything: 3000 slots, more than the launch has workgroups."""
    spec = wl.RoundSpec("lst2", 94, 1, 1, 128, 16, 1.0e6, 3, 10, 1, 1600, 0, 200, frac)
    rnd = wl.make_round(spec)
    od = _encode_both(tdo, rnd, 3000)
    assert int(od.offset[-1]) == (3000 if frac else 0)


@pytest.mark.parametrize("cap", [0, 1, 7])
def test_capacity_below_the_lists(tdo, cap):
    import torch
    from paper_2604_03143_amd import tdk
    import gpu_helpers as gh
    spec = wl.RoundSpec("lst3", 95, 1, 2, 128, 16, 1.0e6, 2, 3, 2, 60, 0, 90, 0.5)
    rnd = wl.make_round(spec)
    o = OracleRun(tdo, rnd)
    o.rerotate(); o.perturb()
    full = tdo.diff_encode(o.g, o.hr, o.mk, o.mv, o.pk, o.pv, spec.eps, 100)
    n = int(full.offset[-1])
    assert n > 7
    g = gh.GpuRun(rnd, mk=o.mk, mv=o.mv, pk=o.pk, pv=o.pv)
    try:
        idx = torch.full((100,), -5, dtype=torch.int32, device="cuda")
        pay = torch.full((100, 2 * 16 * spec.row_elems), 77, dtype=torch.int16, device="cuda")
        cnt, off, ovf = (torch.full((8,), -1, dtype=t, device="cuda") for t in (torch.int32, torch.int64, torch.int32))
        tdk.tdk_diff_encode(g.r, 0, g.io, spec.eps, tdk.diff(cnt, off, idx, pay, cap, ovf), g.stream)
        torch.cuda.synchronize()
        assert np.array_equal(cnt.cpu().numpy()[:6], full.count) and np.array_equal(off.cpu().numpy()[:7], full.offset)
        assert int(ovf[0]) == 1
        assert np.array_equal(idx.cpu().numpy()[:cap], full.idx[:cap]) and (idx[cap:] == -5).all() and (pay[cap:] == 77).all()
        assert np.array_equal(gh.down16(pay)[:cap].ravel(), full.payload[:cap].ravel())
    finally:
        g.close()


def test_sessions_of_unequal_size_and_heads_that_do_not_divide(tdo):
    for H, T in ((3, 16), (5, 32), (7, 16)):
        spec = wl.RoundSpec("lst4", 96, 2, H, 128, T, 1.0e6, 1, 2, 1, 100, 3, 150, 0.3)
        run_pipeline(tdo, wl.make_round(spec, spans=[100, 1, 0, 333], agents=[2, 3, 2, 4]))


@pytest.mark.parametrize("H,T", [(8, 16), (8, 32), (7, 16), (6, 32), (5, 32), (4, 32), (3, 16)])
@pytest.mark.parametrize("agents,listed", [(1, 1), (3, 1), (7, 3), (40, 3)])
def test_few_slots_are_shared_out(tdo, H, T, agents, listed):
    """One to 120 listed pages, fewer than there are workgroups: a slot of two or three whole batches of accesses (8 heads and 16
    tokens, 4 to 6 and 32) is copied by up to two of them, one of four (8 and 32) by up to four, a smaller one (3 and 7 and 16) by one,
    when it is stored and when it is restored."""
    spec = wl.RoundSpec("lst5", 97, 1, H, 128, T, 1.0e6, 1, agents, 1, 4 * T + 3, 0, 40, 0.0)
    run_pipeline(tdo, wl.make_round(spec, perturbed_per_agent=listed))
