"""The three step calls only enqueue kernels (no allocation, no synchronisation, no memset), so a
caller can capture a whole multi-layer step in a HIP graph.  Every replay must give the eager result."""
import numpy as np
import pytest

from paper_2604_03143_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("queues", [False, True])
def test_step_captured_in_a_graph_replays_exactly(tdo, queues):
    """queues: the write kernels in their looping form (work queues whose counters the kernels put back to zero
    themselves); otherwise static launches with a shared tail (one more such counter)."""
    import torch
    from paper_2604_03143_amd import tdk
    import gpu_helpers as gh
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    spec = wl.RoundSpec("graph", 58, 3, 8, 128, 16, 1.0e6, 2, 6, 3, 70, 5, 300, 0.2)
    rnd = wl.make_round(spec)
    L = spec.num_layers
    runs = [gh.GpuRun(rnd, layer=l) for l in range(L)]
    r = runs[0].r
    if queues:
        tdk.tdk_round_tune(r, 0, tdk.TUNE_DEFAULT | tdk.TUNE_QUEUES_ANY_SIZE)
    stored, fresh = [], []
    for l, g in enumerate(runs):                     # eager set-up: the mirrors each layer stores
        tdk.tdk_rerotate_round(r, l, g.io, g.stream)
        wl.perturb_device(rnd, l, g.pk, g.pv)
        stored.append(g.encode())
        fresh.append(g.new_diff())
    want = [(g.pk.clone(), g.pv.clone()) for g in runs]

    def step(stream):
        for l, g in enumerate(runs):
            tdk.tdk_rerotate_round(r, l, g.io, stream)
            tdk.tdk_diff_decode(r, l, g.io, stored[l].c, stream)
            tdk.tdk_diff_encode(r, l, g.io, spec.eps, fresh[l].c, stream)

    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        step(side.cuda_stream)                       # warm-up on the capture stream
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            step(torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    try:
        for rep in range(3):
            for l, g in enumerate(runs):             # eager work between replays: wipe what the step writes
                g.pk.zero_(); g.pv.zero_()
                fresh[l].idx.fill_(-1); fresh[l].payload.zero_(); fresh[l].count.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            mask = torch.from_numpy(wl.shared_row_mask(rnd)).cuda()
            for l, g in enumerate(runs):
                assert torch.equal(g.pk[mask], want[l][0][mask]) and torch.equal(g.pv[mask], want[l][1][mask]), (rep, l)
                n = int(stored[l].offset.cpu()[-1])
                assert torch.equal(fresh[l].count, stored[l].count) and torch.equal(fresh[l].offset, stored[l].offset)
                assert torch.equal(fresh[l].idx[:n], stored[l].idx[:n])
                assert torch.equal(fresh[l].payload[:n], stored[l].payload[:n])
    finally:
        torch.cuda.synchronize()
        for g in runs[1:]:
            g.r.destroy()
        runs[0].close()


@pytest.mark.parametrize("group", [2, 32])
@pytest.mark.parametrize("queues", [False, True])
def test_captured_step_replays_after_the_work_lists_were_replaced(tdo, queues, group):
    """A captured call names the places and lengths of the lists of its time: tuned to somewhat shorter and much shorter ones, the round
    must leave whole lists there."""
    import torch
    from paper_2604_03143_amd import tdk
    import gpu_helpers as gh
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    spec = wl.RoundSpec("graph3", 60, 1, 8, 128, 16, 1.0e6, 2, 5, 4, 70, 5, 300, 0.2)
    rnd = wl.make_round(spec)
    g = gh.GpuRun(rnd, flags=tdk.TUNE_DEFAULT | (tdk.TUNE_QUEUES_ANY_SIZE if queues else 0))
    try:
        assert tdk.tdk_round_agents_per_group(g.r) == 1
        g.rerotate()
        wl.perturb_device(rnd, 0, g.pk, g.pv)
        stored, fresh = g.encode(), g.new_diff()
        want_k, want_v = g.pk.clone(), g.pv.clone()
        side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
            st = torch.cuda.current_stream().cuda_stream
            tdk.tdk_rerotate_round(g.r, 0, g.io, st)
            tdk.tdk_diff_decode(g.r, 0, g.io, stored.c, st)
            tdk.tdk_diff_encode(g.r, 0, g.io, spec.eps, fresh.c, st)
        tdk.tdk_round_tune(g.r, group, tdk.TUNE_DEFAULT)
        mask = torch.from_numpy(wl.shared_row_mask(rnd)).cuda()
        n = int(stored.offset.cpu()[-1])
        for rep in range(3):
            for again in (False, True):              # replayed, then eagerly with the lists as they are now
                g.pk.zero_(); g.pv.zero_()
                fresh.idx.fill_(-1); fresh.payload.zero_(); fresh.count.zero_()
                torch.cuda.synchronize()
                if again:
                    g.rerotate()
                    g.decode(stored)
                    g.encode(d=fresh)
                else:
                    graph.replay()
                torch.cuda.synchronize()
                assert torch.equal(g.pk[mask], want_k[mask]) and torch.equal(g.pv[mask], want_v[mask]), (rep, again)
                assert torch.equal(fresh.count, stored.count) and torch.equal(fresh.offset, stored.offset), (rep, again)
                assert torch.equal(fresh.idx[:n], stored.idx[:n]) and torch.equal(fresh.payload[:n], stored.payload[:n]), (rep, again)
    finally:
        torch.cuda.synchronize()
        g.close()


def test_a_round_owns_what_its_lists_take():
    """100 agents x 25600 tokens in items of several agents: no room for items of one agent until they are asked for."""
    import torch
    from paper_2604_03143_amd import tdk
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    pages, agents = 1600, 100
    bt = np.arange(pages + 1, dtype=np.int32)
    r = tdk.tdk_round_create(tdk.model(1), [pages * 16], [0], [0] * agents, [0] * agents, [bt] * agents)
    try:
        before = tdk.tdk_scratch_bytes(r)
        assert tdk.tdk_round_agents_per_group(r) > 4 and before < 64 * pages * agents
        for group in (32, 1, 2, 0, 1):
            tdk.tdk_round_tune(r, group, tdk.TUNE_DEFAULT)
            assert tdk.tdk_scratch_bytes(r) == before + (0 if group == 32 else 4 * 48 * pages * agents)
            before = tdk.tdk_scratch_bytes(r) if group == 32 else before
    finally:
        r.destroy()


@pytest.mark.parametrize("n_q", [1, 7])
def test_attention_call_captured_in_a_graph_replays_exactly(tdo, n_q):
    """tdk_attend_shared only enqueues kernels too (one launch for both passes with one query token, the separate
    kernels with seven); every replay, with the workspace and the outputs wiped in between, gives the eager bits."""
    import torch
    from paper_2604_03143_amd import tdk
    import gpu_helpers as gh
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    spec = wl.RoundSpec("graph2", 59, 1, 4, 128, 16, 1.0e6, 2, 5, 4, 90, 3, 400, 0.25)
    rnd = wl.make_round(spec)
    g = gh.GpuRun(rnd, layer=0)
    try:
        g.rerotate()
        wl.perturb_device(rnd, 0, g.pk, g.pv)
        d = g.encode()
        Hq = 12
        gen = torch.Generator(device="cuda"); gen.manual_seed(5)
        q = torch.randn((rnd.n_agents, n_q, Hq, 128), generator=gen, device="cuda").to(torch.bfloat16).view(torch.int16)
        nbytes = tdk.tdk_attend_workspace_bytes(g.r, n_q, Hq)
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        out = torch.empty((rnd.n_agents, n_q, Hq, 128), dtype=torch.float32, device="cuda")
        lse = torch.empty((rnd.n_agents, n_q, Hq), dtype=torch.float32, device="cuda")
        a = tdk.attend_io(q, n_q, Hq, 0.09, out, lse, ws, nbytes)
        tdk.tdk_attend_shared(g.r, 0, g.io, d.c, a, g.stream)
        torch.cuda.synchronize()
        want_o, want_l = out.clone(), lse.clone()
        assert torch.isfinite(want_o).all() and torch.isfinite(want_l).all()
        side = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            tdk.tdk_attend_shared(g.r, 0, g.io, d.c, a, side.cuda_stream)
            side.synchronize()
            with torch.cuda.graph(graph, stream=side):
                tdk.tdk_attend_shared(g.r, 0, g.io, d.c, a, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        for rep in range(3):
            ws.fill_(0xFF); out.fill_(float("nan")); lse.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want_o) and torch.equal(lse, want_l), rep
    finally:
        torch.cuda.synchronize()
        g.close()
