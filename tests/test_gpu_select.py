"""Selection and master choice of the check layer at the sizes where the kernel's passes end: spans around multiples of
its 1024 threads, past the 16384 keys it keeps in LDS, sessions without agents, and several calls on one round (the
per-session tickets must be back at zero)."""
import numpy as np
import pytest

from paper_2604_03143_amd import workload as wl
from test_gpu_check_layer import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("span,ratio", [(1, 1.0), (1023, 0.3), (1024, 0.05), (1025, 1.0), (2049, 0.5), (16384, 0.1), (16385, 0.7), (20011, 0.02)])
def test_spans_around_the_passes(tdo, span, ratio):
    spec = wl.RoundSpec("sel1", 87, 1, 1, 128, 16, 1.0e6, 1, 2, 1, span, 3, 60, 0.2)
    run_case(tdo, wl.make_round(spec), ratio, 0.0, noise_everywhere=0.02)


def test_few_distinct_scores_on_a_long_span(tdo):
    """Ties across the threads' token ranges and past the keys kept in LDS."""
    spec = wl.RoundSpec("sel2", 88, 1, 1, 128, 16, 1.0e6, 1, 2, 1, 17000, 3, 60, 0.0)
    def fill(o):
        o.rerotate()
        for i in range(o.rnd.n_agents):
            rows = o.rnd.dst_rows(i)
            o.pk[rows[::3], 5] = np.uint16(0x4000)
    run_case(tdo, wl.make_round(spec), 0.2, 0.0, fill=fill)


def test_sessions_without_agents(tdo):
    spec = wl.RoundSpec("sel3", 89, 1, 2, 128, 16, 1.0e6, 1, 2, 1, 100, 3, 60, 0.2)
    run_case(tdo, wl.make_round(spec, spans=[100, 40, 0, 70], agents=[2, 0, 0, 3]), 0.2, 0.0, noise_everywhere=0.02)
    run_case(tdo, wl.make_round(spec, spans=[100, 40], agents=[0, 0]), 0.2, 0.0)


def test_repeated_calls_on_one_round():
    import torch
    from paper_2604_03143_amd import tdk
    import gpu_helpers as gh
    spec = wl.RoundSpec("sel4", 90, 1, 2, 128, 16, 1.0e6, 3, 9, 2, 150, 3, 90, 0.2)
    rnd = wl.make_round(spec)
    pk, pv = wl.pool_host(rnd, 0)
    g = gh.GpuRun(rnd, pk=pk, pv=pv)
    try:
        A, k = rnd.n_agents, 75
        first = None
        for call in range(6):
            t = [torch.zeros(A * spec.span_tokens, dtype=torch.float32, device="cuda"), torch.full((A, k), -1, dtype=torch.int32, device="cuda"),
                 torch.zeros(A, dtype=torch.int32, device="cuda"), torch.zeros(A, dtype=torch.float32, device="cuda"),
                 torch.full((3,), -7, dtype=torch.int32, device="cuda")]
            # (every second call with a threshold that lets nothing through: the early way out)
            tdk.tdk_check_layer(g.r, 0, g.io, 0.25, 3.0e38 if call % 2 else 0.0, tdk.reuse_plan(t[0], t[1], k, *t[2:]), g.stream)
            torch.cuda.synchronize()
            if first is None:
                first = t
            assert torch.equal(t[0], first[0]) and torch.equal(t[3], first[3]) and torch.equal(t[4], first[4])
            assert (t[2] == 0).all() if call % 2 else torch.equal(t[1], first[1])
    finally:
        g.close()


@pytest.mark.parametrize("spans,ratio", [([255, 256], 0.3), ([257, 511], 1.0), ([512, 3], 0.05), ([513, 512], 0.4), ([130, 0], 0.2)])
def test_short_spans(tdo, spans, ratio):
    """The form with 4 wavefronts (no span above 512 tokens), at the edges of its passes and of its range."""
    spec = wl.RoundSpec("sel5", 93, 1, 2, 128, 16, 1.0e6, 2, 2, 1, max(spans), 3, 60, 0.2)
    run_case(tdo, wl.make_round(spec, spans=spans, agents=[2, 3]), ratio, 0.0, noise_everywhere=0.02)
    run_case(tdo, wl.make_round(spec, spans=spans, agents=[2, 3]), ratio, 3.0e38, noise_everywhere=0.02)
