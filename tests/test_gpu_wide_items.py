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
