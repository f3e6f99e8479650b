"""Few KV heads per device (1, 2, 4: several rows share a wavefront's accesses; 3: one row each), every page size, pair
style and layout, with spans whose last page ends at every place inside a shared group of rows: collect, store and restore
(paired and single planes) bit for bit, the check layer's scores within their bound."""
import pytest

from paper_2604_03143_amd import workload as wl
from test_gpu_check_layer import run_case
from test_gpu_parity import run_pipeline
from test_gpu_planes import test_single_plane_encode_decode as planes_case

pytestmark = pytest.mark.gpu


def _round(H, T, tail, permuted):
    spec = wl.RoundSpec("pack", 91, 2, H, 128, T, 1.0e6, 2, 3, 1, 3 * T + tail, 3, 90, 0.3)
    if permuted:
        spec = wl.RoundSpec("pack", 92, 2, H, 128, T, 1.0e6, 1, 4, 3, T + tail, 3, 90, 0.3)
    rnd = wl.make_round(spec)
    return wl.permute_blocks(rnd, seed_tag=7) if permuted else rnd


@pytest.mark.parametrize("T", [16, 32])
@pytest.mark.parametrize("H", [1, 2, 3, 4])
def test_every_tail_of_a_page(tdo, H, T):
    for tail in (1, 2, 3, 5, 7, 8, 9, 15) + ((17, 23, 31) if T == 32 else ()):
        run_pipeline(tdo, _round(H, T, tail, False), style=tail & 1)


@pytest.mark.parametrize("H,T,style", [(1, 16, 1), (1, 32, 0), (2, 16, 0), (2, 32, 1), (4, 16, 1), (4, 32, 0)])
def test_own_block_orders(tdo, H, T, style):
    for tail in (1, 6, 11):
        run_pipeline(tdo, _round(H, T, tail, True), style=style)


@pytest.mark.parametrize("H,T", [(1, 16), (1, 32), (2, 16), (2, 32), (4, 32)])
def test_launch_forms(tdo, H, T):
    """Work queues, a shared tail, plain stores, one agent per item."""
    for group, flags in ((1, 0), (2, 128 + 512), (0, 4095), (3, 1024 + 2048)):
        run_pipeline(tdo, _round(H, T, 5, False), group=group, flags=flags)


@pytest.mark.parametrize("T,style,H", [(16, 0, 1), (32, 1, 1), (16, 1, 2), (32, 0, 2), (32, 0, 4), (16, 0, 3)])
def test_single_planes(tdo, T, style, H):
    planes_case(tdo, T, style, H)


@pytest.mark.parametrize("H,T,style,permuted", [(1, 16, 0, False), (1, 32, 1, True), (2, 16, 1, True), (2, 32, 0, False),
                                                (4, 16, 0, True), (4, 32, 1, False)])
def test_check_layer_scores(tdo, H, T, style, permuted):
    for tail in (1, 9, 14):
        run_case(tdo, _round(H, T, tail, permuted), 0.3, 0.0, noise_everywhere=0.02, style=style)
