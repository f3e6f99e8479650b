"""Restore: is a page in an agent's list?  The lanes of a workgroup share out the agents of its group, so groups at both
sides of 4, 8, 16 and 32 agents take different numbers of lanes per list; lists from one page to more than lanes squared,
and all pages listed.  Every stage bit for bit against the oracle."""
import pytest

from paper_2604_03143_amd import workload as wl
from test_gpu_parity import run_pipeline

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group", [1, 4, 5, 8, 9, 16, 17, 32])
@pytest.mark.parametrize("pages,frac", [(7, 0.1), (90, 0.95), (301, 0.3), (66, 1.0)])
def test_lists_of_every_length(tdo, group, pages, frac):
    spec = wl.RoundSpec("lookup", 107, 1, 1, 128, 16, 1.0e6, 1, 33, 1, 16 * pages - 3, 3, 90, frac)
    run_pipeline(tdo, wl.make_round(spec), group=group)
