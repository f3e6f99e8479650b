"""Attention with a wavefront per 32 rows of an agent: lists that are empty, end inside a tile or are longer than 64 pages, spans
of less than one step, workgroups that hold one agent, two agents or idle wavefronts, a last wavefront with one to 32 rows
(results leave by way of LDS, whole rows at a time, eight rows per turn).  Bounds as in test_gpu_attend.py."""
import pytest

from paper_2604_03143_amd import workload as wl
from test_gpu_attend import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [16, 32])
@pytest.mark.parametrize("n_q", [33, 40, 71, 97, 130])
@pytest.mark.parametrize("span,frac", [(5, 1.0), (64, 1.0), (300, 0.0), (333, 0.06), (1500, 0.9)])
def test_lists_and_rows_of_every_length(tdo, T, n_q, span, frac):
    """One query head per KV head: 2, 3, 4 and 5 wavefronts per agent, five agents."""
    spec = wl.RoundSpec("lists1", 111, 1, 1, 128, T, 1.0e6, 1, 5, 1, span, 3, 200, frac)
    _case(tdo, spec, n_q, 1, perturb=frac > 0)


@pytest.mark.parametrize("span,n_q,Hq,H,frac", [(500, 1, 8, 2, 0.3), (900, 1, 8, 2, 0.9), (2600, 1, 20, 1, 0.5), (6000, 1, 4, 1, 0.7), (6000, 1, 4, 1, 0.0)])
def test_many_parts_are_merged(tdo, span, n_q, Hq, H, frac):
    """Spans cut into few and many chunks and lists into few and many pieces: 8 to 32 chunks and up to 47 pieces, so that the
    parts of a row fall into one or several groups of 64 and most slots between them do not exist."""
    spec = wl.RoundSpec("lists2", 112, 1, H, 128, 16, 1.0e6, 1, 3, 1, span, 3, 200, frac)
    _case(tdo, spec, n_q, Hq, perturb=frac > 0)
