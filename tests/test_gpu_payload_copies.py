"""Payload copies of the restore in their two load policies: ordinary reads, and streamed reads where payload and masters
exceed 80 MB.  The round is larger than that, so the policy is the streamed one; with the streaming of the copies switched
off it is the ordinary one.  The pools must be the same, bit for bit, and hold the payload
in the listed rows."""
import numpy as np
import pytest

from paper_2604_03143_amd import tdk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,moved", [(16, 0), (32, 5)])
def test_streamed_and_ordinary_reads(T, moved):
    import torch
    H, D, span, agents, listed = 8, 128, 60003, 3, 5000 // T
    g = np.random.default_rng([7, T])
    pos0 = g.integers(40, 400, size=agents)
    first = pos0 // T
    touch = (pos0 + span - 1) // T - first + 1
    perm = g.permutation(int(touch.sum()) + 1).astype(np.int32)
    tables, at = [], 1
    for i in range(agents):
        bt = np.full(int(first[i] + touch[i]), perm[0], np.int32)
        bt[first[i]:] = perm[at:at + touch[i]]
        at += int(touch[i])
        tables.append(bt)
    pages = -(-span // T)
    lists = [np.sort(g.choice(pages, size=listed, replace=False)).astype(np.int32) for _ in range(agents)]
    assert (span * 2 + agents * listed * T * 2) * H * D * 2 > 80 << 20
    r = tdk.tdk_round_create(tdk.model(1, H, D, T, 1.0e6, tdk.ROPE_HALF), [span], [0], [0] * agents, pos0, tables, pos0 - moved, None, None)
    try:
        bits = lambda *shape: torch.randint(0, 0x7000, shape, dtype=torch.int16, device="cuda")
        mk, mv = bits(span, H, D), bits(span, H, D)
        pay = bits(agents * listed, 2, T, H, D)
        cnt = torch.full((agents,), listed, dtype=torch.int32, device="cuda")
        off = torch.arange(agents + 1, dtype=torch.int64, device="cuda") * listed
        idx = torch.from_numpy(np.concatenate(lists)).cuda()
        d = tdk.diff(cnt, off, idx, pay, agents * listed, torch.zeros(1, dtype=torch.int32, device="cuda"))
        pools = []
        for flags in (tdk.TUNE_DEFAULT, tdk.TUNE_DEFAULT & ~8):
            tdk.tdk_round_tune(r, 0, flags)
            pk, pv = (torch.zeros((len(perm) * T, H, D), dtype=torch.int16, device="cuda") for _ in range(2))
            tdk.tdk_diff_decode(r, 0, tdk.layer_io(mk, mv, pk, pv, len(perm)), d, torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            pools.append((pk, pv))
        assert torch.equal(pools[0][0], pools[1][0]) and torch.equal(pools[0][1], pools[1][1])
        for i in range(agents):
            m = (lists[i].astype(np.int64)[:, None] * T + np.arange(T)).reshape(-1)
            pos = m + int(pos0[i])
            ok = m < span
            rows = torch.from_numpy(np.where(ok, tables[i][np.where(ok, pos, pos0[i]) // T].astype(np.int64) * T + pos % T, 0)).cuda()
            ok = torch.from_numpy(ok).cuda()
            want = pay[i * listed:(i + 1) * listed]
            assert torch.equal(pools[0][1][rows][ok], want[:, 1].reshape(-1, H, D)[ok])
            if not moved:
                assert torch.equal(pools[0][0][rows][ok], want[:, 0].reshape(-1, H, D)[ok])
    finally:
        r.destroy()
