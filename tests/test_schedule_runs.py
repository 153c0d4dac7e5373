"""Host logic: the queue of the tiled factorisation without L^-1 (chains of up to
six or beyond 24 tiles, and every chain of a multi-chain pass), as the device
takes it: by items, of one task or of several updates of one tile.

A block that claims an item waits for the inputs of all its updates at once, adds
them up, claims its next item and moves the tile's version on by their number.
Replayed here with random durations: every replay ends, every tile is written in
step order by one item at a time, and ends final."""
import heapq

import numpy as np
import pytest

from paper_1608_04329_amd import hsp
from test_schedule import GEMM, PANEL, POTRF, decode, expected_tasks, reads_ok, write

MOST = 16  # updates of one item


def schedule(nt, gp):
    """(block 0's chain, items of the others); with one block, its items alone."""
    tasks, off = hsp.hsp_tile_schedule(nt, gp, False)
    starts = hsp.hsp_tile_runs(nt, gp)
    dec = [decode(int(c)) for c in tasks]
    n0 = 0 if gp == 1 else int(off[1])
    if len(dec) == n0:  # one tile
        assert list(starts) == [n0]
        return dec, []
    assert starts[0] == n0 and starts[-1] == len(dec) and np.all(np.diff(starts.astype(np.int64)) >= 1)
    return dec[:n0], [dec[a:b] for a, b in zip(starts[:-1], starts[1:])]


def inputs_ready(item, vU, vL):
    if len(item) == 1:
        return reads_ok(item[0], vU, vL)
    k, i, j = item[0][2:]
    return vU[i, j] >= k and all(vU[t[2], i] >= t[2] + 1 and vU[t[2], j] >= t[2] + 1 for t in item)


def replay(chain, items, blocks, nt, rng):
    vU, vL = np.zeros((nt, nt), np.int64), np.zeros((nt, nt), np.int64)
    claimed = [0]

    def claim():
        claimed[0] += 1
        return claimed[0] - 1

    at = [0] + [claim() for _ in range(blocks - 1)] if chain else [claim()]
    busy, running, now = [False] * len(at), [], 0.0
    left = len(chain) + len(items)

    def item_of(b):
        own = [[t] for t in chain] if chain and b == 0 else items
        return own[at[b]] if at[b] < len(own) else None

    while left:
        for b in range(len(at)):
            it = item_of(b)
            if not busy[b] and it is not None and inputs_ready(it, vU, vL):
                heapq.heappush(running, (now + rng.uniform(0.3, 3.0) * (4.0 if it[0][0] in (POTRF, PANEL) else len(it)), b))
                busy[b] = True
        assert running, f"deadlock with {left} items left"
        now, b = heapq.heappop(running)
        for t in item_of(b):
            write(t, vU, vL)
        at[b] = at[b] + 1 if chain and b == 0 else claim()
        busy[b] = False
        left -= 1
    for i in range(nt):
        assert vL[i, i] == 1 and all(vU[i, j] == i + 1 for j in range(i, nt))


@pytest.mark.parametrize("nt,gp", [(1, 1), (2, 1), (2, 2), (3, 3), (5, 10), (6, 15), (6, 4), (16, 32), (16, 1), (25, 7),
                                   (33, 128), (40, 256), (70, 384)])
def test_items_cover_every_task_and_never_deadlock(nt, gp):
    chain, items = schedule(nt, gp)
    flat = chain + [t for it in items for t in it]
    assert len(flat) == len(set(flat)) and set(flat) == expected_tasks(nt, gp > 1, False)
    for it in items:
        assert len(it) <= MOST
        if len(it) > 1:
            k, i, j = it[0][2:]
            assert it == [(GEMM, 0, k + q, i, j) for q in range(len(it))]
            # the last update before the tile is taken up is an item of its own
            assert k + len(it) < i
    rng = np.random.default_rng(nt + gp)
    for _ in range(3 if nt < 30 else 1):
        replay(chain, items, gp, nt, rng)


def test_a_tile_is_summed_alike_whatever_the_group():
    for nt in (6, 25, 40):
        runs = [sorted((it[0][2:], len(it)) for it in schedule(nt, gp)[1] if it[0][0] == GEMM and it[0][3] != it[0][2] + 1)
                for gp in (2, 48, 300)]
        assert runs[0] == runs[1] == runs[2]


def test_lone_chains_carry_the_inverse_from_7_to_24_tiles():
    assert [nt for nt in range(1, 40) if hsp.hsp_lone_inverse(nt)] == list(range(7, 25))


def test_bad_arguments():
    for nt, gp in [(0, 4), (hsp.hsp_max_p() // 64 + 1, 4), (4, 0), (4, 5000)]:
        with pytest.raises(hsp.HspError):
            hsp.hsp_tile_runs(nt, gp)
