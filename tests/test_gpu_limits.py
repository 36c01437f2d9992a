"""Rules of the step and analysis kernels at their limits: the one-block sort at its most slots and
cells and just past them, bubble grids of more segments than a block has threads, and steps
enqueued ahead over a chunk's end, on row tiles and on boxes that go one step ahead."""
import numpy as np
import pytest

import oracle
from paper_1210_3450_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


@pytest.mark.parametrize("n,cells", [
    (16384, (20, 20, 20)), (16383, (20, 20, 20)), (16385, (20, 20, 20)),   # 16,384 slots, and 16,448
    (9000, (24, 32, 16)), (9000, (23, 89, 6)), (9000, (24, 32, 17)),       # 12,288 cells, 12,282, 13,056
    (16384, (24, 32, 16)),
])
def test_one_block_sort_at_its_limits(n, cells):
    from paper_1210_3450_amd import binding as B
    L = np.array([2.81 * k for k in cells])
    q = rng(91).uniform(0.0, 1.0, (n, 3)) * L
    q[:50] -= L  # wrapped on binning
    with B.Context(B.make_params(n, L)) as c:
        c.set_state(q, np.zeros_like(q))
        c.build_cells()
        cell, nc = c.get_cells()
        assert tuple(nc) == cells
        w = np.mod(q, L)
        k = np.minimum((w * (np.array(cells) / L)).astype(int), np.array(cells) - 1)
        np.testing.assert_array_equal(cell.cpu().numpy(), (k[:, 2] * cells[1] + k[:, 1]) * cells[0] + k[:, 0])
        c.build_neighbors()
        kp, pl = c.get_neighbors()
    kpr, plr = oracle.neighbors(w, L, 2.8)
    np.testing.assert_array_equal(kp.cpu().numpy(), kpr)
    np.testing.assert_array_equal(pl.cpu().numpy(), plr)


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("shape", [(80, 82, 80), (101, 100, 103)])   # 257 and 508 segments
def test_bubble_grids_of_many_segments(shape, noalloc):
    from paper_1210_3450_amd import binding as B
    L = np.array([3.0 * k + 0.5 for k in shape[::-1]])
    gas, counts = inputs.bubble_field(shape, 0.29, 92, border=False)
    q = inputs.subcell_field_positions(counts, L, 92)
    with B.Context(B.make_params(q.shape[0], L)) as c:
        c.set_state(q, np.zeros_like(q))
        got = c.bubbles(noalloc=noalloc)
    ref = oracle.bubbles(q, L)
    assert got["nbubbles"] == len(ref.roots) > 1000
    np.testing.assert_array_equal(got["labels"].cpu().numpy().ravel(), np.asarray(ref.labels).ravel())
    np.testing.assert_array_equal(got["roots"], ref.roots)
    np.testing.assert_array_equal(got["sizes"], ref.sizes)


def run(q, v, L, copies, calls, every, T, **kw):
    """State, series and builds of box 0 after the md_step calls."""
    from paper_1210_3450_amd import binding as B
    n = q.shape[0]
    p = [B.make_params(n, L, **kw) for _ in range(copies)]
    with B.Context(p if copies > 1 else p[0]) as c:
        c.set_state(np.tile(q, (copies, 1)), np.tile(v, (copies, 1)))
        if T:
            c.set_thermostat(T, 0.5)
        for k in calls:
            c.step(k, energy_every=every)
        x, w = c.get_state()
        ke, pe = c.energy_series()
        st = c.stats()
        assert st["steps"] == sum(calls)
    return (x[:n].cpu().numpy(), w[:n].cpu().numpy(), ke[:, 0], pe[:, 0]), (st["rebuilds"] / copies, st["row_tiles"])


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("m,tiles,calls,every,hot,T", [
    (7, True, [3, 421, 1], 7, 1.0, 0.0),     # two chunk ends in one call, on row tiles
    (7, True, [40], 0, 6.0, 0.0),            # a build at nearly every step: steps left out
    (7, True, [230], 5, 1.0, 1.1),
    (7, False, [405], 9, 1.0, 0.0),
    (41, True, [12], 4, 5.0, 0.0),           # 275,684 particles: one step ahead
    (41, False, [12], 0, 5.0, 0.0),
    (41, True, [12], 0, 3.0, 1.1),
])
def test_run_ahead_equals_the_full_sequence(precision, m, tiles, calls, every, hot, T):
    from paper_1210_3450_amd import binding as B
    a = 2.0
    q = inputs.jittered(inputs.fcc_positions(m, a), 0.1, m * a, rng(93))
    v = hot * inputs.maxwell_boltzmann(q.shape[0], 1.0, 1.0, rng(94))
    kw = dict(precision=precision, dt=0.004, threads_per_key=1, flags=B.MD_F_TILE_ON if tiles else B.MD_F_TILE_OFF)
    one, s1 = run(q, v, m * a, 1, calls, every, T, **kw)
    two, s2 = run(q, v, m * a, 2, calls, every, T, **kw)
    assert s1 == s2 and s1[1] == (1 if tiles else 0) and s1[0] > 2
    for x, y in zip(one, two):
        np.testing.assert_array_equal(x, y)
