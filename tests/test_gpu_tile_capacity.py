"""Row tiles up to the staging capacity: crowded cells either side of the FP64 capacity's line
(30 to a cell) and near both capacities against the oracle, beyond them the gather format, and a
rescaled box that crosses the line."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def liquid(cells, rc, spacing, seed):
    """A jittered lattice in a box of `cells` cells a little wider than rc + 0.3."""
    r = np.random.Generator(np.random.PCG64(seed))
    L = np.array([(rc + 0.32) * n for n in cells])
    m = np.floor(L / spacing).astype(int)
    g = np.stack(np.meshgrid(*[(np.arange(k) + 0.5) / k for k in m], indexing="ij"), -1).reshape(-1, 3) * L
    return np.mod(g + r.uniform(-0.08, 0.08, g.shape), L), L


# cells, cutoff, spacing: named by the particles to a cell
CASES = {"22": ((5, 6, 4), 2.8, 1.06, 81), "32": ((6, 5, 5), 3.2, 1.08, 82), "56": ((5, 5, 7), 3.65, 1.0, 83),
         "64": ((7, 5, 4), 4.0, 1.07, 84), "74": ((5, 4, 7), 4.2, 1.06, 86), "89": ((5, 4, 4), 4.5, 1.06, 85)}
# the fullest one-cell slice and its neighbours hold 898, 1300, 2160, 2304, 2873 and 3407
HOLD = {0: ("22", "32", "56", "64"), 1: ("22", "32", "56", "64", "74")}


def check(c, q, L, rc, precision, Fr, per, A, tiles):
    F = c.compute_forces().cpu().numpy()
    assert c.stats()["row_tiles"] == tiles
    kp, pl = c.get_neighbors()
    kpr, plr = oracle.neighbors(q, L, rc + 0.3)
    np.testing.assert_array_equal(kp.cpu().numpy(), kpr)
    np.testing.assert_array_equal(pl.cpu().numpy(), plr)
    tol = 1e-5 if precision == 1 else 1e-12
    assert (np.linalg.norm(F - Fr, axis=1) / np.maximum(A, 1.0)).max() <= tol
    _, pe = c.energy()
    assert abs(pe - per) <= tol * (abs(per) + A.sum() / 14.0)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", sorted(CASES))
def test_crowded_cells_equal_the_oracle(name, precision):
    from paper_1210_3450_amd import binding as B
    cells, rc, spacing, seed = CASES[name]
    q, L = liquid(cells, rc, spacing, seed)
    Fr, per, A = oracle.forces(q, L, rc, skin=0.3)
    with B.Context(B.make_params(q.shape[0], L, rc=rc, precision=precision, flags=B.MD_F_TILE_ON)) as c:
        c.set_state(q, np.zeros_like(q))
        check(c, q, L, rc, precision, Fr, per, A, 1 if name in HOLD[precision] else 0)


@pytest.mark.parametrize("precision", [0, 1])
def test_rescaled_across_the_line(precision):
    from paper_1210_3450_amd import binding as B
    cells, rc, spacing, seed = CASES["32"]
    q, L = liquid(cells, rc, spacing, seed)
    with B.Context(B.make_params(q.shape[0], L, rc=rc, precision=precision, flags=B.MD_F_TILE_ON)) as c:
        c.set_state(q, np.zeros_like(q))
        c.compute_forces()
        for a in (1.19, 1.0 / 1.19):
            c.rescale_box(a)
            q, L = q * a, L * a
            Fr, per, A = oracle.forces(q, L, rc, skin=0.3)
            check(c, q, L, rc, precision, Fr, per, A, 1)
