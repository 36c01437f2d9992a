"""Thermostat steps with kinetic-energy partials alone (no sample recorded) against steps
that leave all partials (a sample each): the same run."""
import numpy as np
import pytest

from paper_1210_3450_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("copies,tpk,flags", [
    (1, 1, 8), (1, 4, 8), (1, 1, 4), (1, 1, 32),   # gathers, row tiles, half lists
    (2, 2, 8), (2, 1, 4),                          # ensembles: every step with the rebuild chain
])
def test_steps_without_a_sample_follow_the_same_run(precision, copies, tpk, flags):
    from paper_1210_3450_amd import binding as B
    L = 7 * 1.75
    q = inputs.jittered(inputs.fcc_positions(7, 1.75), 0.1, L, np.random.Generator(np.random.PCG64(41)))
    v = inputs.maxwell_boltzmann(q.shape[0], 1.0, 1.0, np.random.Generator(np.random.PCG64(42)))
    out = []
    for every in (0, 1):
        p = [B.make_params(q.shape[0], L, precision=precision, threads_per_key=tpk, flags=flags)] * copies
        with B.Context(p if copies > 1 else p[0]) as c:
            c.set_state(np.tile(q, (copies, 1)), np.tile(v, (copies, 1)))
            c.set_thermostat(1.3, 0.3)
            c.step(12, energy_every=every)
            x, w = c.get_state()
            xi, eta = c.get_thermostat()
            ke, pe = c.batch_energy()
            out.append([x.cpu().numpy(), w.cpu().numpy(), xi, eta, ke / q.shape[0], pe / q.shape[0], c.pressure()])
            assert c.energy_series()[0].shape[0] == (12 if every else 0)
    # the two passes differ at most by the rounding of a force sum: FP64 some 1e-14 of forces
    # below 1e3, FP32 some 1e-7 of sums below 1e2; times dt and 12 steps
    tol = 2e-6 if precision == 1 else 1e-11
    for a, b in zip(*out):
        d = np.abs(a - b)
        if a.shape == q.shape or a.shape == (copies * q.shape[0], 3):
            d = np.minimum(d, np.abs(L - d))
        assert d.max() <= tol * max(1.0, np.abs(a).max())
