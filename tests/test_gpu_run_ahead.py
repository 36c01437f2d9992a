"""Steps enqueued ahead of the rebuild decision (one box) against steps that each carry the
rebuild chain (the same box inside an ensemble): bit for bit the same run."""
import numpy as np
import pytest

from paper_1210_3450_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def run(q, v, L, copies, steps, T, **kw):
    """State, series and builds of box 0 after the md_step calls `steps`."""
    from paper_1210_3450_amd import binding as B
    n = q.shape[0]
    every = kw.pop("every")
    p = [B.make_params(n, L, **kw) for _ in range(copies)]
    with B.Context(p if copies > 1 else p[0]) as c:
        c.set_state(np.tile(q, (copies, 1)), np.tile(v, (copies, 1)))
        if T:
            c.set_thermostat(T, 0.5)
        for k in steps:
            c.step(k, energy_every=every)
        x, w = c.get_state()
        ke, pe = c.energy_series()
        xi, _ = c.get_thermostat()
        st = c.stats()
        assert st["steps"] == sum(steps)
    return (x[:n].cpu().numpy(), w[:n].cpu().numpy(), ke[:, 0], pe[:, 0], xi[0]), st["rebuilds"] / copies


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("policy,T,every,hot", [
    (0, 0.0, 0, 1.0), (0, 0.0, 3, 1.0), (0, 1.1, 4, 1.0), (1, 0.0, 0, 1.0), (1, 1.1, 0, 1.0),
    (0, 0.0, 0, 6.0),   # a build at nearly every step: the steps enqueued ahead are left out each time
    (3, 0.0, 5, 0.2),   # never
])
def test_run_ahead_equals_the_full_sequence(precision, policy, T, every, hot):
    a = 2.0
    q = inputs.jittered(inputs.fcc_positions(7, a), 0.1, 7 * a, np.random.Generator(np.random.PCG64(31)))
    v = hot * inputs.maxwell_boltzmann(q.shape[0], 1.0, 1.0, np.random.Generator(np.random.PCG64(32)))
    kw = dict(precision=precision, rebuild=policy, every=every, dt=0.004 if hot > 1 else 0.005)
    steps = [1, 2, 37]
    one, builds1 = run(q, v, 7 * a, 1, steps, T, **kw)
    two, builds2 = run(q, v, 7 * a, 2, steps, T, **kw)
    assert builds1 == builds2
    for x, y in zip(one, two):
        np.testing.assert_array_equal(x, y)


def test_timing_counts_executed_passes_only():
    q = inputs.jittered(inputs.fcc_positions(7, 2.0), 0.1, 14.0, np.random.Generator(np.random.PCG64(33)))
    v = inputs.maxwell_boltzmann(q.shape[0], 1.0, 1.0, np.random.Generator(np.random.PCG64(34)))
    from paper_1210_3450_amd import binding as B
    with B.Context(B.make_params(q.shape[0], 14.0)) as c:
        c.set_state(q, v)
        c.compute_forces()
        c.set_timing(True)
        before = c.stats()["rebuilds"]
        c.step(40)
        st = c.stats()
    assert st["force_launches"] == 40
    assert st["rebuild_launches"] == st["rebuilds"] - before > 0
