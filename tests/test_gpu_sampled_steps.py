"""Samples inside a run, whose step opens the next one in the same pass, against samples at the
end of a call, whose pass stores the forces: the same run and the same energies."""
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
@pytest.mark.parametrize("copies,tpk,flags,policy", [
    (1, 1, 8, 0), (1, 4, 8, 1), (1, 1, 4, 0), (1, 1, 4, 1),   # gathers, row tiles, both rebuild rules
    (1, 1, 32, 0),                                            # half lists: passes of their own
    (2, 2, 8, 0), (2, 1, 4, 0), (1, 2, 10, 2),                # the full sequence; graphs between samples
])
def test_samples_inside_a_run_equal_samples_at_its_end(precision, copies, tpk, flags, policy):
    from paper_1210_3450_amd import binding as B
    L = 7 * 1.75
    q = inputs.jittered(inputs.fcc_positions(7, 1.75), 0.1, L, np.random.Generator(np.random.PCG64(61)))
    v = inputs.maxwell_boltzmann(q.shape[0], 1.0, 1.0, np.random.Generator(np.random.PCG64(62)))
    out = []
    for calls in ([15], [3] * 5):
        p = [B.make_params(q.shape[0], L, precision=precision, threads_per_key=tpk, flags=flags,
                           rebuild=policy)] * copies
        with B.Context(p if copies > 1 else p[0]) as c:
            c.set_state(np.tile(q, (copies, 1)), np.tile(v, (copies, 1)))
            for k in calls:
                c.step(k, energy_every=3)
            x, w = c.get_state()
            ke, pe = c.energy_series()
            vir, _ = c.observable_series()
            assert ke.shape[0] == 5
            out.append([x.cpu().numpy(), w.cpu().numpy(), ke / q.shape[0], pe / q.shape[0], vir / q.shape[0]])
    # the passes differ at most by the rounding of a force sum: FP64 some 1e-14 of forces
    # below 1e3, FP32 some 1e-7 of sums below 1e2; times dt and 15 steps
    tol = 2e-6 if precision == 1 else 1e-11
    for i, (a, b) in enumerate(zip(*out)):
        d = np.abs(a - b)
        if i == 0:
            d = np.minimum(d, np.abs(L - d))
        assert d.max() <= tol * max(1.0, np.abs(a).max())
