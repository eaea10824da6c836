"""The sorted one-sided local kernel, which runs above 2^20 particles (far-tile bits, expanded far form,
launch shapes), on sampled rows against the oracle; and the symmetric local kernel on coincident
particles, whose i-groups have zero boxes.  Gates as in gpu_helpers; potentials as in the parity
tests of the local mode."""
import numpy as np
import pytest

import oracle
from paper_1003_3896_amd import inputs, nbody

pytestmark = pytest.mark.gpu

N = (1 << 20) + 65


def _sampled(b, a, pot):
    from gpu_helpers import TOL, TOL_MEDIAN, rel_errors, stats
    err, dpot = [], []
    for r in ((0, 24), (N // 2, N // 2 + 24), (N - 24, N)):
        ref, rpot, scale = oracle.accel(b.pos, b.mass, b.G, b.eps[0], rows=r, want_pot=True, want_abs=True)
        s = slice(*r)
        err.append(rel_errors(a[s], ref, scale))
        if pot is not None:
            dpot.append(np.abs(pot[s] - rpot).max() / np.abs(rpot).max())
    err = np.concatenate(err)
    print("\n[fp32dl N=%d] %s %s" % (N, stats(err), dpot), flush=True)
    assert err.max() <= TOL["fp32dl"] and np.median(err) <= TOL_MEDIAN["fp32dl"]
    assert all(d <= 2e-6 for d in dpot)


@pytest.mark.parametrize("tile", [(1, 4, 256, 8), (2, 4, 128, 4), (2, 2, 256, 8), (1, 2, 128, 4)])
def test_shapes_above_the_symmetric_path(tile):
    from gpu_helpers import make_sim, torch_dev
    torch_dev()
    b = inputs.single(*inputs.plummer(N, 4721), 1e-4, False)
    sim = make_sim(b, "fp32dl")
    nbody.nbody_set_tile(sim.ctx, "fp32dl", 3, *tile, 0)
    a = sim.accel().cpu().numpy().copy()
    _sampled(b, a, None)
    nbody.nbody_set_tile(sim.ctx, "fp32dl", 3, *tile[:3], 2, 0)  # the grid changes nothing
    assert np.array_equal(sim.accel().cpu().numpy(), a)
    sim.close()


@pytest.mark.parametrize("salpeter,eps", [(False, 0.0), (True, 0.0), (True, 1e-4)])
def test_masses_softening_and_potential_above_the_symmetric_path(salpeter, eps):
    from gpu_helpers import make_sim, torch_dev
    torch_dev()
    b = inputs.single(*inputs.plummer(N, 4722, salpeter=salpeter), eps, False)
    sim = make_sim(b, "fp32dl")
    a = sim.accel(pot=True).cpu().numpy()
    pot = sim.pot.cpu().numpy()
    assert np.isfinite(a).all() and np.isfinite(pot).all()
    _sampled(b, a, pot)
    sim.close()


@pytest.mark.parametrize("n", [4097, 9000])
def test_coincident_particles_on_the_symmetric_path(n):
    from gpu_helpers import TOL, make_sim, oracle_reference, rel_errors, stats, torch_dev
    torch_dev()
    p, v, m = inputs.plummer(n, 4723, salpeter=True)
    p = p.copy()
    p[:1100] = p[0]             # whole chunks of the sorted order at one point
    p[n // 2:n // 2 + 20] = p[0]
    b = inputs.single(p, v, m, 1e-3, False)
    ref, scale, rpot = oracle_reference(b, want_pot=True)
    for prec in ("fp32dl", "fp32ds"):
        sim = make_sim(b, prec)
        a = sim.accel(pot=True).cpu().numpy()
        assert np.isfinite(a).all()
        err = rel_errors(a, ref, scale)
        print("\n[%s coincident N=%d] %s" % (prec, n, stats(err)), flush=True)
        assert err.max() <= TOL[prec]
        assert np.abs(sim.pot.cpu().numpy() - rpot).max() <= 2e-6 * np.abs(rpot).max()
        sim.close()
