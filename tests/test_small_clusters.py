"""Clusters of fewer than 4096 particles: no separate reduction or sort pass (the pair kernel reduces the
chunk partials; the local mode runs the double-single kernel there), one pass between two integrator
stages, and fewer i-particles per lane where there are few items.  Everything bitwise against the ways
that do not take these shortcuts, in batches that mix all sizes and paths."""
import numpy as np
import pytest

from paper_1003_3896_amd import inputs, nbody

pytestmark = pytest.mark.gpu


def _batch(sizes, galaxy=None, eps=1e-3):
    cl = []
    for c, n in enumerate(sizes):
        p, v, m = inputs.plummer(n, 910 + c, salpeter=c % 2 == 1)
        if c % 3 == 0:
            p, v = inputs.on_orbit(p, v)
        cl.append(inputs.single(p, v, m, eps, c % 3 == 0))
    b = inputs.concat(cl)
    if galaxy:
        b.galaxy = galaxy
    return b


def test_local_mode_of_small_clusters_is_double_single():
    """Sizes around a chunk, a range and the path's end, alone and beside a sorted cluster: FP32DL gives
    the FP32DS bits for the small ones."""
    from gpu_helpers import make_sim, torch_dev
    torch_dev()
    sizes = (1, 255, 257, 1023, 2049, 4095, 4096, 63)
    b = _batch(sizes)
    local, ds = make_sim(b, "fp32dl"), make_sim(b, "fp32ds")
    for pot in (False, True):
        a1, a2 = local.accel(pot=pot).cpu().numpy().copy(), ds.accel(pot=pot).cpu().numpy().copy()
        for c, n in enumerate(sizes):
            s = slice(b.offsets[c], b.offsets[c + 1])
            if n < 4096:
                assert np.array_equal(a1[s], a2[s]), n
                assert not pot or np.array_equal(local.pot.cpu().numpy()[s], ds.pot.cpu().numpy()[s]), n
    local.close()
    ds.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp32c", "fp32dl"])
@pytest.mark.parametrize("sizes,galaxy", [((700, 64, 255, 1300), None), ((300, 5000, 77, 9000, 2500), None),
                                          ((300, 5000, 200), inputs.ALLEN_SANTILLAN)])
def test_stages_chained_equal_stages_one_by_one(prec, sizes, galaxy):
    """A step function, the same stages as one substeps call and as single substep calls (which never
    fuse the end of a stage with the next one's start), with and without graphs: the same bits."""
    from gpu_helpers import make_sim, torch_dev
    torch = torch_dev()
    b = _batch(sizes, galaxy)
    dt, steps = 1.0 / 600, 2
    d, k = nbody.nbody_sym6_coefficients()
    for integ in ("leapfrog", "sym6"):
        rounds = ([(0.5 * dt, dt, 0.5 * dt)] if integ == "leapfrog" else
                  [(k[s] * dt, d[s] * dt, k[7] * dt if s == 6 else 0.0) for s in range(7)]) * steps
        coef = np.array([[r] * b.B for r in rounds])
        got = []
        for how in ("step", "step, no graph", "substeps", "substeps, no graph", "substep"):
            s = make_sim(b, prec)
            nbody.nbody_use_graphs(s.ctx, "no graph" not in how)
            s.accel()
            if how.startswith("step"):
                s.step(integ, dt, steps)
            elif how.startswith("substeps"):
                nbody.nbody_substeps(s.ctx, s.sys, s.pos, s.vel, s.mass, s.acc, coef, s.ws_addr, s.ws_bytes)
            else:
                for r in coef:
                    s.substep(r[:, 0], r[:, 1], r[:, 2])
            torch.cuda.synchronize()
            got.append([x.cpu().numpy() for x in (s.pos, s.vel, s.acc)])
            for x, y in zip(got[0], got[-1]):
                assert np.array_equal(x, y), (integ, how)
            s.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32ds", "fp32c"])
def test_few_items_take_one_particle_per_lane(prec):
    """One cluster alone (few items) and 40 copies of it (many): the same bits."""
    from gpu_helpers import make_sim, torch_dev
    torch_dev()
    one = _batch((2100,))
    many = inputs.concat([one] * 40)
    many.galaxy = one.galaxy
    a, m = make_sim(one, prec).accel().cpu().numpy(), make_sim(many, prec).accel().cpu().numpy()
    assert np.array_equal(np.concatenate([a] * 40), m)
