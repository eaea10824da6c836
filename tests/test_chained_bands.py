"""Chained integrator stages on batches whose clusters need different numbers of bands of partial-sum
rows: one band up to about 67,500 particles, two at 70000, more from there, one thread per
particle in the combine pass from 131072 on.  Every cluster's stage must end exactly once, whichever pass adds its
last rows."""
import numpy as np
import pytest

from paper_1003_3896_amd import inputs, nbody

pytestmark = pytest.mark.gpu


def _batch(sizes, eps=1e-3):
    cl = []
    for c, n in enumerate(sizes):
        p, v, m = inputs.plummer(n, 8500 + c, salpeter=c % 2 == 1)
        if c % 2 == 0:
            p, v = inputs.on_orbit(p, v)
        cl.append(inputs.single(p, v, m, eps, c % 2 == 0))
    return inputs.concat(cl)


def _rounds(integ, dt, steps):
    if integ == "leapfrog":
        return [(0.5 * dt, dt, 0.5 * dt)] * steps
    d, k = nbody.nbody_sym6_coefficients()
    return [(k[s] * dt, d[s] * dt, k[7] * dt if s == 6 else 0.0) for s in range(7)] * steps


def _run(b, prec, integ, how, dt, steps):
    from gpu_helpers import make_sim
    s = make_sim(b, prec)
    nbody.nbody_use_graphs(s.ctx, "no graph" not in how)
    nbody.nbody_timing_enable(s.ctx, "timed" in how)
    s.accel()
    if how.startswith("step"):
        s.step(integ, dt, steps)
    elif how.startswith("substeps"):
        coef = np.array([[r] * b.B for r in _rounds(integ, dt, steps)])
        nbody.nbody_substeps(s.ctx, s.sys, s.pos, s.vel, s.mass, s.acc, coef, s.ws_addr, s.ws_bytes)
    else:
        for pre, drift, post in _rounds(integ, dt, steps):
            s.substep([pre] * b.B, [drift] * b.B, [post] * b.B)
    s.torch.cuda.synchronize()
    out = [x.cpu().numpy() for x in (s.pos, s.vel, s.acc)]
    s.close()
    return out


@pytest.mark.parametrize("prec", ["fp64", "fp32ds", "fp32dl", "fp32"])
@pytest.mark.parametrize("sizes", [(70000, 5000, 300), (140000, 70000, 9000), (5000, 100, 200000)])
def test_unequal_band_counts_chained_equal_single_stages(prec, sizes):
    """Step functions and substeps calls, with and without graphs, against single substep calls: the same
    bits; and a cluster stepped alone gives the bits of the cluster in the batch."""
    from gpu_helpers import torch_dev
    torch_dev()
    b = _batch(sizes)
    dt, steps = 1.0 / 600, 2
    for integ in ("leapfrog", "sym6"):
        want = _run(b, prec, integ, "single", dt, steps)
        for how in ("step", "step, no graph", "step, timed", "substeps", "substeps, no graph"):
            got = _run(b, prec, integ, how, dt, steps)
            for name, x, y in zip(("pos", "vel", "acc"), got, want):
                assert np.array_equal(x, y), (integ, how, name)
    small = min((n, c) for c, n in enumerate(sizes) if n >= 4096)[1]
    s = slice(b.offsets[small], b.offsets[small + 1])
    one = inputs.single(b.pos[s], b.vel[s], b.mass[s], b.eps[small], bool(b.field[small]))
    one.galaxy = b.galaxy
    for x, y in zip(_run(one, prec, "sym6", "step", dt, steps), want):
        assert np.array_equal(x, y[s])
