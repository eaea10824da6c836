"""Clusters of fewer than 4096 particles take their reference point and common mass from the pair kernel
itself (few items), or from the reduction kernel (many items, or a larger cluster in the batch): the
same bits by all three ways."""
import numpy as np
import pytest

from paper_1003_3896_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp32c", "fp32ds", "fp32dl"])
def test_frames_of_small_clusters_by_either_kernel(prec):
    from gpu_helpers import make_sim, torch_dev
    torch_dev()
    cl = []
    for c, n in enumerate((2100, 3841, 2304)):
        p, v, m = inputs.plummer(n, 8700 + c, salpeter=c == 1)
        p, v = inputs.on_orbit(p, v)
        cl.append(inputs.single(p, v, m, 1e-3, c != 2))
    three = inputs.concat(cl)
    big = inputs.single(*inputs.plummer(5000, 8710), 1e-3, False)

    def run(batch):
        s = make_sim(batch, prec)
        s.accel(pot=True)
        out = [s.acc.cpu().numpy().copy(), s.pot.cpu().numpy().copy()]
        s.step("sym6", 1.0 / 600, 2)
        out += [x.cpu().numpy() for x in (s.pos, s.vel, s.acc)]
        s.close()
        return out

    few, many, beside = run(three), run(inputs.concat(cl * 20)), run(inputs.concat([big] + cl))
    for x, y, z in zip(few, many, beside):
        assert np.isfinite(x).all()
        assert np.array_equal(np.concatenate([x] * 20), y)
        assert np.array_equal(x, z[5000:])
