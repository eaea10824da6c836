"""The i-particles per lane of the kernels for clusters of fewer than 4096 particles follow the number of items
of the batch (one, two or four): the same bits."""
import numpy as np
import pytest

from paper_1003_3896_amd import inputs, nbody

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp32c", "fp32ds", "fp32dl", "fp64"])
@pytest.mark.parametrize("eps", [1e-3, 0.0])
@pytest.mark.parametrize("sizes", [(700, 1999, 64, 255, 1), (1025, 2047, 513), (2049, 4095, 300)])
def test_few_and_many_copies_same_bits(prec, eps, sizes):
    from gpu_helpers import make_sim, torch_dev
    torch_dev()
    cl = [inputs.single(*inputs.plummer(n, 8900 + c, salpeter=c % 2 == 1), eps, False) for c, n in enumerate(sizes)]
    want = None
    for copies in (1, 15, 150):
        s = make_sim(inputs.concat(cl * copies), prec)
        for w4 in (False, True):  # the tuned shape, and four waves to a group
            if w4:
                for ncl in range(nbody.N_CLASSES):
                    nbody.nbody_set_tile(s.ctx, prec, ncl, 2, 4, 128, 8)
            s.accel()
            a0 = s.acc.cpu().numpy().copy()
            s.accel(pot=True)
            got = [a0, s.acc.cpu().numpy(), s.pot.cpu().numpy()]
            if want is None:
                want = {}
            if w4 not in want:
                want[w4] = [g.copy() for g in got]
            for g, w in zip(got, want[w4]):
                assert np.array_equal(g, np.concatenate([w] * copies)), (copies, w4)
        s.close()
