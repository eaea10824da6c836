"""The no-allocation entry point takes batches of up to 38,836 small clusters: 4 MiB of tables at 108 bytes
for a cluster of one item (its descriptor counted as 72 bytes, a chunk, an item, a counter)."""
import numpy as np
import pytest

from paper_1003_3896_amd import inputs, nbody

LAST = (4 << 20) // 108


def test_many_small_clusters_are_within_the_limits():
    """The last counts inside and the first outside, for every mode without sort tables."""
    for prec in ("fp32", "fp32c", "fp32ds", "fp64"):
        for n in (1, 60):
            for B, match in ((33000, "context is NULL"), (36000, "context is NULL"), (LAST - 8, "context is NULL"),
                             (LAST + 1, "staging")):
                with pytest.raises(nbody.NBodyError, match=match):
                    nbody.nbody_accel_noalloc(None, nbody.System(np.arange(B + 1) * n, 1e-3, prec=prec), None, None,
                                              None, None, 0)


def test_whatever_the_limits_accept_fits():
    """Random batches near both limits: accepted or rejected by the limits, never for lack of room."""
    rng = np.random.default_rng(77)
    seen = set()
    for _ in range(100):
        hi = int(np.exp(rng.uniform(0.5, np.log(1200000))))
        total = rng.uniform(0.2, 1.3) * (256 << 20) / rng.uniform(130, 700)
        sizes = []
        while sum(sizes) < total and len(sizes) < 40000:
            sizes += np.maximum(1, np.rint(np.exp(rng.uniform(0, np.log(hi), 2000 if hi < 200 else 1)))).astype(int).tolist()
        offs = np.concatenate([[0], np.cumsum(sizes)])
        with pytest.raises(nbody.NBodyError) as e:
            nbody.nbody_accel_noalloc(None, nbody.System(offs, 1e-3, prec=["fp64", "fp32dl"][int(rng.integers(2))]), None,
                                      None, None, None, 0)
        msg = str(e.value)
        assert "does not fit" not in msg, (len(sizes), hi)
        seen.add("context" in msg)
    assert seen == {True, False}


@pytest.mark.gpu
def test_noalloc_of_many_small_clusters_equals_accel():
    from gpu_helpers import make_sim, torch_dev
    torch = torch_dev()
    B = LAST - 8
    offs = np.concatenate([[0], np.cumsum(1 + np.arange(B) % 5)])
    rng = np.random.default_rng(5)
    n = int(offs[-1])
    b = inputs.single(rng.normal(size=(n, 3)), np.zeros((n, 3)), rng.uniform(0.5, 1.0, n), 1e-3, False)
    b.offsets, b.eps, b.field = offs, np.full(B, 1e-3), np.zeros(B, np.uint8)
    sim = make_sim(b, "fp64")
    sim.accel(pot=True)
    acc, pot = torch.zeros_like(sim.acc), torch.zeros_like(sim.pot)
    nbody.nbody_accel_noalloc(sim.ctx, sim.sys, sim.pos, sim.mass, acc, pot)
    torch.cuda.synchronize()
    assert torch.equal(acc, sim.acc) and torch.equal(pot, sim.pot)
    assert bool((acc[offs[1]:] != 0).any())
    sim.close()
