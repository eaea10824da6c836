"""The room for partial-sum rows that a whole batch may take: 2 GiB above the least that its clusters
need, so that no batch asks for more than that above what j-ranges (32 bytes per particle and range) would;
where the room is short, clusters take their rows in more bands, with the same bits."""
import numpy as np
import pytest

from paper_1003_3896_amd import inputs, nbody

RANGES = {4096: 8, 8191: 8, 16384: 8, 65536: 16, 131072: 16, 262144: 16, 600000: 4, 1 << 20: 4}


@pytest.mark.parametrize("n,B", [(4096, 10000), (8191, 8192), (16384, 4096), (65536, 100), (65536, 1500), (131072, 500),
                                 (262144, 200), (600000, 100), (1 << 20, 64)])
def test_batches_ask_for_little_more_than_their_ranges(n, B):
    offs = np.arange(B + 1) * n
    for prec, sort in (("fp64", 0), ("fp32dl", 56)):
        ws = nbody.nbody_workspace_bytes(None, nbody.System(offs, 1e-3, prec=prec))
        assert ws <= (2 << 30) + B * (n * (32 + 32 * RANGES[n] + sort + 4) + 8192), (prec, ws)
        assert ws <= nbody.nbody_workspace_bytes_max(B * n, B)


def test_bound_of_random_mixes():
    """Batches of one-sided and symmetric clusters, few or many, up to several GiB of rows: the
    batch-independent bound holds."""
    rng = np.random.default_rng(3)
    for _ in range(200):
        hi = np.exp(rng.uniform(np.log(300), np.log(3e6)))
        B = int(rng.integers(1, 400))
        sizes = np.maximum(1, np.rint(np.exp(rng.uniform(np.log(hi / 300), np.log(hi), B)))).astype(np.int64)
        sizes[rng.random(B) < 0.2] = rng.choice([4095, 4096, 4097, 131071, 1 << 20, (1 << 20) + 1])
        offs = np.concatenate([[0], np.cumsum(sizes)])
        field = rng.integers(0, 2, B).astype(np.uint8)
        for prec in ("fp64", "fp32dl"):
            for galaxy in ((), (inputs.ALLEN_SANTILLAN,)):
                sys = nbody.System(offs, 1e-3, field, 1.0, *galaxy, prec=prec)
                assert nbody.nbody_workspace_bytes(None, sys) <= nbody.nbody_workspace_bytes_max(int(offs[-1]), B)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32dl"])
def test_short_room_same_bits(prec):
    from gpu_helpers import make_sim, torch_dev
    torch_dev()
    cl = [inputs.single(*inputs.plummer(n, 8800 + c, salpeter=c % 2 == 1), 1e-3, c % 2 == 0)
          for c, n in enumerate((16384, 70000, 5000, 300))]
    many = inputs.concat(cl[:1] * 200 + cl[1:])
    full = nbody.nbody_workspace_bytes(None, nbody.System([0, 16384], 1e-3, prec=prec))
    a = make_sim(many, prec)
    assert a.ws_bytes < 200 * full  # the batch has less room than its clusters alone
    a.accel(pot=True)
    acc, pot = a.acc.cpu().numpy().copy(), a.pot.cpu().numpy().copy()
    a.step("leapfrog", 1.0 / 600, 3)
    got = [acc, pot] + [x.cpu().numpy() for x in (a.pos, a.vel, a.acc)]
    a.close()
    for b, k in ((cl[0], 0), (cl[0], 199), (cl[1], 200), (cl[2], 201), (cl[3], 202)):
        s = make_sim(b, prec)
        s.accel(pot=True)
        want = [s.acc.cpu().numpy().copy(), s.pot.cpu().numpy().copy()]
        s.step("leapfrog", 1.0 / 600, 3)
        want += [x.cpu().numpy() for x in (s.pos, s.vel, s.acc)]
        s.close()
        sl = slice(many.offsets[k], many.offsets[k + 1])
        for x, y in zip(got, want):
            assert np.array_equal(x[sl], y), (k, b.n)
