"""Sums of the pairwise gravity kernel where a particle's own sum is small
against the largest that any particle can have: the one particle (or the few
at one place) that outweighs all others feels only these.  Each such particle
is compared by itself with the oracle.

Bounds: the light particles lie on one side, so their terms add up without
cancellation; a term carries a few roundings of the form's arithmetic and the
sum of 20000 of them no more than its FP64 partial sums do.  FP64: 64 units of
2^-53; FP32C: the form's own 1e-6.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = {0: 64 * 2.0 ** -53, 1: 1e-6}


@pytest.fixture(scope="module")
def sg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1807_08116_amd import sphgrav
    sphgrav.lib()
    return sphgrav


@pytest.fixture(scope="module")
def orc():
    import oracle
    oracle.lib()
    return oracle


def star_and_disk(n, heavy, light, ratio, eps=0.01, seed=11):
    """`heavy` particles of mass 1 / heavy at the origin; the others, of mass
    `light` together, in x > 0 out to ratio * eps from them."""
    rng = np.random.default_rng(seed)
    p = rng.normal(0.0, 1.0, (n, 3)) * rng.uniform(0.2, 1.0, (n, 1))
    p[:, 0] = np.abs(p[:, 0]) + 0.2
    p *= ratio * eps / np.abs(p).max()
    m = rng.uniform(0.5, 1.5, n)
    at = rng.choice(n, heavy, replace=False)
    p[at] = 0.0
    m *= light / np.delete(m, at).sum()
    m[at] = 1.0 / heavy
    z = np.zeros(n)
    return dict(ng=0, x=p[:, 0].copy(), y=p[:, 1].copy(), z=p[:, 2].copy(), vx=z, vy=z, vz=z, m=m,
                h=np.zeros(0), e=np.zeros(0)), np.sort(at)


def evaluate(sg, st, precision, pot=True, **kw):
    eng = sg.Engine(st, precision=precision, **kw)
    eng.ctx.compute_accel(sg.SG_GRAV | (sg.SG_POT if pot else 0))
    eng.ctx.sync()
    out = np.stack([eng.numpy(f) for f in ("ax", "ay", "az")], 1), eng.numpy("pot")
    eng.ctx.close()
    return out


def one_by_one(a, ref):
    return (np.linalg.norm(a - ref, axis=1) / np.linalg.norm(ref, axis=1)).max()


@pytest.mark.parametrize("precision,heavy,light,ratio", [
    (0, 1, 1e-6, 1e5), (0, 1, 1e-8, 1e5), (0, 1, 1e-10, 1e5), (0, 1, 1e-6, 5e5), (0, 1, 1e-10, 5e5),
    (0, 1, 1e-14, 1e3), (0, 7, 1e-8, 1e5), (0, 300, 1e-10, 1e5), (1, 1, 1e-10, 1e8), (1, 5, 1e-6, 5e8)])
def test_heavy_particles(sg, orc, precision, heavy, light, ratio):
    st, at = star_and_disk(20001, heavy, light, ratio)
    t = np.unique(np.concatenate([at, np.arange(0, 20001, 97)]))
    gx, gy, gz, gp = orc.gravity(st["x"], st["y"], st["z"], st["m"], 1.0, 0.01, targets=t)
    ref = np.stack([gx, gy, gz], 1)
    own = np.isin(t, at)
    for pot in (True, False):
        a, phi = evaluate(sg, st, precision, pot=pot, eps=0.01)
        print("heavy: %.2e, others: %.2e" % (one_by_one(a[t][own], ref[own]),
                                             one_by_one(a[t][~own], ref[~own])))
        assert one_by_one(a[t][own], ref[own]) < TOL[precision]
        assert np.linalg.norm(a[t] - ref) < (1e-12, 1e-6)[precision] * np.linalg.norm(ref)
        if pot:                       # (a heavy one's is the rest of a sum that holds its m / eps)
            assert np.linalg.norm(phi[t][~own] - gp[~own]) < (1e-12, 1e-6)[precision] * np.linalg.norm(gp[~own])


def test_ensemble_heavy_particles(sg):
    states = [star_and_disk(n, 1, 1e-10, 1e8, seed=n)[0] for n in (12289, 20001)]
    ens = sg.Ensemble(states, grav_ipl=2, grav_tile=256, eps=0.01)
    ens.gravity(sg.SG_GRAV | sg.SG_POT)
    ens.sync()
    for st, e in zip(states, ens.engines):
        a, phi = evaluate(sg, st, sg.SG_FP32C, grav_ipl=2, grav_tile=256, grav_split=1, eps=0.01)
        np.testing.assert_array_equal(np.stack([e.numpy(f) for f in ("ax", "ay", "az")], 1), a)
        np.testing.assert_array_equal(e.numpy("pot"), phi)
    ens.close()
