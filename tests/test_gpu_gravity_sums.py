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


def test_short_lengths_fp64(sg):
    """Separations whose r^-3 is no FP64 number although m r^-3 is: closest
    pairs at 1e-104 in a system of 1e-101.  All lengths and masses are a
    power of two times those of an ordinary system, so its accelerations,
    scaled, are the reference (the two differ by the kernel that serves them:
    the forms' 1e-12)."""
    rng = np.random.default_rng(3)
    n, eps = 13312, 0.001                 # whole tiles of the one-sided kernel
    p = rng.uniform(-0.5, 0.5, (n, 3))
    z = np.zeros(n)
    ls, ms = 2.0 ** -335, 2.0 ** -200

    def state(k, q):
        return dict(ng=0, x=k * p[:, 0], y=k * p[:, 1], z=k * p[:, 2], vx=z, vy=z, vz=z,
                    m=np.full(n, q / n), h=np.zeros(0), e=np.zeros(0))

    ref, rphi = evaluate(sg, state(1.0, 1.0), 0, eps=eps)
    got, phi = evaluate(sg, state(ls, ms), 0, eps=eps * ls)
    assert np.isfinite(got).all() and np.isfinite(phi).all()
    assert np.linalg.norm(got * (ls / ms) * ls - ref) < 1e-12 * np.linalg.norm(ref)
    assert np.linalg.norm(phi * (ls / ms) - rphi) < 1e-12 * np.linalg.norm(rphi)


@pytest.mark.parametrize("precision,scale,eps", [(0, 1e101, 1e98), (1, 3e12, 1e9)])
def test_long_lengths(sg, precision, scale, eps):
    """Extents at which r^-3 leaves the normal range: the one-sided kernel's
    answers, which are numbers there."""
    rng = np.random.default_rng(5)
    n = 12500
    p = scale * rng.uniform(-0.5, 0.5, (n, 3))
    z = np.zeros(n)
    st = dict(ng=0, x=p[:, 0].copy(), y=p[:, 1].copy(), z=p[:, 2].copy(), vx=z, vy=z, vz=z,
              m=np.full(n, 1.0 / n), h=np.zeros(0), e=np.zeros(0))
    got = evaluate(sg, st, precision, eps=eps, grav_ipl=1)
    ref = evaluate(sg, st, precision, eps=eps, grav_ipl=1, grav_variant=1 if precision else 4)
    assert np.isfinite(ref[0]).all() and (np.abs(ref[0]).max(axis=1) > 0.0).all()
    np.testing.assert_array_equal(got[0], ref[0])
    np.testing.assert_array_equal(got[1], ref[1])


def tiles_and_period(n, t):
    """The launch rule: tiles of the longest source list, and tiles between two
    roundings of the target-side sums."""
    nb = -(-n // (256 * t))
    tiles = t * (1 + nb // 2)
    s = min(max(-(-16384 // nb), tiles // 32), 128)
    return tiles, -(-tiles // s) if s < tiles else 1


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,ipl", [(66000, 1), (100001, 4)])
def test_parts_with_longer_periods(sg, orc, precision, n, ipl):
    """Sizes whose target-side sums span several tiles: parts that do not end
    with a period are rounded up to one, so every cut gives the same bits."""
    tiles, period = tiles_and_period(n, ipl)
    splits = (1, 3, 7, 64)
    assert period > 1 and any(-(-tiles // s) % period for s in splits)
    rng = np.random.default_rng(n)
    p = rng.normal(0.0, 1.0, (n, 3))
    z = np.zeros(n)
    st = dict(ng=0, x=p[:, 0].copy(), y=p[:, 1].copy(), z=p[:, 2].copy(), vx=z, vy=z, vz=z,
              m=rng.uniform(0.5, 1.5, n) / n, h=np.zeros(0), e=np.zeros(0))
    ref, rphi = evaluate(sg, st, precision, grav_ipl=ipl)
    t = np.arange(0, n, 331)
    gx, gy, gz, gp = orc.gravity(st["x"], st["y"], st["z"], st["m"], 1.0, 0.01, targets=t)
    a = np.stack([gx, gy, gz], 1)
    tol = (1e-12, 1e-6)[precision]
    assert np.linalg.norm(ref[t] - a) < tol * np.linalg.norm(a)
    assert np.linalg.norm(rphi[t] - gp) < tol * np.linalg.norm(gp)
    for split in splits:
        got, phi = evaluate(sg, st, precision, grav_ipl=ipl, grav_split=split)
        np.testing.assert_array_equal(got, ref)
        np.testing.assert_array_equal(phi, rphi)
