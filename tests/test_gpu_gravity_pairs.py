"""The symmetric gravity kernel (each pair once) against the oracle.

Sizes sit at the edges of its blocks (256 T targets), 256-source tiles,
64-source runs and the parity of the number of blocks, with each number T of
targets per lane.  Bounds are the forms' own: FP64 normwise 1e-12 (only the
order of summation differs from the oracle's), FP32C 1e-6.  The fixed-point
sums make results independent of the parts a source list is cut into, and
inputs they cannot hold go to the one-sided kernel bit for bit.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = {0: 1e-12, 1: 1e-6}


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


def halo(n, seed=5, scale=1.0, masses="equal"):
    rng = np.random.default_rng(seed)
    p = rng.normal(0.0, 1.0, (n, 3)) * rng.lognormal(0.0, 1.0, (n, 1)) * scale
    if masses == "zero":
        m = np.zeros(n)
    else:
        m = np.full(n, 1.0 / n) if masses == "equal" else rng.lognormal(0.0, 2.5, n) / n
    z = np.zeros(n)
    return dict(ng=0, x=p[:, 0].copy(), y=p[:, 1].copy(), z=p[:, 2].copy(), vx=z, vy=z, vz=z, m=m,
                h=np.zeros(0), e=np.zeros(0))


def evaluate(sg, st, precision, pot=True, **kw):
    eng = sg.Engine(st, precision=precision, **kw)
    eng.ctx.compute_accel(sg.SG_GRAV | (sg.SG_POT if pot else 0))
    eng.ctx.sync()
    out = np.stack([eng.numpy(f) for f in ("ax", "ay", "az")], 1), eng.numpy("pot")
    eng.ctx.close()
    return out


def err(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def check(sg, orc, st, precision, eps=0.01, **kw):
    n = len(st["x"])
    a, phi = evaluate(sg, st, precision, eps=eps, **kw)
    t = np.unique(np.concatenate([np.arange(0, n, 37), np.arange(n - 300, n)]))
    gx, gy, gz, gp = orc.gravity(st["x"], st["y"], st["z"], st["m"], 1.0, eps, targets=t)
    assert err(a[t], np.stack([gx, gy, gz], 1)) < TOL[precision]
    assert err(phi[t], gp) < TOL[precision]
    a2, _ = evaluate(sg, st, precision, pot=False, eps=eps, **kw)
    assert err(a2[t], np.stack([gx, gy, gz], 1)) < TOL[precision]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,ipl", [(12288, 0), (12289, 1), (12287 + 256, 1), (12800, 2),
                                   (12800 + 512 - 1, 2), (13312, 4), (13312 + 65, 4), (12351, 4),
                                   (14336, 4), (24577, 0)])
def test_edges(sg, orc, precision, n, ipl):
    check(sg, orc, halo(n), precision, grav_ipl=ipl)


@pytest.mark.parametrize("precision", [0, 1])
def test_unequal_masses_and_coincident(sg, orc, precision):
    st = halo(13000, masses="unequal")
    for f in ("x", "y", "z"):
        st[f][2000:4600] = st[f][2000]        # whole blocks of one position
    check(sg, orc, st, precision, grav_ipl=2)


@pytest.mark.parametrize("precision", [0, 1])
def test_parts_do_not_matter(sg, precision):
    st = halo(16000)
    ref = evaluate(sg, st, precision, grav_ipl=1)
    for split in (1, 3, 64):
        got = evaluate(sg, st, precision, grav_ipl=1, grav_split=split)
        np.testing.assert_array_equal(got[0], ref[0])
        np.testing.assert_array_equal(got[1], ref[1])


@pytest.mark.parametrize("precision,eps,scale", [(0, 1e-7, 1.0), (0, 1e3, 1e160), (1, 1e-9, 10.0),
                                                 (1, 1e-3, 1e16)])
def test_out_of_range_is_one_sided(sg, precision, eps, scale):
    st = halo(12500, scale=scale)
    got = evaluate(sg, st, precision, eps=eps, grav_ipl=1)
    ref = evaluate(sg, st, precision, eps=eps, grav_ipl=1, grav_variant=1 if precision else 4)
    np.testing.assert_array_equal(got[0], ref[0])
    np.testing.assert_array_equal(got[1], ref[1])


@pytest.mark.parametrize("precision", [0, 1])
def test_no_mass_and_no_number(sg, precision):
    a, phi = evaluate(sg, halo(12400, masses="zero"), precision)
    assert not a.any() and not phi.any()
    st = halo(12400)
    st["y"][7777] = np.nan
    eng = sg.Engine(st, precision=precision)
    eng.ctx.compute_accel(sg.SG_GRAV | sg.SG_POT)
    with pytest.raises(sg.SGError) as e:
        eng.ctx.sync()
    assert e.value.code == sg.SG_ENONFINITE
    assert np.isnan(eng.numpy("ax")).all()
    eng.ctx.close()
    st = halo(12400)
    st["m"][17] = np.nan
    a, _ = evaluate(sg, st, precision)
    assert np.isnan(a).all()


def test_ensemble_equals_single(sg):
    states = [halo(n, seed=n) for n in (300, 12287, 12289, 17000)]
    for ipl in (1, 2, 4):
        ens = sg.Ensemble(states, grav_ipl=ipl, grav_tile=256)
        for rep in range(2):
            ens.gravity(sg.SG_GRAV | sg.SG_POT)
        ens.sync()
        for st, e in zip(states, ens.engines):
            a, phi = evaluate(sg, st, sg.SG_FP32C, grav_ipl=ipl, grav_tile=256, grav_split=1)
            np.testing.assert_array_equal(np.stack([e.numpy(f) for f in ("ax", "ay", "az")], 1), a)
            np.testing.assert_array_equal(e.numpy("pot"), phi)
        ens.close()
