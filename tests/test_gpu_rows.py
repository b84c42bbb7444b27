"""Density and force passes over neighbour rows of every length around the
group's step of eight entries, and long ones, against the oracle.  Clumps far
apart give their members rows of one length; each length is compared by itself
(FP64 normwise 1e-12, FP32C 1e-6: the forms' bounds)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LENGTHS = list(range(0, 27)) + [31, 32, 33, 95, 96, 97, 700]


@pytest.fixture(scope="module")
def sg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1807_08116_amd import sphgrav
    sphgrav.lib()
    return sphgrav


@pytest.mark.parametrize("precision", [0, 1])
def test_row_lengths(sg, precision):
    import oracle as orc
    from paper_1807_08116_amd import ic
    prm = ic.DEFAULT_PARAMS
    rng = np.random.default_rng(17)
    pos, row = [], []
    for q, k in enumerate(LENGTHS):
        at = np.array([10.0 * (q % 6), 10.0 * (q // 6), 0.0])
        pos.append(at + rng.uniform(-0.5, 0.5, (k + 1, 3)))
        row += [k] * (k + 1)
    pos, row = np.concatenate(pos), np.array(row)
    n = len(pos)
    mix = rng.permutation(n)
    pos, row = pos[mix], row[mix]
    x, y, z = (np.ascontiguousarray(pos[:, d]) for d in range(3))
    h = rng.uniform(0.9, 1.1, n)          # (a clump's members lie within 3^1/2 < h_i + h_j)
    v = rng.normal(0.0, 0.1, (3, n))
    m, e = rng.uniform(0.5, 1.5, n) / n, rng.uniform(0.04, 0.06, n)
    st = dict(ng=n, x=x, y=y, z=z, vx=v[0], vy=v[1], vz=v[2], m=m, h=h, e=e)
    off, idx = orc.nbrs(x, y, z, h)
    np.testing.assert_array_equal(np.diff(off), row)
    rho = orc.density(x, y, z, m, h, off, idx)
    ref = orc.sph_force(x, y, z, v[0], v[1], v[2], m, h, rho, e, prm["gamma"], prm["alpha"],
                        prm["beta"], prm["eta"], off, idx)
    eng = sg.Engine(st, precision=precision)
    eng.build_neighbors()
    eng.ctx.compute_density()
    eng.ctx.compute_accel(sg.SG_SPH)
    eng.ctx.sync()
    got = [eng.numpy(f) for f in ("rho", "ax", "ay", "az", "dedt")]
    eng.ctx.close()
    tol = 1e-6 if precision else 1e-12
    for k in LENGTHS:
        s = row == k
        assert np.linalg.norm(got[0][s] - rho[s]) < tol * np.linalg.norm(rho[s]), k
        a, b = (np.stack([q[s] for q in c]) for c in (got[1:4], ref[:3]))
        if k == 0:
            assert not a.any() and not got[4][s].any()
            continue
        assert np.linalg.norm(a - b) < tol * np.linalg.norm(b), k
        assert np.linalg.norm(got[4][s] - ref[3][s]) < tol * np.linalg.norm(ref[3][s]), k


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("ng", [700, 65537])
def test_time_step_between_forces(sg, precision, ng):
    """The time-step rule's records share the force pass's memory and hold the
    sound speed where those have the mass: its value against the oracle's rule
    on the same state, and forces before and after it alike, bit for bit."""
    import oracle as orc
    from paper_1807_08116_amd import ic
    prm = ic.DEFAULT_PARAMS
    rng = np.random.default_rng(ng)
    x, y, z = rng.uniform(0.0, 1.0, (3, ng))
    v = rng.normal(0.0, 0.1, (3, ng))
    h = ng ** (-1 / 3) * rng.uniform(0.8, 1.2, ng)
    m, e = rng.uniform(0.5, 1.5, ng) / ng, rng.uniform(0.02, 0.06, ng)
    st = dict(ng=ng, x=x, y=y, z=z, vx=v[0], vy=v[1], vz=v[2], m=m, h=h, e=e)
    eng = sg.Engine(st, precision=precision)
    eng.build_neighbors()
    eng.ctx.compute_density()
    eng.ctx.compute_accel(sg.SG_SPH | sg.SG_GRAV)
    dt = float(eng.ctx.cfl_dt(0.3))
    eng.ctx.sync()
    F = ("ax", "ay", "az", "dedt", "rho")
    before = {f: eng.numpy(f).copy() for f in F}
    rho = before["rho"]
    c = np.sqrt(prm["gamma"] * (prm["gamma"] - 1.0) * e)
    off, idx = orc.nbrs(x, y, z, h)
    ref = orc.cfl_dt(x, y, z, v[0], v[1], v[2], h, c, before["ax"], before["ay"], before["az"],
                     before["dedt"], 0.3, prm["alpha"], prm["beta"], prm["eta"], off, idx)
    assert abs(dt - ref) < 1e-12 * ref
    eng.ctx.compute_accel(sg.SG_SPH | sg.SG_GRAV)
    eng.ctx.sync()
    for f in F:
        np.testing.assert_array_equal(eng.numpy(f), before[f], err_msg=f)
    eng.ctx.close()
