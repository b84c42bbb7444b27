"""Neighbour lists at the sizes where the search changes its number of
targets per wavefront (1, 2, 4, 8, 16, 32), and one off a whole wavefront:
bit for bit against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1807_08116_amd import sphgrav
    sphgrav.lib()
    return sphgrav


@pytest.mark.parametrize("ng", [1, 5, 9499, 9503, 15999, 16001, 21999, 22003, 25003, 39999, 45001,
                                119999, 120007, 149999, 150017, 450031])
def test_lists_match_oracle(sg, ng):
    import oracle as orc
    from paper_1807_08116_amd import ic
    rng = np.random.default_rng(ng)
    p, m = ic.plummer(ng, 1.0, 0.1, rng)
    r2 = np.sum(p * p, 1)
    h = 0.6 * (np.pi / (3.0 * ng)) ** (1 / 3) * (1.0 + r2) ** (5 / 6) * rng.uniform(0.7, 1.3, ng)
    z = np.zeros(ng)
    st = dict(ng=ng, x=p[:, 0].copy(), y=p[:, 1].copy(), z=p[:, 2].copy(), vx=z, vy=z, vz=z, m=m,
              h=h, e=z + 0.05)
    eng = sg.Engine(st, precision=sg.SG_FP64)
    eng.build_neighbors()
    s = orc.sort_gas(st["x"], st["y"], st["z"], h)
    soff, sidx = orc.rows_to_slots(s["perm"], *orc.nbrs(st["x"], st["y"], st["z"], h))
    np.testing.assert_array_equal(eng.ctx.export(sg.SG_X_PERM), s["perm"])
    np.testing.assert_array_equal(eng.ctx.export(sg.SG_X_OFFSETS), s["off"])
    np.testing.assert_array_equal(eng.ctx.export(sg.SG_X_NBR_OFF), soff)
    np.testing.assert_array_equal(eng.ctx.export(sg.SG_X_NBR_IDX), sidx)
    eng.ctx.close()


# Where the FP32 pretest cannot decide, or must not: ties (a lattice whose
# neighbours sit at exactly h_i + h_j), scales whose squares underflow or
# overflow, and particles far from the origin.
@pytest.mark.parametrize("case", ["ties", 1e-17, 1e-21, 1e-26, 1e12, 3e18, 1e25, "far"])
def test_pretest_edges(sg, case):
    import oracle as orc
    rng = np.random.default_rng(5)
    k = 31
    g = np.stack(np.meshgrid(*[np.arange(k, dtype=np.float64)] * 3), -1).reshape(-1, 3)
    ng = len(g)
    if case == "ties":
        p, h = g, np.full(ng, 0.5)
        p = p[rng.permutation(ng)]
        h[::7] = 1.0
    else:
        p = g + rng.uniform(-0.4, 0.4, g.shape)
        h = rng.uniform(0.45, 1.1, ng)
        if case == "far":
            p = p + np.array([1e9, -3e10, 7e5])
        else:
            p, h = p * case, h * case
    z = np.zeros(ng)
    st = dict(ng=ng, x=p[:, 0].copy(), y=p[:, 1].copy(), z=p[:, 2].copy(), vx=z, vy=z, vz=z,
              m=z + 1.0, h=h, e=z + 0.05)
    eng = sg.Engine(st, precision=sg.SG_FP32C)
    eng.build_neighbors()
    s = orc.sort_gas(st["x"], st["y"], st["z"], h)
    soff, sidx = orc.rows_to_slots(s["perm"], *orc.nbrs(st["x"], st["y"], st["z"], h))
    np.testing.assert_array_equal(eng.ctx.export(sg.SG_X_NBR_OFF), soff)
    np.testing.assert_array_equal(eng.ctx.export(sg.SG_X_NBR_IDX), sidx)
    eng.ctx.close()
