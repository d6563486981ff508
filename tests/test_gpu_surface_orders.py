"""Surface quads of every order on the GPU against the oracle, in both
precisions: several elements to a wave in the face and resolve kernels (a node
block of an odd number of values for odd N), every point in the first
interpolation pass of the one call, values in list order or scattered, and the
one call and the two calls bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2501_12349_amd import workloads as W
from tests.parity import compare_eval, compare_find, to_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _points(rng, om, nel, n):
    """Points beside the surface: 40 % anywhere on an element and up to 1e-3 off
    it, the others 1e-5 to 1e-1 (in reference units) from an element's edge and
    up to 1e-7 off it; and some far away."""
    e = rng.integers(0, nel, n)
    r = rng.uniform(-1.0, 1.0, (2, n))
    edge = rng.uniform(size=n) > 0.4
    d = rng.integers(0, 2, n)
    near = np.sign(rng.uniform(-1, 1, n)) * (1.0 - 10.0 ** rng.uniform(-5, -1, n))
    r[d[edge], np.nonzero(edge)[0]] = near[edge]
    pts = np.empty((3, n))
    for p in range(n):
        x, G, _ = om.map(int(e[p]), r[:, p])
        G = np.asarray(G).reshape(3, 2)
        nrm = np.cross(G[:, 0], G[:, 1])
        off = rng.uniform(-1.0, 1.0) * (1e-7 if edge[p] else 1e-3)
        pts[:, p] = x + off * nrm / np.linalg.norm(nrm)
    pts[:, :n // 50] *= 1.7
    return pts


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("N", list(range(2, 11)))
def test_surface_every_order(N, precision):
    from paper_2501_12349_amd import fpts
    ne = 4
    rng = np.random.default_rng(1100 + N)
    nodes = W.sphere(n_pts=64, ne=ne, N=N)["nodes"]
    om = oracle.Mesh(nodes, 3, 2, N)
    pts = _points(rng, om, nodes.shape[0], 3000)
    orc = om.find(pts)
    gm = fpts.Mesh(nodes, N)
    tp = torch.from_numpy(np.ascontiguousarray(pts)).cuda()
    two = gm.find(tp, precision=precision)
    g = to_np(two)
    rep = compare_find(om, pts, orc, g, (np.pi / 2) / ne, surface=True)
    rep["codes"] = np.bincount(g["code"], minlength=3).tolist()
    print("surface N=%d %s" % (N, precision), rep, flush=True)
    assert min(rep["codes"]) > 30
    for Nf, nf in ((N, 1), (N, 3), (N, 4), (N, 5), (5, 4), (6, 3)):
        fields = np.stack([W.nodal_field(nodes, W.poly_coeffs(3, min(N - 1, 3), rng))
                           for _ in range(nf)]) if Nf == N else \
            rng.standard_normal((nf, nodes.shape[0], Nf * Nf))
        tf = torch.from_numpy(np.ascontiguousarray(fields)).cuda()
        u2 = gm.eval(two, tf, field_nodes_1d=Nf)
        one, u1 = gm.find_eval(tp, tf, precision=precision, field_nodes_1d=Nf)
        torch.cuda.synchronize()
        for k in two:
            assert torch.equal(one[k], two[k]), (Nf, nf, k)
        assert torch.equal(torch.isnan(u1), torch.isnan(u2)), (Nf, nf)
        assert torch.equal(torch.nan_to_num(u1), torch.nan_to_num(u2)), (Nf, nf)
        if Nf == N:
            same = g["elem"] == orc["elem"]
            compare_eval(om.eval(orc, fields)[:, same], u1.cpu().numpy()[:, same],
                         orc["code"][same])
