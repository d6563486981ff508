"""A NaN or an infinity in one field of a call (a masked or an overflowed
component) stays in that field: the others' values are those of the same call
with that field finite, bit for bit, whichever fields a launch takes together."""
import numpy as np
import pytest

from paper_2501_12349_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _mesh(kind, N):
    from paper_2501_12349_amd import fpts
    if kind == "hex":
        nodes = W.curve_hex(W.box_mesh(3, 3, N), 0.1)
    elif kind == "quad":
        nodes = W.curve_quad2d(W.box_mesh(2, 5, N), 5)
    else:
        nodes = W.sphere(n_pts=64, ne=2, N=N)["nodes"]
    return fpts.Mesh(nodes, N, ref_dim=3 if kind == "hex" else 2), nodes


def _points(kind, nodes, N, rng, n):
    if kind != "surface":
        return W.uniform_points(rng, n, nodes.shape[1], -0.02, 1.02)
    # nodes of the mesh, moved a little
    D = nodes.shape[1]
    x = nodes.transpose(1, 0, 2).reshape(D, -1)
    return x[:, rng.integers(0, x.shape[1], n)] * (1.0 + 1e-7 * rng.standard_normal(n))


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("Nf", [2, 3, 5, 6, 7, 8, 9, 10])
@pytest.mark.parametrize("kind", ["hex", "quad", "surface"])
def test_bad_field_stays_alone(kind, Nf, bad):
    rng = np.random.default_rng(900 + Nf)
    gm, nodes = _mesh(kind, 4)
    pts = torch.from_numpy(np.ascontiguousarray(_points(kind, nodes, 4, rng, 777))).cuda()
    R = gm.ref_dim
    res = gm.find(pts)
    assert int((res["code"] != 2).sum()) > 300
    for nf in (2, 3, 4, 5):
        f = torch.from_numpy(rng.standard_normal((nf, gm.n_elem, Nf ** R))).cuda()
        for which in range(nf):
            g = f.clone()
            g[which, :, 0] = bad
            keep = [k for k in range(nf) if k != which]
            for fused in (False, True):
                if fused:
                    ref = gm.find_eval(pts, f, field_nodes_1d=Nf)[1]
                    got = gm.find_eval(pts, g, field_nodes_1d=Nf)[1]
                else:
                    ref = gm.eval(res, f, field_nodes_1d=Nf)
                    got = gm.eval(res, g, field_nodes_1d=Nf)
                torch.cuda.synchronize()
                assert torch.equal(torch.isnan(got[keep]), torch.isnan(ref[keep])), (nf, which)
                assert torch.equal(torch.nan_to_num(got[keep]), torch.nan_to_num(ref[keep]))
