"""Interpolate in the smallest workspace it takes (13 bytes per point, 16 per
element and 4 KiB): the bits of the call with the workspace it asks for."""
import numpy as np
import pytest

from paper_2501_12349_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 64, 5000, 70001])
@pytest.mark.parametrize("N,nf", [(3, 4), (6, 3), (8, 5)])
@pytest.mark.parametrize("kind", ["hex", "quad", "surface", "line"])
def test_small_workspace(kind, N, nf, n):
    from paper_2501_12349_amd import fpts
    rng = np.random.default_rng(1000 + n)
    if kind == "hex":
        wl = dict(nodes=W.curve_hex(W.box_mesh(3, 4, N), 0.1))
        wl["pts"] = W.uniform_points(rng, n, 3, -0.01, 1.01)
    elif kind == "quad":
        wl = dict(nodes=W.curve_quad2d(W.box_mesh(2, 30, N), 30))
        wl["pts"] = W.uniform_points(rng, n, 2, -0.01, 1.01)
    elif kind == "surface":
        wl = W.sphere(n_pts=n, ne=4, N=N, offset=1e-6)
    else:
        wl = W.line2d(level=2, per_elem=1, N=N)
        wl["pts"] = wl["pts"][:, rng.integers(0, wl["pts"].shape[1], n)]
    R = {"hex": 3, "quad": 2, "surface": 2, "line": 1}[kind]
    gm = fpts.Mesh(wl["nodes"], N, ref_dim=R)
    pts = torch.from_numpy(np.ascontiguousarray(wl["pts"])).cuda()
    f = torch.from_numpy(rng.standard_normal((nf, gm.n_elem, N ** R))).cuda()
    res = gm.find(pts)
    ref = gm.eval(res, f)
    small = 13 * n + 16 * gm.n_elem + 4096
    if n > 1000 and R > 1:
        assert small < gm.eval_workspace_bytes(n) // 3
    ws = torch.full((small,), 0xff, dtype=torch.uint8, device="cuda")
    got = gm.eval(res, f, ws=ws)
    torch.cuda.synchronize()
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    assert torch.equal(torch.nan_to_num(got), torch.nan_to_num(ref))
    # a workspace without room for the point ids is refused
    with pytest.raises(fpts.FptsError):
        gm.eval(res, f, ws=ws[:4 * n])


@pytest.mark.parametrize("N,nf", [(2, 3), (4, 4), (6, 7)])
@pytest.mark.parametrize("kind", ["hex", "quad", "surface"])
def test_many_points(kind, N, nf):
    # enough points that the values go through list order, in the call of its
    # own (2.5 million) and in the fused one (half a million); the call in a
    # small workspace writes them where they go
    from paper_2501_12349_amd import fpts
    n = 2500001
    rng = np.random.default_rng(1200 + N)
    if kind == "hex":
        nodes = W.curve_hex(W.box_mesh(3, 6, N), 0.1)
    elif kind == "quad":
        nodes = W.curve_quad2d(W.box_mesh(2, 20, N), 20)
    else:
        nodes = W.sphere(n_pts=64, ne=4, N=N)["nodes"]
    D = nodes.shape[1]
    if kind == "surface":
        x = nodes.transpose(1, 0, 2).reshape(D, -1)
        pts = x[:, rng.integers(0, x.shape[1], n)] * (1.0 + 1e-6 * rng.standard_normal(n))
    else:
        pts = W.uniform_points(rng, n, D, -0.01, 1.01)
    gm = fpts.Mesh(nodes, N, ref_dim=3 if kind == "hex" else 2)
    tp = torch.from_numpy(np.ascontiguousarray(pts)).cuda()
    f = torch.from_numpy(rng.standard_normal((nf, gm.n_elem, N ** gm.ref_dim))).cuda()
    res, one = gm.find_eval(tp, f)
    full = gm.eval(res, f)
    ws = torch.full((13 * n + 16 * gm.n_elem + 4096,), 0xff, dtype=torch.uint8, device="cuda")
    small = gm.eval(res, f, ws=ws)
    torch.cuda.synchronize()
    assert int((res["code"] == 2).sum()) < n // 2
    for got in (one, full):
        assert torch.equal(torch.isnan(got), torch.isnan(small))
        assert torch.equal(torch.nan_to_num(got), torch.nan_to_num(small))
