"""The sizes at which a call changes its way through the library: element
counts at the edges of the scans' tiles and of the spread counters, a few
points to the element and hundreds of thousands in one, ragged point counts,
every number of fields per launch, long cell lists in the device setup, more
requests than one batch copy takes."""
import numpy as np
import pytest

import oracle
from paper_2501_12349_amd import workloads as W
from tests.parity import compare_eval, compare_find, to_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _fpts():
    from paper_2501_12349_amd import fpts
    return fpts


def _check(nodes, D, N, pts, nf, precision, h, sample=None):
    """One call and two calls give the same bits; both meet the oracle."""
    rng = np.random.default_rng(nf)
    fields = np.stack([W.nodal_field(nodes, W.poly_coeffs(D, min(N - 1, 3), rng))
                       for _ in range(nf)])
    gm = _fpts().Mesh(nodes, N)
    tp = torch.from_numpy(np.ascontiguousarray(pts)).cuda()
    tf = torch.from_numpy(fields).cuda()
    two = gm.find(tp, precision=precision)
    u2 = gm.eval(two, tf)
    one, u1 = gm.find_eval(tp, tf, precision=precision)
    torch.cuda.synchronize()
    for k in two:
        assert torch.equal(one[k], two[k]), k
    assert torch.equal(torch.isnan(u1), torch.isnan(u2))
    assert torch.equal(torch.nan_to_num(u1), torch.nan_to_num(u2))
    g, ug = to_np(one), u1.cpu().numpy()
    if sample is not None:
        g = {k: (v[:, sample] if v.ndim == 2 else v[sample]) for k, v in g.items()}
        ug, pts = ug[:, sample], np.ascontiguousarray(pts[:, sample])
    om = oracle.Mesh(nodes, D, D, N)
    orc = om.find(pts)
    compare_find(om, pts, orc, g, h)
    same = g["elem"] == orc["elem"]
    compare_eval(om.eval(orc, fields)[:, same], ug[:, same], orc["code"][same])


@pytest.mark.parametrize("where", ["spread", "one element"])
@pytest.mark.parametrize("n", [1, 65, 4097])
@pytest.mark.parametrize("side", [22, 23, 91, 129])
def test_element_counts(side, n, where):
    # 484, 529, 8281 and 16641 elements: either side of 512 (scan parts), past
    # 8192 (two tiles of the scans) and past 16384 (counters not spread)
    nodes = W.curve_quad2d(W.box_mesh(2, side, 3), side)
    rng = np.random.default_rng(side + n)
    lo, hi = (-0.02, 1.02) if where == "spread" else (0.5 + 0.1 / side, 0.5 + 0.6 / side)
    _check(nodes, 2, 3, W.uniform_points(rng, n, 2, lo, hi), 1 + n % 3, "fp64", 1.0 / side)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("N", list(range(2, 11)))
def test_few_points_per_element(N, precision):
    # one to five fields: one or two launches, values scattered or spread
    nodes = W.curve_hex(W.box_mesh(3, 6, N), 0.1)
    rng = np.random.default_rng(600 + N)
    _check(nodes, 3, N, W.uniform_points(rng, 333, 3, -0.01, 1.01), 1 + N % 5, precision, 1 / 6)


@pytest.mark.parametrize("N,nf", [(4, 4), (6, 3), (7, 2), (8, 3)])
def test_crowded_element(N, nf):
    # even parts of one element's list, in the Newton passes and the
    # interpolation (more than 64 points to a part)
    nodes = W.curve_hex(W.box_mesh(3, 3, N), 0.1)
    rng = np.random.default_rng(700 + N)
    n = 600001
    _check(nodes, 3, N, W.uniform_points(rng, n, 3, 0.36, 0.63), nf, "fp64", 1 / 3,
           sample=rng.choice(n, 300, replace=False))


@pytest.mark.parametrize("hash_n", [0, 1, 2])
@pytest.mark.parametrize("N", [2, 5, 8, 10])
@pytest.mark.parametrize("kind", ["hex", "quad", "surface", "line"])
def test_device_setup(kind, N, hash_n):
    # hash_n = 1, 2: cells with more elements than sixteen lanes hold
    if kind == "hex":
        nodes = W.curve_hex(W.box_mesh(3, 5, N), 0.1)
    elif kind == "quad":
        nodes = W.curve_quad2d(W.box_mesh(2, 12, N), 12)
    elif kind == "surface":
        nodes = W.sphere(n_pts=64, ne=4, N=N)["nodes"]
    else:
        nodes = W.line2d(level=1, per_elem=1, N=N)["nodes"]
    D = nodes.shape[1]
    R = {"hex": 3, "quad": 2, "surface": 2, "line": 1}[kind]
    moved = nodes.copy()
    for d in range(D):
        moved[:, d] += 0.01 * np.sin(3.0 * nodes[:, (d + 1) % D] + d)
    fpts = _fpts()
    a = fpts.Mesh(nodes, N, dim=D, ref_dim=R, hash_n=hash_n)
    a.update_nodes(torch.from_numpy(np.ascontiguousarray(moved)).cuda())
    b = fpts.Mesh(moved, N, dim=D, ref_dim=R, hash_n=hash_n)
    for x, y in zip(a.boxes(), b.boxes()):
        assert np.array_equal(x, y)
    for x, y in zip(a.cells(), b.cells()):
        assert np.array_equal(np.asarray(x), np.asarray(y))


def test_more_requests_than_one_copy():
    N, nf = 4, 2
    nodes = W.curve_hex(W.box_mesh(3, 4, N), 0.1)
    rng = np.random.default_rng(800)
    field = torch.from_numpy(np.stack([W.nodal_field(nodes, W.poly_coeffs(3, 3, rng))
                                       for _ in range(nf)])).cuda()
    fpts = _fpts()
    mesh = fpts.Mesh(nodes, N)
    server = fpts.Server(1 << 30, n_streams=1, max_batch_points=1 << 20)
    mid = server.add_mesh(mesh, field)
    pts = [torch.from_numpy(W.uniform_points(rng, int(k), 3, -0.02, 1.02)).cuda()
           for k in rng.integers(1, 700, 37)]
    torch.cuda.synchronize()
    got = [server.submit(mid, p) for p in pts]
    server.drain()
    for p, (rid, out) in zip(pts, got):
        ref, u = mesh.find_eval(p, field)
        torch.cuda.synchronize()
        for k in ref:
            assert torch.equal(out[k], ref[k]), k
        key = [k for k in out if k not in ref][0]
        assert torch.equal(torch.nan_to_num(out[key]), torch.nan_to_num(u))
        server.release(rid)
    server.close()
