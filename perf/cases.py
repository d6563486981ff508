"""The calls that programs built on this library spend their time in, as
cases that can be prepared, run and checked.

Every case is one pass through the public Python entry points
(``paper_2501_12349_amd.fpts``): Find + Interpolate in one call or in two,
Interpolate alone, a particle-tracking step, a search after the mesh moved,
and a burst of requests to the serving loop, on quad, hex, surface and line
meshes of the orders and sizes of the repository's workloads.

Points are made from known reference coordinates (element, r), so that
``exact`` can state what Find and Interpolate have to return in 64 bits
without searching: interior points are the element map at (element, r);
points outside a box-shaped mesh have their closest point on one of its flat
sides; points beside a surface or a curve lie on the element's normal.
"""
import math

import numpy as np
import torch

# --------------------------------------------------------------------------
# The cases.
# --------------------------------------------------------------------------

BASE = {"path": "find_eval", "mesh": "hex", "order": 7, "side": 8, "points": 1000, "fields": 1,
        "field_order": 0, "precision": "fp64"}


def _case(name=None, **kw):
    c = dict(BASE)
    c.update(kw)
    if not c["field_order"]:
        c["field_order"] = c["order"]
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a probe of a small 2D mesh (a boundary rake, a few sensors): the
        # smallest call, where launches count
        _case("quad_p4_1k", mesh="quad", order=4, side=8, points=1000, fields=2),
        # an ordinary request against a resident high-order mesh
        _case("hex_p9_20k_mixed", order=9, side=12, points=20000, precision="mixed"),
        # grid-to-grid transfer: a million points of another mesh, a few per
        # cent of them outside; Find once, then Interpolate
        _case("hex_p5_1m_two_calls", path="find_then_eval", order=5, side=16, points=1020000),
        # the cubic 3D mesh of the triple-point kind (65 thousand elements)
        _case("hex_p3_4m", order=3, side=40, points=4000000),
        # the large high-order search with a velocity field
        _case("hex_p7_5m", order=7, side=32, points=5000000, fields=3),
        # the same with FP32 Newton + FP64 polish, at a ragged size
        _case("hex_p7_1m3_mixed", order=7, side=24, points=1300021, fields=3, precision="mixed"),
        # fixed points, a new field every time step: Interpolate alone, the
        # field two orders below the geometry (pressure), four of them
        _case("eval_p7_q5_3m", path="eval", order=7, side=24, points=3000000, fields=4,
              field_order=5),
        # points on and near a curved surface
        _case("surface_p6_2m", mesh="surface", order=6, side=32, points=2000000, fields=2),
        # points along interfaces (line elements in 2D), in element order
        _case("line_p3_5m", mesh="line", order=3, side=5376, points=5376000),
        # one time step of particles in a channel
        _case("lpt_p7_2m", path="lpt", mesh="channel", order=7, side=12, points=2000000, fields=3),
        # a mesh that moves between searches (r-adaptivity)
        _case("moving_p5_200k", path="update", order=5, side=18, points=200000),
        # a burst of requests to two resident meshes
        _case("serve_8_requests", path="serve", order=5, side=20, points=100000,
              precision="mixed"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same paths: orders 1 to 9, both precisions, point
    counts spread over their logarithm (nearly all odd and ragged)."""
    path = rng.choice(["find_eval", "find_eval", "find_eval", "find_then_eval", "eval", "lpt",
                       "update", "serve"])
    prec = rng.choice(["fp64", "mixed"])
    if path == "lpt":
        return _case(path=path, mesh="channel", order=rng.choice([3, 5, 7]),
                     side=rng.randint(6, 12), points=_log_int(rng, 5e3, 2e6), fields=3,
                     precision=prec, hint=rng.random() < 0.4)
    if path == "serve":
        return _case(path=path, order=rng.choice([3, 5, 7]), side=rng.randint(8, 18),
                     points=_log_int(rng, 1e3, 2e5), precision=prec)
    if path == "update":
        return _case(path=path, mesh=rng.choice(["quad", "hex"]), order=rng.randint(2, 7),
                     side=rng.randint(6, 18), points=_log_int(rng, 1e3, 5e5), precision=prec)
    mesh = rng.choice(["hex", "hex", "hex", "quad", "surface", "line"])
    order = rng.randint(1, 9) if mesh in ("hex", "quad") else rng.randint(3, 7)
    top = {"hex": 3e6 if order <= 7 else 1e6, "quad": 3e6, "surface": 1e6, "line": 4e6}[mesh]
    side = {"hex": lambda: rng.randint(4, 24 if order <= 7 else 16),
            "quad": lambda: _log_int(rng, 8, 300),
            "surface": lambda: rng.randint(8, 32),
            "line": lambda: 84 * _log_int(rng, 1, 128)}[mesh]()
    c = _case(path=path, mesh=mesh, order=order, side=side, points=_log_int(rng, 1e3, top),
              fields=rng.randint(1, 4), precision=prec)
    if path == "eval" and rng.random() < 0.5:
        c["field_order"] = rng.randint(1, 9)
    return c


# --------------------------------------------------------------------------
# Tensor-product elements in torch, FP64.
# --------------------------------------------------------------------------

def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _gll(N):
    """GLL nodes on [-1, 1]."""
    if N == 2:
        return np.array([-1.0, 1.0])
    inner = np.polynomial.legendre.Legendre.basis(N - 1).deriv().roots().real
    z = np.concatenate([[-1.0], np.sort(inner), [1.0]])
    return 0.5 * (z - z[::-1])


def _bases(N, r):
    """phi_i(r): [N][n]."""
    z = _gll(N)
    out = []
    for i in range(N):
        v = torch.ones_like(r)
        for m in range(N):
            if m != i:
                v = v * ((r - z[m]) / (z[i] - z[m]))
        out.append(v)
    return torch.stack(out)


def _diff(N):
    """D[m][i] = phi_i'(z_m)."""
    z = _gll(N)
    D = np.zeros((N, N))
    for i in range(N):
        for m in range(N):
            if m == i:
                D[m, i] = sum(1.0 / (z[i] - z[k]) for k in range(N) if k != i)
            else:
                D[m, i] = np.prod([(z[m] - z[k]) / (z[i] - z[k]) for k in range(N)
                                   if k not in (i, m)]) / (z[i] - z[m])
    return torch.from_numpy(D).to(_dev())


def _interp(vals, elem, r):
    """vals [nel][C][N^R] at (elem [n], r [R][n]): [C][n], the tensor sum
    taken directly, in chunks."""
    R, n = r.shape
    C, NP = vals.shape[1], vals.shape[2]
    N = int(round(NP ** (1.0 / R)))
    out = torch.empty((C, n), dtype=torch.float64, device=vals.device)
    step = max(1024, (1 << 25) // (C * NP))
    for s in range(0, n, step):
        sl = slice(s, min(n, s + step))
        e, v = elem[sl].long(), None
        v = vals[e]                                         # [k][C][NP]
        for d in range(R):
            phi = _bases(N, r[d, sl]).t()                   # [k][N]
            v = (v.reshape(v.shape[0], C, -1, N) * phi[:, None, None, :]).sum(-1)
        out[:, sl] = v.reshape(v.shape[0], C).t()
    return out


def _gen(seed, salt):
    g = torch.Generator(device=_dev())
    g.manual_seed(1000003 * int(seed) + salt)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, dtype=torch.float64, device=_dev())


def _box_params(dim, side, N):
    """Parameter-space node coordinates of a side^dim box mesh of [0,1]^dim:
    [nel][dim][N^dim], first index fastest, and each element's cell."""
    t = torch.from_numpy(0.5 * (_gll(N) + 1.0)).to(_dev())
    ax = (torch.arange(side, dtype=torch.float64, device=_dev())[:, None] + t[None, :]) / side
    # element id a + side (b + side c); node i + N j + N^2 k
    comps = []
    for d in range(dim):
        es = [1] * dim
        ns = [1] * dim
        es[dim - 1 - d] = side
        ns[dim - 1 - d] = N
        comps.append(ax.reshape(es + ns).expand([side] * dim + [N] * dim)
                     .reshape(side ** dim, N ** dim))
    return torch.stack(comps, dim=1).contiguous()


def _curve(X, amp, side):
    """The workloads' curving maps: the identity on the sides of the box."""
    if X.shape[1] == 2:
        d = amp / side * torch.sin(2 * math.pi * X[:, 0]) * torch.sin(2 * math.pi * X[:, 1])
    else:
        d = amp * torch.sin(math.pi * X[:, 0]) * torch.sin(math.pi * X[:, 1]) * \
            torch.sin(math.pi * X[:, 2])
    return X + d[:, None, :]


CHANNEL_L = (2.0 * math.pi, 2.0, math.pi)


def _channel_y(eta):
    return torch.tanh(1.5 * eta) / math.tanh(1.5)


def _channel_cells(side):
    """Elements per direction: 1.5 : 1 : 1.5, as in the 36 x 24 x 36 channel."""
    return (3 * side // 2, side, 3 * side // 2)


def _nodes(case, seed):
    """Node coordinates [nel][dim][N^R]."""
    N, side, kind = case["order"] + 1, case["side"], case["mesh"]
    if kind in ("quad", "hex"):
        amp = (0.05 if kind == "quad" else 0.1) * (1.0 + 0.2 * ((seed % 7) / 7.0))
        return _curve(_box_params(2 if kind == "quad" else 3, side, N), amp, side)
    t = torch.from_numpy(0.5 * (_gll(N) + 1.0)).to(_dev())
    if kind == "channel":
        cells = _channel_cells(side)
        ax = [(torch.arange(m, dtype=torch.float64, device=_dev())[:, None] + t[None, :]) / m
              for m in cells]
        ax = [CHANNEL_L[0] * ax[0], _channel_y(2.0 * ax[1] - 1.0), CHANNEL_L[2] * ax[2]]
        comps = []
        for d in range(3):
            es, ns = [1, 1, 1], [1, 1, 1]
            es[2 - d], ns[2 - d] = cells[d], N
            comps.append(ax[d].reshape(es + ns).expand([cells[2], cells[1], cells[0], N, N, N])
                         .reshape(-1, N ** 3))
        return torch.stack(comps, dim=1).contiguous()
    if kind == "line":
        # a closed wavy curve
        s = (torch.arange(side, dtype=torch.float64, device=_dev())[:, None] + t[None, :]) / side
        th = 2.0 * math.pi * s
        rad = 1.0 + 0.2 * torch.cos(3.0 * th + 0.1 * (seed % 11))
        return torch.stack([rad * torch.cos(th), rad * torch.sin(th)], dim=1).contiguous()
    # surface: cubed sphere, equiangular faces, radius 1 + a small cubic bump
    P = _box_params(2, side, N)
    X, Y = torch.tan((P[:, 0] - 0.5) * math.pi / 2), torch.tan((P[:, 1] - 0.5) * math.pi / 2)
    o = torch.ones_like(X)
    out = []
    for f in ((o, X, Y), (-o, -X, Y), (-X, o, Y), (X, -o, Y), (-Y, X, o), (Y, X, -o)):
        u = torch.stack(f, dim=1)
        u = u / u.norm(dim=1, keepdim=True)
        a = 0.1 * (seed % 11)
        bump = u[:, 0] * u[:, 1] * u[:, 2] + 0.3 * u[:, 2] ** 3 + 0.2 * a * u[:, 0] ** 2 * u[:, 1]
        out.append((1.0 + 0.05 * bump)[:, None, :] * u)
    return torch.cat(out).contiguous()


def _ref_dim(case):
    return {"quad": 2, "hex": 3, "channel": 3, "surface": 2, "line": 1}[case["mesh"]]


def _dim(case):
    return {"quad": 2, "hex": 3, "channel": 3, "surface": 3, "line": 2}[case["mesh"]]


def _field_nodes(case, seed):
    """Coordinates at which the field's nodal values are taken (the mesh's
    own nodes, or those of the field's order on the same mesh)."""
    return _nodes(dict(case, order=case["field_order"]), seed)


def _fields(case, seed):
    """[fields][nel][Nf^R]: smooth waves at the nodes, a few per domain; the
    channel's are its velocity."""
    X = _field_nodes(case, seed)
    if case["mesh"] == "channel":
        w = 1.0 - X[:, 1] ** 2
        p = 0.3 * (seed % 13)
        sx, cx = torch.sin(X[:, 0] + p), torch.cos(X[:, 0] + p)
        u = 1.5 * w - 0.2 * w * X[:, 1] * sx
        v = -0.05 * w * w * cx
        return torch.stack([u, v, 0.05 * w * sx]).contiguous()
    g = _gen(seed, 7)
    out = []
    for f in range(case["fields"]):
        k = 1.0 + 2.0 * _rand(g, X.shape[1]) + 0.3 * f
        ph = 6.0 * _rand(g, 1)
        out.append(torch.sin((X * k[None, :, None]).sum(1) + ph))
    return torch.stack(out).contiguous()


# --------------------------------------------------------------------------
# Points and the answers that go with them.
# --------------------------------------------------------------------------

def _points(case, seed, nodes, n, salt=0):
    """Query points of the case and what Find has to say of them: pts
    [dim][n], code, elem, r, dist."""
    g = _gen(seed, 11 + salt)
    dim, R, nel = _dim(case), _ref_dim(case), nodes.shape[0]
    code = torch.zeros(n, dtype=torch.int32, device=_dev())
    dist = torch.zeros(n, dtype=torch.float64, device=_dev())
    # about two in a hundred lie outside the mesh: half of them just off it,
    # half in no element's boxes
    n_near, n_far = n // 100, n // 100
    if case["mesh"] == "line":
        # a run of points per element, along the curve
        elem = torch.arange(n, device=_dev()) * nel // n
    else:
        elem = torch.randint(nel, (n,), generator=g, device=_dev())
    margin = 1e-6 if R == dim else 1e-3
    r = (2.0 * _rand(g, R, n) - 1.0) * (1.0 - margin)
    x = _interp(nodes, elem, r)
    where = torch.randperm(n, generator=g, device=_dev())
    if R == dim:
        side = case["side"]
        off, far = where[:n_near], where[n_near:n_near + n_far]
        for idx, lo, hi in ((off, 0.002, 0.02), (far, 0.6, 1.2)):
            k = idx.numel()
            if not k:
                continue
            c = 0.02 + 0.96 * _rand(g, dim, k)          # place on the side
            d = torch.randint(dim, (k,), generator=g, device=_dev())
            up = torch.randint(2, (k,), generator=g, device=_dev())
            gap = (lo + (hi - lo) * _rand(g, k)) / side
            c[d, torch.arange(k, device=_dev())] = up.double()
            cell = torch.clamp((c * side).floor(), 0, side - 1)
            mul = torch.tensor([side ** a for a in range(dim)], device=_dev(),
                               dtype=torch.float64)
            elem[idx] = (cell * mul[:, None]).sum(0).long()
            r[:, idx] = torch.clamp(2.0 * (c * side - cell) - 1.0, -1.0, 1.0)
            y = c.clone()
            y[d, torch.arange(k, device=_dev())] += torch.where(up > 0, gap, -gap)
            x[:, idx] = y
            code[idx] = 1
            dist[idx] = gap
    else:
        # along the normal of the element
        Dm = _diff(case["order"] + 1)
        N = case["order"] + 1
        if R == 1:
            t = _interp(torch.matmul(nodes, Dm.t().contiguous()), elem, r)
            nrm = torch.stack([-t[1], t[0]])
            h = 2.0 * math.pi / case["side"]
            near = min(5e-6, 0.002 * h)
            off = 0.005 * h if 0.005 * h > 4e-5 else 0.0
            share = 0.1
        else:
            V = nodes.reshape(nel, 3, N, N)
            t1 = _interp(torch.matmul(V, Dm.t().contiguous()).reshape(nel, 3, -1), elem, r)
            t2 = _interp(torch.matmul(Dm, V).reshape(nel, 3, -1).contiguous(), elem, r)
            nrm = torch.linalg.cross(t1, t2, dim=0)
            near, off, share = 5e-6, min(1e-3, 0.006 * math.pi / 2 / case["side"]), 0.7
        nrm = nrm / nrm.norm(dim=0)
        s = torch.where(_rand(g, n) < 0.5, -1.0, 1.0)
        a = near * (0.05 + 0.95 * _rand(g, n))
        if off:
            out = _rand(g, n) < share
            a = torch.where(out, 2e-5 + (off - 2e-5) * _rand(g, n), a)
            code = torch.where(out, 1, 0).to(torch.int32)
        dist = a
        x = x + s * a * nrm
        far = where[:n_far]
        u = torch.randn((dim, far.numel()), generator=g, dtype=torch.float64, device=_dev())
        x[:, far] = u / u.norm(dim=0) * (1.5 + 0.5 * _rand(g, far.numel()))
    elem = elem.to(torch.int32)
    code[far], elem[far], dist[far] = 2, -1, math.inf
    r[:, far] = 0.0
    return x.contiguous(), code, elem, r.contiguous(), dist


def _expected(case, seed, nodes, fields, n, salt=0):
    x, code, elem, r, dist = _points(case, seed, nodes, n, salt)
    u = _interp(fields.transpose(0, 1).contiguous(), elem.clamp(min=0), r)
    u[:, code == 2] = math.nan
    return {"code": code, "elem": elem, "r": r, "dist": dist, "u": u}


def _particles(case, seed):
    """Particles of the channel: positions (one in a hundred just beyond a
    wall of the mesh), velocities and the box they live in."""
    g = _gen(seed, 17)
    n = case["points"]
    L = CHANNEL_L
    x = torch.stack([L[0] * _rand(g, n), 2.0 * _rand(g, n) - 1.0, L[2] * _rand(g, n)])
    cells = _channel_cells(case["side"])
    gap = 0.02 * (1.0 - float(_channel_y(torch.tensor(1.0 - 2.0 / cells[1],
                                                      dtype=torch.float64))))
    k = n // 100
    x[1, :k] = torch.where(_rand(g, k) < 0.5, -1.0, 1.0) * (1.0 + gap * (0.2 + 0.6 * _rand(g, k)))
    x = x[:, torch.randperm(n, generator=g, device=_dev())].contiguous()
    v = torch.stack([1.5 * (1.0 - x[1] ** 2), 0.02 * torch.sin(x[0]), 0.02 * torch.cos(x[2])])
    return x, v.contiguous(), (0.0, -1.0 - gap, 0.0), (L[0], 1.0 + gap, L[2])


TAU, DT = 5.0, 1e-3


def _locate_channel(case, x):
    """(elem, r, distance) of the closest points of the channel to x."""
    cells, N = _channel_cells(case["side"]), case["order"] + 1
    L, rs, ix = CHANNEL_L, [], []
    y = x[1].clamp(-1.0, 1.0)
    for d, s in ((0, x[0] / L[0]), (2, x[2] / L[2])):
        c = (s * cells[d]).floor().clamp(0, cells[d] - 1)
        ix.append(c.long())
        rs.append((2.0 * (s * cells[d] - c) - 1.0).clamp(-1.0, 1.0))
    m = cells[1]
    edge = _channel_y(2.0 * torch.arange(m + 1, dtype=torch.float64, device=x.device) / m - 1.0)
    b = (torch.searchsorted(edge, y, right=True) - 1).clamp(0, m - 1)
    t = torch.from_numpy(0.5 * (_gll(N) + 1.0)).to(x.device)
    yn = _channel_y(2.0 * (torch.arange(m, dtype=torch.float64, device=x.device)[:, None] +
                           t[None, :]) / m - 1.0)                      # [m][N]
    dyn = torch.matmul(yn, _diff(N).t().contiguous())
    r = (2.0 * (y - edge[b]) / (edge[b + 1] - edge[b]) - 1.0).clamp(-1.0, 1.0)
    for _ in range(8):
        p = _bases(N, r).t()
        r = (r + (y - (yn[b] * p).sum(1)) / (dyn[b] * p).sum(1)).clamp(-1.0, 1.0)
    r = torch.where(y >= 1.0, torch.ones_like(r), torch.where(y <= -1.0, -torch.ones_like(r), r))
    elem = ix[0] + cells[0] * (b + cells[1] * ix[1])
    return elem, torch.stack([rs[0], r, rs[1]]), (x[1] - y).abs()


def _requests(case):
    """(mesh, points) of eight requests: sizes spread over their logarithm
    up to the case's, alternating between two meshes."""
    rng = np.random.default_rng(23 + case["points"])
    n = case["points"]
    sizes = np.exp(rng.uniform(np.log(n / 32.0), np.log(n), size=8)).astype(np.int64) + 1
    sizes[0] = n
    return [(int(k % 2), int(s)) for k, s in enumerate(sizes)]


def _serve_case(case, k):
    """Resident mesh k of the serving case: the case's own, and a cubic one."""
    return case if k == 0 else _case(mesh="hex", order=3, side=case["side"],
                                     precision=case["precision"])


# --------------------------------------------------------------------------
# prepare, run, work, exact.
# --------------------------------------------------------------------------

def prepare(case, seed):
    from paper_2501_12349_amd import fpts
    path, N = case["path"], case["order"] + 1
    state = {"case": dict(case)}
    if path == "serve":
        server = fpts.Server(budget_bytes=1 << 30, n_streams=4, max_batch_points=1 << 20)
        nodes = []
        for k in range(2):
            c = _serve_case(case, k)
            nodes.append(_nodes(c, seed))
            mesh = fpts.Mesh(nodes[k].cpu().numpy(), c["order"] + 1)
            server.add_mesh(mesh, _fields(c, seed))
        state["requests"] = [
            (k, _points(_serve_case(case, k), seed, nodes[k], n, salt=31 + i)[0])
            for i, (k, n) in enumerate(_requests(case))]
        state["server"] = server
        return state
    nodes = _nodes(case, seed)
    if path == "update":
        # set up on the straight-sided mesh; the moved nodes come from the
        # application, on the device
        straight = _box_params(_dim(case), case["side"], N)
        state["mesh"] = fpts.Mesh(straight.cpu().numpy(), N)
        state["nodes"] = nodes
    else:
        state["mesh"] = fpts.Mesh(nodes.cpu().numpy(), N, ref_dim=_ref_dim(case))
    state["field"] = _fields(case, seed)
    if path == "lpt":
        x, v, lo, hi = _particles(case, seed)
        P = fpts.Particles(x, v, TAU, DT, lo, hi, (1, 0, 1), hint=bool(case.get("hint")))
        state["particles"] = P.start(state["mesh"], precision=case["precision"])
        P.hist[0].copy_(v)                       # as a step before this one left it
        return state
    state["pts"] = _points(case, seed, nodes, case["points"])[0]
    if path == "eval":
        state["found"] = state["mesh"].find(state["pts"], precision=case["precision"])
    return state


def run(state):
    case, prec = state["case"], state["case"]["precision"]
    path = case["path"]
    if path == "serve":
        server = state["server"]
        got = [server.submit(k, pts, precision=prec) for k, pts in state["requests"]]
        server.drain()
        for rid, _ in got:
            server.release(rid)
        return [out for _, out in got]
    mesh = state["mesh"]
    if path == "lpt":
        P = state["particles"]
        mesh.lpt_step(P, state["field"], precision=prec)
        return dict(x=P.x, v=P.v, hist=P.hist, **P.find)
    if path == "eval":
        return {"u": mesh.eval(state["found"], state["field"],
                               field_nodes_1d=case["field_order"] + 1)}
    if path == "find_then_eval":
        res = mesh.find(state["pts"], precision=prec)
        return dict(res, u=mesh.eval(res, state["field"]))
    if path == "update":
        mesh.update_nodes(state["nodes"])
    res, u = mesh.find_eval(state["pts"], state["field"], precision=prec)
    return dict(res, u=u)


def _element_count(case):
    s = case["side"]
    if case["mesh"] == "channel":
        a, b, c = _channel_cells(s)
        return a * b * c
    return {"quad": s * s, "hex": s ** 3, "surface": 6 * s * s, "line": s}[case["mesh"]]


def _one(case, n, find=True, interp=True):
    """Bytes and FLOPs of one search and / or interpolation of n points: the
    points, results and touched elements once; three evaluations of the map
    and its derivatives per point, sum-factorised, and the contraction of
    each field."""
    D, R, N, Nf = _dim(case), _ref_dim(case), case["order"] + 1, case["field_order"] + 1
    nel = min(_element_count(case), n)
    b = f = 0.0
    if find:
        b += n * (8.0 * D + 4 + 4 + 8.0 * R + 8) + 8.0 * D * nel * N ** R
        rows = sum(N ** k for k in range(R))       # length-N dot products per coordinate
        f += 3.0 * n * 2.0 * D * N * (rows + R * max(rows - 1, 1))
    if interp:
        b += n * (0.0 if find else 8.0 + 8.0 * R) + 8.0 * case["fields"] * (n + nel * Nf ** R)
        f += n * 2.0 * case["fields"] * Nf * sum(Nf ** k for k in range(R))
    return b, f


def work(case):
    path, n = case["path"], case["points"]
    if path == "serve":
        parts = [_one(_serve_case(case, k), m) for k, m in _requests(case)]
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    b, f = _one(case, n, find=path != "eval")
    if path == "lpt":
        b += n * 8.0 * 3 * 8                        # x, v and the history, read and written
    if path == "update":
        b += 8.0 * _dim(case) * _element_count(case) * (case["order"] + 1) ** _ref_dim(case)
    return {"bytes": b, "flops": f}


def exact(case, seed):
    path = case["path"]
    if path == "serve":
        out = []
        cases = [_serve_case(case, k) for k in range(2)]
        nodes = [_nodes(c, seed) for c in cases]
        fields = [_fields(c, seed) for c in cases]
        for i, (k, n) in enumerate(_requests(case)):
            out.append(_expected(cases[k], seed, nodes[k], fields[k], n, salt=31 + i))
        return out
    nodes, fields = _nodes(case, seed), _fields(case, seed)
    if path == "lpt":
        # one step of Adams-Bashforth 2 on x' = v, v' = (u - v) / tau (the
        # step before had the same v and no drag), the box, then the search
        x, v, lo, hi = _particles(case, seed)
        elem, r, _ = _locate_channel(case, x)
        u = _interp(fields.transpose(0, 1).contiguous(), elem, r)
        a = (u - v) / TAU
        x1, v1 = x + DT * v, v + DT * 1.5 * a
        hv, ha = v.clone(), a.clone()
        for d in (0, 2):
            x1[d] = x1[d] - (hi[d] - lo[d]) * torch.floor((x1[d] - lo[d]) / (hi[d] - lo[d]))
        for end, out in ((hi[1], x1[1] > hi[1]), (lo[1], x1[1] < lo[1])):
            x1[1] = torch.where(out, 2.0 * end - x1[1], x1[1])
            for q in (v1, hv, ha):
                q[1] = torch.where(out, -q[1], q[1])
        elem, r, dist = _locate_channel(case, x1)
        code = (dist > 0).to(torch.int32)
        return {"x": x1, "v": v1, "hist": torch.stack([hv, ha]), "code": code,
                "elem": elem.to(torch.int32), "r": r, "dist": dist}
    want = _expected(case, seed, nodes, fields, case["points"])
    return {"u": want["u"]} if path == "eval" else want
