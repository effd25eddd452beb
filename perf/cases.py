"""Performance cases of the DG solver: what a user's program asks of it.

A case is one pass through the public entry points (``Mesh``, ``DeviceMesh``,
``Batch``), in one of four paths:

``step``   a state in the mesh's own element numbering is moved into the
           layout order on the device, advanced by a few SSP-RK3 steps and
           moved back (a solver run between two outputs);
``rhs``    the right-hand side of Eq. (2), volume and surface term, of a state
           held in layout order, handed back in the mesh's own numbering (a
           user's own time integrator, or a residual monitor);
``adapt``  the solution is transferred onto a locally refined mesh (hanging
           faces, six colors) and advanced there;
``batch``  several meshes of mixed sizes advanced together by batched steps
           (the serving loop).

Meshes are jittered periodic or walled grids, numbered by the grid or at
random (as an unstructured generator numbers them); states are a smooth
density wave in the constant mode and seeded noise in the others.
"""

from __future__ import annotations

import itertools
import math

import numpy as np
import torch

import paper_1601_07613_amd as dgc

GAMMA = 1.4
DIM = {"tri": 2, "quad": 2, "mixed": 2, "tet": 3}
FACES = {"tri": 3, "quad": 4, "mixed": 4, "tet": 4}


def _case(name, path, elem, n, p, precision="f64", variant="colored", layout="paired", walls=False,
          numbering="grid", steps=1, members=0, n_lo=0):
    return {"name": name, "path": path, "elem": elem, "n": n, "p": p, "precision": precision, "variant": variant,
            "layout": layout, "walls": walls, "numbering": numbering, "steps": steps, "members": members,
            "n_lo": n_lo}


def listed():
    return [
        # the smallest call: 512 triangles, where launches and latency are all there is
        _case("tri_p1_512_step", "step", "tri", 16, 1, layout="paper", steps=10),
        # one serving-sized solve in the library's default layout
        _case("tri_p3_65k_step", "step", "tri", 181, 3, layout="paper", steps=4),
        # the benchmark's size and order, an unstructured numbering, walls as on its mesh
        _case("tri_p2_991k_step", "step", "tri", 704, 2, walls=True, numbering="random", steps=2),
        # the f32 form of the same step
        _case("tri_p2_500k_step_f32", "step", "tri", 500, 2, precision="f32", walls=True, numbering="random", steps=2),
        # the same mesh's right-hand side through the colored surface pass
        _case("tri_p2_991k_rhs", "rhs", "tri", 704, 2, walls=True, numbering="random"),
        # the highest order
        _case("tri_p5_39k_step", "step", "tri", 141, 5, steps=2),
        # three dimensions, the benchmark's Kuhn mesh at a middle size
        _case("tet_p1_511k_step", "step", "tet", 44, 1, steps=2),
        # three dimensions at the highest order, closed box
        _case("tet_p2_57k_step", "step", "tet", 21, 2, walls=True, steps=1),
        # parallelograms at the benchmark's order
        _case("quad_p2_590k_step", "step", "quad", 768, 2, steps=2),
        # a hybrid mesh: triangles and parallelograms, padded records
        _case("mixed_p2_step", "step", "mixed", 301, 2, walls=True, steps=2),
        # refinement under a running solution: transfer, then steps with hanging faces
        _case("adapt_p2_step", "adapt", "tri", 200, 2, layout="paper", steps=2),
        # the serving loop's iteration: meshes of 2e3 to 2e5 elements, f32 form
        _case("batch_p2_f32_step", "batch", "tri", 316, 2, precision="f32", layout="paper", steps=2, members=8,
              n_lo=32),
    ]


def draw(rng):
    path = rng.choice(["step", "step", "step", "rhs", "rhs", "adapt", "batch"])
    if path == "adapt":
        elem = "tri"
    elif path == "batch":
        elem = rng.choice(["tri", "tri", "quad", "tet"])         # mixed meshes are not batched
    else:
        elem = rng.choice(["tri", "tri", "tri", "quad", "mixed", "tet"])
    p = rng.choice({"tri": [1, 2, 2, 3, 4, 5], "quad": [1, 2, 3], "mixed": [1, 2, 3], "tet": [1, 1, 2]}[elem])
    precision = rng.choice(["f64", "f64", "f32"])
    variant = "colored"
    if path in ("step", "rhs"):
        variant = rng.choice(["colored"] * 6 + ["compact", "gather"])
    cap = 9e6 / (_modes(elem, p) * (DIM[elem] + 2))       # elements whose state a drawn case may hold
    K = math.exp(rng.uniform(math.log(300.0), math.log(min(6e5, cap) / (2.5 if path == "adapt" else 1.0))))
    per_cell = {"tri": 2, "quad": 1, "mixed": 1.3, "tet": 6}[elem]
    n = max(4, int(round((K / per_cell) ** (1.0 / DIM[elem]))))
    members = n_lo = 0
    if path == "batch":
        members = rng.randint(2, 12)
        n = max(4, int(n / members ** (1.0 / DIM[elem])))
        n_lo = max(4, n // 8)
    # refinement starts from a periodic mesh in the default layout
    return {"path": path, "elem": elem, "n": n, "p": p, "precision": precision, "variant": variant,
            "layout": "paper" if path == "adapt" else rng.choice(["paired", "paper", "paper_sfc"]),
            "walls": path != "adapt" and rng.random() < 0.4, "numbering": rng.choice(["grid", "random"]),
            "steps": rng.randint(1, 3), "members": members, "n_lo": n_lo}


# -- sizes -------------------------------------------------------------------
def _modes(elem, p):
    if elem == "tet":
        return (p + 1) * (p + 2) * (p + 3) // 6
    return (p + 1) * (p + 2) // 2 if elem == "tri" else (p + 1) ** 2


def _points(elem, p):
    """Quadrature points of a face and of an element."""
    if elem == "tet":
        return (3 if p <= 1 else (p + 1) ** 2), (p + 1) ** 3
    return p + 1, (p + 1) ** 2


def _member_sizes(case):
    if not case["members"]:
        return [case["n"]]
    m, lo, hi = case["members"], case["n_lo"], case["n"]
    return [int(round(lo * (hi / lo) ** (i / max(1, m - 1)))) for i in range(m)]


def _refine_flags(xyz, n):
    """The triangles to refine, by their cells' places on the unjittered grid."""
    return _in_circle((np.rint(xyz * n) / n).mean(axis=1))


def _in_circle(centers):
    return np.hypot(centers[:, 0] - 0.5, centers[:, 1] - 0.5) < 0.25


def _counts(case, n):
    """Elements and faces of one mesh."""
    if case["path"] == "adapt":
        fl = int(_refine_flags(_mesh(case, n, 0)[1], n).sum())
        K = 2 * n * n
        return K + 3 * fl, (3 * (K + 3 * fl)) // 2         # hanging faces are few
    if case["elem"] == "tet":
        return 6 * n ** 3, 12 * n ** 3 + (6 * n * n if case["walls"] else 0)
    if case["elem"] == "tri":
        return 2 * n * n, 3 * n * n + (2 * n if case["walls"] else 0)
    if case["elem"] == "quad":
        return n * n, 2 * n * n + (2 * n if case["walls"] else 0)
    split = math.pi * 0.25 ** 2 * n * n
    return int(n * n + split), int(2 * n * n + split) + (2 * n if case["walls"] else 0)


def work(case):
    """Bytes: the state in and out (and its move between the numberings); per
    stage of a step the stage's input and the step's initial state read and
    its output written, and the mesh's geometry read.  Operations: traces,
    fluxes, projections at the quadrature points."""
    elem, p = case["elem"], case["p"]
    dim, M, NP = DIM[elem], DIM[elem] + 2, _modes(elem, p)
    Q, QV = _points(elem, p)
    nbytes = flops = 0
    for n in _member_sizes(case):
        K, E = _counts(case, n)
        geo = K * (dim * dim + 1) * 8 + E * ((dim + 3) * 8 + 10)
        f1 = (K * QV * (2 * M * NP * (1 + dim) + 2 * dim * dim * M + 10 * dim + 15)
              + E * Q * (8 * M * NP + 80))
        rec = K * M * NP * (4 if case["path"] == "rhs" and case["precision"] == "f32" else 8)
        if case["path"] == "rhs":
            nbytes += 2 * rec + geo + 2 * rec + 4 * K
            flops += f1
            continue
        nbytes += case["steps"] * (8 * rec + 3 * geo)
        flops += case["steps"] * (3 * f1 + 14 * K * M * NP)
        nbytes += 4 * rec + 8 * K          # in and out of the numbering (or the transfer)
    return {"bytes": int(nbytes), "flops": int(flops)}


# -- meshes ------------------------------------------------------------------
def _mesh(case, n, seed):
    """Vertex ids ``[K, nv]`` and own coordinates ``[K, nv, dim]``."""
    rng = np.random.default_rng([seed, n, 7])
    elem, walls = case["elem"], case["walls"]
    nv, h = (n + 1 if walls else n), 1.0 / n
    if elem == "tet":
        d = rng.uniform(-0.05 * h, 0.05 * h, size=(nv, nv, nv, 3))
        if walls:
            for ax in range(3):
                np.moveaxis(d, ax, 0)[[0, -1]] = 0.0
        k, j, i = (a.ravel() for a in np.meshgrid(*[np.arange(n)] * 3, indexing="ij"))
        ev = np.empty((6 * n ** 3, 4), dtype=np.int32)
        xyz = np.empty((6 * n ** 3, 4, 3))
        for s, perm in enumerate(itertools.permutations(range(3))):
            off, corners = np.zeros(3, dtype=int), [np.zeros(3, dtype=int)]
            for ax in perm:
                off = off.copy()
                off[ax] += 1
                corners.append(off)
            if sum(perm[a] > perm[b] for a in range(3) for b in range(a + 1, 3)) % 2:
                corners[1], corners[2] = corners[2], corners[1]
            for v, o in enumerate(corners):
                a, b, c = i + o[0], j + o[1], k + o[2]
                ev[s::6, v] = a % nv + nv * (b % nv) + nv * nv * (c % nv)
                xyz[s::6, v] = np.stack([a * h, b * h, c * h], axis=1) + d[a % nv, b % nv, c % nv]
    else:
        j, i = (a.ravel() for a in np.meshgrid(np.arange(n), np.arange(n), indexing="ij"))
        if elem == "tri":
            d = rng.uniform(-0.1 * h, 0.1 * h, size=(nv, nv, 2))
            if walls:
                d[[0, -1]] = d[:, [0, -1]] = 0.0

            def pos(a, b):
                return np.stack([a * h, b * h], axis=1) + d[a % nv, b % nv]
        else:
            # column and row offsets keep every cell a parallelogram
            a0, b0, s0, t0 = rng.uniform(-0.1 * h, 0.1 * h, size=(4, n + 1))
            if walls:
                a0[[0, -1]] = b0[[0, -1]] = 0.0
                s0[:] = t0[:] = 0.0
            else:
                for a in (a0, b0, s0, t0):
                    a[n] = a[0]

            def pos(a, b):
                return np.stack([a * h + a0[a] + t0[b], b * h + b0[b] + s0[a]], axis=1)
        corner = [(i, j), (i + 1, j), (i + 1, j + 1), (i, j + 1)]
        cv = np.stack([a % nv + nv * (b % nv) for a, b in corner], axis=1).astype(np.int32)
        cx = np.stack([pos(a, b) for a, b in corner], axis=1)
        if elem == "quad":
            ev, xyz = cv, cx
        elif elem == "tri":
            ev = cv[:, [0, 1, 2, 0, 2, 3]].reshape(-1, 3)
            xyz = cx[:, [0, 1, 2, 0, 2, 3]].reshape(-1, 3, 2)
        else:
            # the cells near the center are split into two triangles
            split = _in_circle(np.stack([(i + 0.5) * h, (j + 0.5) * h], axis=1))
            start = np.cumsum(np.where(split, 2, 1)) - np.where(split, 2, 1)
            K = int(np.where(split, 2, 1).sum())
            ev = np.full((K, 4), -1, dtype=np.int32)
            xyz = np.zeros((K, 4, 2))
            ev[start[~split]], xyz[start[~split]] = cv[~split], cx[~split]
            for r, t in enumerate(([0, 1, 2], [0, 2, 3])):
                ev[start[split] + r, :3] = cv[split][:, t]
                xyz[start[split] + r, :3] = cx[split][:, t]
    if case["numbering"] == "random":
        perm = np.random.default_rng([seed, n, 8]).permutation(len(ev))
        ev, xyz = ev[perm], xyz[perm]
    return np.ascontiguousarray(ev), np.ascontiguousarray(xyz)


def _det(ev, xyz):
    """Jacobian determinant, measure and centroid of every element."""
    x0 = xyz[:, 0]
    if xyz.shape[2] == 3:
        J = np.stack([xyz[:, a] - x0 for a in (1, 2, 3)], axis=2)
        det = (J[:, :, 0] * np.cross(J[:, :, 1], J[:, :, 2])).sum(axis=1)
        return J, det, det / 6.0, xyz.mean(axis=1)
    quad = np.full(len(ev), ev.shape[1] == 4) & (ev[:, -1] >= 0)
    last = xyz[np.arange(len(ev)), np.where(quad, 3, 2)]
    J = np.stack([xyz[:, 1] - x0, last - x0], axis=2)
    det = J[:, 0, 0] * J[:, 1, 1] - J[:, 0, 1] * J[:, 1, 0]
    cen = np.where(quad[:, None], xyz.mean(axis=1), xyz[:, :3].mean(axis=1))
    return J, det, det * np.where(quad, 1.0, 0.5), cen


def _state(case, n, seed, ev, xyz):
    """Modal state ``[K, M, N_p]`` (f64) in the mesh's own numbering."""
    rng = np.random.default_rng([seed, n, 9])
    dim = DIM[case["elem"]]
    _, _, meas, cen = _det(ev, xyz)
    phase, amp = rng.uniform(0, 2 * math.pi), rng.uniform(0.1, 0.25)
    vel = rng.uniform(-0.6, 0.6, size=dim)
    rho = 1.0 + amp * np.sin(2 * math.pi * cen.sum(axis=1) + phase)
    u = np.stack([rho] + [rho * v for v in vel] + [1.0 / (GAMMA - 1.0) + 0.5 * rho * (vel ** 2).sum()], axis=1)
    c = np.zeros((len(ev), dim + 2, _modes(case["elem"], case["p"])))
    sq = np.sqrt(meas)[:, None]
    c[:, :, 0] = sq * u
    if c.shape[2] > 1:
        c[:, :, 1:] = (0.01 * sq * (np.abs(u) + 0.1))[:, :, None] * rng.standard_normal(c[:, :, 1:].shape)
    if case["elem"] == "mixed":
        c[ev[:, 3] < 0, :, _modes("tri", case["p"]):] = 0.0
    return c


def _dt(case, n):
    return 0.05 / (n * (2 * case["p"] + 1))


def _color(mesh, case):
    for seed in range(8):          # the coloring heuristic may give up on a seed
        try:
            return mesh.color(seed=seed, layout=case["layout"])
        except dgc.DgcError:
            if seed == 7:
                raise


# -- a pass ------------------------------------------------------------------
def prepare(case, seed):
    st = {"case": case, "members": []}
    for n in _member_sizes(case):
        ev, xyz = _mesh(case, n, seed)
        U0 = _state(case, n, seed, ev, xyz)
        mesh = dgc.Mesh.build(ev, xyz)
        _color(mesh, case)
        dev = dgc.DeviceMesh(mesh, case["p"])
        m = {"dt": _dt(case, n)}
        if case["path"] == "adapt":
            m["old"], m["U0"] = dev, torch.from_numpy(dev.to_layout(U0)).cuda()
            fine, _ = mesh.refine(_refine_flags(xyz, n))
            dev = dgc.DeviceMesh(fine, case["p"])
            dev.adapt_arrays()
            m["dt"] *= 0.5
        elif case["path"] == "rhs":
            dt = torch.float64 if case["precision"] == "f64" else torch.float32
            m["U0"] = torch.from_numpy(dev.to_layout(U0)).to("cuda", dt)
            m["ws"] = dev.workspace("surface", case["variant"], case["precision"])
        elif case["path"] == "batch":
            m["U0"] = torch.from_numpy(dev.to_layout(U0)).cuda()
            m["U"] = m["U0"].clone()
        else:
            m["U0"] = torch.from_numpy(U0).cuda()
        dev.to_layout_device(torch.zeros((dev.K, 1), device="cuda"))   # keeps the permutation on the device
        if case["path"] != "rhs":
            m["ws"] = dev.workspace("rk", case["variant"], case["precision"])
        m["dev"] = dev
        st["members"].append(m)
    if case["path"] == "batch":
        st["batch"] = dgc.Batch([(m["dev"], m["U"], m["ws"], m["dt"]) for m in st["members"]],
                                precision=case["precision"])
    return st


def run(st):
    case = st["case"]
    if case["path"] == "batch":
        for m in st["members"]:
            m["U"].copy_(m["U0"])
        for _ in range(case["steps"]):
            st["batch"].rk_step()
        return [m["dev"].from_layout_device(m["U"]) for m in st["members"]]
    m = st["members"][0]
    dev = m["dev"]
    if case["path"] == "rhs":
        rhs = dev.alloc(case["precision"], zero=False)
        dev.volume_rhs(m["U0"], rhs, case["precision"])
        dev.surface_rhs(m["U0"], rhs, case["variant"], case["precision"], ws=m["ws"])
        return dev.from_layout_device(rhs)
    U = dev.transfer_from(m["U0"]) if case["path"] == "adapt" else dev.to_layout_device(m["U0"])
    for _ in range(case["steps"]):
        dev.rk_step(U, m["dt"], case["variant"], case["precision"], ws=m["ws"])
    return dev.from_layout_device(U)


# -- the same in 64 bits with plain torch ------------------------------------
def _gauss_jacobi(n, a):
    """Gauss points on [-1, 1] for the weight (1 - x)^a (Golub-Welsch)."""
    k = np.arange(n, dtype=np.float64)
    diag = -a * a / np.where((2 * k + a) * (2 * k + a + 2) == 0, 1, (2 * k + a) * (2 * k + a + 2))
    k = k[1:]
    off = np.sqrt(4 * k * (k + a) * k * (k + a) / ((2 * k + a) ** 2 * (2 * k + a + 1) * (2 * k + a - 1)))
    x, v = np.linalg.eigh(np.diag(diag) + np.diag(off, 1) + np.diag(off, -1))
    return x, v[0] ** 2 * 2.0 ** (a + 1) / (a + 1)


def _volume_rule(kind, n):
    (x, wx), (y, wy), (z, wz) = (_gauss_jacobi(n, a) for a in (0, 1, 2))
    if kind == "quad":
        X, Y = np.meshgrid(0.5 * (x + 1), 0.5 * (x + 1), indexing="xy")
        return np.stack([X.ravel(), Y.ravel()], axis=1), 0.25 * np.outer(wx, wx).ravel()
    if kind == "tri":
        a, b = (g.ravel() for g in np.meshgrid(x, y, indexing="ij"))
        return np.stack([0.25 * (1 + a) * (1 - b), 0.5 * (1 + b)], axis=1), np.outer(wx, wy).ravel() / 8.0
    a, b, c = (g.ravel() for g in np.meshgrid(x, y, z, indexing="ij"))
    pts = np.stack([(1 + a) * (1 - b) * (1 - c) / 8.0, 0.25 * (1 + b) * (1 - c), 0.5 * (1 + c)], axis=1)
    return pts, (wx[:, None, None] * wy[:, None] * wz).ravel() / 64.0


def _jac(n, a, x, order):
    """Orthonormal Jacobi polynomial of degree n for (1 - x)^a, or its derivative."""
    def poly(n, a, b):
        p0, p1 = torch.ones_like(x), 0.5 * ((a + b + 2) * x + (a - b))
        if n == 0:
            return p0
        for k in range(1, n):
            c = 2 * k + a + b
            p0, p1 = p1, (((c + 1) * (a * a - b * b) + c * (c + 1) * (c + 2) * x) * p1
                          - 2 * (k + a) * (k + b) * (c + 2) * p0) / (2 * (k + 1) * (k + a + b + 1) * c)
        return p1
    norm = math.sqrt(2.0 ** (a + 1) / (2 * n + a + 1))
    if order == 0:
        return poly(n, a, 0) / norm
    return (0.5 * (n + a + 1) * poly(n - 1, a + 1, 1) / norm) if n else torch.zeros_like(x)


def _basis(kind, p, X, grad=False):
    """Basis values at reference points ``X [..., dim]`` -> ``[..., N_p]``, or
    the reference gradients ``[..., dim, N_p]``."""
    out = []
    if kind == "quad":
        x, y = 2 * X[..., 0] - 1, 2 * X[..., 1] - 1
        for b in range(p + 1):
            for a in range(p + 1):
                P = [_jac(a, 0, x, 0), _jac(b, 0, y, 0)]
                if not grad:
                    out.append(2.0 * P[0] * P[1])
                else:
                    out.append(torch.stack([4.0 * _jac(a, 0, x, 1) * P[1], 4.0 * P[0] * _jac(b, 0, y, 1)], dim=-1))
        return torch.stack(out, dim=-1)
    # collapsed coordinates; the points used are away from their poles
    if kind == "tri":
        xi, eta = X[..., 0], X[..., 1]
        e1 = 1.0 - eta
        a, b = 2.0 * xi / e1 - 1.0, 2.0 * eta - 1.0
        for d in range(p + 1):
            for j in range(d + 1):
                i = d - j
                A, B = _jac(i, 0, a, 0), _jac(j, 2 * i + 1, b, 0)
                w = 2.0 ** i * e1 ** i
                s = 2.0 * math.sqrt(2.0)
                if not grad:
                    out.append(s * A * B * w)
                    continue
                dA, dB = _jac(i, 0, a, 1), _jac(j, 2 * i + 1, b, 1)
                dw = -i * 2.0 ** i * e1 ** (i - 1) if i else torch.zeros_like(e1)
                out.append(s * torch.stack([dA * (2.0 / e1) * B * w,
                                            dA * (2.0 * xi / e1 ** 2) * B * w + A * (2.0 * dB * w + B * dw)], dim=-1))
        return torch.stack(out, dim=-1)
    x, y, z = X[..., 0], X[..., 1], X[..., 2]
    f1, f2 = 1.0 - y - z, 1.0 - z
    a, b, c = 2.0 * x / f1 - 1.0, 2.0 * y / f2 - 1.0, 2.0 * z - 1.0
    s = 8.0
    for d in range(p + 1):
        for k in range(d + 1):
            for j in range(d - k + 1):
                i = d - j - k
                A, B, Cc = _jac(i, 0, a, 0), _jac(j, 2 * i + 1, b, 0), _jac(k, 2 * i + 2 * j + 2, c, 0)
                # (1-b)^i (1-c)^(i+j) = 2^(2i+j) f1^i f2^j
                w = 2.0 ** (2 * i + j)
                if not grad:
                    out.append(s * A * B * Cc * w * f1 ** i * f2 ** j)
                    continue
                dA, dB, dC = _jac(i, 0, a, 1), _jac(j, 2 * i + 1, b, 1), _jac(k, 2 * i + 2 * j + 2, c, 1)
                zero = torch.zeros_like(x)
                da = [2.0 / f1, 2.0 * x / f1 ** 2, 2.0 * x / f1 ** 2]
                db = [zero, 2.0 / f2, 2.0 * y / f2 ** 2]
                g1 = i * f1 ** (i - 1) if i else zero
                g2 = j * f2 ** (j - 1) if j else zero
                df1, df2 = [0.0, -1.0, -1.0], [0.0, 0.0, -1.0]
                P = f1 ** i * f2 ** j
                g = []
                for e in range(3):
                    t = (dA * da[e] * B * Cc + A * dB * db[e] * Cc) * P
                    if e == 2:
                        t = t + A * B * dC * 2.0 * P
                    g.append(s * w * (t + A * B * Cc * (g1 * df1[e] * f2 ** j + f1 ** i * g2 * df2[e])))
                out.append(torch.stack(g, dim=-1))
    return torch.stack(out, dim=-1)


REF = {"tri": [[0, 0], [1, 0], [0, 1]], "quad": [[0, 0], [1, 0], [1, 1], [0, 1]],
       "tet": [[0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1]]}
LOCAL = {"tri": [[0, 1], [1, 2], [2, 0]], "quad": [[0, 1], [1, 2], [2, 3], [3, 0]],
         "tet": [[1, 2, 3], [0, 2, 3], [0, 1, 3], [0, 1, 2]]}


def _match(ev, kinds, kind):
    """Faces of a conforming mesh: left and right (element, local face, the
    places of the left side's face vertices among the element's); right
    element -1 at walls."""
    el, lf, vid = [], [], []
    for k, name in enumerate(kinds):
        rows = np.nonzero(kind == k)[0]
        for f, loc in enumerate(LOCAL[name]):
            el.append(rows)
            lf.append(np.full(len(rows), f))
            vid.append(ev[rows][:, loc])
    el, lf, vid = np.concatenate(el), np.concatenate(lf), np.concatenate(vid).astype(np.int64)
    s = np.sort(vid, axis=1)
    order = np.lexsort(tuple([lf, el] + [s[:, c] for c in range(s.shape[1])][::-1]))
    s, el, lf, vid = s[order], el[order], lf[order], vid[order]
    same = (s[1:] == s[:-1]).all(axis=1)
    first = np.concatenate([[True], ~same])
    paired = first & np.concatenate([same, [False]])
    i = np.nonzero(first)[0]
    j = np.where(paired[i], i + 1, i)
    R = np.where(paired[i], el[j], -1)
    return el[i], lf[i], R, lf[j], vid[i]


class _Exact:
    """The semi-discrete system of one mesh, from vertex ids and coordinates."""

    def __init__(self, case, ev, xyz, refine=None):
        self.p = case["p"]
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        kinds = {"mixed": ["tri", "quad"]}.get(case["elem"], [case["elem"]])
        kind = (ev[:, 3] >= 0).astype(int) if case["elem"] == "mixed" else np.zeros(len(ev), dtype=int)
        dim = xyz.shape[2]
        L, fL, R, fR, vid = _match(ev, kinds, kind)
        ref = [np.array(REF[k], dtype=np.float64) for k in kinds]

        def places(e):
            """Reference coordinates, in element e, of the faces' vertices."""
            pos = (ev[e][:, None, :] == vid[:, :, None]).argmax(axis=2)
            out = np.zeros((len(e), vid.shape[1], dim))
            for k in range(len(kinds)):
                rows = kind[e] == k
                out[rows] = ref[k][pos[rows]]
            return out

        refL, refR = places(L), places(np.where(R >= 0, R, L))
        if refine is not None:
            ev, xyz, L, R, refL, refR = _refined(xyz, refine, L, fL, R, fR)
            kind = np.zeros(len(xyz), dtype=int)
        J, det, _, _ = _det(ev, xyz)
        corner = xyz[L, 0][:, None, :] + (refL[:, :, None, :] * J[L][:, None, :, :]).sum(axis=3)
        if dim == 2:
            t = corner[:, 1] - corner[:, 0]
            meas = np.hypot(t[:, 0], t[:, 1])
            normal = np.stack([t[:, 1], -t[:, 0]], axis=1) / meas[:, None]
            s, w = _gauss_jacobi(self.p + 1, 0)
            bary, wf = np.stack([0.5 * (1 - s), 0.5 * (1 + s)], axis=1), 0.5 * w
        else:
            c = np.cross(corner[:, 1] - corner[:, 0], corner[:, 2] - corner[:, 0])
            area = np.sqrt((c ** 2).sum(axis=1))
            normal, meas = c / area[:, None], 0.5 * area
            flip = ((corner[:, 0] - xyz[L].mean(axis=1)) * normal).sum(axis=1) < 0
            normal[flip] *= -1.0
            if self.p <= 1:
                bary, wf = np.full((3, 3), 1 / 6) + 0.5 * np.eye(3), np.full(3, 1 / 3)
            else:
                pts, w = _volume_rule("tri", self.p + 1)
                bary, wf = np.column_stack([1 - pts.sum(axis=1), pts]), 2 * w

        def t(a):
            return torch.from_numpy(np.ascontiguousarray(a)).to(self.dev)

        self.NP = max(_modes(k, self.p) for k in kinds)
        self.L, self.R, self.wall = t(L), t(np.where(R >= 0, R, L)), t(R < 0)
        self.inner = (~self.wall).nonzero()[:, 0]
        self.n, self.meas, self.sq = t(normal), t(meas), t(np.sqrt(det))
        self.Ji = torch.linalg.inv(t(J))
        self.wf, tk = t(wf), t(kind)
        bary = t(bary)
        self.phi = []
        for e, rf in ((self.L, t(refL)), (self.R, t(refR))):
            X = (bary[None, :, :, None] * rf[:, None, :, :]).sum(dim=2)
            phi = torch.zeros(len(X), len(wf), self.NP, dtype=torch.float64, device=self.dev)
            for k, name in enumerate(kinds):
                rows = (tk[e] == k).nonzero()[:, 0]
                phi[rows, :, :_modes(name, self.p)] = _basis(name, self.p, X[rows])
            self.phi.append(phi)
        self.vol = []
        for k, name in enumerate(kinds):
            pts, w = _volume_rule(name, self.p + 1)
            B, D = _basis(name, self.p, t(pts)), _basis(name, self.p, t(pts), grad=True)
            self.vol.append(((tk == k).nonzero()[:, 0], B, D * t(w)[:, None, None]))

    def rhs(self, U):
        dim = self.n.shape[1]
        out = torch.zeros_like(U)
        for rows, B, D in self.vol:
            n = B.shape[1]
            sq = self.sq[rows][:, None, None]
            u = (U[rows][:, :, :n] @ B.t().contiguous()) / sq
            vel, pres = _primitive(u)
            acc = torch.zeros_like(U[rows][:, :, :n])
            F = []
            for e in range(dim):
                f = u * vel[e][:, None]
                f[:, 1 + e] += pres
                f[:, -1] += pres * vel[e]
                F.append(f)
            for d in range(dim):
                G = sum(self.Ji[rows, d, e][:, None, None] * F[e] for e in range(dim))
                acc += G @ D[:, d].contiguous()
            out[rows, :, :n] = acc * sq
        tr = [torch.bmm(U[e], ph.transpose(1, 2).contiguous()) / self.sq[e][:, None, None]
              for e, ph in ((self.L, self.phi[0]), (self.R, self.phi[1]))]
        a = tr[0]
        n = self.n[:, :, None]
        ghost = a.clone()
        ghost[:, 1:-1] -= 2.0 * (a[:, 1:-1] * n).sum(dim=1, keepdim=True) * n
        b = torch.where(self.wall[:, None, None], ghost, tr[1])
        f, lam = [], []
        for u in (a, b):
            vel, pres = _primitive(u)
            un = sum(vel[e] * self.n[:, e, None] for e in range(dim))
            g = u * un[:, None]
            g[:, 1:-1] += pres[:, None] * n
            g[:, -1] += pres * un
            f.append(g)
            lam.append(un.abs() + torch.sqrt(GAMMA * pres / u[:, 0]))
        F = 0.5 * (f[0] + f[1]) - 0.5 * torch.maximum(lam[0], lam[1])[:, None] * (b - a)
        F = F * (self.wf * self.meas[:, None])[:, None, :]
        out.index_add_(0, self.L, torch.bmm(F, self.phi[0]) / self.sq[self.L][:, None, None], alpha=-1.0)
        i = self.inner
        out.index_add_(0, self.R[i], torch.bmm(F[i], self.phi[1][i]) / self.sq[self.R[i]][:, None, None])
        return out

    def step(self, U, dt):
        a = U + dt * self.rhs(U)
        b = 0.75 * U + 0.25 * (a + dt * self.rhs(a))
        return U / 3.0 + 2.0 / 3.0 * (b + dt * self.rhs(b))


def _primitive(u):
    vel = [u[:, 1 + e] / u[:, 0] for e in range(u.shape[1] - 2)]
    return vel, (GAMMA - 1.0) * (u[:, -1] - 0.5 * sum(u[:, 1 + e] * vel[e] for e in range(len(vel))))


CHILD = np.array([[[0, 0], [.5, 0], [0, .5]], [[.5, 0], [1, 0], [.5, .5]], [[0, .5], [.5, .5], [0, 1]],
                  [[.5, .5], [0, .5], [.5, 0]]])


def _refined(xyz, flags, L, fL, R, fR):
    """One 4-way split of the flagged triangles: the leaves replace their
    parent in place (corner children at its vertices, then the center
    child); an edge split on one side only becomes two hanging faces."""
    size = np.where(flags, 4, 1)
    start = np.cumsum(size) - size
    out = np.empty((int(size.sum()), 3, 2))
    out[start[~flags]] = xyz[~flags]
    x = xyz[flags]
    J = np.stack([x[:, 1] - x[:, 0], x[:, 2] - x[:, 0]], axis=2)
    for c in range(4):
        out[start[flags] + c] = x[:, :1] + (CHILD[c][None, :, None, :] * J[:, None]).sum(axis=3)
    V = np.array(REF["tri"], dtype=np.float64)
    faces = []

    def edge(f, t0, t1):
        a, d = V[f], V[(f + 1) % 3] - V[f]
        return np.stack([a + t0 * d, a + t1 * d], axis=1)

    def add(l, rl, r, rr):
        faces.append((l, r, rl, rr))

    refL, refR = flags[L], flags[R]
    s = ~refL & ~refR
    add(start[L[s]], edge(fL[s], 0, 1), start[R[s]], edge(fR[s], 1, 0))
    s = refL & refR
    for h in (0, 1):
        # half h of the left edge lies on its corner child f + h, and on the right element's f + 1 - h
        add(start[L[s]] + (fL[s] + h) % 3, edge(fL[s], 0, 1), start[R[s]] + (fR[s] + 1 - h) % 3, edge(fR[s], 1, 0))
    for fine, ff, coarse, fc, s in ((L, fL, R, fR, refL & ~refR), (R, fR, L, fL, refR & ~refL)):
        for h in (0, 1):
            add(start[fine[s]] + (ff[s] + h) % 3, edge(ff[s], 0, 1), start[coarse[s]],
                edge(fc[s], 1 - 0.5 * h, 0.5 - 0.5 * h))
    par = np.nonzero(flags)[0]
    for k in range(3):
        kk = np.full(len(par), k)
        add(start[par] + 3, edge(kk, 0, 1), start[par] + (k + 2) % 3, edge(kk, 1, 0))
    l, r, rl, rr = (np.concatenate([f[i] for f in faces]) for i in range(4))
    return np.zeros((len(out), 3), dtype=np.int64), out, l, r, rl, rr


def _transfer(p, U, flags):
    """L2 projection onto the children of the flagged elements."""
    pts, w = _volume_rule("tri", p + 1)
    B = _basis("tri", p, torch.from_numpy(pts))
    size = np.where(flags, 4, 1)
    start = np.cumsum(size) - size
    out = torch.empty((int(size.sum()),) + U.shape[1:], dtype=torch.float64)
    out[start[~flags]] = U[~flags]
    for c in range(4):
        v = CHILD[c]
        X = v[0] + pts[:, :1] * (v[1] - v[0]) + pts[:, 1:] * (v[2] - v[0])
        P = 0.5 * (B * torch.from_numpy(w)[:, None]).t().contiguous() @ _basis("tri", p, torch.from_numpy(X))
        out[start[flags] + c] = U[flags] @ P.t().contiguous()
    return out


def exact(case, seed):
    outs = []
    for n in _member_sizes(case):
        ev, xyz = _mesh(case, n, seed)
        U = torch.from_numpy(_state(case, n, seed, ev, xyz))
        flags, dt = None, _dt(case, n)
        if case["path"] == "adapt":
            flags = _refine_flags(xyz, n)
            U, dt = _transfer(case["p"], U, flags), 0.5 * dt
        ex = _Exact(case, ev, xyz, flags)
        if case["path"] == "rhs" and case["precision"] == "f32":
            U = U.float().double()
        U = U.to(ex.dev)
        if case["path"] == "rhs":
            U = ex.rhs(U)
        else:
            for _ in range(case["steps"]):
                U = ex.step(U, dt)
        outs.append(U)
    return outs if case["path"] == "batch" else outs[0]
