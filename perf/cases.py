"""What users of the library have it do, as timed cases.

A case is one call of a public entry point on one mesh (or batch of meshes): a box of
nx x ny x nz cells, each one brick or six tetrahedra.  ``prepare`` makes the mesh on the
GPU from a seed (jittered nodes, log-uniform coefficients, optionally random numbering)
and the reusable context a program keeps; ``run`` is one call; ``exact`` gives the same
outputs from plain torch in 64 bits.
"""
from __future__ import annotations

import math
import random

import torch

import paper_1501_04784_amd as kb

DEV = "cuda"

#: the fields of a case that is one mesh, with the values most cases share
_MESH = {"order": "natural", "jitter": 0.2, "coef_lo": 1e-2, "coef_hi": 1e2, "prec": "fp32fb64", "op": "stiffness"}


def _case(name, call, elem, nx, ny, nz, **more):
    return {"name": name, "call": call, "elem": elem, "nx": nx, "ny": ny, "nz": nz, **_MESH, **more}


def listed():
    return [
        # a small mesh in an interactive or optimisation loop: launches and latency count
        _case("build_hex_1k_fp64", "build", 8, 10, 10, 10, prec="fp64", coef_lo=1.0, coef_hi=1.0),
        # a script's single call, allocations and the final synchronisation included
        _case("onecall_hex_64k", "onecall", 8, 40, 40, 40),
        # a mesh generator's randomly numbered bricks, a context kept over many builds
        _case("build_hex_1m", "build", 8, 100, 100, 100, order="nodes", jitter=0.25),
        # the benchmark's mesh: 20.25M tetrahedra, nodes and elements in random order
        _case("build_tet_20m", "build", 4, 150, 150, 150, order="both", coef_lo=1e-3, coef_hi=1e3),
        # the largest table row: 27M undistorted bricks in grid order, double precision
        _case("build_hex_27m_fp64", "build", 8, 300, 300, 300, prec="fp64", jitter=0.0),
        # a data set of 256 boxes of unlike sizes built in one call
        {"name": "batch_256_hex", "call": "batch", "elem": 8, "meshes": 256, "lo": 8, "hi": 64, "shapes": 4,
         **_MESH},
        # the adjoint of a brick mesh, as one step of a gradient loop with its own context
        _case("adjoint_hex_262k", "adjoint", 8, 64, 64, 64, prec="fp64", coef_lo=1e-1, coef_hi=1e1),
        # forward and backward through torch.autograd on a mid-size tetrahedral mesh
        _case("autograd_tet_162k", "autograd", 4, 30, 30, 30, order="both", prec="fp64", jitter=0.15,
              coef_lo=1e-3, coef_hi=1e3),
        # a vector problem's element matrices (3 components per node) assembled
        _case("assemble_dof3_hex_1m", "assemble", 8, 100, 100, 100, order="nodes", dof=3),
        # the mass matrix of a box of odd sides, double precision
        _case("mass_tet_1m4_fp64", "build", 4, 61, 47, 83, op="mass", prec="fp64"),
        # element groups with carried sums (the form that meshes beyond one pass take)
        _case("grouped_tet_20m", "grouped", 4, 150, 150, 150, groups=2, coef_lo=1e-3, coef_hi=1e3),
        # the element integrals alone, for a program that assembles them itself
        _case("integrate_hex_1m_fp64", "integrate", 8, 100, 100, 100, order="nodes", prec="fp64"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def box(lo, hi):  # about log-uniform cells, sides of unlike lengths
        side = math.exp(rng.uniform(math.log(lo), math.log(hi)) / 3)
        a, b = rng.uniform(0.7, 1.4), rng.uniform(0.7, 1.4)
        return [max(1, int(side * a)), max(1, int(side * b)), max(1, int(side / (a * b)))]

    call = rng.choice(["build", "build", "build", "onecall", "batch", "adjoint", "autograd", "assemble", "grouped",
                       "integrate"])
    elem = rng.choice([8, 4])
    hi_c = 10.0 ** rng.choice([1, 2, 3])
    common = {"order": rng.choice(["natural", "nodes", "both"]),
              "jitter": rng.choice([0.0, 0.1, 0.2 if elem == 8 else 0.15]),
              "coef_lo": 1.0 / hi_c, "coef_hi": hi_c, "prec": rng.choice(["fp64", "fp32", "fp32fb64"]),
              "op": "stiffness"}
    if call == "batch":
        lo = rng.randint(2, 8)
        return {"call": call, "elem": elem, "meshes": log_int(4, 256), "lo": lo,
                "hi": rng.randint(lo + 4, 64 if elem == 8 else 32), "shapes": rng.randrange(1 << 20), **common}
    #: cells, from the smallest to the largest listed case of each call
    most = {"build": 27e6 if elem == 8 else 3.375e6, "onecall": 1e6 if elem == 8 else 2e5, "adjoint": 1e6,
            "autograd": 2e5, "assemble": 1e6 if elem == 8 else 4e5, "grouped": 5e6 if elem == 8 else 3.375e6,
            "integrate": 4e6}[call]
    nx, ny, nz = box(1000 if elem == 8 else 170, most * 0.9)
    case = {"call": call, "elem": elem, "nx": nx, "ny": ny, "nz": nz, **common}
    if call in ("build", "onecall", "integrate"):
        case["op"] = rng.choice(["stiffness", "stiffness", "mass"])
    if call in ("adjoint", "autograd"):
        case["prec"] = "fp64"
    if call == "assemble":
        case["dof"] = rng.randint(1, 3)
    if call == "grouped":
        case["groups"] = rng.randint(2, 5)
    return case


# ------------------------------------------------------------------------- meshes
# corner offsets of a brick, and of the six tetrahedra of a cell (one per order of the
# axes; the last two corners swapped for odd orders, so every volume is positive)
_HEX = ((0, 0, 0), (1, 0, 0), (1, 1, 0), (0, 1, 0), (0, 0, 1), (1, 0, 1), (1, 1, 1), (0, 1, 1))


def _tets():
    out = []
    for p, odd in (((0, 1, 2), 0), ((0, 2, 1), 1), ((1, 0, 2), 1), ((1, 2, 0), 0), ((2, 0, 1), 0), ((2, 1, 0), 1)):
        v = [[0, 0, 0]]
        for axis in p[:2]:
            nxt = list(v[-1])
            nxt[axis] = 1
            v.append(nxt)
        v.append([1, 1, 1])
        if odd:
            v[2], v[3] = v[3], v[2]
        out.append([tuple(x) for x in v])
    return out


_TETS = _tets()


def _sizes(elem, nx, ny, nz):
    """(elements, nodes, entries of the lower triangle)"""
    cells, x, y, z = nx * ny * nz, nx + 1, ny + 1, nz + 1
    nn = x * y * z
    if elem == 8:
        return cells, nn, ((3 * nx + 1) * (3 * ny + 1) * (3 * nz + 1) + nn) // 2
    edges = nx * y * z + x * ny * z + x * y * nz
    return 6 * cells, nn, nn + edges + nx * ny * z + nx * y * nz + x * ny * nz + cells


def _mesh(elem, nx, ny, nz, order, jitter, coef_lo, coef_hi, gen):
    """conn int32 [n_elem, elem], coords float64 [n_node, 3], coef float64 [n_elem] on the GPU."""
    h = 1.0 / max(nx, ny, nz)
    ax = [torch.arange(n + 1, device=DEV) for n in (nx, ny, nz)]
    k, j, i = torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    ijk = torch.stack((i, j, k), -1).reshape(-1, 3)
    top = torch.tensor([nx, ny, nz], device=DEV)
    coords = ijk.to(torch.float64) * h
    if jitter:
        inner = ((ijk > 0) & (ijk < top)).all(1, keepdim=True)
        coords = coords + inner * (torch.rand(coords.shape, generator=gen, device=DEV, dtype=torch.float64) * 2 - 1) * (
            jitter * h)
    cell = ((ijk < top).all(1)).nonzero().reshape(-1)  # each cell by its first corner's node
    at = lambda c: c[0] + (nx + 1) * (c[1] + (ny + 1) * c[2])  # noqa: E731
    if elem == 8:
        conn = torch.stack([cell + at(c) for c in _HEX], 1)
    else:
        conn = torch.stack([cell + at(c) for t in _TETS for c in t], 1).reshape(-1, 4)
    if order != "natural":
        perm = torch.randperm(coords.shape[0], generator=gen, device=DEV)
        moved = torch.empty_like(coords)
        moved[perm] = coords
        coords, conn = moved, perm[conn]
    if order == "both":
        conn = conn[torch.randperm(conn.shape[0], generator=gen, device=DEV)]
    u = torch.rand(conn.shape[0], generator=gen, device=DEV, dtype=torch.float64)
    coef = torch.exp(u * math.log(coef_hi / coef_lo) + math.log(coef_lo))
    return conn.to(torch.int32).contiguous(), coords.contiguous(), coef


def _one_mesh(case, gen):
    return _mesh(case["elem"], case["nx"], case["ny"], case["nz"], case["order"], case["jitter"], case["coef_lo"],
                 case["coef_hi"], gen)


def _boxes(case):
    """The cells per axis of each mesh of a batch."""
    r = random.Random(case["shapes"])
    return [tuple(r.randint(case["lo"], case["hi"]) for _ in range(3)) for _ in range(case["meshes"])]


def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _inputs(case, seed):
    """Everything that is drawn: the mesh (or the meshes packed back to back, with offsets),
    given element values, weights."""
    gen = _generator(seed)
    if case["call"] == "batch":
        parts, eo, no = [], [0], [0]
        for n in _boxes(case):
            parts.append(_mesh(case["elem"], *n, case["order"], case["jitter"], case["coef_lo"], case["coef_hi"], gen))
            eo.append(eo[-1] + parts[-1][0].shape[0])
            no.append(no[-1] + parts[-1][1].shape[0])
        conn, coords, coef = (torch.cat(x).contiguous() for x in zip(*parts))
        return {"conn": conn, "coords": coords, "coef": coef, "eo": eo, "no": no}
    conn, coords, coef = _one_mesh(case, gen)
    got = {"conn": conn, "coords": coords, "coef": coef}
    nnz = _sizes(case["elem"], case["nx"], case["ny"], case["nz"])[2]
    if case["call"] == "assemble":
        nd = case["elem"] * case["dof"]
        got["klow"] = torch.randn((conn.shape[0], nd * (nd + 1) // 2), generator=gen, device=DEV,
                                  dtype=kb.value_dtype(case["prec"]))
    if case["call"] in ("adjoint", "autograd"):
        got["w"] = torch.randn(nnz, generator=gen, device=DEV, dtype=torch.float64)
    return got


# ------------------------------------------------------------------- the calls timed
def _dof_nnz(case):
    """Entries of the lower triangle with dof components per node: each pair of nodes a
    dof x dof block, of the diagonal pairs only the lower triangle."""
    _, nn, nnz = _sizes(case["elem"], case["nx"], case["ny"], case["nz"])
    d = case["dof"]
    return (nnz - nn) * d * d + nn * (d * (d + 1) // 2)


def prepare(case, seed):
    s = _inputs(case, seed)
    call, elem, prec = case["call"], case["elem"], case["prec"]
    s["case"] = case
    if call == "batch":
        s["batch"] = kb.Batch(elem, s["conn"], s["coords"], s["coef"],
                              torch.tensor(s["eo"], dtype=torch.int64, device=DEV),
                              torch.tensor(s["no"], dtype=torch.int64, device=DEV), tuple(s["eo"]), tuple(s["no"]))
        s["ctx"] = kb.BatchBuilder(s["batch"], prec=prec, cap=sum(_sizes(elem, *n)[2] for n in _boxes(case)))
        return s
    n_elem, n_node, nnz = _sizes(elem, case["nx"], case["ny"], case["nz"])
    if call == "build":
        s["ctx"] = kb.Builder(elem, n_elem, n_node, prec=prec, cap=nnz, op=case["op"])
    elif call == "assemble":
        s["ctx"] = kb.Builder(elem, n_elem, n_node, prec=prec, cap=_dof_nnz(case), dof=case["dof"])
    elif call == "grouped":
        s["ctx"] = kb.GroupedBuilder(elem, n_elem, n_node, -(-n_elem // case["groups"]), nnz, prec=prec)
    elif call == "adjoint":
        k = kb.build_lower_csr(s["conn"], s["coords"], s["coef"], elem, prec="fp64", cap=nnz)
        s["row_ptr"], s["col_idx"] = k.row_ptr, k.col_idx
        s["ctx"] = kb.AdjointBuilder(elem, n_elem, n_node)
    elif call == "autograd":
        s["coords"].requires_grad_(True)
        s["coef"].requires_grad_(True)
    return s


def run(s):
    case, conn, coords, coef = s["case"], s["conn"], s["coords"], s["coef"]
    call, ctx = case["call"], s.get("ctx")
    if call in ("build", "grouped"):
        ctx.run(conn, coords, coef)
        return {"row_ptr": ctx.row_ptr, "col_idx": ctx.col_idx, "vals": ctx.vals, "nnz": ctx.nnz_dev,
                "status": ctx.status}
    if call == "onecall":
        k = kb.build_lower_csr(conn, coords, coef, case["elem"], prec=case["prec"], op=case["op"])
        return {"row_ptr": k.row_ptr, "col_idx": k.col_idx, "vals": k.vals, "status": k.status}
    if call == "batch":
        ctx.run()
        return {"row_ptr": ctx.row_ptr, "col_idx": ctx.col_idx, "vals": ctx.vals, "nnz": ctx.nnz_off,
                "status": ctx.status}
    if call == "assemble":
        ctx.run(conn, None, None, klow=s["klow"])
        return {"row_ptr": ctx.row_ptr, "col_idx": ctx.col_idx, "vals": ctx.vals, "nnz": ctx.nnz_dev,
                "status": ctx.status}
    if call == "adjoint":
        ctx.run(conn, coords, coef, s["row_ptr"], s["col_idx"], s["w"])
        return {"grad_coef": ctx.grad_coef, "grad_coords": ctx.grad_coords, "status": ctx.status}
    if call == "autograd":
        vals, row_ptr, col_idx = kb.lower_csr_values(coords, coef, conn, case["elem"])
        gx, gc = torch.autograd.grad(vals, (coords, coef), s["w"])
        return {"row_ptr": row_ptr, "col_idx": col_idx, "vals": vals, "grad_coef": gc, "grad_coords": gx}
    out, status = kb.integrate_lower(conn, coords, coef, case["elem"], prec=case["prec"], op=case["op"])
    return {"vals": out, "status": status}


# -------------------------------------------------------------------------- work
def _element_flops(elem, op):
    """Operations of one element's integral (multiplications and additions)."""
    if elem == 8:  # per point: J 3x3 over 8 nodes, determinant and adjugate, then B and B^T B (or N N^T)
        return 8 * (144 + 32 + (120 + 24 + 36 * 6 if op == "stiffness" else 36 * 2)) + 36
    return 9 + 32 + (9 + 12 + 10 * 5 if op == "stiffness" else 2) + 10


def work(case):
    elem, call = case["elem"], case["call"]
    v = 8 if case["prec"] == "fp64" else 4
    boxes = _boxes(case) if call == "batch" else [(case["nx"], case["ny"], case["nz"])]
    n_elem, n_node, nnz = (sum(x) for x in zip(*(_sizes(elem, *n) for n in boxes)))
    te = elem * (elem + 1) // 2
    mesh = 4 * elem * n_elem + 8 * n_elem + 24 * n_node
    csr = 4 * (n_node + 1) + (4 + v) * nnz
    flops = n_elem * _element_flops(elem, case["op"])
    # P = G S G^T and the gradient of each corner at every point, beside J and G
    back = n_elem * (8 * (144 + 32 + 120 + 384 + 144 + 192) if elem == 8 else 50 + 96 + 72 + 96)
    if call == "integrate":
        return {"bytes": mesh + n_elem * te * v, "flops": flops}
    if call == "assemble":
        nd = elem * case["dof"]
        pairs = n_elem * nd * (nd + 1) // 2
        return {"bytes": 4 * elem * n_elem + v * pairs + 4 * (case["dof"] * n_node + 1) + (4 + v) * _dof_nnz(case),
                "flops": pairs}
    if call == "adjoint":
        return {"bytes": mesh + csr + 8 * n_elem + 24 * n_node, "flops": back}
    if call == "autograd":
        return {"bytes": mesh + csr + mesh + csr + 8 * n_elem + 24 * n_node, "flops": flops + n_elem * te + back}
    return {"bytes": mesh + csr, "flops": flops + n_elem * te}


# ------------------------------------------------------- the same in 64 bits, by torch
def _dn(elem):
    """(derivatives [points, 3, nodes], values [points, nodes], weight) of the rule."""
    if elem == 4:
        d = torch.tensor([[[-1.0, 1, 0, 0], [-1, 0, 1, 0], [-1, 0, 0, 1]]], dtype=torch.float64, device=DEV)
        return d, torch.full((1, 4), 0.25, dtype=torch.float64, device=DEV), 1.0 / 6.0
    c = torch.tensor(_HEX, dtype=torch.float64, device=DEV) * 2 - 1  # natural corner signs
    g = 1.0 / math.sqrt(3.0)
    pts = torch.tensor([(a, b, d) for a in (-g, g) for b in (-g, g) for d in (-g, g)], dtype=torch.float64, device=DEV)
    f = 1 + pts[:, None, :] * c[None]  # [points, nodes, 3]
    d = torch.stack([c[None, :, 0] * f[..., 1] * f[..., 2], c[None, :, 1] * f[..., 0] * f[..., 2],
                     c[None, :, 2] * f[..., 0] * f[..., 1]], 1) / 8
    return d, f.prod(-1) / 8, 1.0


def _matrices(x, elem, op):
    """Element matrices [n, nodes, nodes] of corner coordinates x [n, nodes, 3] (coefficient 1)."""
    d, val, w = _dn(elem)
    x = x - x[:, :1].detach()  # (K and the gradients are those of any translate)
    m = 0.0
    for q in range(d.shape[0]):
        j = [[(x[:, :, c] * d[q, r]).sum(1) for c in range(3)] for r in range(3)]
        cof = [[j[(r + 1) % 3][(c + 1) % 3] * j[(r + 2) % 3][(c + 2) % 3]
                - j[(r + 1) % 3][(c + 2) % 3] * j[(r + 2) % 3][(c + 1) % 3] for c in range(3)] for r in range(3)]
        det = j[0][0] * cof[0][0] + j[0][1] * cof[0][1] + j[0][2] * cof[0][2]
        if op == "mass":
            if elem == 4:  # exact: V (1 + delta) / 20
                one = torch.ones((4, 4), dtype=torch.float64, device=DEV) + torch.eye(4, dtype=torch.float64,
                                                                                     device=DEV)
                return (det / 120)[:, None, None] * one
            m = m + det[:, None, None] * (val[q][:, None] * val[q][None])
            continue
        for c in range(3):  # row c of B = J^-1 dN, J^-1 = cofactors^T / det
            b = sum(cof[r][c][:, None] * d[q, r] for r in range(3))
            m = m + (w / det)[:, None, None] * (b[:, :, None] * b[:, None, :])
    return m


def _tril(n):
    a, b = torch.tril_indices(n, n, device=DEV)
    return a, b


def _packed(s, case, chunk=1 << 18):
    """Lower triangles [n_elem, pairs] of c k_e."""
    a, b = _tril(case["elem"])
    out = torch.empty((s["conn"].shape[0], a.numel()), dtype=torch.float64, device=DEV)
    for e in range(0, out.shape[0], chunk):
        x = s["coords"][s["conn"][e:e + chunk].long()]
        out[e:e + chunk] = _matrices(x, case["elem"], case["op"])[:, a, b] * s["coef"][e:e + chunk, None]
    return out


def _assembled(conn, k, n_node, most=1 << 27):
    """(row_ptr, col_idx, vals) of the lower pairs of conn [n, m] with values k, equal
    (row, column) summed; by ranges of rows, to bound the memory of the sort."""
    a, b = _tril(conn.shape[1])
    ea, eb = conn[:, a], conn[:, b]
    row, col, k = torch.maximum(ea, eb).reshape(-1), torch.minimum(ea, eb).reshape(-1), k.reshape(-1)
    counts = torch.zeros(n_node, dtype=torch.int64, device=DEV).index_add_(
        0, row.long(), torch.ones((), dtype=torch.int64, device=DEV).expand(row.numel()))
    ends = torch.cumsum(counts, 0)
    cols, vals, per_row, lo = [], [], [], 0
    while lo < n_node:
        done = int(ends[lo - 1]) if lo else 0
        hi = max(lo + 1, int(torch.searchsorted(ends, torch.tensor(done + most, device=DEV), right=True)))
        at = ((row >= lo) & (row < hi)).nonzero().reshape(-1) if hi - lo < n_node else slice(None)
        key, to = torch.unique(row[at].long() * n_node + col[at], return_inverse=True)
        vals.append(torch.zeros(key.numel(), dtype=torch.float64, device=DEV).index_add_(0, to, k[at].double()))
        cols.append((key % n_node).to(torch.int32))
        per_row.append(torch.bincount(key // n_node - lo, minlength=hi - lo))
        lo = hi
    rp = torch.zeros(n_node + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.cumsum(torch.cat(per_row), 0)
    return rp.to(torch.int32), torch.cat(cols), torch.cat(vals)


def _gradients(s, case, row_ptr, col_idx, chunk=1 << 16):
    """(dL/dcoef, dL/dcoords) of L = sum w K over the lower pattern, by torch.autograd."""
    elem, n_node = case["elem"], s["coords"].shape[0]
    a, b = _tril(elem)
    rows = torch.repeat_interleave(torch.arange(n_node, device=DEV), (row_ptr[1:] - row_ptr[:-1]).long())
    keys = rows * n_node + col_idx
    gc = torch.empty_like(s["coef"])
    gx = torch.zeros((n_node, 3), dtype=torch.float64, device=DEV)
    for e in range(0, gc.numel(), chunk):
        conn = s["conn"][e:e + chunk].long()
        ea, eb = conn[:, a], conn[:, b]
        wk = s["w"][torch.searchsorted(keys, torch.maximum(ea, eb) * n_node + torch.minimum(ea, eb))]
        x = s["coords"][conn].detach().requires_grad_(True)
        part = (_matrices(x, elem, "stiffness")[:, a, b] * wk).sum(1)
        c = s["coef"][e:e + chunk].detach()
        g, = torch.autograd.grad((part * c).sum(), x)
        gc[e:e + chunk] = part.detach()
        gx.index_add_(0, conn.reshape(-1), g.reshape(-1, 3))
    return gc, gx


def exact(case, seed):
    s = _inputs(case, seed)
    call = case["call"]
    with torch.no_grad():
        if call == "integrate":
            return {"vals": _packed(s, case), "status": None}
        conn, n_node = s["conn"], s["coords"].shape[0]
        if call == "batch":
            eo, no = (torch.tensor(x, device=DEV) for x in (s["eo"], s["no"]))
            base = torch.repeat_interleave(no[:-1], eo[1:] - eo[:-1])
            conn = (conn + base[:, None]).to(torch.int32)
            s = dict(s, conn=conn)
        if call == "assemble":
            d = case["dof"]
            conn = (conn[:, :, None] * d + torch.arange(d, device=DEV, dtype=torch.int32)).reshape(conn.shape[0], -1)
            n_node *= d
        k = s["klow"] if call == "assemble" else _packed(s, case)
        row_ptr, col_idx, vals = _assembled(conn, k, n_node)
        del k
    if call in ("adjoint", "autograd"):
        gc, gx = _gradients(s, case, row_ptr, col_idx)
        if call == "adjoint":
            return {"grad_coef": gc, "grad_coords": gx, "status": None}
        return {"row_ptr": row_ptr, "col_idx": col_idx, "vals": vals, "grad_coef": gc, "grad_coords": gx}
    if call == "batch":  # each mesh's rows counted from its own first entry, columns in its own ids
        first = row_ptr[no[:-1]]
        parts = [row_ptr[lo:hi + 1] - row_ptr[lo] for lo, hi in zip(s["no"][:-1], s["no"][1:])]
        per_mesh = torch.diff(torch.cat([first, row_ptr[-1:]])).long()
        col_idx = (col_idx - torch.repeat_interleave(no[:-1], per_mesh)).to(torch.int32)
        return {"row_ptr": torch.cat(parts), "col_idx": col_idx, "vals": vals,
                "nnz": torch.cat([first, row_ptr[-1:]]).long(), "status": None}
    out = {"row_ptr": row_ptr, "col_idx": col_idx, "vals": vals, "status": None}
    if call != "onecall":
        out["nnz"] = row_ptr[-1:].long()
    return out
