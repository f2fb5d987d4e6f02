"""Meshes in random order, large enough for the launches that only those take."""
import numpy as np
import pytest
import torch

import meshgen
import paper_1501_04784_amd as kb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32fb64"])
def test_a_workgroup_per_tile(prec):
    """Bricks in random order in more than 512 buckets (of 2^11 rows here): pass 1 takes a
    workgroup per tile, 4269 of them (odd, so the last of FP64's pairs of tiles is half empty,
    and not a multiple of the XCDs); the two levels set by hand walk the same tiles with
    persistent workgroups."""
    m = meshgen.box_mesh(8, 103, 103, 103, jitter=0.2, coef=(0.01, 100.0), permute_nodes=True, permute_elems=True,
                         seed=11)
    assert -(-m.n_node // 2**11) > 512 and -(-m.n_elem // 256) == 4269
    mesh = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (m.conn, m.coords, m.coef)]
    print(f"[workgroup per tile] {prec}", flush=True)
    a, b = (kb.build_lower_csr(*mesh, 8, prec=prec, tuning=t)
            for t in (kb.Tuning(sub_bits=1), kb.Tuning(sub_bits=1, seg_pairs=4096)))
    assert a.nnz == b.nnz == meshgen.box_nnz(8, 103, 103, 103) and a.n_fallback == b.n_fallback
    assert torch.equal(a.row_ptr, b.row_ptr) and torch.equal(a.col_idx, b.col_idx) and torch.equal(a.vals, b.vals)


@pytest.mark.parametrize("elem,n,prec", [(8, (129, 131, 128), "fp64"), (8, (129, 131, 128), "fp32fb64"),
                                         (4, (60, 61, 59), "fp32")])
@pytest.mark.parametrize("elements", ["in grid order", "random"])
def test_renumbered(elem, n, prec, elements):
    """A mesh renumbered at random, which takes the two levels, is the mesh in grid order, which
    goes direct, with rows and columns renumbered: bit for bit, since the sums are exact."""
    m = meshgen.box_mesh(elem, *n, jitter=0.15, coef=(0.01, 100.0), seed=12)
    conn, coords, coef = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (m.conn, m.coords, m.coef))
    print(f"[renumbered] {elem} {n} {prec} {elements}", flush=True)
    a = kb.build_lower_csr(conn, coords, coef, elem, prec=prec)
    gen = torch.Generator("cuda").manual_seed(13)
    to = torch.randperm(m.n_node, generator=gen, device="cuda")  # node i becomes to[i]
    moved = torch.empty_like(coords)
    moved[to] = coords
    conn = to[conn.long()].to(torch.int32)
    if elements == "random":
        by = torch.randperm(m.n_elem, generator=gen, device="cuda")
        conn, coef = conn[by].contiguous(), coef[by]
    b = kb.build_lower_csr(conn, moved, coef, elem, prec=prec)
    assert a.nnz == b.nnz == meshgen.box_nnz(elem, *n) and a.n_fallback == b.n_fallback

    def keys(k, number):
        rows = torch.repeat_interleave(torch.arange(m.n_node, device="cuda"), (k.row_ptr[1:] - k.row_ptr[:-1]).long())
        r, c = number(rows), number(k.col_idx.long())
        return torch.maximum(r, c) * m.n_node + torch.minimum(r, c)

    key, at = keys(a, lambda i: to[i]).sort()
    assert torch.equal(key, keys(b, lambda i: i))  # (rows and their columns ascend)
    assert torch.equal(a.vals[at], b.vals)
