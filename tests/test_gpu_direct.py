"""Pass 1 writing straight to the sub-buckets (few sub-buckets, or elements numbered with
locality) against the two-level partition: the sums are exact, so the matrices must be
equal bit for bit.  Widths set by hand (``seg_pairs``) force the two levels."""
import numpy as np
import pytest
import torch

import meshgen
import paper_1501_04784_amd as kb

pytestmark = pytest.mark.gpu

TWO_LEVEL = kb.Tuning(seg_pairs=4096)


def on_gpu(m):
    return tuple(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (m.conn, m.coords, m.coef))


def assert_same(a, b):
    assert a.nnz == b.nnz and a.flags == b.flags and a.n_fallback == b.n_fallback
    assert torch.equal(a.row_ptr, b.row_ptr) and torch.equal(a.col_idx, b.col_idx) and torch.equal(a.vals, b.vals)


# cells per axis: one element; a tile and one more; about the 1024 sub-buckets of the array
# (16384 brick nodes at 16 rows each) and one layer more; many sub-buckets (the hash)
SHAPES = {8: [(1, 1, 1), (64, 1, 1), (65, 2, 2), (31, 31, 15), (31, 31, 16), (40, 39, 41)],
          4: [(1, 1, 1), (11, 1, 1), (12, 8, 2), (31, 31, 31), (31, 31, 32), (40, 39, 41)]}


@pytest.mark.parametrize("prec", ["fp64", "fp32fb64"])
@pytest.mark.parametrize("op", ["stiffness", "mass"])
@pytest.mark.parametrize("order", ["natural", "random"])
@pytest.mark.parametrize("elem", [8, 4])
def test_direct_equals_two_level(elem, order, op, prec):
    for i, (nx, ny, nz) in enumerate(SHAPES[elem]):
        m = meshgen.box_mesh(elem, nx, ny, nz, jitter=0.15, coef=(0.01, 100.0), seed=i,
                             permute_nodes=order == "random", permute_elems=order == "random")
        print(f"[direct] {elem} {nx}x{ny}x{nz} {order} {op} {prec}", flush=True)
        conn, coords, coef = on_gpu(m)
        a = kb.build_lower_csr(conn, coords, coef, elem, prec=prec, op=op)
        assert_same(a, kb.build_lower_csr(conn, coords, coef, elem, prec=prec, op=op, tuning=TWO_LEVEL))


@pytest.mark.parametrize("elem,prec", [(8, "fp64"), (8, "fp32"), (4, "fp64"), (4, "fp32fb64")])
def test_rows_without_a_slot(elem, prec):
    """Grid-ordered elements (so the samples choose the hash) but for one tile's worth from
    all over the mesh, which touches more sub-buckets than the hash has slots: those rows
    take their places one by one."""
    m = meshgen.box_mesh(elem, 56, 56, 60, jitter=0.1, coef=(0.1, 10.0), seed=3)
    conn, coef = m.conn.copy(), m.coef.copy()
    n, k = conn.shape[0], 1500
    at = np.random.default_rng(7).choice(n, k, replace=False)
    to = np.arange(n // 16, n // 16 + k)  # between the sampled tiles (at multiples of n / 8)
    for a in (conn, coef):
        a[to], a[at] = a[at].copy(), a[to].copy()
    conn, coords, coef = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (conn, m.coords, coef))
    print(f"[no slot] {elem} {prec}", flush=True)
    a = kb.build_lower_csr(conn, coords, coef, elem, prec=prec)
    assert_same(a, kb.build_lower_csr(conn, coords, coef, elem, prec=prec, tuning=TWO_LEVEL))
    g = kb.build_lower_csr_grouped(conn, coords, coef, elem, -(-n // 3), a.nnz, prec=prec)
    h = kb.build_lower_csr_grouped(conn, coords, coef, elem, -(-n // 3), a.nnz, prec=prec, tuning=TWO_LEVEL)
    assert_same(g, h)


@pytest.mark.parametrize("elem,dof", [(8, 1), (8, 2), (8, 3), (4, 1), (4, 2), (4, 3)])
@pytest.mark.parametrize("n", [3, 22])
def test_given_values(elem, dof, n):
    m = meshgen.box_mesh(elem, n, n + 1, n + 2, seed=1)
    nd = elem * dof
    klow = torch.randn((m.n_elem, nd * (nd + 1) // 2), dtype=torch.float64, device="cuda",
                       generator=torch.Generator("cuda").manual_seed(n))
    conn = torch.from_numpy(m.conn).cuda()
    print(f"[direct values] {elem} dof {dof} n {n}", flush=True)
    a = kb.assemble_lower_csr(conn, m.n_node, klow, elem, dof=dof)
    assert_same(a, kb.assemble_lower_csr(conn, m.n_node, klow, elem, dof=dof, tuning=TWO_LEVEL))


def test_bad_elements_are_left_out_either_way():
    m = meshgen.box_mesh(8, 30, 30, 30, jitter=0.1, seed=2)
    conn = m.conn.copy()
    conn[5, 3], conn[77, 0], conn[900, 7] = m.n_node, -4, conn[900, 1]
    args = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (conn, m.coords, m.coef)]
    print("[direct flags]", flush=True)
    a, b = (kb.build_lower_csr(*args, 8, prec="fp64", check=False, tuning=t) for t in (None, TWO_LEVEL))
    assert a.flags == 3
    assert_same(a, b)
