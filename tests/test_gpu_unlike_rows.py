"""Meshes numbered with locality whose rows are not those of a box: long rows in some ranges of
ids (the direct way's wider sub-buckets overflow there and are reduced in parts, or go on to
the heavy path), and rows shared by few elements.  The sums are exact, so the matrices equal
those of the two-level partition (``seg_pairs`` set by hand) bit for bit."""
import numpy as np
import pytest
import torch

import meshgen
import paper_1501_04784_amd as kb

pytestmark = pytest.mark.gpu

TWO_LEVEL = kb.Tuning(seg_pairs=4096)


def assert_same(a, b):
    assert a.nnz == b.nnz and a.flags == b.flags
    assert torch.equal(a.row_ptr, b.row_ptr) and torch.equal(a.col_idx, b.col_idx) and torch.equal(a.vals, b.vals)


def with_windows(elem, n):
    """A box's connectivity, then windows of consecutive ids whose nodes are joined at random:
    (ids, elements) of each kind and their number."""
    box = meshgen.box_mesh(elem, n, n, n)
    rng = np.random.default_rng(elem)
    conn, at = [box.conn], box.n_node
    for ids, elems, count in ((64, 60, 24),    # twice the entries of the box's rows: parts
                              (400, 400, 3),   # more than a part's table holds: the heavy path
                              (64, 5000, 1)):  # many pairs, more than one pass adds up
        for _ in range(count):
            conn.append(at + np.argsort(rng.random((elems, ids)), axis=1)[:, :elem])
            at += ids
    return np.concatenate(conn).astype(np.int32), at


@pytest.mark.parametrize("elem,dof,prec", [(8, 1, "fp64"), (8, 1, "fp32"), (8, 3, "fp64"), (4, 1, "fp32"),
                                           (4, 3, "fp64")])
def test_long_rows_in_ranges(elem, dof, prec):
    conn, n_node = with_windows(elem, 40 if dof == 1 else 24)
    nd = elem * dof
    klow = torch.randn((conn.shape[0], nd * (nd + 1) // 2), dtype=kb.value_dtype(prec), device="cuda",
                       generator=torch.Generator("cuda").manual_seed(dof))
    c = torch.from_numpy(conn).cuda()
    print(f"[long rows] {elem} dof {dof} {prec}", flush=True)
    a, b = (kb.assemble_lower_csr(c, n_node, klow, elem, prec=prec, dof=dof, tuning=t) for t in (None, TWO_LEVEL))
    assert_same(a, b)


@pytest.mark.parametrize("prec", ["fp64", "fp32fb64"])
def test_long_rows_in_a_grouped_build(prec):
    """The same with residuals (running sums of the groups before)."""
    conn, n_node = with_windows(8, 30)
    rng = np.random.default_rng(3)
    mesh = [torch.from_numpy(x).cuda() for x in (conn, rng.random((n_node, 3)), rng.uniform(0.5, 2, conn.shape[0]))]
    print(f"[long rows, grouped] {prec}", flush=True)
    a = kb.build_lower_csr(*mesh, 8, prec=prec, check=False)
    assert_same(a, kb.build_lower_csr(*mesh, 8, prec=prec, check=False, tuning=TWO_LEVEL))
    g, h = (kb.build_lower_csr_grouped(*mesh, 8, -(-conn.shape[0] // 3), a.nnz, prec=prec, check=False, tuning=t)
            for t in (None, TWO_LEVEL))
    assert_same(g, h)


def milliseconds(builder, mesh):
    builder.run(*mesh)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    torch.cuda.synchronize()
    ev[0].record()
    for _ in range(3):
        builder.run(*mesh)
    ev[1].record()
    torch.cuda.synchronize()
    return ev[0].elapsed_time(ev[1]) / 3


def apart(m):
    return meshgen.Mesh(m.elem, np.arange(m.conn.size, dtype=np.int32).reshape(m.conn.shape),
                        np.ascontiguousarray(m.coords[m.conn.reshape(-1)]), m.coef)


SHAPES = {"sheet": (300, 300, 1), "beam": (60000, 1, 1), "two by two": (30000, 2, 2), "apart": (40, 40, 40)}


@pytest.mark.parametrize("shape", sorted(SHAPES))
@pytest.mark.parametrize("elem", [8, 4])
def test_rows_of_few_elements(elem, shape):
    """Entries shared by few elements: more of them for a mesh's pairs than a box has.  The
    tables hold them: the build takes no longer than the two levels do (three times as long
    is allowed; overflowing tables took up to four hundred times)."""
    m = meshgen.box_mesh(elem, *SHAPES[shape], jitter=0.1, coef=(0.1, 10.0), seed=4)
    if shape == "apart":
        m = apart(m)
    mesh = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (m.conn, m.coords, m.coef)]
    print(f"[few elements] {elem} {shape}", flush=True)
    b = [kb.Builder(elem, m.n_elem, m.n_node, prec="fp32fb64", tuning=t) for t in (None, TWO_LEVEL)]
    ms = [milliseconds(x, mesh) for x in b]
    assert_same(*(x.result() for x in b))
    assert ms[0] < 3 * ms[1], ms


@pytest.mark.parametrize("n_node,prec", [(161, "fp64"), (161, "fp32"), (1000, "fp64")])
def test_rows_of_every_length(n_node, prec):
    """Random tetrahedra over few nodes: rows of every length up to n_node, at the edges of how
    many columns the ordering takes at a time, against numpy's sums of whole numbers."""
    rng = np.random.default_rng(n_node)
    # (of 161 nodes every pair occurs, some 20 times)
    conn = np.argsort(rng.random((48000 if n_node < 200 else 20000, n_node)), axis=1)[:, :4]
    klow = rng.integers(-8, 9, (len(conn), 10)).astype(np.float64)
    a, b = np.tril_indices(4)
    row, col = (f(conn[:, a], conn[:, b]).astype(np.int64) for f in (np.maximum, np.minimum))
    key, to = np.unique(row * n_node + col, return_inverse=True)
    print(f"[every length] {n_node} {prec}", flush=True)
    k = kb.assemble_lower_csr(torch.from_numpy(conn.astype(np.int32)).cuda(), n_node,
                              torch.from_numpy(klow).to("cuda", kb.value_dtype(prec)), 4, prec=prec)
    assert np.array_equal(k.row_ptr.cpu().numpy(), np.searchsorted(key, np.arange(n_node + 1) * n_node))
    assert np.array_equal(k.col_idx.cpu().numpy(), key % n_node)
    assert np.array_equal(k.vals.cpu().numpy().astype(np.float64), np.bincount(to.reshape(-1), klow.reshape(-1)))
    if n_node < 200:
        assert np.array_equal(np.diff(k.row_ptr.cpu().numpy()), np.arange(1, n_node + 1))


def test_small_boxes_in_random_order():
    """A batch of small boxes, whose last rows are twice the average: with few sub-buckets their
    tables are not filled further than the two levels' (they took 1.3 times as long)."""
    rng = np.random.default_rng(8)
    boxes = [meshgen.box_mesh(4, *(int(x) for x in rng.integers(3, 15, 3)), jitter=0.1, coef=(0.1, 10.0), seed=i,
                              permute_nodes=True, permute_elems=True) for i in range(64)]
    batch = kb.pack_batch([(m.conn, m.coords, m.coef) for m in boxes], 4, "cuda")
    print("[small boxes]", flush=True)
    b = [kb.BatchBuilder(batch, prec="fp32fb64", tuning=t) for t in (None, TWO_LEVEL)]
    ms = [milliseconds(x, ()) for x in b]
    for x, y in zip(*(x.results() for x in b)):
        assert_same(x, y)
    assert ms[0] < 1.1 * ms[1], ms
