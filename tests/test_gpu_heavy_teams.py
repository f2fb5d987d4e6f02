"""Heavy sub-buckets of builds of at most 2^16 pairs, which teams of workgroups of one launch
reduce: against sums of whole numbers by numpy, and no slower than the same rows in a build
just too large for the teams."""
import numpy as np
import pytest
import torch

import meshgen
import paper_1501_04784_amd as kb

pytestmark = pytest.mark.gpu


def assembled(conn, klow, n_node):
    """(row_ptr, col_idx, vals) by numpy."""
    a, b = np.tril_indices(conn.shape[1])
    ea, eb = conn[:, a].astype(np.int64), conn[:, b].astype(np.int64)
    key, to = np.unique(np.maximum(ea, eb) * n_node + np.minimum(ea, eb), return_inverse=True)
    vals = np.bincount(to.reshape(-1), klow.reshape(-1))
    return np.searchsorted(key, np.arange(n_node + 1) * n_node), key % n_node, vals


def check(conn, n_node, prec, tuning=None):
    rng = np.random.default_rng(conn.size)
    te = conn.shape[1] * (conn.shape[1] + 1) // 2
    klow = rng.integers(-8, 9, (conn.shape[0], te)).astype(np.float64)
    k = kb.assemble_lower_csr(torch.from_numpy(conn).cuda(), n_node,
                              torch.from_numpy(klow).to("cuda", kb.value_dtype(prec)), conn.shape[1], prec=prec,
                              tuning=tuning)
    row_ptr, col, vals = assembled(conn, klow, n_node)
    assert np.array_equal(k.row_ptr.cpu().numpy(), row_ptr) and np.array_equal(k.col_idx.cpu().numpy(), col)
    assert np.array_equal(k.vals.cpu().numpy().astype(np.float64), vals)


def fans(count, tets):
    conn = [meshgen.fan_mesh(tets, seed=i).conn.astype(np.int64) + i * (3 * tets + 1) for i in range(count)]
    return np.concatenate(conn).astype(np.int32), count * (3 * tets + 1)


@pytest.mark.parametrize("prec", ["fp64", "fp32fb64"])
@pytest.mark.parametrize("count,tets", [(1, 342), (1, 2000), (1, 6553), (3, 1500), (10, 650)])
def test_fans(count, tets, prec):
    """One sub-bucket and a team of 64; its most pairs; teams that do not divide the grid."""
    print(f"[teams] {count} x {tets} {prec}", flush=True)
    check(*fans(count, tets), prec)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_more_sub_buckets_than_teams(prec):
    """Tetrahedra that share no node with a table too small for their 640 entries in 256 rows:
    103 sub-buckets, of which teams take 64."""
    conn = np.random.default_rng(1).permutation(4 * 6553).reshape(-1, 4).astype(np.int32)
    print(f"[teams, many] {prec}", flush=True)
    check(conn, conn.size, prec, kb.Tuning(table_slots=512))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_digits_wider_than_a_leaf(prec):
    """1500 tetrahedra around the last of 2^24 nodes: the digits of its row are 8192 columns
    wide, those of the other rows 2^23, and their keys lie far apart."""
    n_node = 1 << 24
    rng = np.random.default_rng(2)
    conn = np.concatenate([rng.choice(n_node - 600, (1500, 3), replace=False),
                           np.full((1500, 1), n_node - 1)], 1)
    conn[:300, 2] = n_node - 2 - rng.integers(0, 200, 300)  # and rows beside it
    assert all(len(set(c)) == 4 for c in conn)
    print(f"[teams, wide] {prec}", flush=True)
    check(conn.astype(np.int32), n_node, prec)


def test_grouped_fan():
    """Residuals: the sums of two groups, both of them the teams'."""
    m = meshgen.fan_mesh(1200)
    mesh = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (m.conn, m.coords, m.coef)]
    print("[teams, grouped]", flush=True)
    a = kb.build_lower_csr(*mesh, 4, prec="fp32fb64")
    g = kb.build_lower_csr_grouped(*mesh, 4, 700, a.nnz, prec="fp32fb64")
    assert torch.equal(a.row_ptr, g.row_ptr) and torch.equal(a.col_idx, g.col_idx)
    assert (a.vals - g.vals).abs().max() <= 2.0 ** -23 * a.vals.abs().max()


def milliseconds(conn, n_node, klow, elem=4):
    b = kb.Builder(elem, conn.shape[0], n_node, prec="fp64")
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    b.run(conn, None, None, klow=klow)
    torch.cuda.synchronize()
    ev[0].record()
    for _ in range(5):
        b.run(conn, None, None, klow=klow)
    ev[1].record()
    torch.cuda.synchronize()
    return ev[0].elapsed_time(ev[1]) / 5


@pytest.mark.parametrize("count,tets", [(1, 500), (1, 4000), (10, 650)])
def test_time(count, tets):
    """Fans beside as many tetrahedra that share no node as it takes to leave the teams: that
    build's time is the whole device's, which the teams' may exceed by half at most."""
    conn, n = fans(count, tets)
    more = 6600 - len(conn)
    beside = np.concatenate([conn + 4 * more, np.arange(4 * more, dtype=np.int32).reshape(-1, 4)])
    print(f"[teams, time] {count} x {tets}", flush=True)
    ms = [milliseconds(torch.from_numpy(c).cuda(), nn, torch.ones((len(c), 10), dtype=torch.float64, device="cuda"))
          for c, nn in ((conn, n), (beside, n + 4 * more))]
    assert ms[0] < 1.5 * ms[1], ms
