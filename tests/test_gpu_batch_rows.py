"""A batch's rows and columns, written in each mesh's own numbering as the union matrix is
copied out: against the union mesh's own build, whose blocks they are (the sums are exact,
so the values must be equal bit for bit)."""
import numpy as np
import pytest
import torch

import meshgen
import paper_1501_04784_amd as kb

pytestmark = pytest.mark.gpu


# numbers of meshes about the 64 and 4096 that one and two searches by a wave tell apart
@pytest.mark.parametrize("n_mesh", [1, 64, 65, 4096, 4097])
@pytest.mark.parametrize("elem", [8, 4])
def test_batch_rows_against_the_union(elem, n_mesh):
    rng = np.random.default_rng(n_mesh)
    kinds = [meshgen.box_mesh(elem, *c, jitter=0.15, coef=(0.1, 10.0), permute_nodes=True, seed=i)
             for i, c in enumerate([(1, 1, 1), (1, 2, 1), (3, 2, 2), (5, 4, 6)])]
    no_node = meshgen.Mesh(elem, np.zeros((0, elem), np.int32), np.zeros((0, 3)), np.zeros(0))
    no_elem = meshgen.Mesh(elem, np.zeros((0, elem), np.int32), np.ones((3, 3)), np.zeros(0))
    kinds += [no_node, no_elem]
    pick = rng.choice(6, size=n_mesh, p=[0.5, 0.2, 0.1, 0.05, 0.1, 0.05])
    pick[0] = 2
    meshes = [kinds[k] for k in pick]
    print(f"[batch rows] elem={elem} n_mesh={n_mesh}", flush=True)
    got = kb.build_lower_csr_batched([(m.conn, m.coords, m.coef) for m in meshes], elem, prec="fp64")
    off = np.concatenate([[0], np.cumsum([m.n_node for m in meshes])])
    union = [np.concatenate([m.conn + o for m, o in zip(meshes, off)]).astype(np.int32),
             np.concatenate([m.coords for m in meshes]), np.concatenate([m.coef for m in meshes])]
    one = kb.build_lower_csr(*(torch.from_numpy(a).cuda() for a in union), elem, prec="fp64")
    rp, col, val = (t.cpu().numpy() for t in (one.row_ptr, one.col_idx, one.vals))
    assert len(got) == n_mesh
    for r, a, b in zip(got, off[:-1], off[1:]):
        first, last = rp[a], rp[b]
        np.testing.assert_array_equal(r.row_ptr.cpu().numpy(), rp[a:b + 1] - first)
        np.testing.assert_array_equal(r.col_idx.cpu().numpy(), col[first:last] - a)
        np.testing.assert_array_equal(r.vals.cpu().numpy(), val[first:last])
