"""Meshes of so many tiles that a workgroup of the counting kernel takes several of them, a
ragged last group among them: the number of entries is known in closed form, the sums are
exact, so the two ways of partitioning give the same bits, and small whole numbers as
element values add up to the same total in the matrix."""
import numpy as np
import pytest
import torch

import meshgen
import paper_1501_04784_amd as kb

pytestmark = pytest.mark.gpu

TWO_LEVEL = kb.Tuning(seg_pairs=4096)


def couplings(nx, ny, nz):
    """Ordered pairs of nodes that share a brick."""
    return (3 * nx + 1) * (3 * ny + 1) * (3 * nz + 1)


@pytest.mark.parametrize("prec", ["fp64", "fp32fb64"])
@pytest.mark.parametrize("order", ["natural", "random"])
def test_brick_build(order, prec):
    nx, ny, nz = 129, 131, 128  # 2.16M bricks: more than 16 groups per CU of 256-element tiles
    m = meshgen.box_mesh(8, nx, ny, nz, permute_nodes=order == "random", permute_elems=order == "random", seed=5)
    print(f"[count groups] bricks {order} {prec}", flush=True)
    t = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (m.conn, m.coords, m.coef)]
    a, b = (kb.build_lower_csr(*t, 8, prec=prec, tuning=tu) for tu in (None, TWO_LEVEL))
    assert a.nnz == b.nnz == (couplings(nx, ny, nz) + m.n_node) // 2
    assert torch.equal(a.row_ptr, b.row_ptr) and torch.equal(a.col_idx, b.col_idx) and torch.equal(a.vals, b.vals)


@pytest.mark.parametrize("order", ["natural", "random"])
def test_three_component_assembly(order):
    nx, ny, nz = 65, 63, 67  # 274,365 bricks of 24 rows, a few dozen a tile
    m = meshgen.box_mesh(8, nx, ny, nz, permute_nodes=order == "random", seed=6)
    conn = m.conn.copy()
    conn[100000, 3] = conn[100000, 4]   # an element left out: an id twice
    conn[200000, 0] = m.n_node          # and one with an id out of range
    print(f"[count groups] three components {order}", flush=True)
    klow = torch.randint(1, 9, (m.n_elem, 300), dtype=torch.int32, device="cuda",
                         generator=torch.Generator("cuda").manual_seed(1)).to(torch.float64)
    c = torch.from_numpy(conn).cuda()
    a, b = (kb.assemble_lower_csr(c, m.n_node, klow, 8, prec="fp64", tuning=tu, check=False, dof=3)
            for tu in (None, TWO_LEVEL))
    assert a.flags == b.flags == 3  # an id out of range, an id repeated
    assert torch.equal(a.row_ptr, b.row_ptr) and torch.equal(a.col_idx, b.col_idx) and torch.equal(a.vals, b.vals)
    assert a.nnz <= (9 * couplings(nx, ny, nz) + 3 * m.n_node) // 2
    assert a.vals.sum().item() == klow.sum().item() - klow[100000].sum().item() - klow[200000].sum().item()
