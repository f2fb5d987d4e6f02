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
