"""The adjoint's node buckets against the FP64 oracle, at their edges: bucket sizes changing
with the node count, a node of more corners than one workgroup sums, more buckets than the
counting kernel's LDS array holds.  Tolerance as the other adjoint tests: 1e-12 of the
largest gradient (both FP64; the GPU's node sums are exact, the oracle's sequential)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import meshgen
from tests.gpu_common import say
from tests.test_gpu_adjoint import TOL, rel_err, run_both

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def scattered_tets(n_tets, n_node, seed):
    """Disjoint well-shaped tets whose corners are drawn from all over n_node ids."""
    rng = np.random.default_rng(seed)
    conn = rng.choice(n_node, (n_tets, 4), replace=False).astype(np.int32)
    X = np.zeros((n_node, 3))
    unit = np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1]], float)
    X[conn] = unit + rng.uniform(-0.1, 0.1, (n_tets, 4, 3))
    return meshgen.Mesh(4, conn, X, np.exp(rng.uniform(-2, 2, n_tets)))


CASES = {
    # nodes: 64 and 80 (one and two buckets of 64); 32768 and 33792 (buckets of 64, then 128)
    "hex_64_nodes": lambda: meshgen.box_mesh(8, 3, 3, 3, jitter=0.2, coef=(0.1, 10.0), seed=1),
    "hex_80_nodes": lambda: meshgen.box_mesh(8, 3, 3, 4, jitter=0.2, coef=(0.1, 10.0), permute_nodes=True, seed=2),
    "hex_32768_nodes": lambda: meshgen.box_mesh(8, 31, 31, 31, jitter=0.2, coef=(0.1, 10.0), seed=3),
    "tet_33792_nodes": lambda: meshgen.box_mesh(4, 31, 31, 32, jitter=0.15, coef=(0.1, 10.0), permute_nodes=True,
                                                permute_elems=True, seed=4),
    # one node in every element: 65,536 corners in its bucket and more (one, two, three workgroups)
    "fan_60000": lambda: meshgen.fan_mesh(60000, False, seed=5),
    "fan_65600": lambda: meshgen.fan_mesh(65600, True, seed=6),
    "fan_150000": lambda: meshgen.fan_mesh(150000, False, seed=7),
    # 8,399 buckets, a workgroup's corners in more of them than its hash has slots
    "scattered": lambda: scattered_tets(3000, 8_600_000, 8),
}


@pytest.mark.parametrize("name", list(CASES))
def test_bucket_edges(name):
    m = CASES[name]()
    say(f"[adjoint buckets] {name} nel={m.n_elem} nodes={m.n_node}")
    gc, gx, ogc, ogx = run_both(m, seed=9)
    ec, ex = rel_err(gc, ogc), rel_err(gx, ogx)
    say(f"  dL/dc {ec:.2e}  dL/dX {ex:.2e}")
    assert ec <= TOL and ex <= TOL
