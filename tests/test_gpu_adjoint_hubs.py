"""The adjoint's sums at nodes of thousands of elements, which waves with most lanes at one node
form in registers: against the FP64 oracle (tolerance as the other adjoint tests), and the
time of such a mesh."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import meshgen
import paper_1501_04784_amd as kb
from tests.gpu_common import say
from tests.test_gpu_adjoint import TOL, rel_err, run_both

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def hubs(of):
    """A tetrahedron around hub of[e] per element e; the hubs have the last ids, and so one
    bucket (with some of the other nodes)."""
    n = len(of)
    m = meshgen.fan_mesh(n, center_last=True, seed=int(np.sum(of)))
    conn = m.conn.copy()
    hub = conn == 3 * n
    conn[hub] = 3 * n + np.repeat(of, hub.sum(1))
    coords = np.concatenate([m.coords[:-1], np.zeros((int(np.max(of)) + 1, 3))])
    return meshgen.Mesh(4, conn, coords, m.coef)


CASES = {
    # a chunk of records, one more, two chunks and one more
    "32768": lambda: hubs(np.zeros(32768, int)),
    "32769": lambda: hubs(np.zeros(32769, int)),
    "65537": lambda: hubs(np.zeros(65537, int)),
    # two hubs in turn (32 lanes each), three, and runs that change within a wave's records
    "in turn": lambda: hubs(np.arange(20000) % 2),
    "of three": lambda: hubs(np.arange(20000) % 3),
    "runs": lambda: hubs(np.arange(70000) // 100 % 2),
}


@pytest.mark.parametrize("name", list(CASES))
def test_hubs(name):
    m = CASES[name]()
    say(f"[adjoint hubs] {name} nel={m.n_elem}")
    gc, gx, ogc, ogx = run_both(m, seed=9)
    ec, ex = rel_err(gc, ogc), rel_err(gx, ogx)
    say(f"  dL/dc {ec:.2e}  dL/dX {ex:.2e}")
    assert ec <= TOL and ex <= TOL


def milliseconds(m):
    mesh = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (m.conn, m.coords, m.coef)]
    k = kb.build_lower_csr(*mesh, 4, prec="fp64")
    a = kb.AdjointBuilder(4, m.n_elem, m.n_node)
    args = (*mesh, k.row_ptr, k.col_idx, torch.ones(k.nnz, dtype=torch.float64, device="cuda"))
    a.run(*args)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    torch.cuda.synchronize()
    ev[0].record()
    for _ in range(5):
        a.run(*args)
    ev[1].record()
    torch.cuda.synchronize()
    return ev[0].elapsed_time(ev[1]) / 5


def test_time():
    """60,000 tetrahedra around a node against as many that share none: what the node's records
    add is two workgroups' reading of them, and an atomic per address would be ten times it."""
    hub = meshgen.fan_mesh(60000)
    apart = meshgen.Mesh(4, np.arange(240000, dtype=np.int32).reshape(-1, 4), hub.coords[hub.conn.reshape(-1)],
                         hub.coef)
    say("[adjoint hubs] time")
    ms = milliseconds(hub), milliseconds(apart)
    assert ms[0] < 5 * ms[1], ms
