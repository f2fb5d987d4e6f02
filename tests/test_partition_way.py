"""Which way a build's pairs take, as the benchmark reports it: from the plan, or from the word
that the device leaves in the workspace; and the bytes and kernels that go with it."""
import ctypes
import os
import re

import numpy as np
import pytest

import bench
import meshgen
import paper_1501_04784_amd as kb
from paper_1501_04784_amd import _lib


def plan_way(elem, n_elem, n_node, prec="fp32fb64", tuning=None):
    way, tile, at = ctypes.c_int32(), ctypes.c_int32(), ctypes.c_size_t()
    rc = _lib.lib().kb_plan_way(ctypes.byref(kb._mesh(elem, n_elem, n_node)), kb._prec(prec),
                                ctypes.byref((tuning or kb.Tuning()).to_c()), ctypes.byref(way), ctypes.byref(tile),
                                ctypes.byref(at))
    return rc, way.value, tile.value, at.value


def test_plan():
    # few sub-buckets: direct, and tiles small enough for every compute unit
    assert plan_way(8, 1000, 1331, "fp64")[:3] == (0, _lib.KB_WAY_DIRECT, bench.SMALL_TILE)
    # many: the elements are sampled; widths set by hand mean the two levels
    rc, way, _, at = plan_way(8, 1000000, 1030301)
    ws, _ = kb.plan(8, 1000000, 1030301, "fp32fb64")
    assert (rc, way) == (0, _lib.KB_WAY_SAMPLED) and at % 4 == 0 and at + 4 <= ws
    assert plan_way(8, 1000000, 1030301, tuning=kb.Tuning(seg_pairs=4096))[1] == _lib.KB_WAY_BUCKETS
    assert plan_way(8, -1, 8)[0] == _lib.KB_EINVAL
    header = open(os.path.join(os.path.dirname(bench.__file__), "include", "kbuild.h")).read()
    for name in ("KB_WAY_BUCKETS", "KB_WAY_DIRECT", "KB_WAY_SAMPLED"):
        assert int(re.search(rf"#define {name} (\d)", header).group(1)) == getattr(_lib, name)


def test_bytes_by_hand():
    # one tet, four nodes, 10 pairs, 10 entries, FP32: (key, value) after pass 1, no pass 2
    b, two = (bench.algorithmic_bytes(4, 1, 4, 10, "fp32", d) for d in (True, False))
    assert b["integrate"] == 16 + 8 + 24 * 4 + 8 * 10 and b["histogram"] == b["partition"] == 0
    assert all(b[k] == two[k] for k in ("count", "reduce", "compress", "path"))


def test_small_tiles_of_fp64_bricks_take_the_plain_kernel():
    assert bench.pass1_kernel(8, "fp64", "stiffness", bench.SMALL_TILE) == "k_pass1"
    assert bench.pass1_kernel(8, "fp64", "stiffness", 128) == "k_pass1_two"
    assert bench.pass1_kernel(8, "fp32", "stiffness", bench.SMALL_TILE) == "k_pass1_pair"


@pytest.mark.gpu
@pytest.mark.parametrize("order", ["grid", "random"])
def test_reported_from_the_device(order):
    """Grid order goes direct, random numbers take the two levels: as the device left it."""
    import torch

    m = meshgen.box_mesh(8, 40, 41, 42, permute_nodes=order == "random")
    mesh = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (m.conn, m.coords, m.coef)]
    print(f"[way] {order}", flush=True)
    b = kb.Builder(8, m.n_elem, m.n_node, prec="fp32fb64")
    b.run(*mesh)
    b.result()
    assert plan_way(8, m.n_elem, m.n_node)[1] == _lib.KB_WAY_SAMPLED
    assert bench.partition_way(kb, b, m, "fp32fb64", None)[0] == (order == "grid")
