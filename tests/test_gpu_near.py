"""Near sets and internal order at the sizes where the search changes its sort
(4,096 wires), its scan (8,192) and its candidate walk (a cell with more than
32 wires, one cell for everything, several clouds): integers, equal to the
oracle's."""
import math

import numpy as np
import pytest

from oracle import mom, precond
from paper_2410_03060_amd import workloads as W
from parity_util import gpu_pairs, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_03060_amd import binding
    binding.lib()
    return binding


def _cloud(name):
    if name == "several":
        return W.concat_clouds([W.random_cloud(3, n, box_lam=b, d_c_lam=1.0)
                                for n, b in ((33, 2.0), (1, 1.0), (900, 3.0), (64, 40.0))])
    n, box, d_c = {"one": (1, 1.0, 1.0), "31": (31, 2.0, 1.0), "4096": (4096, 14.0, 1.0), "4097": (4097, 14.0, 1.0),
                   "8192": (8192, 30.0, 1.0), "8193": (8193, 30.0, 1.0), "crowded": (700, 2.0, 1.0),
                   "one_cell": (333, 2.0, 5.0), "dense": (257, 3.0, math.inf)}[name]
    return W.random_cloud(17, n, box_lam=box, d_c_lam=d_c)


@pytest.mark.parametrize("name", ["one", "31", "4096", "4097", "8192", "8193", "crowded", "one_cell", "dense",
                                  "several"])
def test_near_sets(B, name):
    cloud = _cloud(name)
    cl = B.build_cloud(cloud)
    row_ptr, col, perm, diag = cl.pattern()
    assert np.array_equal(perm, precond.cell_order(cloud))
    row = np.repeat(np.arange(cl.n), np.diff(row_ptr))
    assert np.array_equal(np.lexsort((col, row)), np.arange(cl.nnzb))   # ascending columns in every row
    assert np.array_equal(row[diag], np.arange(cl.n)) and np.array_equal(col[diag], np.arange(cl.n))
    I, J = mom.near_pairs(cloud.center, cloud.cloud_off, cloud.d_c)
    assert 2 * cl.n_pairs == len(I)   # the oracle lists both orders of a pair
    got = {(min(a, b), max(a, b)) for a, b in zip(perm[row], perm[col]) if a != b}
    assert got == {(min(a, b), max(a, b)) for a, b in zip(I.tolist(), J.tolist())}
    say(f"[near] {name}: N={cl.n} pairs={cl.n_pairs} equal")
