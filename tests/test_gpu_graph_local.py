"""Graph partition where its two ways of splitting a segment meet: segments of
one workgroup from the start, at and just past the largest such segment, parts
too large for it; graphs whose BFS leaves vertices unreached, reaches all of
them in one level or takes one level per vertex.  Labels and numbering bit
for bit against the oracle."""

import numpy as np
import pytest

import oracle as O
from problems import grid_graph, unstructured_problem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU machines, skipped by marker
    pytest.skip("no GPU", allow_module_level=True)

import paper_2508_04917_amd as P  # noqa: E402


def from_pairs(n, a, b):
    r = np.concatenate([a, b, np.arange(n)])
    c = np.concatenate([b, a, np.arange(n)])
    k = np.unique(r.astype(np.int64) * n + c)
    ptr = np.zeros(n + 1, dtype=np.int32)
    np.cumsum(np.bincount(k // n, minlength=n), out=ptr[1:])
    return ptr, (k % n).astype(np.int32)


def shuffled(ptr, col, seed):
    n = ptr.size - 1
    perm = np.random.default_rng(seed).permutation(n)
    rows = np.repeat(np.arange(n), np.diff(ptr))
    return from_pairs(n, perm[rows], perm[col])


def knn(n, seed):
    p = unstructured_problem(n, seed, bs=1)
    return p.brow_ptr, p.bcol


def islands(n, size, seed):
    """Disjoint paths of `size` vertices in a random numbering."""
    i = np.arange(n - 1)
    i = i[(i + 1) % size != 0]
    return shuffled(*from_pairs(n, i, i + 1), seed)


CASES = {
    "knn_one_workgroup": (lambda: knn(6000, 61), 500),
    "knn_at_limit": (lambda: knn(36864, 62), 4096),
    "knn_past_limit": (lambda: knn(40960, 63), 4096),
    "knn_two_general_depths": (lambda: knn(110592, 64), 2048),
    "large_parts": (lambda: knn(40000, 65), 20000),
    "odd_parts": (lambda: knn(7 * 333, 66), 333),
    "grid_shuffled": (lambda: shuffled(*grid_graph(24, 20, 18), 67), 270),
    "path": (lambda: from_pairs(5000, np.arange(4999), np.arange(1, 5000)), 100),
    "star_of_leaves": (lambda: from_pairs(3000, np.zeros(60, dtype=np.int64), np.arange(1, 61)), 300),
    "islands": (lambda: islands(12000, 37, 68), 400),
    "single_rows": (lambda: knn(700, 69), 1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_labels(name):
    make, S = CASES[name]
    ptr, col = make()
    n = ptr.size - 1
    print(f"[graph] {name}: {n} vertices, parts of {S}", flush=True)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")  # noqa: E731
    val = torch.ones(col.size, dtype=torch.float64, device="cuda")
    h = P.ddilu.dd_partition_graph(n, 1, t(ptr), t(col), val, part_rows=S)
    pid, n2o, o2n = (x.cpu().numpy() for x in P.dd_get_partition(h))
    ref = O.graph_partition(n, ptr, col, S)
    assert np.array_equal(pid, ref)
    assert np.array_equal(n2o, np.argsort(ref, kind="stable"))
    assert np.array_equal(o2n[n2o], np.arange(n))
    h.close()
