"""Assignment of fp32 and fp16 rows to many clusters (kmeans_blocks.hip) at the sizes where its tiles, its runs of records
and its place in the workspace turn over, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_01000_amd import embedpart as ep
from parity import DEV, Kmeans, label_mismatches, to_np32

pytestmark = pytest.mark.gpu


def _rows(n, d, k, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    comps = max(2, min(k, 40))
    x = 2.0 * torch.randn(comps, d, generator=g)[torch.randint(0, comps, (n,), generator=g)] + torch.randn(n, d, generator=g)
    unit = 4 if dtype == torch.float32 else 8
    padded = torch.full((n, (d + unit - 1) // unit * unit + unit), float("nan"), dtype=dtype)   # never read as data
    padded[:, :d] = x.clamp_(min=0).to(dtype)
    return padded


@pytest.mark.parametrize("n,d,k,dtype", [
    (65, 1, 65, torch.float32),            # one column, k == n, a record with one real centroid
    (1024, 32, 96, torch.float32),         # exactly one block of four point tiles per wave, whole records
    (1025, 33, 97, torch.float16),         # one row and one column more: two blocks, four K-steps
    (513, 64, 128, torch.float32),
    (511, 65, 200, torch.float32),         # six K-steps, one point tile per wave: two blocks
    (70_000, 97, 65, torch.float32),       # more blocks than workgroups: runs that start and end inside a block
    (3_000, 128, 2_500, torch.float32),    # fewer: the records of a block over many workgroups
    (3_001, 127, 2_500, torch.float16),
    (300, 100, 300, torch.float16),
    (20_011, 20, 1_000, torch.float32),
])
def test_blocks_assign(n, d, k, dtype):
    X = _rows(n, d, k, dtype, n + d).to(DEV)[:, :d]
    X32 = to_np32(X)
    rng = np.random.default_rng(n)
    C = X32[oracle.init_indices(n, n, k)].astype(np.float64) + 0.01 * rng.normal(size=(k, d))
    C[k - 1] = C[0]                                        # a tie between the first and the last centroid
    C = C.astype(np.float32).astype(np.float64)
    got, d2, obj = Kmeans(X, k).set_centroids(C).assign()
    want, best, _, obj_or = oracle.assign(X32, C)
    differing, unexcused = label_mismatches(X32, C, got, want, best)
    assert unexcused == 0, f"{unexcused} of {differing} differing labels are not near-ties"
    assert not np.any(got == k - 1)
    terms = (X32.astype(np.float64) ** 2).sum(axis=1) + (C ** 2).sum(axis=1)[got]
    assert np.all(np.abs(d2 - best) <= 1e-5 * terms)      # the size of the terms that the expanded form cancels
    assert abs(obj - obj_or) <= 1e-6 * obj_or + (-(-d // 16) + 4) * 2.0**-24 * terms.sum()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_blocks_infinities_change_their_own_label_only(dtype):
    n, d, k = 3_001, 70, 100
    padded = _rows(n, d, k, dtype, 7)
    C0 = torch.randn(k, d, generator=torch.Generator().manual_seed(8)).numpy()
    clean, clean_d2, _ = Kmeans(padded.to(DEV)[:, :d], k).set_centroids(C0).assign()
    for row, col, value in [(5, 3, float("inf")), (40, d - 1, float("-inf")), (n - 1, 0, float("nan"))]:
        padded[row, col] = value
    got, d2, obj = Kmeans(padded.to(DEV)[:, :d], k).set_centroids(C0).assign()
    rest = np.delete(np.arange(n), [5, 40, n - 1])
    np.testing.assert_array_equal(got[rest], clean[rest])
    np.testing.assert_array_equal(d2[rest], clean_d2[rest])
    assert got[5] == np.nonzero(C0[:, 3] > 0)[0][0] and got[40] == np.nonzero(C0[:, d - 1] < 0)[0][0] and got[n - 1] == 0
    assert np.isfinite(obj) and abs(obj - d2[rest].astype(np.float64).sum()) <= 1e-5 * obj


@pytest.mark.parametrize("n,d,k", [(20_000, 128, 20_000), (60_000, 36, 60_000)])
def test_blocks_static_workspace_in_slices(n, d, k):
    """Records that do not all fit the static workspace are formed and swept a slice at a time: the same bits."""
    X = _rows(n, d, k, torch.float32, d).to(DEV)[:, :d]
    p = ep.problem(X, k)
    idx = ep.kmeans_init_indices(3, n, k)
    out = []
    for static in (False, True):
        ws = ep.workspace(ep.kmeans_workspace_bytes(p), DEV)
        C = torch.empty((k, d), dtype=torch.float32, device=DEV)
        labels = torch.full((n,), -1, dtype=torch.int32, device=DEV)
        counts = torch.zeros(k, dtype=torch.int64, device=DEV)
        hist = torch.zeros(2, dtype=torch.float64, device=DEV)
        ep.kmeans_init(p, X, idx, C, ws)
        if static:
            ep.kmeans_run_noalloc(p, X, 2, C, labels, counts, hist, 0)
        else:
            ep.kmeans_run(p, X, 2, C, labels, counts, hist, 0, ws)
        out.append((C.cpu(), labels.cpu(), counts.cpu(), hist.cpu()))
    for a, b in zip(*out):
        assert torch.equal(a, b)
