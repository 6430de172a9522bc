"""Few flagged queries: their groups are cut into parts that several workgroups walk.  GPU."""
import numpy as np
import pytest
import torch

from oracle import knn_oracle as ko
from paper_2505_15511_amd import knn_in_clusters

pytestmark = pytest.mark.gpu


# `copies` copies of one row: more ties than the filter's list holds, so each of them is flagged (one query's group cut into the
# most parts; a few; as many as half the workgroups and one more, where nothing is cut any longer)
@pytest.mark.parametrize("copies", [26, 60, 256, 257])
@pytest.mark.parametrize("sizes,d,k", [([9000, 700], 40, 15), ([2500, 1100], 20, 1), ([5000], 7, 32), ([1030, 1023, 1025], 300, 16), ([600, 600], 64, 17)])
def test_flagged_queries_are_exact(copies, sizes, d, k):
    print(f"copies={copies} sizes={sizes} d={d} k={k}", flush=True)
    rng = np.random.default_rng(copies + d)
    c = np.repeat(np.arange(len(sizes)), sizes)
    X = rng.normal(size=(len(c), d)).astype(np.float32)
    where = np.sort(rng.choice(sizes[0], copies, replace=False))
    X[where] = X[where[0]]
    if len(sizes) > 1:                                   # an exact tie far away, in another group
        where2 = sizes[0] + np.arange(k + 12)
        X[where2] = X[where2[0]]
    perm = rng.permutation(len(c))
    X, c = X[perm], c[perm]
    out, st = knn_in_clusters(torch.from_numpy(X).cuda(), torch.from_numpy(c.astype(np.int32)).cuda(), len(sizes), k, return_stats=True)
    print(f"  flagged {st['fallback_queries']}", flush=True)
    assert st["fallback_queries"] >= (copies if copies > k + 8 else 1) if k + 9 <= copies else True
    ref, _ = ko.in_cluster_knn(X, c, k)
    assert np.array_equal(out.cpu().numpy().astype(np.int64), ref)
