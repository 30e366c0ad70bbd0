"""The one-launch forms of short steps on both sides of the sizes where they end: the counting sort
(8192 ids, 512 buckets), the objective's sum (4096 and 16,384 rows), the segments' few pieces, the
reseeding's search (16,384 rows) and the centre norms that a fit's update leaves for its next assignment."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1704_06363_amd import hmoe
from paper_1704_06363_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 65, 1023, 1025, 4096, 8191, 8192, 8193])
@pytest.mark.parametrize("K", [1, 2, 50, 511, 512, 513])
def test_dispatch(n, K):
    ids = np.random.default_rng(n + K).integers(0, K, n).astype(np.int32)
    if K > 1:
        ids[ids == K // 2] = 0  # an empty bucket
    out = hmoe.moe_dispatch(torch.from_numpy(ids).cuda(), K)
    for got, ref in zip((out["counts"], out["offsets"], out["perm"], out["inv"]), O.dispatch(ids, K)):
        assert np.array_equal(got.cpu().numpy(), ref)
    # ids out of range follow every expert, in order
    bad = ids.copy()
    bad[:: 7] = np.where(np.arange(len(bad[:: 7])) % 2, -5, K + 3)
    out = hmoe.moe_dispatch(torch.from_numpy(bad).cuda(), K)
    key = np.where((bad < 0) | (bad >= K), K, bad)
    assert np.array_equal(out["perm"].cpu().numpy(), np.argsort(key, kind="stable"))
    assert np.array_equal(out["counts"].cpu().numpy(), np.bincount(key, minlength=K + 1)[:K])
    assert int(out["offsets"][K]) == int((key < K).sum())


# segments of no, one, a few, 8, 9, 31 .. 33 and 40 pieces of 256 rows: from 2^20 outputs on a thread adds an
# output's pieces, below that eight threads do, in the same order
def test_column_sums_of_uneven_segments():
    K, d = 4096, 256
    pieces = {0: 1, 3: 40, 4: 31, 5: 32, 700: 33, 701: 8, 702: 9, 4094: 3, 4095: 16}
    a = torch.cat([torch.full((256 * p - (e % 2) * 5,), e, dtype=torch.int32, device="cuda") for e, p in pieces.items()])
    a = a[torch.randperm(a.numel(), generator=torch.Generator().manual_seed(1)).cuda()].contiguous()
    X = W.gmm_features(a.numel(), d, 8, seed=3, dtype="f32", device="cuda")
    got = []
    for w in (d, d - 8):
        x = X[:, :w].contiguous()
        sums, counts = torch.ones(K, w, dtype=torch.float64, device="cuda"), torch.zeros(K, dtype=torch.int64, device="cuda")
        hmoe.kmeans_update(x, K, a, None, sums, counts, torch.zeros(K, w, device="cuda"), mode=hmoe.UPDATE_ACCUMULATE)
        ref = torch.ones_like(sums).index_add_(0, a.long(), x.double())
        assert (sums - ref).abs().max() <= a.numel() * 2.0 ** -53 * x.double().abs().sum(0).max()
        assert counts.tolist() == torch.bincount(a.long(), minlength=K).tolist()
        got.append(sums)
    assert torch.equal(got[0][:, : d - 8], got[1])


@pytest.mark.parametrize("n,d,K,dtype", [(40, 16, 9, "f32"), (4096, 8, 2, "f32"), (4097, 8, 2, "f32"), (8192, 72, 50, "bf16"), (8193, 64, 300, "f32"),
                                         (16384, 40, 64, "f32"), (16385, 40, 600, "bf16"), (20000, 1032, 3, "bf16")])
def test_fit_is_its_steps(n, d, K, dtype):
    """A fit and the same iterations through assign and update: the same bits (reseeding included: two
    centres start far from every row)."""
    X = W.gmm_features(n, d, 40, seed=n, dtype=dtype, device="cuda")
    C = X[torch.randperm(n, generator=torch.Generator().manual_seed(1))[:K].cuda()].float().contiguous()
    if K > 4:
        C[1] = 1e3
        C[3] = 2e3
    out = hmoe.kmeans_fit(X, K, 3, C=C)
    C2, obj = C.clone(), []
    sums = torch.empty(K, d, dtype=torch.float64, device="cuda")
    counts = torch.empty(K, dtype=torch.int64, device="cuda")
    for t in range(4):
        a, md = hmoe.kmeans_assign(X, C2.to(X.dtype))
        obj.append(md.double().sum().item())
        if t < 3:
            hmoe.kmeans_update(X, K, a, md, sums, counts, C2)
    assert torch.equal(out["C"], C2) and torch.equal(out["assign"], a) and torch.equal(out["min_dist"], md)
    assert torch.equal(out["counts"].long(), torch.bincount(a.long(), minlength=K))
    # sums of n non-negative terms in fp64, in two orders
    assert np.allclose(out["objective"].cpu().numpy(), obj, rtol=n * 2.0 ** -52)
