"""Rows wider than the 1024 16-byte vectors (4096 fp32, 8192 bf16 columns) that one workgroup of
the segmented column sums covers, in a workspace that holds NaN: every column of the centre sums,
of the bias gradients and of the PCA's mean is written."""
import pytest
import torch

from paper_1704_06363_amd import hmoe

pytestmark = pytest.mark.gpu
F32, BF16 = torch.float32, torch.bfloat16


def _nan_ws(nbytes):
    return torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")


def _randn(*shape, dtype=F32, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(*shape, generator=g, device="cuda").to(dtype)


@pytest.mark.parametrize("dtype,d", [(F32, 4088), (F32, 4096), (F32, 4104), (F32, 8192), (F32, 8200),
                                     (BF16, 8192), (BF16, 8200), (BF16, 16392)])
def test_centre_sums(dtype, d):
    n, K = 700, 3
    X = _randn(n, d, dtype=dtype, seed=d)
    a = torch.arange(n, dtype=torch.int32, device="cuda") % K
    sums = torch.zeros(K, d, dtype=torch.float64, device="cuda")
    counts = torch.zeros(K, dtype=torch.int64, device="cuda")
    ws = _nan_ws(hmoe.kmeans_update_workspace(n, d, K, dtype))
    hmoe.kmeans_update(X, K, a, None, sums, counts, torch.zeros(K, d, device="cuda"), mode=hmoe.UPDATE_ACCUMULATE,
                       reseed=False, ws=ws)
    ref = torch.zeros_like(sums).index_add_(0, a.long(), X.double())
    # fp64 sums of 234 terms: n eps times their magnitude
    assert (sums - ref).abs().max() <= n * 2.0 ** -53 * X.double().abs().sum(0).max()


@pytest.mark.parametrize("dtype,h,o", [(F32, 4096, 64), (F32, 4104, 64), (F32, 8192, 64), (F32, 64, 8192),
                                       (F32, 4104, 4104), (BF16, 8192, 64)])
def test_bias_gradients(dtype, h, o):
    """One row per expert, with a column of ones in the layer's input: the bias gradient is that
    column of the weight gradient, a sum of one term."""
    n = K = 3
    d, V = 16, 24
    p = {"W1": _randn(K, h, d, dtype=dtype, seed=1), "b1": _randn(K, h, dtype=dtype, seed=2),
         "W2": _randn(K, o, h, dtype=dtype, seed=3) * h ** -0.5, "b2": _randn(K, o, dtype=dtype, seed=4),
         "D": _randn(V, o, dtype=dtype, seed=5) * o ** -0.5, "bD": _randn(V, dtype=dtype, seed=6)}
    X = _randn(n, d, dtype=dtype, seed=7)
    X[:, 0] = 1.0
    i32 = dict(dtype=torch.int32, device="cuda")
    off, perm = torch.arange(K + 1, **i32), torch.arange(n, **i32)
    row_ptr, tag = torch.arange(n + 1, **i32), torch.arange(n, **i32)
    f = hmoe.moe_forward(p, X, off, perm, row_ptr, tag, save_logits=True)
    H1 = f["H1_sorted"]
    H1[:, 0] = 1.0
    ws = _nan_ws(hmoe.moe_workspace(hmoe.make_params(p), n))
    g = hmoe.moe_backward(p, X, off, perm, perm, row_ptr, tag, H1, f["H"], f["lse"], logits=f["logits"],
                          logit_anchor=f["logit_anchor"], ws=ws)
    assert torch.equal(g["db1"], g["dW1"][:, :, 0])
    assert torch.equal(g["db2"], g["dW2"][:, :, 0])
    assert bool(torch.isfinite(g["db1"]).all()) and int(torch.count_nonzero(g["db2"])) > K * o // 2


@pytest.mark.parametrize("dtype,d", [(F32, 4104), (BF16, 8200)])
def test_pca_mean(dtype, d):
    n, r = 600, 8
    X = _randn(n, d, dtype=dtype, seed=d) + _randn(d, dtype=dtype, seed=1)
    ws = _nan_ws(hmoe.pca_workspace(n, d, r, dtype))
    mean, _, ev = hmoe.pca_fit(X, r, n_iter=1, ws=ws)
    ref = X.double().mean(0)
    # an fp64 sum rounded to fp32
    assert (mean.double() - ref).abs().max() <= 2.0 ** -23 * ref.abs().max()
    assert bool(torch.isfinite(ev).all())
