"""k-means++ seeding over the 8-bit copy of the rows: every output is the same to the last bit as
without the copy (a workspace without room for it), whose picks are pinned against the oracle."""
import pytest
import torch

from oracle import oracle as O
from paper_1704_06363_amd import hmoe
from paper_1704_06363_amd import workloads as W
from tests.parity import np64

pytestmark = pytest.mark.gpu


def _both(X, K, n_iter, seed):
    n, d = X.shape
    u = W.uniforms(K, seed)
    ws = torch.empty(hmoe.kmeans_fit_workspace(n, d, K, X.dtype), dtype=torch.uint8, device="cuda")
    row = -(-d // 16) * 16 + 20  # the copy: 8-bit row, scale, bound and norm, and its nearest centre
    with_copy = hmoe.kmeans_fit(X, K, n_iter, init_uniforms=u, ws=ws)
    without = hmoe.kmeans_fit(X, K, n_iter, init_uniforms=u, ws=ws[: ws.numel() - n * row])
    with pytest.raises(hmoe.HmoeError):
        hmoe.kmeans_fit(X, K, n_iter, init_uniforms=u, ws=ws[: ws.numel() - n * row - 4096])
    for k in with_copy:
        a, b = with_copy[k].view(torch.uint8), without[k].view(torch.uint8)
        assert torch.equal(a, b), k
    return with_copy, u


# widths of one vector, of no whole 16-entry vector, and odd in both dtypes; 32 MB and up
@pytest.mark.parametrize("n,d,K,dtype", [(70001, 120, 33, "f32"), (40000, 264, 16, "f32"), (20011, 1000, 17, "bf16"),
                                         (131073, 128, 40, "bf16"), (1048577, 8, 17, "f32")])
def test_copy_changes_nothing(n, d, K, dtype):
    X = W.gmm_features(n, d, 24, seed=n, dtype=dtype, device="cuda")
    out, u = _both(X, K, 2, n)
    if n * K < 3_000_000:
        assert out["init_idx"].tolist() == O.kmeanspp(np64(X), K, u).tolist()


def test_copy_with_rows_it_cannot_hold():
    # zero rows, equal rows, rows too large or small for the copy, one entry far above the rest
    n, d, K = 40000, 264, 24
    X = W.gmm_features(n, d, 24, seed=3, dtype="f32", device="cuda")
    X[100:200] = 0.0
    X[200:400] = X[200].clone()
    X[500] *= 1e16
    X[600] *= 1e-20
    X[700:800, 5] = 1e6
    _both(X, K, 0, 7)
    X[900, 3] = float("inf")  # every sum of distances is infinite or NaN: picks by the fallbacks
    _both(X, K, 0, 8)
    X[900, 3] = float("nan")
    _both(X, K, 0, 9)


@pytest.mark.parametrize("d", [133144, 133152, 140000])
def test_rows_past_the_integer_sums_of_the_copy(d):
    """From 133,152 columns on the squares of a row of 8-bit entries near 127 pass 2^31.  16 far
    families of four rows, of which two have one larger entry and so smaller 8-bit entries (whose
    squares do not): a family is picked twice only when the passes miss a distance."""
    K, n = 16, 64
    g = torch.Generator(device="cuda").manual_seed(d)
    sign = torch.randint(0, 2, (K, 1, d), generator=g, device="cuda").float() * 2 - 1
    X = (sign * (1 - 0.005 * torch.rand(K, 1, d, generator=g, device="cuda"))
         + 1e-4 * torch.randn(K, 4, d, generator=g, device="cuda"))
    X[:, 2:, 7] = 1.04
    X = X.reshape(n, d).contiguous()
    u = W.uniforms(K, 3)
    ws = torch.empty(hmoe.kmeans_fit_workspace(n, d, K, X.dtype), dtype=torch.uint8, device="cuda")
    out = hmoe.kmeans_fit(X, K, 0, init_uniforms=u, ws=ws)
    assert out["init_idx"].tolist() == O.kmeanspp(np64(X), K, u).tolist()
    assert len(set(i // 4 for i in out["init_idx"].tolist())) == K
