"""The pipelined tile engine at the edges of its stages: reductions of none to five whole
64-element stages with and without a partial one, tiles with one row or column of vectors left
over, and rows too wide for its 32-bit offsets (which take the register-staged engine)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1704_06363_amd import hmoe
from paper_1704_06363_amd import workloads as W
from tests.parity import anchor_of_columns, assert_assign, np64
from tests.test_gpu_bf16 import _check_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,h,o,V,n", [
    (8, 64, 56, 264, 257), (64, 8, 128, 256, 256), (72, 128, 8, 520, 129), (120, 136, 64, 248, 127),
    (128, 192, 136, 2056, 300), (184, 200, 192, 2048, 1), (192, 264, 200, 1032, 511), (328, 72, 256, 512, 513)])
@pytest.mark.parametrize("saved", [False, True])
def test_step_at_stage_edges(d, h, o, V, n, saved):
    K = 3
    inp = W.skewed_inputs(device="cuda", seed=d + n, n=n, d=d, h=h, o=o, V=V, K=K, bias=True)
    ids = np.random.default_rng(n).integers(0, K, n).astype(np.int32)
    _check_step(inp["X"], ids, K, inp["params"], inp["row_ptr"], inp["tag"], saved=saved)


# more tiles than the persistent forward has workgroups, with reductions of one and two stages, whole and not
@pytest.mark.parametrize("o", [8, 40, 64, 72, 120, 128])
def test_short_reductions_over_many_tiles(o):
    n, V, K = 4400, 4360, 3
    inp = W.skewed_inputs(device="cuda", seed=o, n=n, d=64, h=72, o=o, V=V, K=K, bias=True)
    p = inp["params"]
    p["bD"] = torch.randn(V, generator=torch.Generator().manual_seed(o)).to(torch.bfloat16).cuda()
    ids = torch.from_numpy(np.random.default_rng(o).integers(0, K, n).astype(np.int32)).cuda()
    dd = hmoe.moe_dispatch(ids, K, rows=inp["X"])
    row_ptr, tag = torch.tensor(inp["row_ptr"], device="cuda"), torch.tensor(inp["tag"], device="cuda")
    f = hmoe.moe_forward(p, dd["rows_sorted"], dd["offsets"], dd["perm"], row_ptr, tag, save_logits=True)
    H, D = f["H"].double(), p["D"].double()  # from the stored H: no rounding of it in between
    L = H @ D.T + p["bD"].double()
    # fp32 sums of o products and the bias, and the offset from the anchor rounded to bf16
    sums = (o + 2) * 2.0 ** -24 * (H.abs() @ D.abs().T + p["bD"].double().abs())
    A = torch.from_numpy(anchor_of_columns(f["logit_anchor"], V)).cuda().double()
    got = A + f["logits"].double()
    assert ((got - L).abs() <= 3 * sums + 2.0 ** -8 * (L - A).abs()).all()
    # the exponentials' own error, a few units of 2^-23
    assert (f["lse"].double() - L.logsumexp(1)).abs().max() <= 3 * sums.max() + 2e-6


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [8, 24, 32, 56, 64, 72, 128, 136, 200])
def test_assign_at_stage_edges(d, dtype):
    n, K = 515, 259
    X = W.gmm_features(n, d, 40, seed=d, dtype=dtype, device="cuda")
    C = W.gmm_features(K, d, 40, seed=d, dtype=dtype, device="cuda")
    a, md = hmoe.kmeans_assign(X, C)
    a_ref, d1, d2 = O.assign(np64(X), np64(C))
    assert_assign(a, a_ref, d1, d2)
    # fp32 sums of d products and the final cancellation: a few d eps of the terms' magnitude
    mag = (np64(X) ** 2).sum(1) + (np64(C) ** 2).sum(1).max()
    assert (np.abs(np64(md) - d1) <= (d + 8) * 2.0 ** -23 * mag).all()


def test_assign_takes_the_lowest_of_equal_centres():
    # every centre twice, in both orders of tile, lane group and lane
    X = W.gmm_features(300, 64, 20, seed=4, dtype="bf16", device="cuda")
    half = W.gmm_features(150, 64, 20, seed=5, dtype="bf16", device="cuda")
    C = torch.cat([half, half.flip(0)]).contiguous()
    a, _ = hmoe.kmeans_assign(X, C)
    assert int(a.max()) < 150


def test_rows_beyond_the_offset_range():
    # d_in = 2^23 + 8: 300 rows of X at 2 bytes pass 2^32 bytes; the products against fp64
    d, h, o, V, n = (1 << 23) + 8, 8, 8, 264, 300
    g = torch.Generator(device="cuda").manual_seed(1)
    X = torch.randn(n, d, generator=g, device="cuda", dtype=torch.bfloat16)
    p = W.moe_params(1, d, h, o, V, 2, "bf16", "cuda")
    off = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    perm = torch.arange(n, dtype=torch.int32, device="cuda")
    row_ptr = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    tag = torch.arange(n, dtype=torch.int32, device="cuda") % V
    f = hmoe.moe_forward(p, X, off, perm, row_ptr, tag, save_logits=True)
    b = hmoe.moe_backward(p, X, off, perm, perm, row_ptr, tag, f["H1_sorted"], f["H"], f["lse"],
                          logits=f["logits"], logit_anchor=f["logit_anchor"])
    h1 = sum(x.double() @ w.double().T for x, w in zip(X.split(1 << 20, 1), p["W1"][0].split(1 << 20, 1)))
    h1 = h1.clamp_(min=0)
    # H1 ~ N(0, 1): rounding to bf16 and fp32 sums of 2^23 terms of variance 2^-23
    assert (f["H1_sorted"].double() - h1).abs().max() <= 2.0 ** -8 * h1.abs().max() + 1e-3
    # dX = dZ W1 in bf16, and dW1 = dZ^T X with the same dZ: one fixes the other's scale
    nz = (f["H1_sorted"] > 0).double()
    dZ = torch.linalg.lstsq(p["W1"][0][:, :4096].double().T.cpu(), b["dX"][:, :4096].double().T.cpu()).solution.T
    dZ = dZ.cuda() * nz
    ref = dZ.T @ X[:, -4096:].double()
    err = (b["dW1"][0][:, -4096:].double() - ref).norm() / ref.norm()
    assert err <= 2.0 ** -7


@pytest.mark.parametrize("dtype,K,d", [("f32", 65, 1 << 22), ("bf16", 129, 1 << 23), ("f32", 65, (1 << 22) - 8)])
def test_assign_around_the_offset_range(dtype, K, d):
    # the last row width on the pipelined engine and the first past it, against fp64 by column chunks
    n, tdt = 9, torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(K)
    C = torch.randn(K, d, generator=g, device="cuda", dtype=tdt)
    pick = torch.tensor([0, 1, 31, 63, 64, K - 1, 40, 2, K - 2], device="cuda")
    X = (C[pick].float() + 0.5 * torch.randn(n, d, generator=g, device="cuda")).to(tdt)
    a, md = hmoe.kmeans_assign(X, C)
    d2 = sum(torch.cdist(x.double(), c.double()) ** 2 for x, c in zip(X.split(1 << 18, 1), C.split(1 << 18, 1)))
    assert torch.equal(a.long(), pick) and torch.equal(d2.argmin(1), pick)
    # fp32 sums of d squares and products: at most d / 64 eps of their magnitude in sums of 64 lanes
    mag = (X.double() ** 2).sum(1) + (C.double() ** 2).sum(1).max()
    assert ((md.double() - d2.min(1).values).abs() <= d / 64 * 2.0 ** -24 * mag).all()
