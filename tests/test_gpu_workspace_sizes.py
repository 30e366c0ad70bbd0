"""Workspaces of the sizes that the library asked for before it kept copies and tables that only save
time: accepted, with the same results (the gradient's bias column sums add fewer, larger blocks)."""
import numpy as np
import pytest
import torch

from paper_1704_06363_amd import hmoe
from paper_1704_06363_amd import workloads as W
from tests.parity import assert_close

pytestmark = pytest.mark.gpu


def _ws(size):
    return torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("n,d,K,dtype,fit,update", [
    (4096, 64, 8, "f32", 116176, 56208), (1000, 64, 16, "f32", 58724, 29412), (5000, 64, 512, "bf16", 840788, 339764),
    (70001, 120, 300, "f32", 3892284, 1208264), (100003, 64, 4000, "f32", 22219808, 4675348)])
def test_clustering(n, d, K, dtype, fit, update):
    X = W.gmm_features(n, d, 24, seed=n, dtype=dtype, device="cuda")
    assert hmoe.kmeans_update_workspace(n, d, K, X.dtype) <= update
    u = W.uniforms(K, 1)
    a = hmoe.kmeans_fit(X, K, 2, init_uniforms=u)
    b = hmoe.kmeans_fit(X, K, 2, init_uniforms=u, ws=_ws(fit))
    for k in a:
        assert torch.equal(a[k].view(torch.uint8), b[k].view(torch.uint8)), k
    with pytest.raises(hmoe.HmoeError):
        hmoe.kmeans_fit(X, K, 2, init_uniforms=u, ws=_ws(fit - 64))
    outs = []
    for ws in (None, _ws(update)):
        sums, counts = torch.empty(K, d, dtype=torch.float64, device="cuda"), torch.empty(K, dtype=torch.int64,
                                                                                          device="cuda")
        C, ids = a["C"].clone(), a["assign"].clone()
        hmoe.kmeans_update(X, K, ids, a["min_dist"], sums, counts, C, ws=ws)
        outs.append((sums, counts, C, ids))
    assert all(torch.equal(x, y) for x, y in zip(*outs))


@pytest.mark.parametrize("n,K,d,h,o,V,dtype,own,size", [
    (4096, 8, 64, 128, 64, 1000, "f32", False, 53269760), (8192, 8, 64, 128, 64, 1000, "f32", False, 72943872),
    (5003, 50, 1000, 2056, 520, 10008, "bf16", False, 266409600), (1024, 8, 64, 128, 64, 1000, "bf16", True, 136851492),
    (512, 16, 2048, 4096, 1024, 50000, "bf16", False, 196080384)])
@pytest.mark.parametrize("saved", [True, False])
def test_step(n, K, d, h, o, V, dtype, own, size, saved):
    saved = saved or own  # a decoder for each expert needs the saved logits
    p = W.moe_params(K, d, h, o, V, 3, dtype, "cuda", bias=True, per_expert_decoders=own)
    X = W.rectified_gaussian(n, d, 1, dtype, "cuda")
    ids = torch.from_numpy(np.random.default_rng(2).integers(0, K, n).astype(np.int32)).cuda()
    rp, tg = (torch.from_numpy(a).cuda() for a in W.zipf_labels(n, V, 5, 4))
    dd = hmoe.moe_dispatch(ids, K, rows=X)
    args = (p, dd["rows_sorted"], dd["offsets"], dd["perm"])
    f, g = [], []
    for ws in (None, _ws(size)):
        f.append(hmoe.moe_forward(*args, rp, tg, save_logits=saved, ws=ws))
        r = f[0]
        g.append(hmoe.moe_backward(*args, dd["inv"], rp, tg, r["H1_sorted"], r["H"], r["lse"], logits=r["logits"],
                                   logit_anchor=r["logit_anchor"], ws=ws))
    with pytest.raises(hmoe.HmoeError):
        hmoe.moe_forward(*args, rp, tg, save_logits=saved, ws=_ws(size // 2))
    for k in f[0]:
        assert (f[0][k] is None and f[1][k] is None) or torch.equal(f[0][k], f[1][k]), k
    for k in g[0]:
        if k == "dbD":  # fp32 sums of up to n terms in another order, each below 2 / n
            assert_close(g[1][k], g[0][k], 1e-5, k)
        else:
            assert torch.equal(g[0][k], g[1][k]), k
