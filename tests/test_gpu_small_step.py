"""The fused FP32 step of narrow shapes (D <= 32) on both sides of the batch size
where its kernel changes, at the edges of its 16-document tiles and of the lane
groups that share a document's words, against the oracle's whitening and
gradient (the FP32 bar of the step elsewhere: 1e-5 relative)."""
import numpy as np
import pytest
import torch

from oracle import tlda_oracle as O
from synth import init_phi

pytestmark = pytest.mark.gpu

tl = pytest.importorskip("paper_2511_07809_amd.tlda")

V = 400


def batch(n, seed):
    """Rows of 0, 1, 2, 3, .. words around the groups' 8, 16, 32 and 64 and up to 200."""
    rng = np.random.default_rng(seed)
    sizes = rng.integers(1, 40, n)
    edge = [0, 1, 2, 3, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 129, 200]
    sizes[:len(edge)] = edge[:n]
    rp = np.zeros(n + 1, dtype=np.int32)
    rp[1:] = np.cumsum(sizes)
    ci = np.concatenate([np.sort(rng.choice(V, s, replace=False)) for s in sizes]).astype(np.int32)
    va = rng.integers(1, 4, ci.size).astype(np.float32)
    return rp, ci, va


@pytest.mark.parametrize("n", [1, 4, 15, 16, 17, 300, 16384, 16385])
@pytest.mark.parametrize("D,K", [(1, 1), (4, 3), (5, 5), (8, 16), (9, 17), (16, 33), (17, 64),
                                 (32, 10)])
def test_small_step_matches_oracle(D, K, n):
    if n >= 16384 and (D, K) not in ((1, 1), (5, 5), (9, 17), (32, 10)):
        pytest.skip("one shape per lane-group width at the large sizes")
    rng = np.random.default_rng(D * 100 + K)
    rp, ci, va = batch(n, n + D)
    Q, _ = np.linalg.qr(rng.standard_normal((V, D)))
    W = Q * rng.uniform(5, 30, size=D)[None, :]
    m = rng.dirichlet(np.ones(V))
    ctx = tl.tlda_create(V, K, D, 1.0, 0.5)
    tl.tlda_set_whitening(ctx, W, m)
    Phi = (init_phi(D, K, 2) * 0.5).astype(np.float32)
    P = torch.from_numpy(Phi).cuda()
    g = torch.empty_like(P)
    X = torch.full((n, D), 7.0, device="cuda")
    kept = torch.zeros(1, dtype=torch.int32, device="cuda")
    tl.tlda_whiten_cp_step(ctx, tl.CsrBatch.from_numpy(rp, ci, va), 1e-2, P, g, X, kept)
    L = np.add.reduceat(np.r_[va, 0.0], rp[:-1]) * (np.diff(rp) > 0)
    nk = int((L >= 3).sum())
    assert int(kept.item()) == nk
    Xr = O.whiten_csr(rp, ci, va, V, m, W)
    x = X.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(x - Xr) <= 1e-5 * max(np.linalg.norm(Xr), 1e-30)
    assert not x[L < 3].any()
    if nk == 0:
        assert np.array_equal(P.cpu().numpy(), Phi)
        return
    ref = O.cp_gradient(Xr, Phi.astype(np.float64), nk, 1.0, 0.5)
    assert np.linalg.norm(g.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)
