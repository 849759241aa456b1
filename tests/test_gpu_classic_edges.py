"""The classic-moment step where its kernel can go wrong: documents around the
32 entries that a wave holds at once and their multiples (they are passed over
twice), runs of documents that end inside a batch of 16 rows, D and K around
the matrix tiles of 16 and the split of K at 64, and fewer documents than waves.

Tolerance: 1e-5 of the data term's Frobenius norm, ten times what FP32 products
and sums of a few thousand terms (6e-8 each, about 1e-6 together) lose against
FP64.  (Not of the gradient's norm: at D = 1, n = 3500 the penalty and the data
term cancel to a hundredth.)  BF16: the oracle on the operands that the kernel
rounds, the rest within the entry-wise bound derived in tests/bf16_ref.py."""
import numpy as np
import pytest
import torch

from bf16_ref import assert_within, bf16_round, classic_bf16_bound, z16_like_kernel
from oracle import tlda_oracle as O
from synth import init_phi

pytestmark = pytest.mark.gpu

tl = pytest.importorskip("paper_2511_07809_amd.tlda")

V = 300
EDGE = [0, 1, 3, 4, 15, 16, 17, 31, 32, 33, 35, 36, 48, 63, 64, 65, 96, 97, 128, 200]


def batch(n, seed):
    rng = np.random.default_rng(seed)
    sizes = rng.integers(0, 40, n)
    sizes[:len(EDGE)] = EDGE[:n]
    rng.shuffle(sizes)
    rp = np.zeros(n + 1, dtype=np.int32)
    rp[1:] = np.cumsum(sizes)
    ci = np.concatenate([np.sort(rng.choice(V, s, replace=False)) for s in sizes]).astype(np.int32)
    va = rng.integers(1, 4, ci.size).astype(np.float32)
    return rp, ci, va


def step(ctx, rp, ci, va, Phi):
    Pd = torch.from_numpy(Phi).cuda()
    g = torch.empty_like(Pd)
    kept = torch.zeros(1, dtype=torch.int32, device="cuda")
    tl.tlda_whiten_cp_step(ctx, tl.CsrBatch.from_numpy(rp, ci, va), 1e-3, Pd, g, None, kept)
    torch.cuda.synchronize()
    return g.cpu().numpy().astype(np.float64), int(kept.item())


def check(g, kept, rp, ci, va, V, m, W, Phi, a0):
    P = Phi.astype(np.float64)
    ref = O.classic_cp_gradient(rp, ci, va, V, m, W, P, a0, 0.5)
    data, n_kept = O.classic_data_term(rp, ci, va, V, m, W, P, a0)
    assert kept == n_kept
    if kept == 0:   # a batch without a kept document: no step, a gradient of zero
        ref = np.zeros_like(ref)
    assert np.linalg.norm(g - ref) <= 1e-5 * np.linalg.norm(3.0 / max(kept, 1) * data)


@pytest.mark.parametrize("n", [1, 2, 13, 300, 3500, 20000])
@pytest.mark.parametrize("D,K", [(1, 2), (4, 16), (8, 17), (16, 33), (17, 48), (50, 49), (64, 64),
                                 (65, 65), (97, 20), (128, 127), (112, 32)])
def test_classic_step_matches_oracle(D, K, n):
    if n >= 3500 and (D, K) not in ((1, 2), (50, 49), (65, 65)):
        pytest.skip("one shape per kind at the sizes with several documents a wave")
    rng = np.random.default_rng(D * 100 + K)
    rp, ci, va = batch(n, n + D)
    Q, _ = np.linalg.qr(rng.standard_normal((V, D)))
    W = Q * rng.uniform(5, 30, D)
    m = rng.dirichlet(np.ones(V))
    Phi = (init_phi(D, K, D + K) * 0.3).astype(np.float32)
    ctx = tl.tlda_create(V, K, D, 1.5, 0.5, classic=True)
    tl.tlda_set_whitening(ctx, W, m)
    g, kept = step(ctx, rp, ci, va, Phi)
    g2, _ = step(ctx, rp, ci, va, Phi)
    assert np.array_equal(g, g2)
    check(g, kept, rp, ci, va, V, m, W, Phi, 1.5)


@pytest.mark.parametrize("n", [1, 13, 300, 3500])
@pytest.mark.parametrize("D,K", [(4, 16), (16, 33), (17, 48), (50, 49), (65, 65), (97, 20),
                                 (128, 127), (112, 32)])
def test_classic_bf16_step_within_its_bound(D, K, n):
    if n >= 3500 and (D, K) not in ((50, 49), (65, 65)):
        pytest.skip("one shape per kind at the sizes with several documents a wave")
    rng = np.random.default_rng(D * 100 + K)
    rp, ci, va = batch(n, n + D)
    Q, _ = np.linalg.qr(rng.standard_normal((V, D)))
    W = Q * rng.uniform(5, 30, D)
    m = rng.dirichlet(np.ones(V))
    Phi = (init_phi(D, K, D + K) * 0.3).astype(np.float32)
    ctx = tl.tlda_create(V, K, D, 1.5, 0.5, classic=True, bf16=True)
    tl.tlda_set_whitening(ctx, W, m)
    g, kept = step(ctx, rp, ci, va, Phi)
    g2, _ = step(ctx, rp, ci, va, Phi)
    assert np.array_equal(g, g2)
    P = Phi.astype(np.float64)
    W16 = bf16_round(W)
    Z16 = z16_like_kernel(W16, Phi)
    data, n_kept = O.classic_data_term(rp, ci, va, V, m, W16, P, 1.5, Z=Z16)
    assert kept == n_kept
    G = P.T @ P
    ref = 4.5 * P @ (G * G) - 3.0 / max(kept, 1) * data if kept else np.zeros_like(P)
    bound = 3.0 / max(kept, 1) * classic_bf16_bound(rp, ci, va, W16, Z16, P, m, 1.5)
    assert_within(g, ref, bound + 2.0 ** -22 * np.abs(ref), f"classic BF16 D={D} K={K} n={n}")
