"""The step from X with more than 128 topics and few columns, at the row counts from
which it takes the reduction that pads them to 4 instead of 16, against the
oracle's gradient (the FP32 bar of the step elsewhere: 1e-5 relative)."""
import numpy as np
import pytest
import torch

from oracle import tlda_oracle as O
from synth import init_phi

pytestmark = pytest.mark.gpu

tl = pytest.importorskip("paper_2511_07809_amd.tlda")


@pytest.mark.parametrize("D,K,n", [(1, 256, 1), (4, 233, 65), (3, 250, 8191), (4, 129, 16384),
                                   (4, 129, 16385), (5, 217, 3), (8, 256, 1000), (8, 180, 80001),
                                   (7, 201, 160001), (12, 160, 160001), (20, 144, 160001)])
def test_narrow_step_from_x(D, K, n):
    rng = np.random.default_rng(D + K + n)
    X = rng.standard_normal((n, D)).astype(np.float32)
    X[n // 2] = 0.0
    Phi = (init_phi(D, K, 2) * 0.3).astype(np.float32)
    ctx = tl.tlda_create(300, K, D, 1.0, 0.5)
    kept = torch.tensor([max(1, n - 1)], dtype=torch.int32, device="cuda")
    Xd, got = torch.from_numpy(X).cuda(), []
    for rows in (n, min(n, 5), n):   # and again after a batch that takes another grid
        P = torch.from_numpy(Phi).cuda()
        g = torch.empty_like(P)
        tl.tlda_cp_step(ctx, Xd, rows, kept, 1e-2, P, g)
        got.append(g.cpu().numpy().astype(np.float64))
    ref = O.cp_gradient(X.astype(np.float64), Phi.astype(np.float64), max(1, n - 1), 1.0, 0.5)
    assert np.linalg.norm(got[0] - ref) <= 1e-5 * np.linalg.norm(ref)
    assert np.array_equal(got[0], got[2])
    np.testing.assert_allclose(P.cpu().numpy(), Phi - np.float32(1e-2) * got[2], rtol=2e-6,
                               atol=1e-7)
