"""The encoder's forward pass over more rows than one launch can take (2^32 work
items: 2^27 rows of 16-document blocks): every row is written, and the last
ones as a small call writes them."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

tl = pytest.importorskip("paper_2511_07809_amd.tlda")


def test_forward_past_one_launch():
    d_in, hidden, k_out, n = 1, 640, 2, 2 ** 27 + 4000
    m = tl.tlda_mlp_create(d_in, hidden, k_out, 64)
    rng = np.random.default_rng(1)
    tl.tlda_mlp_set_params(m, rng.standard_normal(m.n_params).astype(np.float32) * 0.1)
    X = torch.randn(n, d_in, device="cuda")
    theta = torch.full((n, k_out), float("nan"), device="cuda")
    tl.tlda_mlp_forward(m, X, theta)
    assert torch.isfinite(theta.view(-1)).all()
    for r in (0, 2 ** 27 - 1000, n - 700):
        rows = X[r:r + 700].contiguous()
        assert torch.equal(theta[r:r + 700], tl.tlda_mlp_forward(m, rows))
