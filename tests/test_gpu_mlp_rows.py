"""The encoder's forward pass over more rows than one launch can take (2^32 work
items: 2^27 rows of 16-document blocks), where every row has to be written, and
the last ones as a small call writes them; and over inputs wide enough to take
their own way into LDS (more than 128 columns), at each tile height, at widths
around its 64 columns, against the oracle (bars as in tests/test_gpu_mlp.py)."""
import numpy as np
import pytest
import torch

from oracle import mlp_oracle as M

from test_gpu_mlp import U, bf16_round, init_params, make_mlp, rel, rounded

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


@pytest.mark.parametrize("d_in,hidden,k_out,n", [
    (129, 16, 8, 32768 + 5), (192, 40, 3, 16384 + 31), (1000, 64, 16, 16391), (449, 700, 9, 35),
    (513, 33, 65, 1), (1024, 16, 256, 17)])
def test_forward_of_wide_inputs(d_in, hidden, k_out, n):
    params = init_params(d_in, hidden, k_out, seed=d_in + hidden)
    X = np.random.default_rng(n).standard_normal((n, d_in)).astype(np.float32)
    m = make_mlp(d_in, hidden, k_out, 16, params)
    P = tl.tlda_mlp_forward(m, torch.from_numpy(X).cuda()).cpu().numpy()
    ref = M.forward(rounded(params), bf16_round(X))["P"]
    assert rel(P, ref) < 5 * U
    row = np.linalg.norm(P - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert row.max() < 20 * U, int(row.argmax())
