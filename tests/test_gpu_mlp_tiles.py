"""The encoder's kernels at the edges of their tiles: rows around the 16, 32
and 64 documents of a block and the gradient chunks, widths around the
32-feature blocks and the hidden units that a wave keeps, the largest widths.

Oracle and bars as in tests/test_gpu_mlp.py (same rounded weights and inputs;
with u = 2^-8, 5u on the outputs, 10u on the gradients, 2u on the loss).
"""
import numpy as np
import pytest
import torch

from oracle import mlp_oracle as M

from test_gpu_mlp import U, bf16_round, init_params, make_mlp, rel, rounded

pytestmark = pytest.mark.gpu

tl = pytest.importorskip("paper_2511_07809_amd.tlda")


@pytest.mark.parametrize("d_in,hidden,k_out,n", [
    (50, 256, 50, 1), (1, 1, 1, 17), (31, 32, 33, 16400), (32, 33, 64, 32768 + 7),
    (50, 257, 65, 65), (128, 512, 128, 16384 + 1), (64, 513, 129, 40), (1024, 1024, 256, 33)])
def test_forward_at_tile_edges(d_in, hidden, k_out, n):
    params = init_params(d_in, hidden, k_out, seed=d_in + 3 * hidden)
    X = np.random.default_rng(n).standard_normal((n, d_in)).astype(np.float32)
    m = make_mlp(d_in, hidden, k_out, 16, params)
    P = tl.tlda_mlp_forward(m, torch.from_numpy(X).cuda()).cpu().numpy()
    ref = M.forward(rounded(params), bf16_round(X))["P"]
    assert rel(P, ref) < 5 * U
    # every row on its own: no row takes part in another's tile
    row = np.linalg.norm(P - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert row.max() < 20 * U, int(row.argmax())


@pytest.mark.parametrize("d_in,hidden,k_out,n", [
    (50, 256, 50, 1), (5, 31, 3, 16), (33, 65, 64, 127), (50, 256, 50, 257), (7, 257, 65, 1000),
    (64, 512, 129, 5000), (1024, 1024, 256, 300)])
def test_gradients_at_tile_edges(d_in, hidden, k_out, n):
    params = init_params(d_in, hidden, k_out, seed=5 * d_in + hidden)
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, d_in)).astype(np.float32)
    T = rng.dirichlet(np.full(k_out, 0.3), size=n).astype(np.float32)
    m = make_mlp(d_in, hidden, k_out, n + 3, params)
    Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    g, loss = tl.tlda_mlp_gradients(m, Xd, Td)
    gref, lref = M.gradients(rounded(params), bf16_round(X), T.astype(np.float64))
    got = M.unpack(g.cpu().numpy().astype(np.float64), d_in, hidden, k_out)
    for k in M.PARAM_ORDER:
        assert rel(got[k], gref[k]) < 10 * U, k
    assert abs(float(loss.item()) - lref) <= 2 * U * abs(lref)
    # a smaller batch after it, in the same scratch
    h = max(1, n // 3)
    g, loss = tl.tlda_mlp_gradients(m, Xd[:h].contiguous(), Td[:h].contiguous())
    gref, _ = M.gradients(rounded(params), bf16_round(X[:h]), T[:h].astype(np.float64))
    got = M.unpack(g.cpu().numpy().astype(np.float64), d_in, hidden, k_out)
    for k in M.PARAM_ORDER:
        assert rel(got[k], gref[k]) < 10 * U, k
