"""The refresh's dense building blocks at the edges of their tiles, through
the refresh itself: its block width p sets the size of the Cholesky factor,
the triangular inverse, the Gram products and the projected eigenproblem.

Whatever p is, the top-D eigenpairs are the same, so every width is compared
with the oracle's.  Bars as for the refresh at this size elsewhere: the
iteration is converged (eigenvalues to 1e-10 relative), the eigen-gaps are
wide (columns to 1e-7), W^T M2~ W = I to 1e-8.
"""
import numpy as np
import pytest

from oracle import tlda_oracle as O
from synth import CorpusSpec, generate, iter_batches

pytestmark = pytest.mark.gpu

tl = pytest.importorskip("paper_2511_07809_amd.tlda")


@pytest.fixture(scope="module")
def corpus():
    spec = CorpusSpec("f", V=640, K=4, N=3000, doc_len_lambda=40.0, alpha0=1.0, topic_conc=0.1,
                      zipf_s=None, zipf_mix=0.0, batch=3000, seed=77)
    rp, ci, va, _ = next(iter_batches(generate(spec)))
    m, N = O.first_moment([(rp, ci, va)], spec.V)
    M2 = O.centered_second_moment([(rp, ci, va)], m, N, spec.alpha0)
    W, lam, _ = O.whitening(M2, spec.K)
    return {"spec": spec, "batch": (rp, ci, va), "M2": M2, "W": W, "lam": lam}


# 16-wide tiles: one, a remainder, whole tiles; 5 / 6 tiles (inverse in the
# same launch or its own), 9 / 10 and 13 / 14 (tiles per wave, then in
# memory), the largest width
@pytest.mark.parametrize("p", [16, 17, 31, 80, 81, 100, 101, 128, 129, 144, 145, 200, 208, 209,
                               288, 289, 511, 512])
def test_refresh_at_every_block_width(corpus, p):
    spec = corpus["spec"]
    ctx = tl.tlda_create(spec.V, spec.K, spec.K, spec.alpha0, eig_iters=200, eig_block=p)
    tl.tlda_update_moments(ctx, tl.CsrBatch.from_numpy(*corpus["batch"]), tl.TLDA_REFRESH_W)
    W, eig, _ = tl.tlda_get_whitening(ctx)
    assert np.linalg.norm(eig - corpus["lam"]) < 1e-10 * np.linalg.norm(corpus["lam"])
    assert np.linalg.norm(W - corpus["W"]) < 1e-7 * np.linalg.norm(corpus["W"])
    np.testing.assert_allclose(W.T @ corpus["M2"] @ W, np.eye(spec.K), atol=1e-8)
