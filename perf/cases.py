"""Performance cases: the calls that a user of the library makes, with sizes over
the range that it serves.

A case is a dict of plain values.  ``prepare`` builds what a program holds
before the call (corpus batches on the GPU, a context with its whitening, the
CP factors), ``run`` is one pass through the public binding, ``exact`` is the
same result in plain 64-bit torch, ``work`` the bytes and operations that the
pass cannot do without.  Documents follow the paper's generative process as
``synth`` draws it (Dirichlet topics over a Zipf background, Poisson lengths),
drawn here on the GPU so that preparing is quick.  The factors start near a
fit's converged ones (a^(1/3) W^T (mu - M1) of the planted topics), where most
of a fit's passes run.

Sizes come from the repository's workloads: 500 words (V = 500, K = 5, batches
of 1000), tweet-shaped (V = 20 000, K = 50, 131 072 documents), streaming
scale (V = 50 000, K = 100, 262 144 documents), 64-slice (V = 20 000, K in
{10, 20, 50}) and the encoder (50 -> 256 -> 256 -> 50, batches of 4096).
"""
import math

import numpy as np
import torch

from paper_2511_07809_amd import tlda as tl

F64 = torch.float64


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # one gradient step of the smallest workload: launches and latency
        dict(name="step_500w", kind="step", bf16=False, V=500, K=5, D=5, docs=1000, length=50,
             alpha0=1.0),
        # one FP32 step of the benchmark's streaming workload: the main path
        dict(name="step_stream_f32", kind="step", bf16=False, V=50000, K=100, D=100, docs=262144,
             length=15, alpha0=2.0),
        # a pass over four resident batches of tweets in BF16, replayed as one graph
        dict(name="pass_tweet_bf16", kind="pass", bf16=True, V=20000, K=50, D=50, docs=131072,
             length=20, alpha0=1.0, batches=4),
        # one step of the classic (alpha0-corrected) estimator on a batch of tweets
        dict(name="classic_tweet", kind="classic", bf16=False, V=20000, K=50, D=50, docs=131072,
             length=20, alpha0=1.0),
        # the two-call form with the whitened batch kept (programs that also use X):
        # an odd vocabulary, D and K apart and past the fused kernel's 128
        dict(name="two_calls_ragged", kind="two", bf16=False, V=12347, K=37, D=150, docs=40001,
             length=30, alpha0=1.0),
        # a whole small fit: moments of five batches, whitening, ten passes, topics, proportions
        dict(name="fit_500w", kind="fit", V=500, K=5, D=5, docs=1000, length=50, alpha0=1.0,
             batches=5, passes=10),
        # the batched method's whitening refresh (cold) over a tweet-sized vocabulary, D = 100
        dict(name="refresh_wide", kind="refresh", V=20000, K=100, D=100, docs=65536, length=20,
             alpha0=1.0),
        # fully online mode, per batch: moments, warm refresh, rebase of Phi, one step
        dict(name="online_tweet", kind="online", V=20000, K=50, D=50, docs=131072, length=20,
             alpha0=1.0),
        # serving: topics from the factors, then proportions of a batch of new documents
        dict(name="infer_tweet", kind="infer", V=20000, K=50, D=50, docs=65536, length=20,
             alpha0=1.0, max_iter=200),
        # encoder training: sixteen Adam steps, then the gradients of a held-out batch
        dict(name="encoder_train", kind="train", D=50, hidden=256, K=50, rows=4096, steps=16),
        # encoder inference over a large batch of whitened documents
        dict(name="encoder_forward", kind="encode", D=50, hidden=256, K=50, rows=131072,
             max_batch=4096),
        # many time slices stepped together: two batch indices in one graph
        dict(name="slices_tweet", kind="slices", V=20000, docs=65536, length=20, alpha0=1.0,
             slices=24, batches=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "pass", "classic", "two", "fit", "refresh", "online",
                       "infer", "train", "encode", "slices"])
    if kind == "train":
        return dict(kind=kind, D=_log(rng, 5, 128), hidden=_log(rng, 33, 512),
                    K=_log(rng, 3, 128), rows=_log(rng, 200, 8192), steps=rng.randint(4, 16))
    if kind == "encode":
        return dict(kind=kind, D=_log(rng, 5, 128), hidden=_log(rng, 33, 512),
                    K=_log(rng, 3, 128), rows=_log(rng, 500, 131072),
                    max_batch=rng.choice([1000, 4096, 16384]))
    if kind == "fit":
        K = rng.randint(3, 12)
        return dict(kind=kind, V=_log(rng, 200, 2000), K=K, D=K, docs=_log(rng, 300, 2000),
                    length=rng.randint(30, 60), alpha0=1.0, batches=rng.randint(2, 6),
                    passes=rng.randint(3, 10))
    if kind == "slices":
        return dict(kind=kind, V=_log(rng, 2000, 20000), docs=_log(rng, 2000, 65536),
                    length=rng.randint(8, 25), alpha0=1.0, slices=rng.randint(3, 24),
                    batches=rng.randint(1, 2))
    alpha0 = rng.choice([1.0, 2.0])
    length = rng.randint(8, 40)
    if kind in ("refresh", "online"):
        V = _log(rng, 700, 20000)
        K = _log(rng, 5, 100 if kind == "refresh" else 60)
        return dict(kind=kind, V=V, K=K, D=K, docs=_log(rng, 4000, 65536), length=length,
                    alpha0=alpha0)
    V = _log(rng, 300, 50000)
    top = 128 if kind in ("pass", "classic", "step") else 120
    D, K = _log(rng, 4, top), _log(rng, 4, top)
    if rng.random() < 0.5:
        K = D
    if kind in ("step", "pass") and max(D, K) > 120:
        D, K = min(D, 120), min(K, 120)
    docs = _log(rng, 700, 200000 if kind == "step" else 65536)
    while docs * length > 4_500_000:
        docs //= 2
    case = dict(kind=kind, V=V, K=K, D=D, docs=docs, length=length, alpha0=alpha0)
    if kind == "step" or kind == "pass" or kind == "classic":
        case["bf16"] = rng.random() < 0.5
    if kind == "two":
        case["bf16"] = False
    if kind == "pass":
        case["batches"] = rng.randint(2, 4)
    if kind == "infer":
        case["max_iter"] = rng.choice([50, 200])
    return case


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _log_dirichlet(g, conc, rows, cols):
    """Dirichlet(conc) rows through log-Gamma variates (small conc underflows otherwise)."""
    a = torch.full((rows, cols), conc + 1.0, dtype=F64, device="cuda")
    lg = torch._standard_gamma(a, generator=g).log()
    lg += torch.rand(rows, cols, dtype=F64, device="cuda", generator=g).clamp_min(1e-300).log() / conc
    lg -= lg.amax(1, keepdim=True)
    p = lg.exp()
    return p / p.sum(1, keepdim=True)


def _topics(g, V, K):
    """[K][V] topics: 0.3 Zipf + 0.7 Dirichlet (Dirichlet(0.1) alone for small vocabularies)."""
    if V < 2000:
        mu = 0.98 * _log_dirichlet(g, 0.1, K, V) + 0.02 / V
    else:
        z = torch.arange(1, V + 1, dtype=F64, device="cuda") ** -1.1
        zipf = torch.empty_like(z)
        zipf[torch.randperm(V, device="cuda", generator=g)] = z / z.sum()
        mu = 0.3 * zipf + 0.7 * _log_dirichlet(g, 0.01, K, V)
    return mu / mu.sum(1, keepdim=True)


def _documents(g, mu, n, length, alpha0):
    """CSR arrays (device) of n documents of 1 + Poisson(length) tokens."""
    K, V = mu.shape
    L = 1 + torch.poisson(torch.full((n,), float(length), device="cuda"), generator=g).long()
    doc = torch.repeat_interleave(torch.arange(n, device="cuda"), L)
    cum_h = _log_dirichlet(g, alpha0 / K, n, K).cumsum(1).clamp_max(1.0)
    cum_h[:, -1] = 1.0
    cum_h += torch.arange(n, device="cuda", dtype=F64)[:, None]
    u = torch.rand(doc.numel(), dtype=F64, device="cuda", generator=g) * (1 - 1e-9)
    topic = torch.searchsorted(cum_h.view(-1), doc + u, right=True) - doc * K
    topic.clamp_(0, K - 1)
    del cum_h
    cum_mu = mu.cumsum(1).clamp_max(1.0)
    cum_mu[:, -1] = 1.0
    cum_mu += torch.arange(K, device="cuda", dtype=F64)[:, None]
    u = torch.rand(doc.numel(), dtype=F64, device="cuda", generator=g) * (1 - 1e-9)
    word = torch.searchsorted(cum_mu.view(-1), topic + u, right=True) - topic * V
    word.clamp_(0, V - 1)
    key, cnt = torch.unique_consecutive((doc * V + word).sort().values, return_counts=True)
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.bincount(key // V, minlength=n).cumsum(0).int()
    return rp, (key % V).int().contiguous(), cnt.float().contiguous()


def _dense(csr, V, lo, hi, counts=False):
    """Rows lo .. hi as dense 64-bit frequencies (or counts), dropped rows zero; and the lengths."""
    rp, ci, va = csr
    a, b = int(rp[lo]), int(rp[hi])
    row = torch.repeat_interleave(torch.arange(hi - lo, device="cuda"),
                                  (rp[lo + 1:hi + 1] - rp[lo:hi]).long())
    F = torch.zeros(hi - lo, V, dtype=F64, device="cuda")
    F[row, ci[a:b].long()] = va[a:b].double()
    L = F.sum(1)
    keep = L >= 3
    F[~keep] = 0
    return (F if counts else F / L.clamp_min(1)[:, None]), L, keep


def _whitening(g, csr, V, D, alpha0, n):
    """W = U diag(l)^(-1/2), l and M1 of the first n documents (64-bit subspace iteration)."""
    F, _, keep = _dense(csr, V, 0, n)
    F = F[keep]
    m = F.mean(0)
    F -= m
    p = min(D + 8, V)
    Q = torch.randn(V, p, dtype=F64, device="cuda", generator=g)
    for _ in range(5):
        Q = F.T @ (F @ Q)
        Q /= Q.norm(dim=0)
        C = torch.linalg.cholesky((Q.T @ Q).cpu() + 1e-13 * p * torch.eye(p, dtype=F64))
        Q = Q @ torch.linalg.inv(C).T.contiguous().cuda()
    B = F @ Q
    l, Z = np.linalg.eigh(((B.T @ B) * ((alpha0 + 1) / F.shape[0])).cpu().numpy())
    l = torch.from_numpy(np.maximum(l[::-1][:D], 1e-6 * l[-1]).copy()).cuda()
    U = Q @ torch.from_numpy(Z[:, ::-1][:, :D].copy()).cuda()
    U /= U.norm(dim=0)
    return (U / l.sqrt()).contiguous(), m


def _factors(g, mu, m, W, alpha0):
    """FP32 factors [D][K] near a fit's converged ones."""
    K, D = mu.shape[0], W.shape[1]
    Phi = K ** (-1.0 / 3.0) * (W.T @ (mu - m).T)
    Phi = Phi / Phi.norm(dim=0, keepdim=True).clamp_min(1e-6)
    Phi += 0.05 * torch.randn(D, K, dtype=F64, device="cuda", generator=g) / math.sqrt(D)
    return Phi.float().contiguous()


def _corpus(case, seed, batches=1):
    """Topics, an injected whitening and the case's batches."""
    g = _gen(seed)
    V, n = case["V"], case["docs"]
    mu = _topics(g, V, case["K"])
    head = _documents(g, mu, 2048, case["length"], case["alpha0"])
    W, m = _whitening(g, head, V, case["D"], case["alpha0"], 2048)
    Phi = _factors(g, mu, m, W, case["alpha0"])
    docs = [_documents(g, mu, n, case["length"], case["alpha0"]) for _ in range(batches)]
    return W, m, Phi, docs


def _mlp_weights(seed, D, H, K):
    rng = np.random.default_rng(seed)
    out = []
    for a, b in ((D, H), (H, H), (H, K)):
        lim = math.sqrt(6.0 / (a + b))
        out += [rng.uniform(-lim, lim, a * b), rng.uniform(-0.05, 0.05, b)]
    return np.concatenate(out).astype(np.float32)


def _mlp_rows(g, n, D, K):
    """Whitened rows (heavier tails than normal) and target proportions."""
    X = torch.randn(n, D, device="cuda", generator=g)
    X *= 0.5 + torch.rand(n, 1, device="cuda", generator=g)
    T = torch.softmax(3.0 * torch.randn(n, K, device="cuda", generator=g), 1)
    return X, T.contiguous()


BETA = 1e-3


def _ctx(case, W, m, **kw):
    ctx = tl.tlda_create(case["V"], case["K"], case["D"], case["alpha0"], 0.0, **kw)
    tl.tlda_set_whitening(ctx, W.cpu().numpy(), m.cpu().numpy())
    return ctx


# ---------------------------------------------------------------------------
# what a program has in hand before the call
# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case)
    if kind in ("step", "classic", "two", "pass", "infer"):
        W, m, Phi, docs = _corpus(case, seed, case.get("batches", 1))
        stream = torch.cuda.Stream() if kind == "pass" else None
        ctx = _ctx(case, W, m, bf16=case.get("bf16", False), classic=kind == "classic",
                   stream=stream)
        b = [tl.CsrBatch(*d) for d in docs]
        s.update(ctx=ctx, batch=b[0], batches=b, Phi=Phi)
        s["grad"] = torch.empty_like(Phi)
        s["kept"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        if kind == "two":
            s["X"] = torch.empty(case["docs"], case["D"], device="cuda")
        if kind == "infer":
            s["theta"] = torch.empty(case["docs"], case["K"], device="cuda")
        if kind == "pass":
            torch.cuda.synchronize()
            s["graph"] = tl.tlda_graph_capture_steps(ctx, b, BETA, Phi)
    elif kind in ("fit", "refresh", "online"):
        g = _gen(seed)
        mu = _topics(g, case["V"], case["K"])
        s["batches"] = [tl.CsrBatch(*_documents(g, mu, case["docs"], case["length"], case["alpha0"]))
                        for _ in range(case.get("batches", 1))]
        s["ctx"] = ctx = tl.tlda_create(case["V"], case["K"], case["D"], case["alpha0"], 0.0)
        s["Phi0"] = torch.linalg.qr(torch.randn(case["D"], case["K"], dtype=F64,
                                                generator=torch.Generator().manual_seed(seed))
                                    )[0].float().contiguous().cuda()
        s["Phi"], s["grad"] = s["Phi0"].clone(), torch.empty_like(s["Phi0"])
        s["kept"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        if kind != "fit":
            tl.tlda_update_moments(ctx, s["batches"][0])
        if kind == "online":
            tl.tlda_update_moments(ctx, None, tl.TLDA_REFRESH_W)
            s["batches"] = [tl.CsrBatch(*_documents(g, mu, case["docs"], case["length"],
                                                    case["alpha0"]))]
    elif kind in ("train", "encode"):
        g = _gen(seed)
        D, H, K, n = case["D"], case["hidden"], case["K"], case["rows"]
        s["mlp"] = tl.tlda_mlp_create(D, H, K, case.get("max_batch", n))
        tl.tlda_mlp_set_params(s["mlp"], _mlp_weights(seed, D, H, K))
        s["rows"] = [_mlp_rows(g, n, D, K) for _ in range(case.get("steps", 0) + 1)]
        s["loss"] = torch.zeros(case.get("steps", 0), device="cuda")
        s["theta"] = torch.empty(n, K, device="cuda")
    else:
        s.update(_slices(case, seed))
    torch.cuda.synchronize()
    return s


def _slice_cases(case):
    """Each slice's own K and batch size, as the slice workload has them."""
    out = []
    for i in range(case["slices"]):
        K = (10, 20, 50)[(7 * i + 1) % 3]
        docs = max(500, int(case["docs"] * (0.12 + 0.88 * ((37 * i) % 24) / 23.0)))
        out.append(dict(V=case["V"], K=K, D=K, docs=docs, length=case["length"],
                        alpha0=case["alpha0"]))
    return out


def _slices(case, seed):
    stream = torch.cuda.Stream()
    ctxs, Phis, batches = [], [], []
    for i, c in enumerate(_slice_cases(case)):
        W, m, Phi, docs = _corpus(c, seed * 100 + i, case["batches"])
        torch.cuda.synchronize()
        ctxs.append(_ctx(c, W, m, bf16=True, stream=stream))
        Phis.append(Phi)
        batches.append([tl.CsrBatch(*d) for d in docs])
    torch.cuda.synchronize()
    plans = [tl.tlda_multi_create(ctxs, [b[j] for b in batches], Phis, [BETA] * len(ctxs))
             for j in range(case["batches"])]
    return dict(ctxs=ctxs, Phis=Phis, plans=plans, graph=tl.tlda_graph_capture(plans))


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind in ("step", "classic"):
        tl.tlda_whiten_cp_step(s["ctx"], s["batch"], BETA, s["Phi"], s["grad"], None, s["kept"])
        return dict(Phi=s["Phi"], grad=s["grad"], kept=s["kept"])
    if kind == "two":
        tl.tlda_whiten_batch(s["ctx"], s["batch"], s["X"], s["kept"])
        tl.tlda_cp_step(s["ctx"], s["X"], case["docs"], s["kept"], BETA, s["Phi"], s["grad"])
        return dict(X=s["X"], Phi=s["Phi"], grad=s["grad"], kept=s["kept"])
    if kind == "pass":
        tl.tlda_graph_launch(s["graph"])
        return dict(Phi=s["Phi"])
    if kind == "fit":
        ctx, Phi = s["ctx"], s["Phi"]
        Phi.copy_(s["Phi0"])
        for i, b in enumerate(s["batches"]):
            tl.tlda_update_moments(ctx, b, tl.TLDA_RESET if i == 0 else 0)
        tl.tlda_update_moments(ctx, None, tl.TLDA_REFRESH_W)
        for _ in range(case["passes"]):
            for b in s["batches"]:
                tl.tlda_whiten_cp_step(ctx, b, 0.03, Phi)
        mu, _, _ = tl.tlda_unwhiten(ctx, Phi, tl.TLDA_PROJECT_SIMPLEX)
        theta = tl.tlda_infer_doc_topics(ctx, s["batches"][-1], mu, 50, 1e-6)
        return dict(Phi=Phi, mu=mu.float(), theta=theta)
    if kind == "refresh":
        tl.tlda_update_moments(s["ctx"], None, tl.TLDA_REFRESH_W)
        W, eig, m = tl.tlda_get_whitening(s["ctx"])
        return dict(W=W, eig=eig, M1=m)
    if kind == "online":
        tl.tlda_update_moments(s["ctx"], s["batches"][0], tl.TLDA_REFRESH_WARM)
        tl.tlda_rebase_phi(s["ctx"], s["Phi"])
        tl.tlda_whiten_cp_step(s["ctx"], s["batches"][0], BETA, s["Phi"], s["grad"], None,
                               s["kept"])
        return dict(Phi=s["Phi"], grad=s["grad"], kept=s["kept"])
    if kind == "infer":
        mu, alpha, lam = tl.tlda_unwhiten(s["ctx"], s["Phi"], tl.TLDA_PROJECT_SIMPLEX)
        tl.tlda_infer_doc_topics(s["ctx"], s["batch"], mu, case["max_iter"], 1e-6, s["theta"])
        return dict(mu=mu, alpha=alpha, lam=lam, theta=s["theta"])
    if kind == "train":
        for i in range(case["steps"]):
            X, T = s["rows"][i]
            tl.tlda_mlp_train_step(s["mlp"], X, T, 2e-3, s["loss"][i:i + 1])
        g, loss = tl.tlda_mlp_gradients(s["mlp"], *s["rows"][-1])
        return dict(losses=s["loss"], grads=g, loss=loss)
    if kind == "encode":
        return dict(theta=tl.tlda_mlp_forward(s["mlp"], s["rows"][0][0], s["theta"]))
    tl.tlda_graph_launch(s["graph"])
    return {"Phi%02d" % i: P for i, P in enumerate(s["Phis"])}


# ---------------------------------------------------------------------------
# the work that a pass cannot do without
# ---------------------------------------------------------------------------
def _nnz(c):
    return c["docs"] * (c["length"] + 1) * (0.62 if c["V"] < 2000 else 0.95)


def _step_work(c, wbytes):
    n, D, K, nnz = c["docs"], c["D"], c["K"], _nnz(c)
    return (4 * n + 8 * nnz + wbytes * c["V"] * D + 8 * D * K,
            n * (4.0 * D * K + K) + 2.0 * nnz * D + 4.0 * D * K * K)


def work(case):
    kind = case["kind"]
    if kind in ("train", "encode"):
        D, H, K, n = case["D"], case["hidden"], case["K"], case["rows"]
        P = D * H + H * H + H * K + 2 * H + K
        if kind == "encode":
            return dict(bytes=4 * n * (D + K) + 2 * P, flops=2.0 * n * (D * H + H * H + H * K))
        t = case["steps"]
        return dict(bytes=(t + 1) * 4 * n * (D + K) + t * 28 * P,
                    flops=(t + 1) * n * (6.0 * H * H + 6.0 * H * K + 4.0 * D * H))
    if kind == "slices":
        w = [_step_work(c, 2) for c in _slice_cases(case)]
        return dict(bytes=case["batches"] * sum(x[0] for x in w),
                    flops=case["batches"] * sum(x[1] for x in w))
    V, D, K, n, nnz = case["V"], case["D"], case["K"], case["docs"], _nnz(case)
    B = case.get("batches", 1)
    step = _step_work(case, 2 if case.get("bf16") else 4)
    pairs = n * (nnz / n) * (nnz / n + 1) / 2
    p = min(V, max(2 * D, D + 16))
    if kind in ("step", "pass"):
        return dict(bytes=B * step[0], flops=B * step[1])
    if kind == "classic":
        return dict(bytes=step[0], flops=2.0 * (nnz + n) * D * K + 2.0 * V * D * K + 6.0 * nnz * K)
    if kind == "two":
        return dict(bytes=step[0] + 4 * n * D, flops=step[1])
    if kind == "fit":
        return dict(bytes=B * (4 * n + 8 * nnz) + 16 * V * V + case["passes"] * B * step[0],
                    flops=B * pairs + 60.0 * 2 * V * V * p + case["passes"] * B * step[1]
                    + 50.0 * n * 2 * K * K)
    if kind == "refresh":
        return dict(bytes=8 * V * V + 8 * V * (D + 1), flops=60.0 * 2 * V * V * p)
    if kind == "online":
        return dict(bytes=step[0] + 8 * nnz + 8 * V * V + 8 * V * (D + 1),
                    flops=pairs + 5.0 * 2 * V * V * p + step[1])
    return dict(bytes=8 * V * (D + K) + 8 * nnz + 4 * n * K + 4 * V * D,
                flops=4.0 * V * D * K + 2.0 * nnz * D + 2.0 * n * D * K
                + case["max_iter"] * n * (2.0 * K * K + 6.0 * K))


# ---------------------------------------------------------------------------
# the same in 64 bits, by plain torch
# ---------------------------------------------------------------------------
def _whitened(csr, V, m, W):
    """X in 64 bits (rows of dropped documents zero) and the kept count."""
    n = csr[0].numel() - 1
    step = max(256, int(2e8 / V))
    X, kept = torch.empty(n, W.shape[1], dtype=F64, device="cuda"), 0
    shift = m @ W
    for lo in range(0, n, step):
        F, _, keep = _dense(csr, V, lo, min(n, lo + step))
        X[lo:lo + step] = (F @ W - shift) * keep[:, None]
        kept += int(keep.sum())
    return X, kept


def _penalty(Phi):
    G = Phi.T @ Phi
    return 3.0 * Phi @ (G * G)


def _gradient(X, n, Phi, alpha0):
    S = X @ Phi
    return _penalty(Phi) - 1.5 * (alpha0 + 1) * (alpha0 + 2) / n * (X.T @ (S * S))


def _classic_gradient(csr, V, m, W, Phi, a0):
    c2, c3 = a0 * (a0 + 1) / 2, (a0 + 1) * (a0 + 2) / 2
    Z, mw = W @ Phi, m @ W
    r = mw @ Phi
    n, step = csr[0].numel() - 1, max(256, int(2e8 / V))
    out, kept = torch.zeros_like(Phi), 0
    for lo in range(0, n, step):
        C, L, keep = _dense(csr, V, lo, min(n, lo + step), counts=True)
        C, L = C[keep], L[keep]
        kept += L.numel()
        l2 = (1 / (L * (L - 1)))[:, None]
        l3 = l2 / (L - 2)[:, None]
        s, q = C @ Z, C @ (Z * Z)
        a = c3 * l3 * (s * s - q) - c2 * l2 * 2 * r * s
        b = -2 * c3 * l3 * s + 2 * c2 * l2 * r
        out += W.T @ (C.T @ a + Z * (C.T @ b)
                      + Z * Z * (C.T @ (2 * c3 * l3).expand(-1, Phi.shape[1]).contiguous()))
        out += torch.outer(mw, (-c2 * l2 * (s * s - q) + a0 * a0 * r * r).sum(0))
    return _penalty(Phi) - 3.0 / kept * out


def _solve(X, A, max_iter, tol):
    G = A.T @ A
    step = 1.0 / float(np.linalg.eigvalsh(G.cpu().numpy())[-1])
    K = A.shape[1]
    b = X @ A
    t = torch.full((X.shape[0], K), 1.0 / K, dtype=F64, device="cuda")
    live = torch.ones(X.shape[0], dtype=torch.bool, device="cuda")
    j = torch.arange(1, K + 1, dtype=F64, device="cuda")
    for _ in range(max_iter):
        y = t - step * (t @ G - b)
        u = y.sort(1, descending=True).values
        tau = (u.cumsum(1) - 1) / j
        rho = ((u > tau) * j).amax(1).long() - 1
        new = (y - tau.gather(1, rho[:, None])).clamp_min(0)
        change = (new - t).abs().sum(1)
        t = torch.where(live[:, None], new, t)
        live &= change >= tol
        if not bool(live.any()):
            break
    return t


def _recover(Phi, U, l, m):
    n2 = (Phi * Phi).sum(0)
    lo, hi = torch.zeros_like(n2), torch.ones_like(n2)
    for _ in range(200):
        mid = 0.5 * (lo + hi)
        low = mid ** (1.0 / 3.0) * n2 + mid < 1
        lo, hi = torch.where(low, mid, lo), torch.where(low, hi, mid)
    a = 0.5 * (lo + hi)
    mu = (U * l.sqrt()) @ (Phi * a ** (-1.0 / 3.0)) + m[:, None]
    mu = mu.clamp_min(0)
    return mu / mu.sum(0), a / a.sum(), n2 ** 1.5


def _top_pairs(M2, D):
    """Top-D eigenpairs, signed so that the largest-magnitude entry is positive."""
    V = M2.shape[0]
    if V <= 1200:
        l, U = np.linalg.eigh(M2.cpu().numpy())
        l, U = l[::-1][:D].copy(), U[:, ::-1][:, :D].copy()
        l, U = torch.from_numpy(l).cuda(), torch.from_numpy(U).cuda()
    else:
        p = min(V, 3 * D + 32)
        Q = torch.randn(V, p, dtype=F64, device="cuda", generator=_gen(5))
        for it in range(150):
            Q = M2 @ Q
            if it % 3 == 2 or it == 149:
                for _ in range(2):
                    Q /= Q.norm(dim=0)
                    C = torch.linalg.cholesky((Q.T @ Q).cpu() + 1e-14 * torch.eye(p, dtype=F64))
                    Q = Q @ torch.linalg.inv(C).T.contiguous().cuda()
        l, Z = np.linalg.eigh((Q.T @ (M2 @ Q)).cpu().numpy())
        l = torch.from_numpy(l[::-1][:D].copy()).cuda()
        U = Q @ torch.from_numpy(Z[:, ::-1][:, :D].copy()).cuda()
        U /= U.norm(dim=0)
    top = U.abs().argmax(0)
    return l, U * U.gather(0, top[None]).sign()


def _second_moment(batches, V, alpha0):
    S, f, N = torch.zeros(V, V, dtype=F64, device="cuda"), 0, 0
    for csr in batches:
        n, step = csr[0].numel() - 1, max(256, int(2e8 / V))
        for lo in range(0, n, step):
            F, _, keep = _dense(csr, V, lo, min(n, lo + step))
            S += F.T @ F
            f, N = f + F.sum(0), N + int(keep.sum())
    m = f / N
    S *= (alpha0 + 1) / N
    S -= (alpha0 + 1) * torch.outer(m, m)
    return S, m


def _forward(P, X):
    Z1 = X @ P[0] + P[1]
    H1 = 0.5 * Z1 * (1 + torch.erf(Z1 / math.sqrt(2.0)))
    Z2 = H1 @ P[2] + P[3]
    H2 = 0.5 * Z2 * (1 + torch.erf(Z2 / math.sqrt(2.0)))
    return torch.log_softmax(H2 @ P[4] + P[5], 1)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "pass", "two", "classic", "infer"):
        W, m, Phi, docs = _corpus(case, seed, case.get("batches", 1))
        P, a0 = Phi.double(), case["alpha0"]
        if kind == "classic":
            G = _classic_gradient(docs[0], case["V"], m, W, P, a0)
            return dict(Phi=P - BETA * G, grad=G, kept=None)
        for d in docs:
            X, n = _whitened(d, case["V"], m, W)
            if kind == "infer":
                l = 1.0 / (W * W).sum(0)
                mu, alpha, lam = _recover(P, W * l.sqrt(), l, m)
                return dict(mu=mu, alpha=alpha, lam=lam,
                            theta=_solve(X, W.T @ (mu - m[:, None]), case["max_iter"], 1e-6))
            G = _gradient(X, n, P, a0)
            P = P - BETA * G
        if kind == "pass":
            return dict(Phi=P)
        out = dict(Phi=P, grad=G, kept=None)
        if kind == "two":
            out["X"] = X
        return out
    if kind in ("fit", "refresh"):
        g = _gen(seed)
        mu = _topics(g, case["V"], case["K"])
        docs = [_documents(g, mu, case["docs"], case["length"], case["alpha0"])
                for _ in range(case.get("batches", 1))]
        M2, m = _second_moment(docs, case["V"], case["alpha0"])
        l, U = _top_pairs(M2, case["D"])
        W = U / l.sqrt()
        if kind == "refresh":
            return dict(W=W, eig=l, M1=m)
        P = torch.linalg.qr(torch.randn(case["D"], case["K"], dtype=F64,
                                        generator=torch.Generator().manual_seed(seed))
                            )[0].float().double().cuda()
        X = [_whitened(d, case["V"], m, W) for d in docs]
        for _ in range(case["passes"]):
            for x, n in X:
                P = P - 0.03 * _gradient(x, n, P, case["alpha0"])
        mu, _, _ = _recover(P, U, l, m)
        return dict(Phi=P, mu=mu, theta=_solve(X[-1][0], W.T @ (mu - m[:, None]), 50, 1e-6))
    if kind == "online":
        return None   # a few iterations from the library's own earlier subspace, not a closed form
    if kind in ("train", "encode"):
        g = _gen(seed)
        D, H, K, n = case["D"], case["hidden"], case["K"], case["rows"]
        flat = torch.from_numpy(_mlp_weights(seed, D, H, K)).cuda().double()
        rows = [_mlp_rows(g, n, D, K) for _ in range(case.get("steps", 0) + 1)]
        sizes = [D * H, H, H * H, H, H * K, K]

        def parts(x):
            p = list(torch.split(x, sizes))
            return [p[0].view(D, H), p[1], p[2].view(H, H), p[3], p[4].view(H, K), p[5]]

        if kind == "encode":
            return dict(theta=_forward(parts(flat), rows[0][0].double()).exp())
        am, av, losses = torch.zeros_like(flat), torch.zeros_like(flat), []
        for t, (X, T) in enumerate(rows, 1):
            flat = flat.detach().requires_grad_(True)
            loss = -(T.double() * _forward(parts(flat), X.double())).sum() / n
            grad, = torch.autograd.grad(loss, flat)
            losses.append(loss.detach())
            am, av = 0.9 * am + 0.1 * grad, 0.999 * av + 0.001 * grad * grad
            flat = flat.detach() - 2e-3 * (am / (1 - 0.9 ** t)) / ((av / (1 - 0.999 ** t)).sqrt()
                                                                 + 1e-8)
        return dict(losses=torch.stack(losses[:-1]), grads=grad, loss=losses[-1].view(1))
    out = {}
    for i, c in enumerate(_slice_cases(case)):
        W, m, Phi, docs = _corpus(c, seed * 100 + i, case["batches"])
        P = Phi.double()
        for d in docs:
            X, n = _whitened(d, c["V"], m, W)
            P = P - BETA * _gradient(X, n, P, c["alpha0"])
        out["Phi%02d" % i] = P
    return out
