"""Drives libtlda's host layer on the runtime stand-in (fake_hip.cpp), without
a GPU.  Usage: python driver.py STAND_IN_SO CHECK; exit status 0 when CHECK
holds.  Run in a process of its own: the stand-in takes the real runtime's
place, so torch (which loads that) must stay out."""
import ctypes
import os
import sys
import types

ROOT = os.path.dirname(os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
sys.path.insert(0, ROOT)
FAKE = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.modules["torch"] = types.ModuleType("torch")   # the binding's import

import numpy as np  # noqa: E402

from paper_2511_07809_amd import tlda as tl  # noqa: E402

LIB = tl._LIB
for name, res in (("fake_kernel", ctypes.c_char_p), ("fake_query", ctypes.c_char_p),
                  ("fake_grid", ctypes.c_uint32), ("fake_block", ctypes.c_uint32),
                  ("fake_arg", ctypes.c_uint64)):
    getattr(FAKE, name).restype = res
FAKE.fake_fail_malloc.argtypes = [ctypes.c_longlong]

NUM_CU = 256


def context(V, K, D, flags=0):
    cfg = tl.tlda_config(V, K, D, flags, 1.0, 0.0, 0, 0, 0, 0)
    h = ctypes.c_void_p()
    # (any stream but the null one, which is never captured)
    assert LIB.tlda_create(ctypes.byref(cfg), ctypes.c_void_p(8), ctypes.byref(h)) == 0
    return h


def set_whitening(h, V, D, seed=0):
    rng = np.random.default_rng(seed)
    W, m = rng.standard_normal((V, D)), np.full(V, 1.0 / V)
    return LIB.tlda_set_whitening(h, W.ctypes.data, m.ctypes.data)


def batch(n, words=4):
    """n documents of `words` words each (arrays that outlive the call)."""
    rp = np.arange(n + 1, dtype=np.int32) * words
    ci = np.tile(np.arange(words, dtype=np.int32), n)
    va = np.ones(n * words, dtype=np.float32)
    batch.keep = getattr(batch, "keep", []) + [(rp, ci, va)]
    return tl.tlda_csr_batch(n, n * words, rp.ctypes.data, ci.ctypes.data, va.ctypes.data, -1, 0)


def step(h, b, D, K):
    """The step's launches, as (kernel, grid in x)."""
    Phi = np.zeros((D, K), dtype=np.float32)
    FAKE.fake_clear()
    assert LIB.tlda_whiten_cp_step(h, ctypes.byref(b), 0.0, Phi.ctypes.data, None, None, None) == 0
    return launches()


def launches():
    return [(FAKE.fake_kernel(i).decode(), FAKE.fake_grid(i, 0))
            for i in range(FAKE.fake_launches())]


def base(kernel):
    return kernel.replace("(anonymous namespace)::", "").split("(")[0].split("<")[0].split("::")[-1]


def check_fused_grid_does_not_depend_on_the_batch_before():
    """The grid of a fused FP32 step is a function of its own batch: one round
    of the blocks of the instance that is launched, whichever batch came first."""
    # every row-tile height its own occupancy: 16 rows (small batches), 32, 64
    for t, n in ((16, 3), (32, 5), (64, 7)):
        for dq in (16, 32):
            for kq in (16, 32, 64):
                FAKE.fake_occupancy(f"k_whiten_cp<{dq}, {kq}, {t},".encode(), n)
    V = 400
    for D, K in ((5, 5), (32, 10), (16, 33)):
        seen = []
        for order in ((1000, 200000), (200000, 1000), (16384, 16385), (16385, 16384)):
            h = context(V, K, D)
            assert set_whitening(h, V, D) == 0
            grids = {}
            for n in order:
                b = batch(n, 1)
                kernel, grid = step(h, b, D, K)[0]
                assert base(kernel) == "k_whiten_cp", kernel
                queried = [FAKE.fake_query(i).decode() for i in range(FAKE.fake_queries())]
                assert all(q == kernel for q in queried), (queried, kernel)
                grids[n] = grid
            seen.append(grids)
            LIB.tlda_destroy(h)
        assert seen[0] == seen[1] and seen[2] == seen[3], (D, K, seen)
        assert seen[0][200000] in (5 * NUM_CU, 7 * NUM_CU), seen   # the round is full


def check_captured_steps_never_regrow_their_partials():
    """A graph of steps keeps the address of the context's partials: neither
    instance's later step may need more than the capture reserved."""
    for t, n in ((16, 8), (32, 1), (64, 1)):
        FAKE.fake_occupancy(f", {t},".encode(), n)
    FAKE.fake_keep_args(b"k_whiten_cp<", 13)
    V, D, K = 400, 5, 5
    Phi = np.zeros((D, K), dtype=np.float32)
    h = context(V, K, D)
    assert set_whitening(h, V, D) == 0
    FAKE.fake_clear()
    arr = (tl.tlda_csr_batch * 1)(batch(200000, 1))
    g = ctypes.c_void_p()
    assert LIB.tlda_graph_capture_steps(h, arr, 1, 0.0, Phi.ctypes.data, ctypes.byref(g)) == 0
    partial = FAKE.fake_arg(0, 11)
    for n in (16384, 1000, 500000):
        step(h, batch(n, 1), D, K)
        assert FAKE.fake_arg(0, 11) == partial, n
    LIB.tlda_graph_destroy(g)
    LIB.tlda_destroy(h)


def check_no_step_regrows_what_a_graph_writes():
    """A graph captured over small batches keeps its partials when the context
    then steps larger ones, from the batch or from X."""
    FAKE.fake_occupancy(b"k_cp_reduce_mfma<", 6)
    freed = []
    for D, K, flags in ((5, 5, 0), (50, 50, 0), (100, 100, 0), (16, 100, 0), (50, 50, tl.TLDA_BF16),
                        (100, 100, tl.TLDA_BF16)):
        V = 400
        Phi = np.zeros((D, K), dtype=np.float32)
        h = context(V, K, D, flags)
        assert set_whitening(h, V, D) == 0
        small, large = batch(1000, 1), batch(300000, 1)
        g = ctypes.c_void_p()
        arr = (tl.tlda_csr_batch * 1)(small)
        assert LIB.tlda_graph_capture_steps(h, arr, 1, 0.0, Phi.ctypes.data, ctypes.byref(g)) == 0
        before = FAKE.fake_frees()
        step(h, large, D, K)
        assert LIB.tlda_cp_step(h, ctypes.c_void_p(1 << 20), 300000, None, 0.0, Phi.ctypes.data,
                                None) == 0
        if FAKE.fake_frees() != before:
            freed.append((D, K, flags))
        LIB.tlda_graph_destroy(g)
        LIB.tlda_destroy(h)
    assert not freed, freed


def check_rebase_after_a_failed_allocation():
    """Out of memory anywhere in keeping the previous whitening leaves a context
    whose next whitening and rebase work: no kernel gets a null buffer."""
    FAKE.fake_keep_args(b"k_gram(", 8)
    FAKE.fake_keep_args(b"k_gram_sum(", 6)
    FAKE.fake_keep_args(b"k_rebase(", 6)
    V, D, K = 300, 6, 5
    Phi = np.zeros((D, K), dtype=np.float32)
    failures = 0
    for after in range(6):
        h = context(V, K, D)
        assert set_whitening(h, V, D, 1) == 0
        FAKE.fake_fail_malloc(after)
        st = set_whitening(h, V, D, 2)
        FAKE.fake_fail_malloc(-1)
        assert st in (0, 6), st   # TLDA_ERR_OOM
        failures += st == 6
        assert set_whitening(h, V, D, 3) == 0
        FAKE.fake_clear()
        assert LIB.tlda_rebase_phi(h, Phi.ctypes.data) == 0
        seen = set()
        for i, (kernel, _) in enumerate(launches()):
            pointers = {"k_gram": (0, 1, 6), "k_gram_sum": (0, 3), "k_rebase": (0, 1, 2, 5)}
            seen.add(base(kernel))
            for a in pointers[base(kernel)]:
                assert FAKE.fake_arg(i, a) != 0, (after, kernel, a)
        assert seen == {"k_gram", "k_gram_sum", "k_rebase"}
        LIB.tlda_destroy(h)
    assert failures == 4


def check_classic_step_after_a_failed_allocation():
    """Out of memory in a classic context's first step: the next one works."""
    FAKE.fake_keep_args(b"k_classic_z", 10)
    FAKE.fake_keep_args(b"k_classic_cp<", 15)
    V, D, K = 300, 6, 5
    for flags in (tl.TLDA_CLASSIC, tl.TLDA_CLASSIC | tl.TLDA_BF16):
        failures = 0
        for after in range(4):
            h = context(V, K, D, flags)
            assert set_whitening(h, V, D, 1) == 0
            Phi, b = np.zeros((D, K), dtype=np.float32), batch(100)
            FAKE.fake_fail_malloc(after)
            st = LIB.tlda_whiten_cp_step(h, ctypes.byref(b), 0.0, Phi.ctypes.data, None, None, None)
            FAKE.fake_fail_malloc(-1)
            assert st in (0, 6), st
            failures += st == 6
            seen = [base(k) for k, _ in step(h, b, D, K)]
            assert seen[1] == "k_classic_cp", seen
            for i, args in ((0, (0, 4, 7, 8, 9)), (1, (4, 6, 8, 9, 14))):
                assert all(FAKE.fake_arg(i, a) != 0 for a in args), (flags, after, i)
            LIB.tlda_destroy(h)
        assert failures == 3


def check_encoder_forward_takes_any_number_of_rows():
    """Every launch stays within the 2^32 work items of a grid, and together they
    take every row once, from the right place of X and theta."""
    FAKE.fake_keep_args(b"k_forward<", 9)
    for d_in, hidden, k_out in ((50, 256, 50), (5, 16, 5), (1, 1024, 2), (1024, 64, 16)):
        m = ctypes.c_void_p()
        assert LIB.tlda_mlp_create(d_in, hidden, k_out, 64, None, ctypes.byref(m)) == 0
        for n in (1, 17, 1 << 20, (1 << 27) - 16, (1 << 27) + 1, (1 << 29) + 5, (1 << 33) + 7):
            FAKE.fake_clear()
            X, theta = 1 << 20, 1 << 50   # never read
            assert LIB.tlda_mlp_forward(m, X, n, theta) == 0, (hidden, n)
            row = 0
            for i, (kernel, grid) in enumerate(launches()):
                assert base(kernel) == "k_forward"
                docs = 16 * int(kernel.split("k_forward<")[1].split(",")[0])
                assert FAKE.fake_arg(i, 0) == X + 4 * d_in * row
                assert FAKE.fake_arg(i, 8) == theta + 4 * k_out * row, (i, kernel)
                rows = FAKE.fake_arg(i, 1)
                assert (grid - 1) * docs < rows <= grid * docs
                assert grid * FAKE.fake_block(i, 0) < 1 << 32
                row += rows
            assert row == n
        LIB.tlda_mlp_destroy(m)


def check_encoder_tiles_fit_what_they_hold():
    """LDS is sized by what each buffer holds, so that a wide input beside narrow
    layers, or a wide output, does not shrink the tile of documents."""
    for d_in, hidden, k_out, docs in ((50, 256, 50, 64), (1024, 64, 16, 32), (16, 16, 256, 64),
                                      (1024, 1024, 256, 16)):
        m = ctypes.c_void_p()
        assert LIB.tlda_mlp_create(d_in, hidden, k_out, 64, None, ctypes.byref(m)) == 0
        FAKE.fake_clear()
        assert LIB.tlda_mlp_forward(m, 1 << 20, 262144, 1 << 40) == 0
        assert [g for _, g in launches()] == [262144 // docs], (d_in, launches())
        LIB.tlda_mlp_destroy(m)


def check_few_blocks_do_not_form_the_gram_entries():
    """Past 128 columns or topics the reduction forms the finish's squared Gram
    entries only where enough blocks share them; else a launch of its own does."""
    FAKE.fake_keep_args(b"k_cp_reduce_wide(", 9)
    for D, K in ((56, 256), (16, 256), (130, 110), (200, 70), (256, 56)):
        h = context(400, K, D)
        Phi = np.zeros((D, K), dtype=np.float32)
        X = np.zeros((100000, D), dtype=np.float32)
        for n, apart in ((1, True), (65, True), (16384, False), (100000, False)):
            FAKE.fake_clear()
            assert LIB.tlda_cp_step(h, X.ctypes.data, n, None, 0.0, Phi.ctypes.data, None) == 0
            names = [base(k) for k, _ in launches()]
            assert names[0] == "k_cp_reduce_wide"
            assert ("k_gram_sq" in names) == apart, (D, K, n, names)
            assert (FAKE.fake_arg(0, 8) == 0) == apart, (D, K, n)
        LIB.tlda_destroy(h)


def check_few_columns_take_the_narrow_reduction():
    """Past 128 topics, few columns take the reduction that does not pad them to
    16; its grid and the other's do not depend on the batch before."""
    FAKE.fake_occupancy(b"k_cp_reduce_narrow", 3)
    Phi = np.zeros(20 * 256, dtype=np.float32)
    X = ctypes.c_void_p(1 << 20)   # never read

    def reduction(h, n):
        FAKE.fake_clear()
        assert LIB.tlda_cp_step(h, X, n, None, 0.0, Phi.ctypes.data, None) == 0
        return base(FAKE.fake_kernel(0).decode()), FAKE.fake_grid(0, 0)

    narrow, wide = "k_cp_reduce_narrow", "k_cp_reduce_wide"
    for D, K, n, want in ((1, 256, 1, narrow), (4, 233, 1, narrow), (4, 232, 16384, wide),
                          (4, 129, 16385, narrow), (5, 217, 1, narrow), (8, 180, 80000, wide),
                          (8, 180, 80001, narrow), (8, 181, 160000, wide), (8, 216, 160001, narrow),
                          (12, 160, 160001, narrow), (12, 161, 500000, wide), (16, 129, 500000, wide),
                          (20, 144, 160001, narrow), (20, 144, 160000, wide), (21, 129, 500000, wide)):
        seen = []
        for order in ((n, 7), (7, n)):
            h = context(400, K, D)
            got = {rows: reduction(h, rows) for rows in order}
            assert got[n][0] == want, (D, K, n, got)
            seen.append(got)
            LIB.tlda_destroy(h)
        assert seen[0] == seen[1], seen
        if n > 100000:
            assert seen[0][n][1] == (3 if want == narrow else 1) * NUM_CU, seen


def check_short_documents_of_many_topics_keep_the_tall_tiles():
    """Past 32 topics, a batch of more than 12288 documents takes 16-row tiles only
    if its documents have words enough."""
    for D, K, n, words, small in ((16, 60, 16384, 3, False), (16, 60, 16384, 12, True),
                                  (16, 60, 12288, 3, True), (4, 33, 12289, 11, False),
                                  (16, 32, 16384, 3, True), (32, 64, 16385, 20, False)):
        h = context(400, K, D)
        assert set_whitening(h, 400, D) == 0
        kernel, grid = step(h, batch(n, words), D, K)[0]
        rows = int(kernel.split("<")[1].split(",")[2])
        assert (rows == 16) == small, (D, K, n, words, kernel)
        assert grid == min((n + rows - 1) // rows, 2 * NUM_CU)
        LIB.tlda_destroy(h)


def check_small_plans_leave_the_gram_entries_to_the_finish():
    """A slice's table entry names a buffer for the squared Gram entries only where
    forming them in the reduction is the faster way."""
    FAKE.fake_keep_args(b"k_cp_bf16_multi<", 2)
    stride, at_nblk, at_gsq = 168, 104, 80   # of the device table's entries

    def gsq(slices, n, K):
        ctxs = []
        for _ in range(slices):
            h = context(400, K, K, tl.TLDA_BF16)
            assert set_whitening(h, 400, K) == 0
            ctxs.append(h)
        Phi = np.zeros((slices, K * K), dtype=np.float32)
        bs = (tl.tlda_csr_batch * slices)(*[batch(n)] * slices)
        P = (ctypes.c_void_p * slices)(*[Phi[i].ctypes.data for i in range(slices)])
        betas = (ctypes.c_float * slices)()
        plan = ctypes.c_void_p()
        assert LIB.tlda_multi_create(slices, (ctypes.c_void_p * slices)(*ctxs), bs, P, betas, None,
                                     ctypes.byref(plan)) == 0
        FAKE.fake_clear()
        assert LIB.tlda_multi_step(plan) == 0
        table, blocks, got = FAKE.fake_arg(0, 0), 0, []
        for i in range(slices):
            at = table + stride * i
            blocks += ctypes.c_int32.from_address(at + at_nblk).value
            got.append(ctypes.c_uint64.from_address(at + at_gsq).value != 0)
        assert blocks == FAKE.fake_grid(0, 0)   # (the table is read where it should be)
        LIB.tlda_multi_destroy(plan)
        for h in ctxs:
            LIB.tlda_destroy(h)
        return got

    assert gsq(1, 1000, 50) == [False] and gsq(2, 1000, 50) == [False] * 2
    assert gsq(1, 20000, 50) == [True] and gsq(1, 4000, 50) == [True]
    assert gsq(12, 1000, 50) == [True] * 12 and gsq(64, 1000, 10) == [False] * 64


def check_steps_only_launch():
    """A step on a warm context makes no runtime call beyond its launches that
    would cost host time on every one of them: no function attributes."""
    V = 400
    for D, K, flags in ((5, 5, 0), (100, 100, 0), (50, 50, tl.TLDA_BF16), (50, 49, tl.TLDA_CLASSIC),
                        (128, 128, tl.TLDA_CLASSIC), (50, 50, tl.TLDA_CLASSIC | tl.TLDA_BF16),
                        (150, 37, 0), (56, 256, 0), (1, 256, 0)):
        h = context(V, K, D, flags)
        assert set_whitening(h, V, D) == 0
        for n in (100, 50000):
            for _ in range(2):
                assert len(step(h, batch(n), D, K)) >= 2
            assert FAKE.fake_set_attribute() == 0, (D, K, flags)
        LIB.tlda_destroy(h)
    for d_in, hidden, k_out in ((50, 256, 50), (1024, 1024, 256)):
        m = ctypes.c_void_p()
        assert LIB.tlda_mlp_create(d_in, hidden, k_out, 5000, None, ctypes.byref(m)) == 0
        FAKE.fake_clear()
        X, T, theta = 1 << 20, 1 << 30, 1 << 40
        for n in (1, 5000):
            assert LIB.tlda_mlp_forward(m, X, 40 * n, theta) == 0
            assert LIB.tlda_mlp_train_step(m, X, T, n, 1e-3, None) == 0
        assert FAKE.fake_set_attribute() == 0, hidden
        LIB.tlda_mlp_destroy(m)


if __name__ == "__main__":
    globals()["check_" + sys.argv[2]]()
