"""GPU parity of the blocked Cholesky factorization (panel step: the
triangular solve of Alg. It-Inv-TRSM with whole inverted diagonal blocks)
through the C ABI against the CPU oracle's column-by-column definition, on the
same seeded inputs.  Tolerance: 1e-12 relative Frobenius error for L and for
the inverted diagonal blocks on the well-conditioned family
A = G G^T / 2n + I (cond(A) < 4, so L's forward error is a few units of
rounding); the ill-conditioned family is checked by its backward error."""
import numpy as np
import pytest

import oracle
from paper_1612_01855_amd import inputs as gen

pytestmark = pytest.mark.gpu

TOL64 = 1e-12
U = 2.0 ** -53


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    assert _t.cuda.is_available(), "GPU tests need a ROCm device"
    return _t


@pytest.fixture(scope="module")
def T():
    from paper_1612_01855_amd import trsm
    return trsm


def log(msg):
    print(msg, flush=True)


def gpu_factor(torch, T, A, nb=0, lda=None, upper=None):
    """Factor the host matrix A on the GPU (only its lower triangle is given:
    the strict upper triangle and any padding columns hold `upper`).  Returns
    (L as stored, the whole device buffer on the host, Linv blocks, the
    factorization object)."""
    n = A.shape[0]
    lda = n if lda is None else lda
    fill = np.nan if upper is None else upper
    Ah = np.full((n, lda), fill)
    Ah[:, :n] = np.where(np.tril(np.ones((n, n), dtype=bool)), A, fill)
    Ad = torch.from_numpy(Ah).cuda()
    c = T.Cholesky(n, nb, device="cuda")
    log(f"chol n={n} nb={c.nb} lda={lda}")
    c.factor(Ad[:, :n] if lda == n else Ad.as_strided((n, n), (lda, 1)))
    torch.cuda.synchronize()
    full = Ad.cpu().numpy()
    L = np.tril(full[:, :n])
    return L, full, c.linv_blocks().cpu().numpy(), c


@pytest.mark.parametrize("n,nb", [(1, 0), (63, 0), (64, 64), (65, 64), (200, 64), (300, 128),
                                  (1000, 128), (1100, 256), (1536, 512), (2048, 256)])
def test_factor_matches_oracle(torch, T, n, nb):
    A = gen.spd(n, n + 7)
    L, full, Vb, c = gpu_factor(torch, T, A, nb)
    assert c.check() == (T.OK, -1)
    Lref, f = oracle.chol(A)
    assert f == -1
    err = oracle.rel_fro_err(L, Lref)
    log(f"  rel err of L {err:.3e}")
    assert err <= TOL64
    # the strict upper triangle is never written
    assert np.all(np.isnan(full[np.triu_indices(n, 1)]))


@pytest.mark.parametrize("n,nb", [(300, 128), (1100, 256), (777, 64)])
def test_inverted_blocks_match_oracle(torch, T, n, nb):
    A = gen.spd(n, 3 * n)
    L, _, Vb, c = gpu_factor(torch, T, A, nb)
    Lref, _ = oracle.chol(A)
    nbu = c.nb
    for j, inv in enumerate(oracle.diag_block_inverses(Lref, nbu)):
        s = inv.shape[0]
        blk = Vb[j]
        err = oracle.rel_fro_err(blk[:s, :s], inv)
        assert err <= TOL64, (j, err)
        assert np.all(blk[np.triu_indices(nbu, 1)] == 0.0)
        if s < nbu:     # ragged last block: identity padding
            assert np.array_equal(blk[s:, s:], np.eye(nbu - s))
            assert np.all(blk[s:, :s] == 0.0)


def test_leaf_sizes_are_exact_on_integer_factors(torch, T):
    # n <= 64: one LDS leaf, no inverse on the factor's path; every
    # intermediate is an integer, so L comes back exactly
    L0 = gen.int_lower_positive(60, 4)
    Li = L0.astype(np.int64)
    A = (Li @ Li.T).astype(np.float64)
    L, _, _, c = gpu_factor(torch, T, A)
    assert c.check() == (T.OK, -1)
    assert np.array_equal(L, L0)


@pytest.mark.parametrize("n", [2, 15, 16, 17, 48, 49, 64, 65, 80, 81, 112, 113, 127, 128])
@pytest.mark.parametrize("scale", [1.0, 2.0 ** -920, 2.0 ** 920])
def test_leaf_tiles(torch, T, n, scale):
    # one block, factored and inverted in LDS in steps of 16 columns (up to 64 rows
    # by 4 waves, up to 128 by 16, the rows below a step in one wave or several):
    # edges of tiles and waves, and pivots outside the range of the fast roots
    # (scale a power of four: every operation scales exactly, so the bound is the same)
    A = gen.spd(n, 11 * n)
    L, full, Vb, c = gpu_factor(torch, T, A * scale, 0 if n <= 64 else 128, lda=n + 3)
    assert c.check() == (T.OK, -1)
    Lref, _ = oracle.chol(A)
    assert oracle.rel_fro_err(L / np.sqrt(scale), Lref) <= TOL64
    assert np.all(np.isnan(full[np.triu_indices(n, 1)])) and np.all(np.isnan(full[:, n:]))
    inv = oracle.diag_block_inverses(Lref, c.nb)[0]
    assert oracle.rel_fro_err(Vb[0][:n, :n] * np.sqrt(scale), inv) <= TOL64
    for bad in {0, n // 2, n - 1}:
        A2 = A.copy()
        A2[bad, bad] = -1.0
        _, _, _, c = gpu_factor(torch, T, A2 * scale, 0 if n <= 64 else 128)
        assert c.check() == (T.ESINGULAR, bad)


@pytest.mark.parametrize("n,nb,bad", [(50, 0, 17), (300, 64, 0), (300, 64, 200),
                                      (1000, 256, 999), (1000, 256, 512)])
def test_not_positive_definite_reports_the_row(torch, T, n, nb, bad):
    A = gen.spd(n, 5)
    A[bad, bad] = -1.0          # pivot bad is -1 - sum l^2 < 0; earlier pivots unchanged
    _, _, _, c = gpu_factor(torch, T, A, nb)
    assert c.check() == (T.ESINGULAR, bad)
    A[bad, bad] = np.nan
    _, _, _, c = gpu_factor(torch, T, A, nb)
    assert c.check() == (T.ESINGULAR, bad)


def test_padded_leading_dimension(torch, T):
    n, lda = 700, 733
    A = gen.spd(n, 2)
    L, full, _, c = gpu_factor(torch, T, A, 128, lda=lda, upper=7.0)
    assert c.check() == (T.OK, -1)
    assert oracle.rel_fro_err(L, oracle.chol(A)[0]) <= TOL64
    assert np.all(full[:, n:] == 7.0)
    assert np.all(full[np.triu_indices(n, 1)] == 7.0)


def test_factor_then_solve_with_its_blocks(torch, T):
    # the Linv blocks are a TRSM_F64 plan's (n0 = nb): solve A X = B as
    # L Y = B (forward) then L^T X = Y (the oracle's backward substitution)
    n, k, nb = 1100, 40, 256
    A = gen.spd(n, 9)
    B = gen.rhs(n, k, 9)
    Ad = torch.from_numpy(A.copy()).cuda()
    c = T.Cholesky(n, nb, device="cuda")
    c.factor(Ad)
    s = T.Solver.create(n, k, "f64", n0=nb)
    try:
        assert s.info.linv_bytes == c.linv_bytes
        Bd = torch.from_numpy(B).cuda()
        Yd = torch.empty_like(Bd)
        T.trsm_solve(s.plan, Ad.data_ptr(), n, c.linv_ptr, Bd.data_ptr(), k, Yd.data_ptr(), k,
                     s.workspace_ptr, torch.cuda.current_stream().cuda_stream, None)
        torch.cuda.synchronize()
    finally:
        s.close()
    L = np.tril(Ad.cpu().numpy())
    Y = Yd.cpu().numpy()
    assert oracle.rel_fro_err(Y, oracle.trsm(L, B)) <= TOL64
    X = oracle.trsm_t(L, Y)
    Xref = np.linalg.solve(A, B)
    assert oracle.rel_fro_err(X, Xref) <= TOL64


def test_graph_capture_replays(torch, T):
    # no allocation and no memset inside: the whole factorization can be
    # captured and replayed; every replay must equal the eager result
    n, nb = 900, 128
    A = gen.spd(n, 21)
    A0 = torch.from_numpy(A).cuda()
    Ad = A0.clone()
    c = T.Cholesky(n, nb, device="cuda")
    c.factor(Ad)
    torch.cuda.synchronize()
    eager = Ad.clone()
    s = torch.cuda.Stream()
    Ag = A0.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            T.trsm_chol_factor(n, Ag.data_ptr(), n, nb, c.linv_ptr, c.workspace_ptr,
                               s.cuda_stream)
    for _ in range(3):
        Ag.copy_(A0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(torch.tril(Ag), torch.tril(eager))
        assert c.check() == (T.OK, -1)


def test_ill_conditioned_backward_error(torch, T):
    n = 1024
    Ad = gen.spd_on(torch, "cuda", n, 13, ratio=1e-12)
    A = Ad.cpu().numpy()
    A = np.tril(A) + np.tril(A, -1).T
    L, _, _, c = gpu_factor(torch, T, A, 256)
    assert c.check() == (T.OK, -1)
    R = A - L @ L.T
    be = np.linalg.norm(R) / np.linalg.norm(A)
    log(f"  hard n={n} backward error {be:.3e}")
    assert be <= 4 * n * U
    Lref, _ = oracle.chol(A)
    log(f"  rel diff vs oracle {oracle.rel_fro_err(L, Lref):.3e}")


def test_empty(torch, T):
    c = T.Cholesky(0, 0, device="cuda")
    Ad = torch.zeros((1, 1), dtype=torch.float64, device="cuda")
    T.trsm_chol_factor(0, Ad.data_ptr(), 1, 0, c.linv_ptr, c.workspace_ptr, 0)
    assert c.check() == (T.OK, -1)


def test_concurrent_factorizations_on_two_streams(torch, T):
    # two host threads, each with its own stream and buffers, share the
    # library's side stream: both results must equal their lone results
    import threading
    n, nb = 1100, 128
    mats = [gen.spd(n, 40 + t) for t in range(2)]
    lone = []
    for A in mats:
        L, _, _, c = gpu_factor(torch, T, A, nb)
        assert c.check() == (T.OK, -1)
        lone.append(L)
    out = [None, None]
    errors = []

    def work(t):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                Ad = torch.from_numpy(mats[t]).cuda()
                c = T.Cholesky(n, nb, device="cuda")
                for _ in range(3):
                    Ad.copy_(torch.from_numpy(mats[t]))
                    T.trsm_chol_factor(n, Ad.data_ptr(), n, nb, c.linv_ptr, c.workspace_ptr,
                                       s.cuda_stream)
                s.synchronize()
                assert c.check() == (T.OK, -1)
                out[t] = np.tril(Ad.cpu().numpy())
        except Exception as e:   # reported below
            errors.append(e)

    th = [threading.Thread(target=work, args=(t,)) for t in range(2)]
    for x in th:
        x.start()
    for x in th:
        x.join()
    assert not errors, errors
    for t in range(2):
        assert np.array_equal(out[t], lone[t])
