"""Blocked Cholesky factor and triangular inverse at the edges of their 64-wide
blocks and doubling levels, through gap_fold_init (T = U) and
gap_predict_variance, against numpy in FP64: |d| <= 1e-10 of the largest value,
the bar of every FP64 comparison here (the matrices are well conditioned)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gapx():
    import paper_2310_03921_amd as g
    assert torch.cuda.is_available(), "GPU tests need a gfx950 device"
    return g


@pytest.fixture(scope="module")
def gap(gapx):
    return gapx.Gap(0)


def points(M, D=24):
    X = np.random.default_rng(M).standard_normal((M, D))
    return X / np.linalg.norm(X, axis=1)[:, None]


@pytest.mark.parametrize("M", [1, 15, 16, 17, 63, 64, 65, 128, 129, 333])
def test_cholesky_blocks(gapx, gap, M):
    Kmm = oracle.build_kmm(points(M), 2, 1.3)
    T = gap.fold_buffer(M, 0)
    gap.fold_init(T, M, torch.tensor(Kmm, device="cuda"), 1e-3)
    U = T[:M, :M].T.cpu().numpy()
    ref = np.linalg.cholesky(Kmm + 1e-3 * np.eye(M)).T
    assert np.abs(U - ref).max() <= 1e-10 * np.abs(ref).max()


@pytest.mark.parametrize("at", [0, 40, 64, 100, 200])
def test_cholesky_reports_a_bad_pivot(gapx, gap, at):
    """In the first column, inside a block, at a block's start and in the cut last block."""
    M = 201
    K = np.eye(M)
    K[at, at] = -0.5
    with pytest.raises(gapx.GapError) as e:
        gap.fold_init(gap.fold_buffer(M, 0), M, torch.tensor(K, device="cuda"), 0.0)
    assert e.value.status == gapx.GAP_E_NOT_PD


@pytest.mark.parametrize("M", [1, 31, 63, 64, 65, 127, 129, 192, 200, 449])
@pytest.mark.parametrize("N", [3, 70])
def test_variance_over_inverse_levels(gapx, gap, M, N):
    rng = np.random.default_rng([M, N])
    X, d = points(M), points(N + 1000)[:N]
    Kmm = oracle.build_kmm(X, 2, 1.0)
    B = rng.standard_normal((2 * M, M))
    R = np.linalg.cholesky(Kmm + 1e-3 * np.eye(M) + B.T @ B).T
    ref = oracle.predict_variance(d, X, Kmm, 1e-3, R, 2, 1.0)
    ld = M + 3  # entries below the diagonal and past M are never read
    buf = np.full((M, ld), np.nan)
    buf[:, :M] = np.where(np.tri(M, dtype=bool), R.T, np.nan)
    atoms = gapx.Atoms.from_host(np.array([0, N]), d, np.zeros(N + 1, np.int64),
                                 np.zeros(0, np.int32), None)
    var = gap.predict_variance(atoms, gapx.Sparse.from_host(X, 2, 1.0),
                               torch.tensor(Kmm, device="cuda"), 1e-3,
                               torch.tensor(buf, device="cuda"))
    assert np.abs(var.cpu().numpy() - ref).max() <= 1e-10


def inverse_rows(U):
    """U^-1 of an upper triangle by substitution, in U's own precision."""
    n = len(U)
    Y = np.eye(n, dtype=U.dtype)
    for c in range(n):
        Y[:, c] /= U[c, c]
        Y[:, c + 1:] -= np.outer(Y[:, c], U[c, c + 1:])
    return Y


@pytest.mark.parametrize("M", [16, 64, 200])
@pytest.mark.parametrize("eps", [1e-4, 1e-8, 1e-12])
def test_variance_with_an_ill_conditioned_factor(gapx, gap, M, eps):
    """R of columns equal up to eps, inside a 16-column block and across blocks (block
    conditions up to 1e13): against extended precision, within what a substitution may
    be off, |dY| <= M u |Y||R||Y| entry by entry, carried through |k Y|^2."""
    rng = np.random.default_rng([M, 7])
    X, d = points(M), points(40 + 1000)[:40]
    Kmm = oracle.build_kmm(X, 2, 1.0)
    B = rng.standard_normal((2 * M, M))
    for a, b in ((1, 0), (9, 4), (M - 1, 2)):
        B[:, a] = B[:, b] + eps * rng.standard_normal(2 * M)
    R = np.linalg.qr(B)[1]
    Y = inverse_rows(R.astype(np.longdouble))
    U = np.linalg.cholesky(Kmm + 1e-3 * np.eye(M)).T.astype(np.longdouble)
    k = (np.longdouble(1) * d @ X.T) ** 2
    z = k @ Y
    kii = (d * d).sum(1) ** 2
    ref = kii - ((k @ inverse_rows(U)) ** 2).sum(1) + (z ** 2).sum(1)
    u = 2.0 ** -53
    dz = M * u * (np.abs(k) @ np.abs(Y) @ np.abs(R) @ np.abs(Y))
    bound = (2 * np.abs(z) * dz + dz ** 2).sum(1) + M * u * (z ** 2).sum(1) + 1e-10
    atoms = gapx.Atoms.from_host(np.array([0, 40]), d, np.zeros(41, np.int64),
                                 np.zeros(0, np.int32), None)
    var = gap.predict_variance(atoms, gapx.Sparse.from_host(X, 2, 1.0),
                               torch.tensor(Kmm, device="cuda"), 1e-3,
                               torch.tensor(np.ascontiguousarray(R.T), device="cuda"))
    assert (np.abs(var.cpu().numpy() - ref) <= bound).all()
