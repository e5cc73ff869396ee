"""Householder QR panels at their edges, through gap_lstsq: widths and heights
around the 64- and 128-wide blocks, square matrices, and panels whose columns
are numerically dependent (factored column by column).

Bounds: a backward-stable QR has |R^T R - A^T A| <= c(m, n) u |A|_F^2 with c a
low-degree polynomial, here taken as 1e-12 / u = 4500 for n <= 300; solutions of
well-conditioned systems agree to 1e-10 as everywhere in these tests."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gapx():
    import paper_2310_03921_amd as g
    assert torch.cuda.is_available(), "GPU tests need a gfx950 device"
    return g


@pytest.fixture(scope="module")
def gap(gapx):
    return gapx.Gap(0)


def device_matrix(gapx, K, y):
    m, n = K.shape
    A = gapx.colmajor(m, n + 1)
    A[:n, :m] = torch.tensor(K.T)
    A[n, :m] = torch.tensor(y)
    return A


def factor_error(A, K):
    n = K.shape[1]
    R = np.triu(A[:n, :n].T.cpu().numpy())
    return np.linalg.norm(R.T @ R - K.T @ K) / np.linalg.norm(K) ** 2


@pytest.mark.parametrize("m,n", [
    (1, 1), (5, 1), (17, 16), (63, 63), (64, 64), (65, 64), (100, 65), (128, 128), (129, 127),
    (400, 129), (1000, 200), (2049, 256), (4100, 63), (30000, 70), (5003, 300)])
def test_lstsq_shapes(gapx, gap, m, n):
    print(f"m {m} n {n}", flush=True)
    rng = np.random.default_rng([m, n])
    # column scales over twelve decades: the factorisation is invariant to them
    scale = 10.0 ** rng.uniform(-6, 6, n)
    K = rng.standard_normal((m, n)) + (np.eye(m, n) * 3 if m < 2 * n else 0)
    y = rng.standard_normal(m)
    A = device_matrix(gapx, K * scale, y)
    x, _ = gap.lstsq(A, m, n)
    ref = np.linalg.lstsq(K, y, rcond=None)[0]
    got = x.cpu().numpy() * scale
    assert np.linalg.norm(got - ref) <= 1e-10 * np.linalg.norm(ref) * np.linalg.cond(K)
    assert factor_error(A, K * scale) <= 1e-12


@pytest.mark.parametrize("m,n", [(300, 64), (700, 100), (5000, 200)])
@pytest.mark.parametrize("eps", [1e-4, 1e-7, 1e-9, 0.0])
def test_dependent_columns_in_a_panel(gapx, gap, m, n, eps):
    """Columns equal up to eps, in the first and in the last panel: the factor stays
    backward stable, and the rest of the matrix is not disturbed."""
    print(f"m {m} n {n} eps {eps}", flush=True)
    rng = np.random.default_rng([m, n])
    K = rng.standard_normal((m, n))
    for a, b in ((3, 40), (n - 1, n - 9)):
        K[:, a] = K[:, b] + eps * rng.standard_normal(m)
    y = rng.standard_normal(m)
    A = device_matrix(gapx, K, y)
    try:
        x, _ = gap.lstsq(A, m, n)
    except gapx.GapError as e:  # an exactly zero pivot is allowed for equal columns only
        assert eps == 0.0 and e.status == gapx.GAP_E_RANK
    assert factor_error(A, K) <= 1e-12
    if eps >= 1e-7:
        r = y - K @ x.cpu().numpy()
        xn = np.linalg.norm(K) * np.linalg.norm(x.cpu().numpy()) + np.linalg.norm(y)
        assert np.linalg.norm(K.T @ r) <= 1e-12 * np.linalg.norm(K) * xn


def test_zero_column_is_reported(gapx, gap):
    rng = np.random.default_rng(5)
    K = rng.standard_normal((500, 90))
    K[:, 70] = 0.0
    with pytest.raises(gapx.GapError) as e:
        gap.lstsq(device_matrix(gapx, K, rng.standard_normal(500)), 500, 90)
    assert e.value.status == gapx.GAP_E_RANK


@pytest.mark.parametrize("m,n", [(12700, 300), (33000, 193), (40001, 256)])
def test_trailing_update_runs_over_row_blocks(gapx, gap, m, n):
    """More 128 x 64 tiles of the trailing columns than compute units: a block's run
    of tiles starts and ends inside row blocks."""
    print(f"m {m} n {n}", flush=True)
    rng = np.random.default_rng([m, n])
    K = rng.standard_normal((m, n))
    y = rng.standard_normal(m)
    A = device_matrix(gapx, K, y)
    x, _ = gap.lstsq(A, m, n)
    ref = np.linalg.lstsq(K, y, rcond=None)[0]
    assert np.linalg.norm(x.cpu().numpy() - ref) <= 1e-10 * np.linalg.norm(ref) * np.linalg.cond(K)
    assert factor_error(A, K) <= 1e-12


def column_error(A, K):
    """max |R^T R - K^T K|_ij / (|k_i| |k_j|): the bound column by column, which Householder
    QR meets whatever the scales of the columns are."""
    n = K.shape[1]
    R = np.triu(A[:n, :n].T.cpu().numpy())
    norms = np.linalg.norm(K, axis=0)
    norms[norms == 0] = 1.0
    return np.abs((R / norms).T @ (R / norms) - (K / norms).T @ (K / norms)).max()


def solve_dependent(gapx, gap, K, y, rank_ok):
    A = device_matrix(gapx, K, y)
    try:
        x, _ = gap.lstsq(A, *K.shape)
    except gapx.GapError as e:
        assert rank_ok and e.status == gapx.GAP_E_RANK
        x = None
    return A, x


@pytest.mark.parametrize("m,n,pairs", [
    (128, 128, ((70, 100),)), (130, 66, ((65, 64),)), (5000, 128, ((70, 100),)),
    (5000, 300, ((70, 100),)), (5000, 300, ((198, 228),)), (5003, 256, ((70, 100), (198, 228))),
    (33001, 193, ((127, 64), (192, 150))), (700, 300, ((3, 40), (64 + 128, 65 + 128)))])
@pytest.mark.parametrize("eps", [1e-9, 1e-13, 0.0])
def test_second_panel_alone_is_dependent(gapx, gap, m, n, pairs, eps):
    """The second 64 columns of a 128-wide block fail alone, in the first and in a later
    block, with trailing columns behind them and without, and over twelve decades of
    column scales."""
    print(f"m {m} n {n} pairs {pairs} eps {eps}", flush=True)
    rng = np.random.default_rng([m, n])
    K = rng.standard_normal((m, n)) + (np.eye(m, n) * 3 if m < 2 * n else 0)
    for a, b in pairs:
        K[:, a] = K[:, b] + eps * rng.standard_normal(m)
    K *= 10.0 ** rng.uniform(-6, 6, n)
    y = rng.standard_normal(m)
    A, x = solve_dependent(gapx, gap, K, y, eps == 0.0)
    assert column_error(A, K) <= 1e-12
    if x is not None:
        # x minimises a problem whose columns are changed by rounding: K^T r column by column
        x = x.cpu().numpy()
        size = np.linalg.norm(K, axis=0)
        r = y - K @ x
        assert (np.abs(K.T @ r) / size).max() <= 1e-12 * ((size * np.abs(x)).sum()
                                                           + np.linalg.norm(y))


@pytest.mark.parametrize("m,n,zero,same", [
    (500, 90, (70,), ()), (500, 90, (3,), ()), (5000, 300, (70,), (3, 40)),
    (33001, 140, (100,), (3, 40)), (100, 100, (99,), (0, 1)), (5000, 200, (), range(0, 200)),
    (5000, 130, (129,), (64, 127))])
def test_columns_that_no_round_can_tell_apart(gapx, gap, m, n, zero, same):
    """Zero columns, alone and behind a panel of equal columns, and a matrix of one column
    repeated, all ones (no rounding error tells them apart): R still reproduces K^T K."""
    print(f"m {m} n {n} zero {zero} same {same}", flush=True)
    rng = np.random.default_rng([m, n])
    K = rng.standard_normal((m, n)) + (np.eye(m, n) * 3 if m < 2 * n else 0)
    if len(same) == n:
        K[:] = 1.0
    for a in same:
        K[:, a] = K[:, same[0]]
    for a in zero:
        K[:, a] = 0.0
    A, x = solve_dependent(gapx, gap, K, rng.standard_normal(m), True)
    assert x is None or not zero
    assert column_error(A, K) <= 1e-12


@pytest.mark.parametrize("m,n", [(2, 2), (16, 16), (60, 9), (2048, 16), (2049, 15), (5000, 17),
                                 (4100, 144), (4100, 145), (300, 133), (524288, 3), (524289, 3)])
@pytest.mark.parametrize("same", [False, True])
def test_narrow_last_block(gapx, gap, m, n, same):
    """A last block of up to sixteen columns has its own panel while its rows fit the
    device's registers; with equal columns among the last sixteen as well."""
    print(f"m {m} n {n} same {same}", flush=True)
    rng = np.random.default_rng([m, n])
    K = rng.standard_normal((m, n)) + (np.eye(m, n) * 3 if m < 2 * n else 0)
    if same:
        K[:, n - 1] = K[:, n - 2]
    K *= 10.0 ** rng.uniform(-6, 6, n)
    y = rng.standard_normal(m)
    A, x = solve_dependent(gapx, gap, K, y, same)
    assert column_error(A, K) <= 1e-12
    if x is not None:
        x = x.cpu().numpy()
        size = np.linalg.norm(K, axis=0)
        assert (np.abs(K.T @ (y - K @ x)) / size).max() <= 1e-12 * (
            (size * np.abs(x)).sum() + np.linalg.norm(y))
