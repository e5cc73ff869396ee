"""A pair whose Jacobian is not finite reaches its own target's force rows and its own
configuration's virial rows, and no others: not the atoms without incoming pairs and
not those of lower in-degree beside it, whose lanes read some pair's rows as well.
Everything else agrees with the sums pair by pair to 1e-10 of the largest finite
entry, the bar of every FP64 comparison here."""
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


def batch(N, D, M, bad):
    """Four pairs an atom; atoms 0, 5 and N - 1 have no incoming pairs.  The one pair of
    target 6, the last of its source's configuration, has `bad` in one component."""
    rng = np.random.default_rng([N, D, M])
    desc, X = rng.standard_normal((N, D)), rng.standard_normal((M, D))
    jac, r = rng.standard_normal((4 * N, 3, D)), rng.standard_normal((4 * N, 3))
    j = rng.choice(np.setdiff1d(np.arange(N), [0, 5, N - 1]), size=4 * N).astype(np.int32)
    p = 4 * (N // 2) - 1          # the last pair of the first configuration
    j[j == 6] = 9
    j[p] = 6
    jac[p, 1, D // 2 - 1] = bad
    return desc, X, jac, r, j, p


def rows(desc, X, jac, r, j, N, M):
    """Force rows [3 N] and the virial rows of the configurations [0, N/2), [N/2, N), zeta 2."""
    src = np.arange(4 * N) // 4
    cfg = (src >= N // 2).astype(int)
    F, V = np.zeros((N, 3, M)), np.zeros((2, 3, 3, M))
    with np.errstate(invalid="ignore"):
        t = (2.0 * (desc @ X.T))[src][:, None, :] * (jac @ X.T)
        np.subtract.at(F, j, t)
        np.subtract.at(V, cfg, r[:, :, None, None] * t[:, None, :, :])
    return F.reshape(3 * N, M), V.reshape(18, M)


def same(got, ref):
    ok = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), ok)
    assert np.abs(got[ok] - ref[ok]).max() <= 1e-10 * np.abs(ref[ok]).max()
    nan = np.isnan(ref)
    assert np.array_equal(np.isnan(got), nan)
    assert np.array_equal(got[~ok & ~nan], ref[~ok & ~nan])


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("N,D,M", [(40, 6, 5), (40, 250, 70), (40, 252, 5), (300, 37, 66),
                                   (4000, 6, 1600), (4000, 8, 1600)])
def test_bad_jacobian_stays_with_its_target(gapx, gap, N, D, M, bad):
    print(f"N {N} D {D} M {M} {bad}", flush=True)
    desc, X, jac, r, j, p = batch(N, D, M, bad)
    cfg = np.array([0, N // 2, N])
    atoms = gapx.Atoms.from_host(cfg, desc, 4 * np.arange(N + 1, dtype=np.int64), j, jac)
    sp = gapx.Sparse.from_host(X, 2, 1.0)
    F, V = rows(desc, X, jac, r, j, N, M)
    got = gap.build_knm(atoms, sp)[:M, 2:2 + 3 * N].T.cpu().numpy()
    same(got, F)
    got = gap.build_virial_rows(atoms, sp, torch.tensor(r, device="cuda"))[:M, :18].T.cpu().numpy()
    same(got, V)
