"""Predict and backward in FP64 at the edges of the small-call forms: row, column
and contraction remainders of the 32 x 32 tiles, contraction slices, descriptor
lengths off the 16-deep chunks, and sizes on both sides of the line to the
staged kernels, against the oracle (which sums in another order: |d| <= 1e-10 of
the largest value, as every FP64 comparison here)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-10


@pytest.fixture(scope="module")
def gapx():
    import paper_2310_03921_amd as g
    assert torch.cuda.is_available(), "GPU tests need a gfx950 device"
    return g


@pytest.fixture(scope="module")
def gap(gapx):
    return gapx.Gap(0)


def close(got, ref, what):
    err = np.abs(got.cpu().numpy() - ref).max() / np.abs(ref).max()
    assert err <= TOL, f"{what}: {err:.3e}"


# (atoms, sparse points, descriptor length): tiles of the staged kernels are 64 x 128
@pytest.mark.parametrize("N,M,D", [
    (1, 1, 1), (1, 129, 3), (31, 33, 15), (32, 32, 16), (33, 31, 17), (64, 2000, 252),
    (65, 1025, 63), (217, 1501, 333), (700, 160, 1030), (5021, 37, 5),
    (3072, 1024, 20), (3071, 900, 21),   # both sides of the staged P-stage's smallest call
    (14336, 33, 7), (14272, 40, 9),      # and of the staged W X's
    (300, 2048, 1024),                   # the staged W^T D's smallest call
    (64, 65600, 6)])                     # many sparse points
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_predict_and_backward(gapx, gap, N, M, D, dt):
    print(f"N {N} M {M} D {D} {dt}", flush=True)
    rng = np.random.default_rng([N, M, D])
    desc = rng.standard_normal((N, D)) / np.sqrt(D)
    if dt == "f32":
        desc = desc.astype(np.float32)
    X, c = rng.standard_normal((M, D)) / np.sqrt(D), rng.standard_normal(M)
    nb = 3 if N > 1 else 0
    pair_ptr = np.arange(N + 1, dtype=np.int64) * nb
    pair_j = rng.integers(0, N, size=N * nb).astype(np.int32)
    jac = rng.standard_normal((N * nb, 3, D)).astype(desc.dtype)
    cfg = np.array([0, N // 3, N], dtype=np.int64)
    zeta, delta = 3, 1.2
    atoms = gapx.Atoms.from_host(cfg, desc, pair_ptr, pair_j, jac)
    if D % 4:  # row padding is never read: it may hold anything
        atoms.desc[:, D:] = float("nan")
        atoms.jac[:, :, D:] = float("nan")
    sp = gapx.Sparse.from_host(X, zeta, delta)
    if D % 4:
        sp.X[:, D:] = float("nan")
    out = gap.predict(atoms, sp, torch.tensor(c, device="cuda"), dEdd=True, forces=nb > 0)
    P = desc.astype(np.float64) @ X.T
    e_ref = oracle.poly_kernel(P, zeta, delta) @ c
    g_ref = (oracle.poly_kernel_grad_scale(P, zeta, delta) * c) @ X
    close(out["e_atom"], e_ref, "e_atom")
    close(out["dEdd"], g_ref, "dEdd")
    if nb:
        F = np.zeros((N, 3))
        np.add.at(F, pair_j, -np.einsum("pad,pd->pa", jac.astype(np.float64),
                                        np.repeat(g_ref, nb, axis=0)))
        close(out["forces"], F, "forces")
    g_e = rng.standard_normal(N)
    refs = oracle.predict_backward(desc, X, c, g_e, zeta, delta)
    got = gap.predict_backward(atoms, sp, torch.tensor(c, device="cuda"),
                               torch.tensor(g_e, device="cuda"))
    for g, r, what in zip(got, refs, ("d_desc", "d_c", "d_X")):
        close(g, r, what)
