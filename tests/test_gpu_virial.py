"""Virial rows through the C ABI against the FP64 oracle:
|gpu - oracle| <= 1e-10 * max|oracle|."""
import numpy as np
import pytest
import torch

import oracle
import synth

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


def close(got, ref, tol, what):
    got, ref = np.asarray(got, np.float64), np.asarray(ref, np.float64)
    scale = max(np.abs(ref).max(), 1e-300)
    err = np.abs(got - ref).max()
    assert err <= tol * scale, f"{what}: rel err {err / scale:.3e}"


def ragged():
    # D and M off the tile sizes, 1-atom configurations, atoms with no pairs
    return synth.Workload("ragged", 29, n_cfg=9, atoms_lo=1, atoms_hi=23, D=37, nb=3, M=23,
                          zeta=3, delta=1.7)


@pytest.mark.parametrize("wname,jdt", [("fit_small", None), ("fit_small", "f32"),
                                       ("ragged", None)])
def test_virial_rows_vs_oracle(gapx, gap, wname, jdt):
    w = ragged() if wname == "ragged" else synth.WORKLOADS[wname]
    b = synth.generate(w)
    X = synth.sparse_points(w, b)
    r = synth.pair_vectors(w, b)
    jac = b.jac.astype(np.float32) if jdt == "f32" else b.jac
    atoms = gapx.Atoms.from_host(b.cfg_ptr, b.desc, b.pair_ptr, b.pair_j, jac,
                                 jac_dtype=torch.float32 if jdt == "f32" else None)
    sp = gapx.Sparse.from_host(X, w.zeta, w.delta)
    Kv = gap.build_virial_rows(atoms, sp, torch.tensor(r, device="cuda"))
    gap.sync()
    ref = oracle.build_virial_rows(b.cfg_ptr, b.desc, b.pair_ptr, jac, r, X, w.zeta, w.delta)
    close(Kv[:w.M, :9 * b.n_cfg].T.cpu().numpy(), ref, TOL, "virial rows")


def test_fit_with_virial_rows(gapx, gap):
    # energies, forces and virials of every configuration in one design buffer
    w = synth.WORKLOADS["fit_small"]
    b = synth.generate(w)
    X = synth.sparse_points(w, b)
    r = synth.pair_vectors(w, b)
    M = w.M
    K = oracle.build_knm(b.cfg_ptr, b.desc, b.pair_ptr, b.pair_j, b.jac, X, w.zeta, w.delta)
    KV = oracle.build_virial_rows(b.cfg_ptr, b.desc, b.pair_ptr, b.jac, r, X, w.zeta, w.delta)
    Kall = np.vstack([K, KV])
    rng = np.random.default_rng(6)
    y = Kall @ synth.hidden_coefficients(w) + 1e-3 * rng.standard_normal(Kall.shape[0])
    sig = np.concatenate([synth.sigma_rows(w, b.counts), np.full(KV.shape[0], 0.05)])
    c_ref = oracle.fit(Kall, oracle.build_kmm(X, w.zeta, w.delta), y, sig, w.jitter)

    atoms = gapx.Atoms.from_host(b.cfg_ptr, b.desc, b.pair_ptr, b.pair_j, b.jac)
    sp = gapx.Sparse.from_host(X, w.zeta, w.delta)
    n = Kall.shape[0]
    A = gapx.colmajor(n + M, M + 1)
    gap.build_knm(atoms, sp, out=A)
    gap.build_virial_rows(atoms, sp, torch.tensor(r, device="cuda"), out=A, row0=b.n_rows)
    c, _ = gap.fit(A, n, gap.build_kmm(sp), torch.tensor(y, device="cuda"),
                   torch.tensor(sig, device="cuda"), w.jitter, sp)
    close(c.cpu().numpy(), c_ref, TOL, "c")


@pytest.mark.parametrize("D", [1, 33, 150, 255, 256])
def test_rows_at_descriptor_edges(gapx, gap, D):
    """Virial and force rows of the LDS-resident kernels at descriptor lengths off
    their 4-, 16- and 32-entry steps, with row padding that is never read, and a
    target of a degree far above the others."""
    w = synth.Workload("edge", 77, n_cfg=5, atoms_lo=1, atoms_hi=40, D=D, nb=6, M=70)
    b = synth.generate(w)
    X = synth.sparse_points(w, b)
    pair_j = b.pair_j.copy()
    first = b.pair_ptr[b.cfg_ptr[3]], b.pair_ptr[b.cfg_ptr[4]]
    pair_j[first[0]:first[1]:2] = b.cfg_ptr[3]
    r = synth.pair_vectors(w, b)
    atoms = gapx.Atoms.from_host(b.cfg_ptr, b.desc, b.pair_ptr, pair_j, b.jac)
    sp = gapx.Sparse.from_host(X, w.zeta, w.delta)
    if D % 4:
        atoms.jac[:, :, D:] = float("nan")
    Kv = gap.build_virial_rows(atoms, sp, torch.tensor(r, device="cuda"))
    ref = oracle.build_virial_rows(b.cfg_ptr, b.desc, b.pair_ptr, b.jac, r, X, w.zeta, w.delta)
    got = Kv[:, :9 * b.n_cfg].T.cpu().numpy()
    assert np.abs(got - ref).max() <= 1e-10 * np.abs(ref).max()
    K = gap.build_knm(atoms, sp)[:w.M, :b.n_rows].T.cpu().numpy()
    kref = oracle.build_knm(b.cfg_ptr, b.desc, b.pair_ptr, pair_j, b.jac, X, w.zeta, w.delta)
    assert np.abs(K - kref).max() <= 1e-10 * np.abs(kref).max()


@pytest.mark.parametrize("n_cfg,per,M", [(1, 63, 40), (1, 64, 40), (1, 128, 70), (3, 129, 300),
                                         (40, 65, 300), (40, 260, 300), (2, 1000, 9)])
def test_rows_over_slices_of_pairs(gapx, gap, n_cfg, per, M):
    """Configurations of `per` pairs on average, around the one or two steps of 64 that a
    slice takes at least, their pairs cut at random."""
    rng = np.random.default_rng([n_cfg, per, M])
    N, D, P = 4 * n_cfg, 21, n_cfg * per
    cut = np.sort(rng.integers(0, P + 1, size=N - 1))
    pair_ptr = np.concatenate([[0], cut, [P]]).astype(np.int64)
    cfg = np.arange(0, N + 1, 4)
    desc, X = rng.standard_normal((N, D)), rng.standard_normal((M, D))
    jac, r = rng.standard_normal((P, 3, D)), rng.standard_normal((P, 3))
    atoms = gapx.Atoms.from_host(cfg, desc, pair_ptr, rng.integers(0, N, P).astype(np.int32), jac)
    K = gap.build_virial_rows(atoms, gapx.Sparse.from_host(X, 2, 1.0), torch.tensor(r, device="cuda"))
    ref = oracle.build_virial_rows(cfg, desc, pair_ptr, jac, r, X, 2, 1.0)
    assert np.abs(K[:M, :9 * n_cfg].T.cpu().numpy() - ref).max() <= 1e-10 * np.abs(ref).max()
