"""Pair transposition at the edges of its forms: the one-block form (up to 1,024
targets and 12,288 pairs) and the general one, segments around the lengths where
the segment sort changes, and the target order of the force rows over several
blocks of targets.  The view is bit-exact against the oracle's."""
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


def pair_list(n_atoms, n_pairs, heavy=()):
    """Random sources and targets; `heavy`: in-degrees forced on targets 0, 1, ..."""
    rng = np.random.default_rng([n_atoms, n_pairs])
    lo = min(len(heavy), n_atoms - 1)
    j = rng.integers(lo, n_atoms, size=n_pairs).astype(np.int32)
    j[:sum(heavy)] = np.repeat(np.arange(len(heavy)), heavy)
    j = rng.permutation(j)
    cut = np.sort(rng.integers(0, n_pairs + 1, size=n_atoms - 1))
    return np.concatenate([[0], cut, [n_pairs]]).astype(np.int64), j


def atoms_of(gapx, pair_ptr, pair_j):
    n = len(pair_ptr) - 1
    return gapx.Atoms.from_host(np.array([0, n]), np.zeros((n, 4)), pair_ptr, pair_j, None)


@pytest.mark.parametrize("n_atoms,n_pairs,heavy", [
    (1, 1, ()), (64, 1900, (64, 65, 1)), (1024, 12288, (63, 64, 65, 129)), (1024, 12289, ()),
    (1025, 5000, (64, 65)), (4096, 9000, (2048, 2049, 0, 3000)), (9001, 30011, (1023, 1024, 1025))])
def test_pair_transpose_edges(gapx, gap, n_atoms, n_pairs, heavy):
    print(f"n_atoms {n_atoms} n_pairs {n_pairs}", flush=True)
    pair_ptr, pair_j = pair_list(n_atoms, n_pairs, heavy)
    tptr, tpair = gap.pair_transpose(atoms_of(gapx, pair_ptr, pair_j))
    rptr, rpair = oracle.pair_transpose(pair_ptr, pair_j, n_atoms)
    assert np.array_equal(tptr.cpu().numpy(), rptr)
    assert np.array_equal(tpair.cpu().numpy(), rpair)


@pytest.mark.parametrize("n_atoms,n_pairs", [(50, 700), (1500, 700)])
def test_dropped_pairs(gapx, gap, n_atoms, n_pairs):
    """Targets out of range are left out, reported, and their slots hold pair 0."""
    pair_ptr, pair_j = pair_list(n_atoms, n_pairs)
    pair_j[[3, 40, 699]] = [-1, n_atoms, n_atoms + 7]
    tptr, tpair = gap.pair_transpose(atoms_of(gapx, pair_ptr, pair_j))
    with pytest.raises(gapx.GapError):
        gap.sync()
    ok = np.flatnonzero((pair_j >= 0) & (pair_j < n_atoms))
    ref = ok[np.argsort(pair_j[ok], kind="stable")]
    assert np.array_equal(tpair.cpu().numpy(), np.concatenate([ref, [0, 0, 0]]))
    assert int(tptr[-1]) == len(ok)


@pytest.mark.parametrize("n_atoms", [1000, 1024, 2100])
def test_force_rows_over_blocks_of_targets(gapx, gap, n_atoms):
    """Every target gets its row: the order by in-degree is a permutation."""
    rng = np.random.default_rng(n_atoms)
    D, M, P = 8, 5, 4 * n_atoms
    pair_ptr, pair_j = pair_list(n_atoms, P, (90, 33))
    desc, jac = rng.standard_normal((n_atoms, D)), rng.standard_normal((P, 3, D))
    X = rng.standard_normal((M, D))
    cfg = np.array([0, n_atoms])
    K = gap.build_knm(gapx.Atoms.from_host(cfg, desc, pair_ptr, pair_j, jac),
                      gapx.Sparse.from_host(X, 2, 1.0))
    ref = oracle.build_knm(cfg, desc, pair_ptr, pair_j, jac, X, 2, 1.0)
    got = K[:M, :len(ref)].T.cpu().numpy()
    assert np.abs(got - ref).max() <= 1e-10 * np.abs(ref).max()


@pytest.mark.parametrize("n_atoms,n_pairs,heavy", [
    (2, 12288, (6144,)), (1, 12288, ()), (40, 12288, (220, 221, 222, 223)), (3, 300, (64, 65, 66)),
    (3000, 50000, (446, 447, 448, 449, 64, 65)), (1100, 40961, (3000, 400, 404, 405)),
    (1500, 1048577, (2047, 2048, 2049, 300000))])
def test_segment_order_where_its_two_forms_meet(gapx, gap, n_atoms, n_pairs, heavy):
    """Segments of n pairs around n^2 = 4 n_pairs, in the one-block form and the general
    one, and lists that are no multiple of the 256 pairs of a step."""
    print(f"n_atoms {n_atoms} n_pairs {n_pairs}", flush=True)
    pair_ptr, pair_j = pair_list(n_atoms, n_pairs, heavy)
    tptr, tpair = gap.pair_transpose(atoms_of(gapx, pair_ptr, pair_j))
    order = np.argsort(pair_j, kind="stable")
    assert np.array_equal(tptr.cpu().numpy(), np.searchsorted(pair_j[order], np.arange(n_atoms + 1)))
    assert np.array_equal(tpair.cpu().numpy(), order)


@pytest.mark.parametrize("n_atoms", [150, 1300])
def test_every_short_segment(gapx, gap, n_atoms):
    """Segments of 0 to 140 pairs, in the one-block form and the general one."""
    pair_ptr, pair_j = pair_list(n_atoms, 12288, tuple(range(141)))
    tptr, tpair = gap.pair_transpose(atoms_of(gapx, pair_ptr, pair_j))
    order = np.argsort(pair_j, kind="stable")
    assert np.array_equal(tptr.cpu().numpy(), np.searchsorted(pair_j[order], np.arange(n_atoms + 1)))
    assert np.array_equal(tpair.cpu().numpy(), order)
