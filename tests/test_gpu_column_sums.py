"""Mass sums, the M inner product and the mass operator at the edges of their splits:
columns of fewer and more layers than the eight wavefronts of a cell and the four layers
of a block, and members of fewer and more columns than the sums take at a time."""

import numpy as np
import pytest

import oracle as O
import paper_2605_16082_amd as P
import workloads as W

pytestmark = pytest.mark.gpu

MESHES = [W.tiny(n=3, n_layers=d, n_fields=f) for d, f in [(1, 4), (3, 1), (4, 2), (5, 3), (7, 2), (8, 1), (9, 4), (17, 2)]]
MESHES += [W.ragged(n=9, n_fields=3, n_min=1, n_max=40, dz=2.0, depth_max=80.0), W.small_ensemble(n_fields=4),
           W.rotating_blob(n=48, n_layers=3)]
IDS = [f"{w.name}-{w.n_cols}x{int(w.nlayers.max())}-{w.n_fields}" for w in MESHES]


# double: sums of at most 1e5 products, each rounded within a few 2^-53 of the sum of
# magnitudes; float state: the double sums of the stored (rounded) values
@pytest.mark.parametrize("precision", [P.SDG_FP64, P.SDG_FP32])
@pytest.mark.parametrize("w", MESHES, ids=IDS)
def test_sums_match_oracle(w, precision):
    s, _, _, state = P.from_workload(w, precision)
    T = s.gather(state)
    m = O.PrismMesh(w.vxy, w.tri, w.nbr, w.nlayers, w.zlev)
    Mp = O.mass_matrix(m)
    MT = np.einsum("nij,fjn->fin", Mp, T)
    absM = np.einsum("nij,fjn->fin", np.abs(Mp), np.abs(T))
    mass, md = s.mass(state), s.m_dot(state, state)
    assert mass.shape == md.shape
    assert np.all(np.abs(mass.sum(axis=0) - MT.sum(axis=(1, 2))) <= 1e-13 * absM.sum(axis=(1, 2)))
    assert np.all(np.abs(md.sum(axis=0) - (MT * T).sum(axis=(1, 2))) <= 1e-13 * (absM * np.abs(T)).sum(axis=(1, 2)))
    assert np.array_equal(mass, s.mass(state)) and np.array_equal(md, s.m_dot(state, state))
    eps = 1e-13 if precision == P.SDG_FP64 else 1.2e-7
    assert np.all(np.abs(s.gather(s.apply_mass(state)) - MT) <= eps * absM.max())
