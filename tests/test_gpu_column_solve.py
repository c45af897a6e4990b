"""The layer-parallel column solve at the edges of its blocks: column groups of
64 down to 4 columns (256 / depth), columns of one layer, ragged groups, the
deepest mesh it takes (64 layers) and the first that the serial sweeps take."""

import numpy as np
import pytest

import oracle as O
import paper_2605_16082_amd as P
import workloads as W

pytestmark = pytest.mark.gpu


def _sigma(n, layers, fields):
    w = W.tiny(n=n, n_layers=layers, n_fields=fields)
    # a stiff diffusion in the upper layers, so that the layers couple
    w.kappa = np.geomspace(1.0, 1e-4, layers) if layers > 1 else np.array([1.0])
    return w


MESHES = [_sigma(3, d, f) for d, f in [(1, 2), (4, 1), (5, 4), (8, 3), (16, 2), (17, 4), (32, 4), (33, 1), (64, 3),
                                       (65, 2)]]
MESHES += [_sigma(6, 20, 4), W.ragged(), W.ragged(n=9, n_fields=4, n_min=1, n_max=40, dz=2.0, depth_max=80.0),
           W.small_ensemble(n_fields=3)]
IDS = [f"{w.name}-{w.n_cols}x{int(w.nlayers.max())}-{w.n_fields}" for w in MESHES]


# double: the bar of every other double result; float state: twice the output's own
# rounding (2^-24).  The all-float form has a bound of its own below.
@pytest.mark.parametrize("precision,tol", [(P.SDG_FP64, 1e-12), (P.SDG_FP32_STATE_FP64_SOLVE, 1.2e-7)])
@pytest.mark.parametrize("w", MESHES, ids=IDS)
def test_solve_matches_oracle(w, precision, tol):
    s, _, _, state = P.from_workload(w, precision)
    T = s.gather(state)                                  # as stored (rounded in the float forms)
    m = O.PrismMesh(w.vxy, w.tri, w.nbr, w.nlayers, w.zlev)
    ref = O.implicit_solve(m, w.kappa, w.dt, T, w.penalty)
    out = s.vertical_implicit_solve(state)
    s.vertical_implicit_solve(state, state)              # in place
    s.sync()
    scale = np.abs(ref).max(axis=(1, 2))
    assert (np.abs(s.gather(out) - ref).max(axis=(1, 2)) <= tol * scale).all()
    assert np.array_equal(s.gather(state), s.gather(out))


def float_bound(w, m, T):
    """Bound of each value's error in the all-float solve, (F, 6, P): to first order
    |S^-1| (|dS| |x| + |db|) with S the column's system and b = M T*.  S and b are sums
    of at most 20 float products each, and the elimination of a layer (two 3x3
    inverses, their products with the couplings and with y) rounds at most 44 more times
    at the size of the system's own terms: 64 * 2^-24 of |S| |x| + |M| |T*| in all."""
    bound = np.empty_like(T)
    for c in range(m.C):
        S, Mc = O.prism_dg.column_system(m, w.kappa, w.dt, c, w.penalty)
        ps = m.off[c] + np.arange(int(m.nl[c]))
        t = T[:, :, ps].transpose(2, 1, 0).reshape(len(S), -1)
        inv = np.linalg.inv(S)
        terms = np.abs(S) @ np.abs(inv @ (Mc @ t)) + np.abs(Mc) @ np.abs(t)
        b = 64 * 2.0 ** -24 * np.abs(inv) @ terms
        bound[:, :, ps] = b.reshape(len(ps), 6, -1).transpose(2, 1, 0)
    return bound


FLOAT_MESHES = MESHES + [_sigma(4, d, f) for d, f in [(1, 1), (1, 4), (2, 1), (2, 2), (2, 3), (2, 4), (3, 4)]]


@pytest.mark.parametrize("w", FLOAT_MESHES, ids=lambda w: f"{w.name}-{w.n_cols}x{int(w.nlayers.max())}-{w.n_fields}")
def test_all_float_solve_matches_oracle(w):
    s, _, _, state = P.from_workload(w, P.SDG_FP32)
    T = s.gather(state)
    m = O.PrismMesh(w.vxy, w.tri, w.nbr, w.nlayers, w.zlev)
    ref = O.implicit_solve(m, w.kappa, w.dt, T, w.penalty)
    out = s.vertical_implicit_solve(state)
    s.vertical_implicit_solve(state, state)
    s.sync()
    assert (np.abs(s.gather(out) - ref) <= float_bound(w, m, T)).all()
    assert np.array_equal(s.gather(state), s.gather(out))


@pytest.mark.parametrize("precision", [P.SDG_FP64, P.SDG_FP32])
def test_right_hand_side_off_the_16_byte_grid(precision):
    import torch
    w = _sigma(5, 9, 2)
    s, _, _, state = P.from_workload(w, precision)
    flat = torch.zeros(state.numel() + 1, dtype=state.dtype, device=state.device)
    off = flat[1:].view_as(state)
    off.copy_(state)
    assert off.data_ptr() % 16 != 0
    a, b = s.vertical_implicit_solve(state), s.vertical_implicit_solve(off)
    s.sync()
    assert torch.equal(a, b)


@pytest.mark.parametrize("w", [w for w in MESHES if w.n_prisms < 6000], ids=lambda w: f"{w.name}-{int(w.nlayers.max())}")
def test_transposed_solve_is_the_transpose(w):
    """With zero velocity a reverse step is the transposed solve alone, and
    (K^-T M z, M t) = (z, M K^-1 M t)."""
    import torch
    s, U, _, state = P.from_workload(w, P.SDG_FP64)
    U.zero_()
    rng = np.random.default_rng(3)
    z = s.scatter(rng.standard_normal((w.n_fields, 6, w.n_prisms)))
    x = s.vertical_implicit_solve(state)
    mu = torch.zeros_like(z)
    s.step_adjoint(z, mu)
    lhs, rhs = s.m_dot(mu, state), s.m_dot(z, x)
    size = np.sqrt(s.m_dot(z, z) * s.m_dot(state, state))
    assert (np.abs(lhs - rhs) <= 1e-12 * size).all()
