"""One-thread-per-prism stages on launches large enough to read the neighbours in the
cell from LDS (forward: more than 4 wavefronts per CU, adjoint: 16): the forward stages
bitwise against the column walk, the adjoint stages by the transpose identity with the
forward step."""

import numpy as np
import pytest

import paper_2605_16082_amd as P
import workloads as W

pytestmark = pytest.mark.gpu


def _mesh(n, fields, w_zero):
    w = W.ragged(n=n, n_fields=fields, n_min=3, n_max=33, dz=2.0, depth_max=66.0)
    if not w_zero:
        w.U = w.U.copy()
        w.U[2] = 1e-3 * np.random.default_rng(5).standard_normal(w.U[2].shape)
    return w


def _build(n, per_cu, fields, precision, w_zero):
    import torch
    w = _mesh(n, fields, w_zero)
    s, _, _, state = P.from_workload(w, precision)
    # the layers of all cells: a launch has as many wavefronts or a few more
    assert s.n_slots // 64 > per_cu * torch.cuda.get_device_properties(0).multi_processor_count
    return w, s, state


@pytest.mark.parametrize("w_zero", [True, False])
@pytest.mark.parametrize("precision", [P.SDG_FP64, P.SDG_FP32])
@pytest.mark.parametrize("fields", [1, 2, 3, 4])
def test_bitwise_the_walk(fields, precision, w_zero):
    w, s, state = _build(46, 4, fields, precision, w_zero)
    Ts = s.scatter(w.T0 + 0.1 * np.random.default_rng(3).standard_normal(w.T0.shape))
    ref = None
    for shape in [(8, 1, 0), (1, 1, 0), (2, 1, 0), (2, 0, 1), (4, 1, 0), (4, 1, 1)]:
        s.set_tuning(*shape)
        out = [s.rk_stage(k, state, Ts) for k in range(3)] + [s.rhs_3d(Ts)]
        s.sync()
        got = [s.gather(o) for o in out]
        ref = ref or got
        for a, b in zip(got, ref):
            assert np.array_equal(a, b), shape


# <A d, M y> = <d, M A* y>, A the (affine) step's linear part: both sides are sums of
# the same order of products, rounded within 1e-15 of their terms' magnitudes; 1e-12 of
# |A d| |M y| leaves a thousandfold for the terms' own rounding through the step.
@pytest.mark.parametrize("w_zero", [True, False])
@pytest.mark.parametrize("fields", [1, 2, 3, 4])
def test_adjoint_step_is_the_transpose(fields, w_zero):
    w, s, state = _build(90, 16, fields, P.SDG_FP64, w_zero)
    rng = np.random.default_rng(11)
    d = s.scatter(rng.standard_normal(w.T0.shape))
    y = s.scatter(rng.standard_normal(w.T0.shape))
    ends = []
    for x0 in (d, s.new_state()):
        x = x0.clone()
        s.set_fields(x)
        s.step()
        ends.append(x)
    ad = ends[0] - ends[1]
    for shape in [(1, 1, 0), (2, 1, 0), (4, 0, 0)]:
        s.set_tuning(*shape)
        z = s.new_state()
        s.step_adjoint(y, z)
        s.sync()
        left = float(s.m_dot(ad, y).sum())
        right = float(s.m_dot(d, z).sum())
        scale = (float(s.m_dot(ad, ad).sum()) * float(s.m_dot(y, y).sum())) ** 0.5
        assert abs(left - right) <= 1e-12 * scale, shape


@pytest.mark.parametrize("w_zero", [True, False])
def test_adjoint_step_of_four_fields_is_the_transpose(w_zero):
    """The same above the line of four fields (28 wavefronts per CU), and the shapes agree
    bitwise."""
    w, s, state = _build(116, 28, 4, P.SDG_FP64, w_zero)
    rng = np.random.default_rng(11)
    d = s.scatter(rng.standard_normal(w.T0.shape))
    y = s.scatter(rng.standard_normal(w.T0.shape))
    ends = []
    for x0 in (d, s.new_state()):
        x = x0.clone()
        s.set_fields(x)
        s.step()
        ends.append(x)
    ad = ends[0] - ends[1]
    ref = None
    for shape in [(2, 1, 0), (1, 1, 0), (4, 0, 0)]:
        s.set_tuning(*shape)
        z = s.new_state()
        s.step_adjoint(y, z)
        s.sync()
        left = float(s.m_dot(ad, y).sum())
        right = float(s.m_dot(d, z).sum())
        scale = (float(s.m_dot(ad, ad).sum()) * float(s.m_dot(y, y).sum())) ** 0.5
        assert abs(left - right) <= 1e-12 * scale, shape
        ref = s.gather(z) if ref is None else ref
        assert np.array_equal(s.gather(z), ref), shape
