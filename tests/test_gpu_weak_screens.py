"""Screens with an absorption coefficient of either sign, and with none that
is a number, at intensities where the plasma and multiphoton terms are close
to vanishing beside 1 in the working precision."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from oracle import march as M

pytestmark = pytest.mark.gpu


def _prop(insts, precision, **kw):
    from paper_2306_15678_amd.march import Propagator, desc_of
    return Propagator([desc_of(i) for i in insts], precision=precision, **kw)


def _beam(order, c_m, peak):
    """A 128^2 beam of peak intensity `peak` (in I_a) whose multiphoton term
    is 1 + c_m x^(order - 1)."""
    base = dataclasses.replace(W.config2()[0], n=128, n_screens=0)
    beta = c_m / ((order - 1) * W.I_A ** (order - 1) * base.dz)
    medium = W.Medium(terms=W.TERM_KERR | W.TERM_MPA, mpa_order=order, beta_k=beta)
    inst = dataclasses.replace(base, medium=medium)
    u = W.initial_field(inst)
    return inst, u * np.sqrt(peak * W.I_A / np.max(np.abs(u) ** 2))


# c_m x^(K-1) is 6e-5 to 6e-3 at the peak, while x^(K-1) itself vanishes
# beside 1 in the working precision (below 2^-26, 2^-55).  Three steps without
# the term are off by 1.6e-4 to 2.1e-4 (FP32 cases) and 2.6e-5 to 4.2e-5 (FP64).
CASES = [(32, 2, 1e5, 3e-9), (32, 8, 1e10, 0.018), (64, 2, 1e13, 6e-18), (64, 8, 1e18, 1e-3)]


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("precision,order,c_m,peak", CASES)
def test_strong_coefficients_of_either_sign(precision, order, c_m, peak, sign):
    """Three steps and their gradient against the oracle.  Bounds: those of
    the other short marches and gradients (field FP64 1e-11, FP32 2e-5;
    gradient FP64 1e-10, FP32 1e-4)."""
    inst, u0 = _beam(order, sign * c_m, peak)
    target = 0.8 * np.abs(u0) ** 2
    ref = M.march(u0, inst, n_steps=3)
    loss, g_u, _ = M.gradient(u0, inst, n_steps=3, cotangent=lambda u: M.fluence_loss(u, target))
    p = _prop([inst], precision, max_steps=3, ckpt_every=2)
    p.set_field(0, u0)
    p.propagate(3)
    err = M.rel_l2(p.field(0), ref.field)
    p.set_field(0, u0)
    p.forward_record(3)
    got = p.fluence_loss(0, target)
    p.backward()
    gerr = max(abs(got / loss - 1), M.rel_l2(p.grad_field(0), g_u))
    p.close()
    print(f"fp{precision} K={order} c_m={sign * c_m:.0e}: field {err:.1e} gradient {gerr:.1e}",
          flush=True)
    assert err < (1e-11 if precision == 64 else 2e-5)
    assert gerr < (1e-10 if precision == 64 else 1e-4)


@pytest.mark.parametrize("precision", [32, 64])
def test_a_coefficient_that_is_no_number_is_reported(precision):
    """A NaN absorption coefficient makes every intensity non-finite, however
    weak the beam: the power trace says so."""
    from paper_2306_15678_amd._lib import ENONFINITE, SsfmError
    inst, u0 = _beam(8, float("nan"), 1e-6)
    p = _prop([inst], precision)
    p.set_field(0, u0)
    p.propagate(2)
    with pytest.raises(SsfmError) as e:
        p.diag(0, 2)
    assert e.value.status == ENONFINITE
    assert not np.any(np.isfinite(p.field(0)))
    p.close()
