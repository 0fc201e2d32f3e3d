"""The even-odd pseudo-fermion parts take fields whose odd half is zero: one that is not has no solution
on the even sites and is refused, whatever the solver, however small its odd part beside tol."""
import numpy as np
import pytest

import synth
from oracle import lattice

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("kind", [1, 2])
@pytest.mark.parametrize("method,inner", [("cg", "f64"), ("cg", "f32"), ("geom", "f32"), ("bicgstab", "f32")])
def test_odd_half_is_refused(gu, kind, method, inner):
    import paper_0710_0066_amd as sap
    L = (8, 4, 4, 6)
    print(f"even source kind {kind} {method} {inner}", flush=True)
    U = synth.gauge_field(L, 0.5, 2001)
    ctx = gu.make_ctx(L, 4, 0.12, U, l0_sub=2)
    psi = synth.gaussian_spinor(L, 3001)
    odd = lattice.site_mask(L, lattice.parity(L) == 1)
    o = sap.solve_opts(tol=1e-8, max_iter=2000, max_outer=8, inner_prec=sap.SAP_F32 if inner == "f32" else sap.SAP_F64,
                       inner_tol=1e-5 if inner == "f32" else 0.0,
                       method={"cg": sap.SAP_CG, "bicgstab": sap.SAP_BICGSTAB, "geom": sap.SAP_GEOM}[method])
    F = ctx.new_momenta()
    S = sap.eo_pf_force(ctx, F, 1.0, gu.to_sap(ctx, psi * ~odd, 1), kind, 0.1, o)
    assert np.isfinite(S) and S > 0
    for scale in (1.0, 1e-6):
        phi = gu.to_sap(ctx, psi * ~odd + scale * psi * odd, 1)
        with pytest.raises(sap.SapError) as e:
            sap.eo_pf_force(ctx, F, 1.0, phi, kind, 0.1, o)
        assert e.value.code == sap.SAP_E_NOCONV
