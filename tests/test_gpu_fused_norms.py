"""The norms that the LDS-staged hop adds to its output, and in FP32 its products, are sums of FP64
products, as those of the norm passes are: sources whose components have no square in FP32 (above 2e19 it
overflows, below 1e-23 it vanishes) are solved in the iterations that their multiples by a
power of two take."""
import numpy as np
import pytest

import synth
from oracle import dirac

pytestmark = pytest.mark.gpu

SLABD = 20


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


# (BiCGstab: the larger sources overflow its first beta = ||r||^2 whatever the mapping)
@pytest.mark.parametrize("method,inner,power", [(m, i, p) for m in ("cg", "geom") for i in ("f32", "f16") for p in (70, -80)]
                         + [("bicgstab", "f32", -80)])
@pytest.mark.parametrize("blocks", [False, True])
def test_sources_without_an_fp32_square(gu, method, inner, power, blocks):
    import paper_0710_0066_amd as sap
    L, l0, k, n = (8, 8, 4, 8), 4, 0.11, 2
    print(f"fused norms {method} {inner} 2**{power} blocks={blocks}", flush=True)
    U = synth.gauge_field(L, 0.5, 1401)
    b = synth.gaussian_spinor(L, 2401, nrhs=n)
    prec = sap.SAP_F32 if inner == "f32" else sap.SAP_F16
    o = sap.solve_opts(tol=1e-6, max_iter=2000, max_outer=20, inner_prec=prec, inner_tol=1e-3,
                       method={"cg": sap.SAP_CG, "bicgstab": sap.SAP_BICGSTAB, "geom": sap.SAP_GEOM}[method])
    ctx = gu.make_ctx(L, l0, k, U, max_rhs=n)
    sap.sap_set_hop_map(ctx, 0, prec, n, SLABD)
    fx = ctx.new_field(n)
    count = []
    for scale in (1.0, 2.0 ** power):
        fb = gu.to_sap(ctx, b * scale, n)
        if blocks:
            info = sap.solve_blocks(ctx, fx, fb, n, 1, sap.SAP_ALL, o)
        else:
            info = sap.solve_full(ctx, fx, fb, n, o)
        count.append([(e.iters, e.outer) for e in info])
        x = gu.from_sap(ctx, fx, n, b.shape) / scale
        r = b - dirac.apply_op(U, x, k, l0 if blocks else None)
        ax = tuple(range(1, r.ndim))
        assert np.all(np.sum(np.abs(r) ** 2, axis=ax) <= 1.001e-12 * np.sum(np.abs(b) ** 2, axis=ax))
    assert count[0] == count[1]
