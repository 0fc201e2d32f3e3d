"""FP16 operators with the default mapping on both sides of the lines between its kernels (split, site,
marching order): right-hand sides that are multiples of one spinor by powers of two give exact
multiples of one result, and that one matches the oracle."""
import numpy as np
import pytest

import synth
from oracle import dirac, lattice

pytestmark = pytest.mark.gpu

# of max |psi|: projection, link and output roundings of eight hops (the bounds of the FP16 operator tests)
F16_M_TOL, F16_HOP_TOL = 16 * 2.0 ** -12, 100 * 2.0 ** -12


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


# sites times rhs: 7.7e4, 1.02e5, 1.41e5, 1.54e5, 4.1e5, 6.1e5 (ragged eighths of a slice), 6.6e5, 1.31e6
@pytest.mark.parametrize("L,l0,nrhs", [((8, 8, 10, 20), 2, 6), ((8, 8, 10, 20), 2, 8), ((8, 8, 10, 20), 2, 11),
                                       ((8, 8, 10, 20), 2, 12), ((8, 16, 16, 20), 4, 10), ((12, 8, 20, 32), 3, 10),
                                       ((8, 16, 16, 32), 4, 10), ((16, 16, 16, 32), 4, 10)])
def test_default_f16_mapping(gu, L, l0, nrhs):
    import paper_0710_0066_amd as sap
    print(f"f16 default L={L} nrhs={nrhs}", flush=True)
    k = 0.15
    U = synth.gauge_field(L, 0.5, 1701)
    one = synth.gaussian_spinor(L, 2701)
    two = 2.0 ** np.arange(nrhs)
    psi = one[None] * two.reshape((nrhs,) + (1,) * one.ndim)
    par = lattice.parity(L)
    ctx = gu.make_ctx(L, l0, k, U, max_rhs=nrhs)
    fin, fout = gu.to_sap(ctx, psi, nrhs, sap.SAP_F16), ctx.new_field(nrhs, sap.SAP_F16)
    big = float(np.max(np.abs(one)))

    def check(ref, tol, mask):
        got = gu.from_sap(ctx, fout, nrhs, psi.shape, sap.SAP_F16) * mask
        assert np.max(np.abs(got[0] - ref * mask)) <= tol * big
        for r in range(1, nrhs):
            assert np.array_equal(got[r], got[0] * two[r]), r

    every = np.ones_like(lattice.site_mask(L, par >= 0))
    for parity in (0, 1):
        sap.apply_Dslash_eo(ctx, fout, fin, nrhs, parity, sap.SAP_F16)
        m = lattice.site_mask(L, par == parity)
        check(dirac.hop(U, one * lattice.site_mask(L, par != parity)), F16_HOP_TOL, m)
    sap.apply_M(ctx, fout, fin, nrhs, sap.SAP_F16)
    check(dirac.apply_M(U, one, k), F16_M_TOL, every)
    W = dirac.apply_W(U, one, k, l0)
    for color, block, mask in ((sap.SAP_ALL, -1, every),
                               (sap.SAP_BLACK, -1, lattice.site_mask(L, lattice.colour_x0_mask(L, l0, "black"))),
                               (sap.SAP_ALL, 1, lattice.site_mask(L, lattice.single_block_mask(L, l0, 1)))):
        sap.apply_W1_block(ctx, fout, fin, nrhs, 1, block, color, sap.SAP_F16)
        check(W * mask, F16_M_TOL, every)
