"""The gauge kernels (plaquettes, force, link update, canonical to tiled links and back)
against the oracle where their work division can go wrong: slices of whole and of ragged
64-site chunks in the slice-by-slice order, the linear order, the smallest lattice."""
import numpy as np
import pytest
import torch

import synth
from oracle import dirac, forces, hmc, lattice

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("L", [(4, 2, 2, 2),
                               (4, 10, 14, 16),     # 17.5 chunks per slice, fewer slices than a workgroup's steps
                               (12, 8, 16, 16),     # 16 whole chunks per slice
                               (8, 6, 10, 12)])     # linear order, ragged
def test_gauge_kernels_match_oracle(gu, L):
    import paper_0710_0066_amd as sap
    print(f"gauge kernels L={L}", flush=True)
    beta, V = 5.6, int(np.prod(L))
    U = synth.gauge_field(L, 0.5, 1301)
    ctx = gu.make_ctx(L, 2, 0.15, U)
    F = ctx.new_momenta()
    ref = forces.gauge_force(U, beta)

    def momenta(f):
        out = torch.zeros(V * 32, dtype=torch.float64, device="cuda")
        ctx.unpack_momenta(out, f)
        return out.cpu().numpy().reshape(tuple(L) + (4, 8))

    # sums of six staples of unit matrices: 1e-12 of the largest entry is some 5000 ulp
    S = sap.gauge_force(ctx, F, 1.0, beta)
    assert np.max(np.abs(momenta(F) - ref)) <= 1e-12 * np.max(np.abs(ref))
    assert abs(S - forces.gauge_action(U, beta)) <= 1e-12 * abs(S)
    assert abs(sap.sap_plaquette(ctx) - forces.mean_plaquette(U)) <= 1e-13
    sap.gauge_force(ctx, F, -3.0, beta)
    assert np.max(np.abs(momenta(F) + 2.0 * ref)) <= 4e-12 * np.max(np.abs(ref))

    # links: stored and read back bit for bit, then moved, with the hop copies following
    got = torch.zeros(U.size, dtype=torch.complex128, device="cuda")
    ctx.get_gauge(got)
    assert np.array_equal(got.cpu().numpy().reshape(U.shape), U)
    p = synth.gaussian_momenta(L, 1302)
    fp = ctx.new_momenta()
    ctx.pack_momenta(fp, gu.dev(p))
    psi = synth.gaussian_spinor(L, 1303)
    for step, field in (("set", U), ("moved", hmc.T_U(U, p, 0.37))):
        if step == "moved":
            sap.sap_update_links(ctx, fp, 0.37)
            ctx.get_gauge(got)
            assert np.max(np.abs(got.cpu().numpy().reshape(U.shape) - field)) <= 1e-13
        want = dirac.apply_M(field, psi, 0.15)
        for prec, tol in ((sap.SAP_F64, 1e-12), (sap.SAP_F32, 2e-5), (sap.SAP_F16, 16 * 2.0 ** -12)):
            fout = ctx.new_field(1, prec)
            sap.apply_M(ctx, fout, gu.to_sap(ctx, psi, 1, prec), 1, prec)
            err = np.max(np.abs(gu.from_sap(ctx, fout, 1, psi.shape, prec) - want))
            assert err <= tol * np.max(np.abs(psi)), (step, prec, err)


def test_links_off_su3_are_refused_wherever_they_are(gu):
    """One link off SU(3) by 1e-8, or not finite, at the first and last site of either parity."""
    import paper_0710_0066_amd as sap
    L = (4, 10, 14, 16)
    U = synth.gauge_field(L, 0.5, 1304)
    ctx = gu.make_ctx(L, 2, 0.15, U)
    last = tuple(n - 1 for n in L)
    for site in ((0, 0, 0, 0), (0, 0, 0, 1), last, last[:3] + (last[3] - 1,)):
        for mu, bad in ((0, 1e-8), (3, np.nan)):
            V = U.copy()
            V[site][mu][2, 1] += bad
            with pytest.raises(sap.SapError) as e:
                ctx.set_gauge(gu.dev(V))
            assert e.value.code == sap.SAP_E_ARG
            with pytest.raises(sap.SapError) as e:
                sap.sap_plaquette(ctx)
            assert e.value.code == sap.SAP_E_STATE
    ctx.set_gauge(gu.dev(U))
    assert abs(sap.sap_plaquette(ctx) - forces.mean_plaquette(U)) <= 1e-13
