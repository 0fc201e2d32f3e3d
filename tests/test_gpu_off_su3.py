"""The gauge force of links that are off SU(3) by less than sap_set_gauge refuses is the derivative
of the action of those links, whichever kernel forms it."""
import numpy as np
import pytest
import torch

import synth
from oracle import forces

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("L", [(4, 2, 2, 2), (4, 10, 14, 16), (8, 6, 10, 12)])
@pytest.mark.parametrize("off", [0.0, 1e-15, 2e-14, 1e-12, 2e-11])
def test_gauge_force_off_su3(gu, L, off):
    import paper_0710_0066_amd as sap
    print(f"force off SU(3) L={L} off={off}", flush=True)
    beta, V = 5.6, int(np.prod(L))
    U = synth.gauge_field(L, 0.5, 1601)
    rng = np.random.default_rng(1602)
    U = U + off * (rng.uniform(-1, 1, U.shape) + 1j * rng.uniform(-1, 1, U.shape))
    ctx = gu.make_ctx(L, 2, 0.15, U)

    def check(field):
        F = ctx.new_momenta()
        S = sap.gauge_force(ctx, F, 1.0, beta)
        out = torch.zeros(V * 32, dtype=torch.float64, device="cuda")
        ctx.unpack_momenta(out, F)
        got, ref = out.cpu().numpy().reshape(tuple(L) + (4, 8)), forces.gauge_force(field, beta)
        # six staples of three links, beta / 6 and the deviation of rounded links: some 500 ulp
        assert np.max(np.abs(got - ref)) <= 1e-13 * np.max(np.abs(ref))
        assert abs(S - forces.gauge_action(field, beta)) <= 1e-12 * abs(S)

    check(U)
    # moved links are unitary again
    fp = ctx.new_momenta()
    ctx.pack_momenta(fp, gu.dev(synth.gaussian_momenta(L, 1603)))
    sap.sap_update_links(ctx, fp, 0.2)
    moved = torch.zeros(U.size, dtype=torch.complex128, device="cuda")
    ctx.get_gauge(moved)
    check(moved.cpu().numpy().reshape(U.shape))
