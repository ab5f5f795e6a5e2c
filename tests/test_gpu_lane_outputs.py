"""Expectation values of one-wavefront packs of small instances (a group of
lanes per instance and operator) against the row kernel at 256 threads, bit
for bit: every dimension the kernel takes, dense and sparse operators, fewer
and more pairs than a round over the lanes holds, a partial last pack."""
import numpy as np
import pytest

from paper_1110_0573_amd import systems as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1110_0573_amd import lme  # noqa: E402


@pytest.mark.parametrize("n", range(1, 9))
@pytest.mark.parametrize("n_inst,n_e", [(1, 1), (33, 3), (6, 40)])
def test_lane_outputs_bitwise_row_kernel(n, n_inst, n_e):
    rng = np.random.default_rng(10 * n + n_e)
    systems = []
    for _ in range(n_inst):
        H = np.diag(rng.normal(size=n)) + np.diag(rng.normal(size=n - 1), 1)
        E = [np.diag(rng.normal(size=n)) if e % 3 == 1 else
             rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n)) for e in range(n_e)]
        systems.append(S.System(S.tidy(H + H.T), [S.tidy(0.3 * S.destroy(n))] if n > 1 else [],
                                [S.tidy(e) for e in E],
                                rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))))
    h = lme.Handle(systems)
    rho0 = h.pack([s.rho0 for s in systems])
    tl = np.linspace(0.0, 1.0, 6)
    a = h.evolve(rho0, tl, nsteps=20, want_states=True)
    b = h.evolve(rho0, tl, nsteps=20, want_states=True, block=256, layout=lme.LME_LAYOUT_ROW)
    torch.cuda.synchronize()
    assert (a["status"].cpu().numpy() == 0).all()
    for k in ("expect", "states", "rho"):
        assert torch.equal(a[k], b[k]), k
