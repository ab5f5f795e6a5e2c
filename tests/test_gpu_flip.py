"""Spin-flip kernels (chains of 7 and 8 spins) over the forms they accept,
against the oracle and the plain streamed kernel: one and several flipping
operators per spin, of either direction, diagonal operators or none, spins
without a flip in H, the adjoint, one instance and several; operators that
flip two spins at once keep the row-block kernel.  Bars as for the row-block
application: 1e-12 of the largest entry against the oracle, 1e-14 against the
plain streamed kernel (the same terms, the diagonal operators summed first:
at most 20 terms of rounding 1e-16 each, relative to the largest entry)."""
import numpy as np
import pytest

import oracle
from paper_1110_0573_amd import systems as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1110_0573_amd import lme  # noqa: E402


def chain(M, rng, fields, lower, upper, diag, pair):
    """Random chain: sigma_x fields on the spins `fields`, diagonal couplings,
    lowering / raising operators on `lower` / `upper`, `diag` dephasing-like
    diagonal operators, and with `pair` a two-spin flip."""
    H = sum(rng.normal() * S.site_op(S.sigmax(), i, M) for i in fields)
    H = H + sum(rng.normal() * (S.site_op(S.sigmaz(), i, M) @ S.site_op(S.sigmaz(), i + 1, M))
                for i in range(M - 1))
    if pair:
        H = H + S.site_op(S.sigmax(), 1, M) @ S.site_op(S.sigmax(), 4, M)
    C = [S.tidy(rng.uniform(0.1, 0.5) * S.site_op(S.sigmam(), i, M)) for i in lower]
    C += [S.tidy(rng.uniform(0.1, 0.5) * S.dag(S.site_op(S.sigmam(), i, M))) for i in upper]
    C += [S.tidy(rng.uniform(0.1, 0.5) * S.site_op(S.sigmaz(), i, M)) for i in diag]
    return S.System(S.tidy(H), C, [S.site_op(S.sigmaz(), 0, M)], S.ket2dm(S.ket(2 ** M, 3)))


@pytest.mark.parametrize("M,n_inst,fields,lower,upper,diag,pair", [
    (8, 1, range(8), range(8), [], range(8), False), (7, 3, range(7), range(7), [], range(7), False),
    (8, 2, range(8), range(8), range(8), [], False), (7, 2, [0, 6], [2, 2, 5], [2], [1], False),
    (8, 2, [3], [0], [7], [], False), (8, 1, [], [4], [], [0, 7], False),
    (7, 1, range(7), [], [], [3], False), (8, 1, range(8), range(8), [], [0], True)])
def test_flip_applications(M, n_inst, fields, lower, upper, diag, pair):
    rng = np.random.default_rng(10 * M + n_inst + len(fields))
    systems = [chain(M, rng, fields, lower, upper, diag, pair) for _ in range(n_inst)]
    ys = [rng.normal(size=(s.n, s.n)) + 1j * rng.normal(size=(s.n, s.n)) for s in systems]
    h = lme.Handle(systems)
    y = h.pack(ys)
    for adjoint, fn in ((False, oracle.apply_L), (True, oracle.apply_Ldag)):
        a = h.apply(y, adjoint=adjoint)
        b = h.apply(y, adjoint=adjoint, form=lme.LME_FORM_OPERATOR_STREAMED)
        torch.cuda.synchronize()
        assert torch.max(torch.abs(a - b)).item() <= 1e-14 * torch.max(torch.abs(b)).item()
        for got, s, x in zip(h.unpack(a), systems, ys):
            want = fn(s, x)
            assert np.max(np.abs(got - want)) <= 1e-12 * np.max(np.abs(want))


@pytest.mark.parametrize("M,n_inst", [(7, 3), (8, 1)])
def test_flip_adaptive_steps(M, n_inst):
    """The streamed adaptive stepper on flip tiles against the oracle: the
    same steps, expectation values within 1e-9 (rtol 1e-7)."""
    rng = np.random.default_rng(M)
    systems = [chain(M, rng, range(M), range(M), [0, 3], range(M), False) for _ in range(n_inst)]
    tl = np.linspace(0.0, 0.4, 4)
    h = lme.Handle(systems)
    out = h.evolve(h.pack([s.rho0 for s in systems]), tl, method="dopri5", rtol=1e-7, atol=1e-10)
    torch.cuda.synchronize()
    assert (out["status"].cpu().numpy() == 0).all()
    for b, s in enumerate(systems):
        r = oracle.dopri5(s, s.rho0, tl, 1e-7, 1e-10)
        assert tuple(out["counts"].cpu().numpy()[b]) == tuple(int(c) for c in r["counts"])
        assert np.max(np.abs(out["expect"].cpu().numpy()[b] - r["expect"])) <= 1e-9
