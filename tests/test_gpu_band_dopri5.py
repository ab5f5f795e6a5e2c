"""The adaptive band kernel where it can go wrong: the smallest dimensions it
takes, odd and even ones, run lengths and packs around the limits of its two
configurations (48 / 49 and 64 / 65), a partial last pack, collapse operators
on diagonals of either sign, three of them, states that are not Hermitian, a
first step so long that it is rejected, and an instance that stops early
beside healthy ones.

Bar: the bits of the row kernel, states, expectation values and step counts;
the kernel does its arithmetic in its order."""
import numpy as np
import pytest

from tests.test_gpu_band import band_system

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1110_0573_amd import lme  # noqa: E402


@pytest.mark.parametrize("dims,offsets,two_sided", [
    ((4, 4, 4), (1, -1), True), ((4, 5, 6, 7), (1, -1), True), ((9, 31, 33), (2, -2, 1), False),
    ((47, 48), (3, -3), True), ((48, 49), (1, 2), False), ((60,), (1, -1), True),
    ((61, 64), (2, 1, -1), False), ((65,), (1, -1), True), ((11,) * 70, (1, -1), True)])
@pytest.mark.parametrize("h0", [0.0, 3.0])
def test_band_dopri5_bits(dims, offsets, two_sided, h0):
    systems = [band_system(n, offsets, two_sided, 100 * b + n) for b, n in enumerate(dims)]
    h = lme.Handle(systems)
    rng = np.random.default_rng(5)
    states = [rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n)) for n in dims]
    tl = np.linspace(0.0, 1.5, 4)

    def run(rho0, layout):
        out = h.evolve(rho0, tl, method="dopri5", rtol=1e-7, atol=1e-9, h0=h0,
                       want_states=True, layout=layout)
        torch.cuda.synchronize()
        return {k: v.cpu().numpy() for k, v in out.items() if v is not None}

    rho0 = h.pack(states)
    got, ref = run(rho0, lme.LME_LAYOUT_AUTO), run(rho0, lme.LME_LAYOUT_ROW)
    assert (got["status"] == 0).all()
    for k in ref:
        assert np.array_equal(got[k], ref[k]), k
    assert h0 == 0.0 or got["counts"][:, 1].min() > 0      # the long first step is rejected

    states[-1] = np.full_like(states[-1], np.inf)
    rho0 = h.pack(states)
    got, ref = run(rho0, lme.LME_LAYOUT_AUTO), run(rho0, lme.LME_LAYOUT_ROW)
    assert got["status"][-1] == lme.LME_ENONFINITE and (got["status"][:-1] == 0).all()
    for k in ("status", "counts"):
        assert np.array_equal(got[k], ref[k]), k
    keep = slice(0, sum(n * n for n in dims[:-1]))
    assert np.array_equal(got["states"][:, keep], ref["states"][:, keep])


@pytest.mark.parametrize("offsets,two_sided", [((1, 9), True), ((-1, -9), True),
                                               ((9, 1), False), ((1, -30, 9), False)])
def test_band_dopri5_diagonals_beyond_an_instance(offsets, two_sided):
    """Small instances without a diagonal that a large one has, packed beside
    one of infinities: the bits of the row kernel."""
    dims = (40,) + (4,) * 600 + (9,) * 5
    from tests.test_gpu_band import short_of_diagonals
    systems = [short_of_diagonals(n, offsets, two_sided, b) for b, n in enumerate(dims)]
    h = lme.Handle(systems)
    rho0 = h.pack([np.full((4, 4), np.inf) if b == 301 else s.rho0
                   for b, s in enumerate(systems)])
    a, r = (h.evolve(rho0, np.linspace(0.0, 1.2, 3), method="dopri5", rtol=1e-7, atol=1e-9,
                     layout=layout) for layout in (lme.LME_LAYOUT_AUTO, lme.LME_LAYOUT_ROW))
    torch.cuda.synchronize()
    status = a["status"].cpu().numpy()
    assert status[301] == lme.LME_ENONFINITE and (np.delete(status, 301) == 0).all()
    for k in ("status", "counts"):
        assert torch.equal(a[k], r[k]), k
    got, ref = h.unpack(a["rho"]), h.unpack(r["rho"])
    for b in range(len(dims)):
        assert b == 301 or np.array_equal(got[b], ref[b]), b
