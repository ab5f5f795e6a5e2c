"""The band kernel (Hermitian RK4 along diagonals) where it can go wrong: the
smallest dimensions it takes, odd and even ones (for even n the last diagonal
is shared), run lengths and packs around its limits, collapse operators on
diagonals of either sign and beyond the neighbours, expectation operators off
the diagonal, and a diverging instance packed beside healthy ones.

Bars: 1e-10 against the oracle (expectation values, trace distance; both
integrate the same RK4 map, differences are rounding over at most 120 steps);
1e-13 against the general path on the same inputs, as for the other Hermitian
kernels."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
from paper_1110_0573_amd import systems as S
from tests import brute

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1110_0573_amd import lme  # noqa: E402


def band_system(n, offsets, two_sided, seed):
    """H real and tridiagonal (or pairs (0,1), (2,3), ... only), C_k real on
    diagonal offsets[k], a random density matrix, one E-op off the diagonal."""
    rng = np.random.default_rng(seed)
    hop = rng.uniform(0.2, 1.0, n - 1)
    if not two_sided:
        hop[1::2] = 0.0
    H = sp.diags([hop, rng.uniform(-1, 1, n), hop], [-1, 0, 1])
    C = [S.tidy(sp.diags(rng.uniform(-0.4, 0.4, n - abs(d)), d)) for d in offsets]
    X = rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))
    rho = X @ X.conj().T
    E = [S.tidy(sp.diags(np.arange(n, dtype=float))),
         S.tidy(sp.diags(rng.normal(size=n - 2) + 0.3j, 2) + sp.diags(np.ones(n - 1), -1))]
    return S.System(S.tidy(H), C, E, rho / np.trace(rho).real)


@pytest.mark.parametrize("dims,offsets,two_sided", [
    ((4, 4, 4), (1,), True), ((4, 5, 6, 7), (1, -1), True), ((4, 6, 8, 10), (2, 1), False),
    ((9, 32, 33), (2, -2, 1), False), ((31, 32), (3, -3), True), ((63, 64, 65), (1, -1), True),
    ((79, 80, 81), (2, 1), False), ((84,), (1,), False), ((20,) * 300, (2, 1), False),
    ((11,) * 70, (1, -1, 0), True), ((4, 4, 4), (1, -1), True), ((82, 84), (2, 1), False),
    ((11,) * 70, (1, -1), True)])
def test_band_kernel(dims, offsets, two_sided):
    systems = [band_system(n, offsets, two_sided, 100 * b + n) for b, n in enumerate(dims)]
    tl = np.linspace(0.0, 1.2, 5)
    h = lme.Handle(systems)
    rho0 = h.pack([s.rho0 for s in systems])
    out = h.evolve(rho0, tl, nsteps=120, hermitian=True, want_states=True)
    ref = h.evolve(rho0, tl, nsteps=120, want_states=True)
    torch.cuda.synchronize()
    assert (out["status"].cpu().numpy() == 0).all()
    assert torch.max(torch.abs(out["states"] - ref["states"])).item() <= 1e-13
    # expectation values: sums of up to n products with entries of up to n
    scale = max(1.0, float(torch.max(torch.abs(ref["expect"]))))
    assert torch.max(torch.abs(out["expect"] - ref["expect"])).item() <= 1e-13 * max(dims) * scale
    rho = h.unpack(out["rho"])
    # the operator shapes with a Hermitian kernel; others run the general path
    herm = (2 if two_sided else 1, len(offsets)) in {(1, 2), (1, 3), (2, 2)}
    for b in sorted({0, len(dims) // 2, len(dims) - 1}):
        assert not herm or np.array_equal(rho[b], rho[b].conj().T)
        ex, st = oracle.rk4(systems[b], systems[b].rho0, tl, 120, store_states=True)
        assert np.max(np.abs(out["expect"].cpu().numpy()[b] - ex)) <= 1e-10
        assert brute.trace_distance(rho[b], st[-1]) <= 1e-10


def test_band_kernel_diverging_neighbour():
    """A step far outside the stability region makes one instance overflow;
    the instances packed with it keep their results."""
    systems = [band_system(10, (1, -1), True, b) for b in range(600)]
    systems[301].H0 = S.tidy(systems[301].H0 * 1e9)
    tl = np.linspace(0.0, 1.2, 3)
    h = lme.Handle(systems)
    out = h.evolve(h.pack([s.rho0 for s in systems]), tl, nsteps=120, hermitian=True)
    torch.cuda.synchronize()
    status = out["status"].cpu().numpy()
    assert status[301] == lme.LME_ENONFINITE
    assert (np.delete(status, 301) == 0).all()
    for b in (300, 302, 299, 303):
        ex, _ = oracle.rk4(systems[b], systems[b].rho0, tl, 120, store_states=True)
        assert np.max(np.abs(out["expect"].cpu().numpy()[b] - ex)) <= 1e-10


def short_of_diagonals(n, offsets, two_sided, seed):
    """band_system() where n may be too small for some of the diagonals: those
    operators have no entries (a nine-photon loss at a cutoff of four)."""
    s = band_system(n, [d if abs(d) < n else 0 for d in offsets], two_sided, seed)
    s.C = [c if abs(d) < n else S.tidy(np.zeros((n, n))) for c, d in zip(s.C, offsets)]
    return s


@pytest.mark.parametrize("offsets,two_sided", [((1, 9), True), ((-1, -9), True),
                                               ((9, 1), False), ((1, -30, 9), False)])
def test_band_kernel_diagonals_beyond_an_instance(offsets, two_sided):
    """Small instances without a diagonal that a large one has, packed beside
    one that overflows: nothing of it reaches them."""
    dims = (40,) + (4,) * 600 + (9,) * 5
    systems = [short_of_diagonals(n, offsets, two_sided, b) for b, n in enumerate(dims)]
    systems[301].H0 = S.tidy(systems[301].H0 * 1e9)
    tl = np.linspace(0.0, 1.2, 3)
    h = lme.Handle(systems)
    rho0 = h.pack([s.rho0 for s in systems])
    out = h.evolve(rho0, tl, nsteps=120, hermitian=True)
    ref = h.evolve(rho0, tl, nsteps=120, layout=lme.LME_LAYOUT_ROW)
    torch.cuda.synchronize()
    status = out["status"].cpu().numpy()
    assert status[301] == lme.LME_ENONFINITE
    assert (np.delete(status, 301) == 0).all()
    rho, want = h.unpack(out["rho"]), h.unpack(ref["rho"])
    for b in range(len(dims)):
        assert b == 301 or np.max(np.abs(rho[b] - want[b])) <= 1e-13, b
    for b in (0, 1, 300, 302, len(dims) - 1):
        ex, _ = oracle.rk4(systems[b], systems[b].rho0, tl, 120, store_states=True)
        assert np.max(np.abs(out["expect"].cpu().numpy()[b] - ex)) <= 1e-10


@pytest.mark.parametrize("dims,offsets,two_sided", [
    ((4, 5, 6, 7), (1, -1), True), ((4, 6, 8, 10), (2, 1), False), ((63, 64, 65), (1, -1), True),
    ((72, 73), (2, -2, 1), False), ((81, 82, 83), (2, 1), False), ((82, 83), (1, -1), True),
    ((20,) * 300, (2, 1), False)])
def test_band_kernel_block_512(dims, offsets, two_sided):
    """The 512-thread configuration (up to 7 diagonals a thread, n <= 83), which
    runs where a caller names that block size: against the general path."""
    systems = [band_system(n, offsets, two_sided, 100 * b + n) for b, n in enumerate(dims)]
    tl = np.linspace(0.0, 1.2, 5)
    h = lme.Handle(systems)
    rho0 = h.pack([s.rho0 for s in systems])
    out = h.evolve(rho0, tl, nsteps=120, hermitian=True, want_states=True, block=512,
                   layout=lme.LME_LAYOUT_COLUMN)
    ref = h.evolve(rho0, tl, nsteps=120, want_states=True)
    torch.cuda.synchronize()
    assert (out["status"].cpu().numpy() == 0).all()
    assert torch.max(torch.abs(out["states"] - ref["states"])).item() <= 1e-13
    for r in h.unpack(out["rho"]):
        assert np.array_equal(r, r.conj().T)
