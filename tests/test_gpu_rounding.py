"""Rounding errors of the kernels that evaluate their sums in another order
than the general ones, against 80-bit references (numpy's long double).

Bars.  Band kernel: per step it rounds each element of the state once, as the
classic form does; of the rest, its last stage's input enters the result with
h L as a whole, the classic form's three with h L / 3, / 3 and / 6, one half
of that in the root of the squares.  So its error stays within twice the
other's, within three times for the largest of some hundreds of elements.
Spin-flip kernel: fewer rounded terms an element than the plain streamed
kernel (the diagonal operators are one factor), so its root mean square error
does not exceed that one's."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_1110_0573_amd import systems as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1110_0573_amd import lme  # noqa: E402

if np.finfo(np.longdouble).nmant < 63:  # pragma: no cover
    pytest.skip("needs an 80-bit long double", allow_module_level=True)


def rows(M):
    """Columns and 80-bit values of a sparse matrix, padded to one width."""
    M = sp.csr_matrix(M)
    w = np.diff(M.indptr)
    c, v = np.zeros((M.shape[0], w.max()), int), np.zeros((M.shape[0], w.max()), np.clongdouble)
    for i, (a, b) in enumerate(zip(M.indptr, M.indptr[1:])):
        c[i, :b - a], v[i, :b - a] = M.indices[a:b], M.data[a:b]
    return c, v


def generator(s, adjoint=False):
    """y -> A y + y A^+ + sum C y C^+ (adjoint: with A^+ and C^+), A folded in 64
    bits as the library does."""
    A, Cs = sp.csr_matrix(-1j * s.H0), [sp.csr_matrix(c) for c in s.C]
    for c in Cs:
        A = A - 0.5 * (c.conj().T @ c)
    A, Cs = (rows(A.conj().T), [rows(c.conj().T) for c in Cs]) if adjoint else \
        (rows(A), [rows(c) for c in Cs])

    def left(M, y):
        return sum(M[1][:, w, None] * y[M[0][:, w]] for w in range(M[0].shape[1]))

    def dag(y):
        return y.conj().T.copy()

    def L(y):
        out = left(A, y) + dag(left(A, dag(y)))
        for c in Cs:
            out = out + dag(left(c, dag(left(c, y))))
        return out
    return L


@pytest.mark.parametrize("N", [5, 10, 20])
def test_band_kernel_rounding(N):
    rng = np.random.default_rng(N)
    systems = [S.jc_system(N, wa=1 + 0.1 * k, g=0.3 + 0.1 * k, kappa=0.05, gamma=0.05)
               for k in range(3)]
    n, steps, T = 2 * N, 500, 12.5
    rho0 = []
    for _ in systems:
        X = rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))
        r = X @ X.conj().T
        rho0.append(0.5 * (r + r.conj().T) / np.trace(r).real)
    h = lme.Handle(systems)
    got = [h.unpack(h.evolve(h.pack(rho0), [0.0, T], nsteps=steps, **kw)["rho"])
           for kw in (dict(hermitian=True), dict(layout=lme.LME_LAYOUT_ROW))]
    dt = np.longdouble(T) / steps
    band, classic = [], []
    for b, s in enumerate(systems):
        L, y = generator(s), rho0[b].astype(np.clongdouble)
        for _ in range(steps):
            k1 = L(y)
            k2 = L(y + dt / 2 * k1)
            k3 = L(y + dt / 2 * k2)
            y = y + dt / 6 * (k1 + 2 * (k2 + k3) + L(y + dt * k3))
        band.append(float(np.max(np.abs(got[0][b] - y))))
        classic.append(float(np.max(np.abs(got[1][b] - y))))
    print("band", band, "classic", classic)
    assert max(band) <= 3.0 * max(classic)


@pytest.mark.parametrize("M", [7, 8])
@pytest.mark.parametrize("adjoint", [False, True])
def test_spin_flip_rounding(M, adjoint):
    rng = np.random.default_rng(M)
    s = S.tfim_system(rng.uniform(0.5, 1.5, M))
    h = lme.Handle([s])
    y = rng.normal(size=(s.n, s.n)) + 1j * rng.normal(size=(s.n, s.n))
    a, b = (h.unpack(h.apply(h.pack([y]), adjoint=adjoint, form=form))[0]
            for form in (lme.LME_FORM_OPERATOR, lme.LME_FORM_OPERATOR_STREAMED))
    L = generator(s, adjoint)
    want = L(y.astype(np.clongdouble))
    rms = [float(np.sqrt(np.mean(np.abs(x - want) ** 2))) for x in (a, b)]
    print("flip, plain:", rms)
    assert rms[0] <= rms[1]
