"""GPU parity of the Monte-Carlo kernel with the operator in registers against
the oracle, at the sizes where its decomposition can go wrong: a row count
just below, at and above the threads times rows of a configuration, the
largest dimension whose two vectors fit LDS (5090, as before it), several
trajectories per workgroup and a partial last one, and each structure of
A = -iH - 1/2 sum C^+C it accepts (all real, imaginary off-diagonal, real
off-diagonal with a complex diagonal), with no, one and two off-diagonal
entries a row.

Bars as for the general kernel: jump counts and operators exact, jump times
within 1e-10 absolute (times of order 1), expectation values within 1e-9 (the
same RK4 map, rounding accumulated over a few hundred steps)."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
from paper_1110_0573_amd import systems as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1110_0573_amd import lme  # noqa: E402


def ladder(n, structure, reach):
    """Bosonic mode of n states: a hop over `reach` levels (0: none) with
    real or imaginary amplitude in H, optionally with level energies."""
    a = S.destroy(n)
    num = S.tidy(S.dag(a) @ a)
    V = sp.diags(np.linspace(0.3, 0.9, n - reach), reach, shape=(n, n), format="csr") if reach \
        else sp.csr_matrix((n, n), dtype=np.complex128)
    H = V + V.T if structure == "imag" else 1j * (V - V.T)      # -iH imaginary, or real
    if structure != "real":
        H = H + 0.7 * sp.diags(np.linspace(0, 1, n))
    C = [S.tidy(np.sqrt(0.3 / n) * a)]
    hop = sp.diags(np.ones(n - 1), 1, shape=(n, n), format="csr") * 0.2
    E = [num, S.tidy(hop + 0.5j * hop.T)]
    return S.System(S.tidy(H), C, E, None)


@pytest.mark.parametrize("n,n_traj,structure,reach", [
    (2, 3, "imag", 1), (3, 70, "real", 1), (10, 300, "offreal", 3), (63, 5, "imag", 0),
    (64, 9, "real", 7), (65, 257, "imag", 1), (511, 3, "offreal", 200), (512, 2, "real", 31),
    (513, 3, "imag", 1), (1025, 2, "real", 300), (5090, 2, "imag", 271)])
def test_mc_registers_parity(n, n_traj, structure, reach):
    s = ladder(n, structure, reach)
    rng = np.random.default_rng(n)
    psi0 = rng.normal(size=n) + 1j * rng.normal(size=n)
    tl = np.linspace(0.0, 1.5, 7)
    draws = S.mc_draws(n_traj, 40, n + 1)
    h = lme.McHandle(s.H0, s.C, s.E)
    g = h.evolve(torch.from_numpy(psi0).cuda(), tl, 300, torch.from_numpy(draws).cuda())
    torch.cuda.synchronize()
    g = {k: v.cpu().numpy() for k, v in g.items()}
    r = oracle.mc(s, psi0, tl, 300, draws, n_threads=8)
    assert np.array_equal(g["status"], r["status"])
    assert np.array_equal(g["n_jumps"], r["n_jumps"])
    for b in range(n_traj):
        nj = r["n_jumps"][b]
        assert np.array_equal(g["jump_op"][b, :nj], r["jump_op"][b, :nj])
        assert np.max(np.abs(g["jump_t"][b, :nj] - r["jump_t"][b, :nj]), initial=0) <= 1e-10
    scale = max(1.0, np.max(np.abs(r["expect_traj"])))
    assert np.max(np.abs(g["expect_traj"] - r["expect_traj"])) <= 1e-9 * scale
