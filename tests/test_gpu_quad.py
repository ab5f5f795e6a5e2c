"""Two-level batches (one instance per quad of lanes) against the row kernel
at 256 threads, bit for bit, over the forms the quad kernel accepts: no, one
and two control terms with and without off-diagonal entries, segments and
closed forms with and without a cosine, no off-diagonal entry in H, collapse
operators whose sources lie at each distance or differ from lane to lane, more
(instance, operator) pairs than lanes, a partial last pack and one instance."""
import numpy as np
import pytest

from paper_1110_0573_amd import systems as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1110_0573_amd import lme  # noqa: E402

JUMPS = {"down": [[0, 1], [0, 0]], "up": [[0, 0], [1, 0]], "flip": [[0, 1], [0.6, 0]],
         "phase": [[1, 0], [0, -0.7j]], "row": [[0, 1], [0, 0.5]], "one": [[0, 0], [0, 1]]}


def two_level(rng, jumps, ctrl, form, off, n_e):
    H = rng.normal(size=(2, 2)) + 1j * rng.normal(size=(2, 2))
    H = H + H.conj().T
    if not off:
        H = np.diag(np.diag(H))
    X = rng.normal(size=(2, 2)) + 1j * rng.normal(size=(2, 2))
    E = [S.tidy(rng.normal(size=(2, 2)) + 1j * rng.normal(size=(2, 2))) for _ in range(n_e)]
    s = S.System(S.tidy(H), [S.tidy(0.3 * np.array(JUMPS[j], complex)) for j in jumps], E, X)
    s.H_ctrl = [S.tidy({"z": S.sigmaz(), "x": S.sigmax(), "y": S.sigmay()}[c]) for c in ctrl]
    if form == "segments":
        s.edges = np.linspace(0.0, 1.0, 6)
        s.u = rng.normal(size=(len(ctrl), 5))
        s.u[:, 2] = 0.0
    elif ctrl:
        s.fn = rng.normal(size=(len(ctrl), 7))
        if form == "polynomial":
            s.fn[:, 4] = 0.0
    return s


@pytest.mark.parametrize("n_inst,jumps,ctrl,form,off,n_e", [
    (1, ["down"], "z", "polynomial", True, 1), (17, ["down", "up"], "z", "cosine", True, 4),
    (33, ["phase"], "x", "segments", True, 5), (40, ["flip", "one"], "zy", "cosine", True, 2),
    (40, ["row", "down"], "xz", "segments", False, 3), (100, [], "", "none", True, 4),
    (21, ["down", "up", "phase", "row"], "", "none", False, 7),
    (5, ["up"], "yx", "polynomial", True, 40)])
def test_two_level_batches_bitwise_row_kernel(n_inst, jumps, ctrl, form, off, n_e):
    rng = np.random.default_rng(n_inst + 7 * n_e)
    h = lme.Handle([two_level(rng, jumps, ctrl, form, off, n_e) for _ in range(n_inst)])
    rho0 = h.pack([rng.normal(size=(2, 2)) + 1j * rng.normal(size=(2, 2)) for _ in range(n_inst)])
    tl = np.linspace(0.0, 1.0, 11)
    a = h.evolve(rho0, tl, nsteps=50, want_states=True)
    b = h.evolve(rho0, tl, nsteps=50, want_states=True, block=256, layout=lme.LME_LAYOUT_ROW)
    torch.cuda.synchronize()
    assert (a["status"].cpu().numpy() == 0).all()
    for k in ("expect", "states", "rho", "counts", "status"):
        assert torch.equal(a[k], b[k]), k


JUMPS["zero"] = [[0, 0], [0, 0]]


@pytest.mark.parametrize("n_inst,jumps,ctrl,form,off", [
    (1, [["zero"]], "z", "polynomial", True), (40, [["zero"], ["down"]], "z", "polynomial", True),
    (1, [["zero"]], "", "none", True), (9, [["zero", "zero"]], "", "none", False),
    (40, [["zero", "zero"], ["down", "zero"], ["zero", "flip"]], "xz", "segments", True),
    (33, [["zero"], ["phase"]], "zx", "cosine", False),
    (5, [["zero"] * 6], "y", "segments", True)])
def test_two_level_batches_with_operators_without_entries(n_inst, jumps, ctrl, form, off):
    """Collapse operators whose entries are all zero (a decay rate of zero in
    a sweep), alone and beside ones with entries: the bits of the row kernel,
    and where every operator is zero those of the batch without operators."""
    rng = np.random.default_rng(n_inst)
    systems = [two_level(rng, jumps[b % len(jumps)], ctrl, form, off, 2) for b in range(n_inst)]
    for s in systems[1:]:
        s.edges = systems[0].edges
    h = lme.Handle(systems)
    rho0 = h.pack([rng.normal(size=(2, 2)) + 1j * rng.normal(size=(2, 2)) for _ in range(n_inst)])
    tl = np.linspace(0.0, 1.0, 11)

    def run(h, **kw):
        out = h.evolve(rho0, tl, nsteps=50, want_states=True, **kw)
        torch.cuda.synchronize()
        assert (out["status"].cpu().numpy() == 0).all()
        return out

    a = run(h)
    others = [run(h, block=256, layout=lme.LME_LAYOUT_ROW)]
    if all(set(j) == {"zero"} for j in jumps):
        for s in systems:
            s.C = []
        others.append(run(lme.Handle(systems)))
    for b in others:
        for k in ("expect", "states", "rho", "counts"):
            assert torch.equal(a[k], b[k]), k
