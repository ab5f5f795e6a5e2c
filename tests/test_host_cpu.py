"""Host code of liblme.so on a machine without a GPU: the HIP runtime is replaced
by tests/fake_hip.cpp (host memory, launches recorded and not run), which
shows the kernel that a call takes, its launch shape, and what is left after a
failed allocation.  Each case is a process of its own."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROLOGUE = """
import ctypes as C, os, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
fake.fake_launches.restype = C.c_char_p
import numpy as np
from paper_1110_0573_amd import lme, systems as S
lib = lme.load()

def launches():
    got = [l.split() for l in fake.fake_launches().decode().splitlines()]
    fake.fake_clear()
    return got

def apply(h):
    y = np.zeros(h.state_elems, complex)
    out = np.zeros_like(y)
    return lib.lme_apply(h._h, 0, 0, 0.0, None, y.ctypes.data, out.ctypes.data, None)
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("needs g++")
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", so,
                    os.path.join(ROOT, "tests", "fake_hip.cpp")], check=True)
    return so


def run(fake, body, **env):
    r = subprocess.run([sys.executable, "-c", PROLOGUE + textwrap.dedent(body), fake], cwd=ROOT,
                       env={**os.environ, **env}, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_spin_flip_tables_after_a_failed_upload(fake):
    """The tables of the adjoint operators do not fit the first time: the next
    call uploads both and launches with tables."""
    run(fake, """
        h = lme.Handle(S.tfim(n_inst=2, M=7).systems)      # created without a device
        for k in range(1, 7):                               # pools and the two tables
            fake.fake_fail_allocation(k)
            assert apply(h) == lme.LME_ENOMEM, k
            assert not launches()
        fake.fake_fail_allocation(0)
        assert apply(h) == 0
        name, _, _, _, tab = launches()[-1]
        assert "apply_flip_kernel" in name and int(tab, 16) != 0, (name, tab)
        """, FAKE_DEVICES="0")


def test_noalloc_band_adaptive_needs_no_stage_derivatives(fake):
    """lme_evolve_noalloc under banded operators: the kernel stores no stage
    derivatives, so none of its scratch is asked for them (300 systems of 48
    states would need 77 MB of 64).  Kernels that store them are still refused."""
    run(fake, """
        w = [S.kerr_system(48, 0.3, 0.2, 0.4, 0.5)] * 300
        h = lme.Handle(w)
        rho = np.zeros(h.state_elems, complex)
        ex = np.zeros((300, 2, 2), complex)
        tl = np.array([0.0, 1.0])

        def noalloc(layout):
            o = lme.default_options(method=lme.LME_DOPRI5, layout=layout)
            return lib.lme_evolve_noalloc(h._h, C.byref(o), 2, tl.ctypes.data_as(lme._PD),
                                          rho.ctypes.data, None, ex.ctypes.data, None,
                                          rho.ctypes.data, None, None, None)
        assert noalloc(lme.LME_LAYOUT_ROW) == lme.LME_ENOTSUP and not launches()
        assert noalloc(lme.LME_LAYOUT_AUTO) == 0, lib.lme_last_error()
        assert "dp5_band_kernel" in launches()[-1][0]
        """)


@pytest.mark.parametrize("n_inst,method,N", [
    (8192, "LME_RK4", 5), (1024, "LME_RK4", 5), (1024, "LME_DOPRI5", 10), (512, "LME_DOPRI5", 10)])
def test_band_packs_rounds_over_the_cus(fake, n_inst, method, N):
    """Packs for the 256 CUs, but no second round over them where full packs
    take less (the last to end are split in two, for a few packs more)."""
    run(fake, f"""
        h = lme.Handle([S.jc_system({N})] * {n_inst})
        rho = np.zeros(h.state_elems, complex)
        ex = np.zeros(({n_inst}, 2, 2), complex)
        tl = np.array([0.0, 1.0])
        o = lme.default_options(method=lme.{method}, nsteps=10, hermitian=1)
        assert lib.lme_evolve(h._h, C.byref(o), 2, tl.ctypes.data_as(lme._PD), rho.ctypes.data, None,
                              ex.ctypes.data, None, rho.ctypes.data, None, None, None) == 0
        name, grid = launches()[-1][:2]
        assert "band_kernel" in name and 200 <= int(grid) <= 260, (name, grid)
        """)
