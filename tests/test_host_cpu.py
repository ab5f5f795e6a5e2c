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
