"""Plan creation when device memory runs short, on a stand-in for the HIP runtime (hip_stub.cpp): the A(k) factors are
allocated once, in the tiles' layout where the plan has tiles; where that finds no room the plan is made for the streaming
kernels, and only where theirs finds none either is it refused."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RUN = """
import ctypes, sys
from paper_2206_09878_amd import lmvd
from paper_2206_09878_amd.workloads import workload
w = workload("small", n=32, n2=65)
L, h, cfg = lmvd.library(), ctypes.c_void_p(), lmvd.make_config(w)
st = L.lmvd_plan_create(ctypes.byref(cfg), ctypes.byref(h))
print("status", st)
if st == 0:
    a = lmvd.SubstepArgs()
    a.stage, a.kf, a.guess_mode = 0, 1, 1
    for i, (name, _) in enumerate(lmvd.SubstepArgs._fields_):
        if name not in ("stage", "kf", "guess_mode", "z_hist", "md", "mc"):
            setattr(a, name, (1 << 40) + 4096 * i)
    print("substep", L.lmvd_substep(h, ctypes.byref(a), ctypes.c_void_p(1 << 44), None))
    print("adjoint", L.lmvd_mc_adjoint(h, 4096, 8192, 12288, 16384, ctypes.c_void_p(1 << 44), None))
    print("check", L.lmvd_factor_check(h, 1e4, None, None, None))
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "libstub.so")
    subprocess.run(["g++", "-O1", "-fPIC", "-shared", "-I/opt/rocm/include", "-o", so,
                    os.path.join(ROOT, "tests", "hip_stub.cpp")], check=True, capture_output=True)
    return so


@pytest.mark.parametrize("fail", [0, 1, 2])
def test_factors_find_room_or_stream(stub, tmp_path, fail):
    log = str(tmp_path / "log")
    once = 8 * 16 * 16 * 66 * 9  # 16 x 16 pairs, 66 rows of 9 entries
    env = dict(os.environ, HIP_STUB_LOG=log, HIP_STUB_FAIL=str(fail), HIP_STUB_LARGE=str(once // 2),
               LD_PRELOAD=" ".join([stub] + os.environ.get("LD_PRELOAD", "").split()))
    r = subprocess.run([sys.executable, "-c", RUN], cwd=ROOT, env=env, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    out = dict(line.split() for line in r.stdout.splitlines() if line)
    with open(log) as f:
        lines = [x.split(maxsplit=1) for x in f.read().splitlines()]
    large = [what for what, _ in lines if what in ("large", "refused")]
    assert large == ["refused"] * fail + ["large"] * (fail < 2)
    assert out["status"] == ("0" if fail < 2 else "-2")
    if fail == 2:
        return
    assert out["substep"] == out["adjoint"] == out["check"] == "0"
    tiles = [x for what, x in lines if what == "launch" and "_tile" in x]
    streaming = [x for what, x in lines if what == "launch" and any(k in x for k in ("4k_mcI", "10k_prologue", "6k_projI", "6k_mc_t"))]
    assert (bool(tiles), bool(streaming)) == ((True, False) if fail == 0 else (False, True)), (tiles, streaming)
