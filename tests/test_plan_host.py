"""The host side of the forwards, the fold and the backward on the CPU (no GPU): plan_check.cpp
compiles vpce_api.cpp with the kernels replaced by recorders, links the built library for the
tiles' sizes and times, and checks what 600 random problems would launch."""
import os
import shutil
import subprocess

import pytest

import paper_2609_14306_amd as vp
from tile_cases import BACKWARD, FORWARD, even

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CXX = shutil.which("g++")

pytestmark = [pytest.mark.skipif(CXX is None, reason="no g++"),
              pytest.mark.skipif(not os.path.exists(vp.LIB_PATH),
                                 reason="libvpce.so not built (run __graft_entry__.build())")]


@pytest.fixture(scope="module")
def plan_check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_check")
    subprocess.run([CXX, "-D__HIP_PLATFORM_AMD__", "-std=c++17", "-O1", "-Wall",
                    "-I", os.path.join(ROOT, "include"), "-I", "/opt/rocm/include",
                    os.path.join(HERE, "plan_check.cpp"), "-o", exe, vp.LIB_PATH,
                    "-L/opt/rocm/lib", "-lamdhip64",
                    f"-Wl,-rpath,/opt/rocm/lib:{os.path.dirname(vp.LIB_PATH)}"], check=True)
    return exe


def test_backward_plans_cover_the_problem(plan_check):
    out = subprocess.run([plan_check, "3"], stdout=subprocess.PIPE, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
    print(out.stdout)


def _plan(exe, dtype, T, d, rows, strip=0):
    out = subprocess.run([exe, "plan", "1" if dtype == "bf16" else "0", str(T), str(d), str(strip)] +
                         [str(r) for r in rows], stdout=subprocess.PIPE, text=True, check=True).stdout.split()
    p = {k: int(v) for k, v in zip(out[:16:2], out[1:16:2])}
    p["folds"] = [int(x) for x in out[17::2]]
    return p


@pytest.mark.parametrize("cls,dtype,T,d,rows,strip", BACKWARD)
def test_backward_case_runs_on_its_class(plan_check, cls, dtype, T, d, rows, strip):
    assert _plan(plan_check, dtype, T, d, rows[::-1], strip)["class"] == cls


@pytest.mark.parametrize("kind,folds,dtype,T,d,rows", FORWARD)
def test_forward_case_runs_on_its_kind(plan_check, kind, folds, dtype, T, d, rows):
    p = _plan(plan_check, dtype, T, d, rows)
    assert (p["kind"], p["folds"]) == (kind, folds)


# The splits a forward takes (the workspace's size tells only how many it has room for).
@pytest.mark.parametrize("dtype,T,d,rows,splits", [
    ("bf16", 512, 2880, [25136] * 8, 114),    # 792 tiles for two token blocks: seven turns
    ("bf16", 2304, 2880, [25136] * 8, 28),    # 9 blocks x 28 splits fill one round; 32 would start a second
    ("bf16", 4096, 2880, [25136] * 8, 16),
    ("bf16", 9000, 2880, [25136] * 8, 7),
    ("bf16", 12000, 2880, [25136] * 8, 5),
    ("bf16", 32768, 2880, [25136] * 8, 4),
    ("bf16", 33000, 4096, even(151936, 16), 4),   # three would save 11% of the turns: less than a fifth
    ("bf16", 65536, 4096, even(151936, 16), 4),
    ("bf16", 38494, 6912, even(142765, 16), 5),   # fewer turns outweigh the H panels' cache
    ("f32", 25549, 5696, even(25891, 16), 5),
    ("f32", 16384, 7168, [25000] * 8, 16),
])
def test_forward_splits(plan_check, dtype, T, d, rows, splits):
    assert _plan(plan_check, dtype, T, d, rows)["splits"] == splits
