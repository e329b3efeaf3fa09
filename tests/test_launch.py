"""The launches of the kernel sources, recorded on the CPU (tests/host_launch.cpp):
shapes and the kernels' allowance of dynamic LDS, which is process-wide and
has to serve launches of several threads."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2006_09616_amd", "csrc")
LDS = 160 * 1024
FIELDS = ["kernel", "grid", "block", "lds", "allowed"]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not shutil.which("hipcc"):
        pytest.skip("no hipcc")
    tmp = tmp_path_factory.mktemp("launch")
    objs = []
    for src in (os.path.join(CSRC, "replay.hip"), os.path.join(CSRC, "replay_log.hip"), os.path.join(HERE, "host_launch.cpp")):
        objs.append(str(tmp / (os.path.basename(src) + ".o")))
        hip = ["--offload-arch=gfx950", "--cuda-host-only"] if src.endswith(".hip") else ["-x", "c++", "-D__HIP_PLATFORM_AMD__"]
        res = subprocess.run(["hipcc", "-std=c++17", "-O1", "-fPIC", *hip, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                              "-I", "/opt/rocm/include", "-c", src, "-o", objs[-1]], capture_output=True, text=True)
        assert res.returncode == 0, res.stderr[-3000:]
    names = subprocess.run(["nm", "-u", *objs[:2]], capture_output=True, text=True).stdout.split()
    images = [f"-Wl,--defsym,{n}=0" for n in names if n.startswith("__hip_fatbin")]
    so = tmp / "liblaunch.so"
    res = subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", *images, "-o", str(so), *objs], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    return C.CDLL(str(so))


def _row(out):
    return dict(zip(FIELDS, out))


def test_log_launches_agree_on_the_lds_allowance(lib):
    """Any two log plans in turn, as two threads would interleave: the kernel's
    allowance is the same for both and holds the larger."""
    seen, out = set(), (C.c_int64 * len(FIELDS))()
    for lds in (163840, 40000, 100000, 65536, 16, 65552, 163840, 1000):
        for waves in (1, 2, 4):
            assert lib.launch_log(7, waves, lds, out) == 0
            r = _row(out)
            assert (r["grid"], r["block"], r["lds"]) == (7, 64 * waves, lds)
            seen.add((r["kernel"], r["allowed"]))
    assert seen == {(r["kernel"], LDS)}
    assert lib.launch_log(7, 1, 0, out) == 0 and _row(out)["lds"] == 0 and _row(out)["kernel"] != r["kernel"]


def test_trace_launches_agree_on_the_lds_allowance(lib):
    """Every group's kernels: one kernel per group and form, launched with the
    plan's LDS, whose allowance is what their static LDS leaves."""
    out, fixed, kernels = (C.c_int64 * len(FIELDS))(), C.c_int64(0), {}
    for group in range(8):
        for small in (0, 2, 604, 2048):
            if group % 4 == 1 and small:
                continue                                  # lane walks have no small form
            for chunks in (1, 2, 19, 32) if group % 4 == 2 else (0,):
                for waves in (1, 2, 4) if group % 4 in (1, 2) else (1,):
                    assert lib.launch_group(group, 9, waves, chunks, small, out, C.byref(fixed)) == 0
                    r = _row(out)
                    assert r["grid"] == (3 if group == 0 else 9) and r["block"] == 64 * (4 if group == 0 else waves)
                    assert r["lds"] <= r["allowed"] and r["allowed"] + fixed.value in (LDS, 65536 + fixed.value)
                    assert (r["lds"] == 0) == (small == 0 and group % 4 != 2)
                    kernels.setdefault((group, small > 0), set()).add((r["kernel"], r["allowed"] if r["lds"] else 0))
    assert all(len(v) == 1 for v in kernels.values()) and len(set.union(*kernels.values())) == len(kernels) == 14
