"""Which kernels a call enqueues on which stream, and which of them use the plan's tally: the library's
host code on a recording stand-in for the HIP runtime."""
import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_03644_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_routes_of_every_call(tmp_path):
    def compile_host(src):
        name = os.path.splitext(os.path.basename(src))[0]
        obj = str(tmp_path / (name + ".o"))
        # the host side alone
        cmd = ["hipcc", "-std=c++17", "-O1", "-w", "-fPIC", "-I", CSRC, "-x", "hip",
               "--offload-host-only", "-c", "-o", obj]
        subprocess.run(cmd + [src], check=True, capture_output=True, text=True)
        return obj

    srcs = [os.path.join(CSRC, s) for s in ("api.hip", "kernels.hip", "blocks.hip", "fused.hip", "layout.cpp")]
    srcs.append(os.path.join(ROOT, "tests", "native", "routes_check.cpp"))
    with ThreadPoolExecutor(len(srcs)) as ex:
        objs = list(ex.map(compile_host, srcs))
    # the device images that the objects would be registered with are absent
    undefined = subprocess.run(["nm", "--undefined-only"] + objs, check=True, capture_output=True, text=True).stdout
    images = sorted({w for w in undefined.split() if w.startswith("__hip_fatbin")})
    exe = str(tmp_path / "routes_check")
    subprocess.run([shutil.which("g++") or "c++", "-o", exe] + objs + ["-Wl,--defsym=%s=0" % i for i in images],
                   check=True, capture_output=True, text=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout + run.stderr
    assert run.stdout.strip().endswith("ok")
