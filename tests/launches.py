"""Which kernels a step launches, found without a GPU: the library's host code runs against a recorder in
place of the HIP runtime (launch_recorder.cpp)."""
import functools
import json
import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
_dir = tempfile.TemporaryDirectory(prefix="lsam_recorder")


@functools.lru_cache(None)
def _recorder():
    so = os.path.join(_dir.name, "recorder.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "launch_recorder.cpp")],
                   check=True)
    return so


def _plain(name):
    """gemm_bf16_kernel<float,128,...> of a mangled name."""
    full = subprocess.run(["c++filt", name.replace("DF16b", "u6__bf16")], capture_output=True, text=True, check=True).stdout.strip()
    full = re.sub(r"\(anonymous namespace\)::|lsam::|^void ", "", full)
    return re.sub(r"\([^()]*\)$", "", full).replace(" ", "")


_plain = functools.lru_cache(None)(_plain)


def record(*models):
    """For each model (workloads.Workload's fields) the launches of one step, in one process and in this order:
    [{rc, error, launches: [{name, grid, block, lds, limit}]}]."""
    r = subprocess.run([sys.executable, os.path.join(HERE, "launch_recorder_driver.py"), _recorder(), json.dumps(models)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    out = json.loads(r.stdout.strip().splitlines()[-1])
    for m in out:
        for l in m["launches"]:
            l["name"] = _plain(l["name"])
    return out


def names(model):
    r = record(model)[0]
    assert r["rc"] == 0, r["error"]
    return [l["name"] for l in r["launches"]]
