"""Runs steps of models in a process whose HIP runtime is launch_recorder.cpp and prints the launches as JSON.

argv: the recorder, then a JSON list of models: workloads.Workload's fields, and for raw vectors d_raw.  Started
by launches.py."""
import ctypes
import json
import os
import sys

import numpy as np

rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # before the library: its HIP calls bind here
rec.recorded_at.restype = ctypes.c_char_p
sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import workloads  # noqa: E402
from paper_2509_03110_amd import lsam  # noqa: E402

FAKE = 1 << 40          # device addresses: handed around, never read
out = []
for model in json.loads(sys.argv[2]):
    model = {k: tuple(v) if isinstance(v, list) else v for k, v in model.items()}
    w = workloads.Workload("recorded", **model)
    cfg, keep = lsam.config_from_workload(w)
    need = lsam.lsam_workspace_bytes(cfg)
    assert need > 0, lsam.last_error()
    init = np.zeros(w.d, dtype=np.float32)
    h = ctypes.c_void_p()
    L = lsam.lib()
    rc = L.lsam_init(ctypes.byref(cfg), init.ctypes.data, init.size, FAKE, need, None, ctypes.byref(h))
    assert rc == 0, lsam.last_error()
    rec.recorded_clear()
    if w.dims:
        rc = L.lsam_step(h, 2 * FAKE, 3 * FAKE, None)
    else:
        rc = L.lsam_step_grads(h, 2 * FAKE, 3 * FAKE)
    got = []
    v = (ctypes.c_uint64 * 8)()
    for i in range(rec.recorded_count()):
        name = rec.recorded_at(i, v).decode()
        got.append(dict(name=name, grid=list(v[0:3]), block=list(v[3:6]), lds=v[6], limit=v[7]))
    out.append(dict(rc=rc, error=lsam.last_error() if rc else "", launches=got))
    L.lsam_destroy(h)
print(json.dumps(out))
