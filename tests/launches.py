"""The launches a run makes, recorded on the CPU: the library's host side in
a child process whose HIP calls are stand-ins (tests/hip_recorder.cpp)."""
import ctypes as C
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def record(tmp_path, runs):
    """runs: dicts with the workload generator's name and arguments
    ("workload", "args"), the replaced fields ("with"), problem overrides
    ("problem"), the step launches' step counts ("steps"), "drain" and
    "fail_at" (the launch that fails).  One dict of the statuses and of the
    launches [name, workgroups, threads, LDS bytes] per call for each."""
    lib = tmp_path / "librecorder.so"
    if not lib.exists():
        subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I/opt/rocm/include", "-o", str(lib),
                        os.path.join(ROOT, "tests", "hip_recorder.cpp"), "-ldl"], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), str(lib)], input=json.dumps(runs),
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    return json.loads(r.stdout.splitlines()[-1])


def _child(lib_path, runs):
    # before torch and the library: their HIP calls find these first
    rec = C.CDLL(lib_path, mode=C.RTLD_GLOBAL)
    rec.recorder_get.restype = C.c_char_p
    rec.recorder_get.argtypes = [C.c_int, C.POINTER(C.c_uint), C.POINTER(C.c_uint), C.POINTER(C.c_size_t)]
    sys.path.insert(0, ROOT)
    import numpy as np

    import workloads
    from paper_2409_07148_amd import restore as R
    lib = R._lib

    def taken():
        out = []
        for i in range(rec.recorder_count()):
            g, b, s = C.c_uint(), C.c_uint(), C.c_size_t()
            out.append([rec.recorder_get(i, C.byref(g), C.byref(b), C.byref(s)).decode(), g.value, b.value, s.value])
        return out

    results = []
    for run in runs:
        wl = getattr(workloads, run["workload"])(**run.get("args", {})).with_(**run.get("with", {}))
        p = R.problem_from_workload(wl, **run.get("problem", {}))
        n = R.restore_state_bytes(p.target, p.mu, p.local, p.cfg)
        buf = np.empty(n + 256, dtype=np.uint8)   # untouched pages take no memory
        ptr = (buf.ctypes.data + 255) // 256 * 256
        image = np.empty(1, dtype=np.float32)
        ctx = C.c_void_p()
        rec.recorder_reset(run.get("fail_at", -1))
        out = {"init": lib.restore_init(C.byref(ctx), C.byref(p.target), C.byref(p.mu), C.byref(p.local),
                                        C.byref(p.cfg), C.c_void_p(ptr), n, C.c_void_p(image.ctypes.data), None)}
        out["init_launches"] = taken()
        if out["init"] == 0:
            rec.recorder_reset(-1)
            out["step"] = [lib.restore_step(ctx, k, None) for k in run.get("steps", [])]
            out["step_launches"] = taken()
            rec.recorder_reset(-1)
            if run.get("drain"):
                out["drain"] = lib.restore_drain(ctx, None)
            out["drain_launches"] = taken()
            lib.restore_destroy(ctx)
        results.append(out)
    print(json.dumps(results))


if __name__ == "__main__":
    _child(sys.argv[1], json.loads(sys.stdin.read()))
