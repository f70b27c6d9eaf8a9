"""The HIP runtime calls of the library's entry points, recorded without a GPU.

``record(scenarios)`` runs each scenario in one child process in which ``hip_recorder.c`` stands in for the HIP runtime
(the process must not have loaded the library before): a dict with the ``params`` of ``make_params``, the ``calls`` to
make on a new handle and optionally ``workgroups_per_cu``, a list of [text, count] that answers the occupancy query of
kernels whose mangled name contains the text.  Returns, per scenario, the recorded lines of dvbm_init and of each call."""

import ctypes
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))


def record(scenarios):
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "hip_recorder.so")
        subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", so, os.path.join(HERE, "hip_recorder.c"), "-ldl"], check=True)
        r = subprocess.run([sys.executable, os.path.abspath(__file__), so], input=json.dumps(scenarios),
                           capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout.strip().splitlines()[-1])


def launches(lines):
    """(kernel name, workgroups) of the recorded launches of the library's own kernels."""
    out = []
    for line in lines:
        if line.startswith("launch _ZN4dvbm"):
            _, name, blocks, _ = line.split()
            name = name[len("_ZN4dvbm"):]
            digits = len(name) - len(name.lstrip("0123456789"))
            out.append((name[digits:digits + int(name[:digits])], int(blocks)))
    return out


def main(so):
    rec = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)  # before the library: its HIP symbols resolve here
    rec.recorder_log.restype = ctypes.c_char_p
    sys.path.insert(0, os.path.dirname(HERE))
    from paper_2510_04197_amd import dvbm

    lib = dvbm.load_library()
    at = [ctypes.c_void_p(4096 * k) for k in range(1, 6)]  # addresses that nothing dereferences

    def lines():
        out = rec.recorder_log().decode().splitlines()
        rec.recorder_clear()
        return out

    results = []
    for sc in json.loads(sys.stdin.read()):
        rec.recorder_forget_workgroups()
        for text, count in sc.get("workgroups_per_cu", []):
            rec.recorder_set_workgroups(text.encode(), int(count))
        p = dvbm.make_params(**sc["params"])
        h = ctypes.c_void_p()
        rec.recorder_clear()
        dvbm._check(lib.dvbm_init(ctypes.byref(p), at[0], at[0], at[0], at[0], at[0], at[1], at[2], None, ctypes.byref(h)))
        calls = {"step": lambda: lib.dvbm_step(h, 1),
                 "step_from": lambda: lib.dvbm_step_from(h, at[0], at[1]),
                 "adjoint": lambda: lib.dvbm_adjoint_step(h, at[0], at[3], at[4], at[2], at[1]),
                 "adjoint_f32": lambda: lib.dvbm_adjoint_step_f32(h, at[0], at[3], at[4], at[2], at[1]),
                 "noalloc": lambda: lib.dvbm_adjoint_step_noalloc(h, at[0], at[3], at[4], at[2])}
        out = [lines()]
        for c in sc["calls"]:
            dvbm._check(calls[c]())
            out.append(lines())
        lib.dvbm_destroy(h)
        results.append(out)
    print(json.dumps(results), flush=True)


if __name__ == "__main__":
    main(sys.argv[1])
