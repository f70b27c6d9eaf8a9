"""What the entry points ask of the HIP runtime, recorded on the CPU (see hip_calls.py)."""

import os

import pytest

from hip_calls import launches, record

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_04197_amd", "libdvbm.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libdvbm.so not built")


def test_steps_and_adjoint_steps_only_launch():
    """On a new handle already the first step and the first adjoint step make no runtime call besides their launches
    (header: dvbm_adjoint_step_noalloc, for callers that cannot allocate, and steps inside a graph capture)."""
    cases = [dict(nx=64, ny=48, split=split, storage=st, dt=1e-5, bc_x=bx, bc_y=by)
             for split in (1, 2) for st in ("f64", "f32", "f32_dev", "bf16_dev")
             for bx in ("periodic", "zero_gradient") for by in ("periodic", "zero_gradient", "wall")]
    cases += [dict(nx=64, ny=48, split=2, storage=st, dt=1e-5, kernel=k, Pr=Pr)
              for st in ("f64", "f32", "fp16_dev") for k in ("sweep", "cell", "tile") for Pr in (0.5, 1.0, 2.0)]

    def calls(p):
        adjoint = p["storage"] in ("f64", "f32", "f32_dev") and p.get("bc_y") != "wall"
        return ["noalloc", "adjoint_f32", "adjoint", "step", "step_from"] if adjoint else ["step", "step_from"]

    scenarios = [dict(params=p, calls=calls(p)) for p in cases]
    for sc, (_, *logs) in zip(scenarios, record(scenarios)):
        for name, lines in zip(sc["calls"], logs):
            assert lines and all(x.startswith("launch ") for x in lines), (sc["params"], name, lines)


@pytest.mark.parametrize("storage,kern", (("f64", "k_adjoint"), ("f32", "k_adjoint"), ("f32_dev", "k_adjoint_relax")))
def test_adjoint_ranges_belong_to_the_cotangent_type(storage, kern):
    """Each cotangent type's kernel gets the row ranges of its own occupancy, whichever is called first."""
    params = dict(nx=256, ny=4096, split=2, storage=storage, dt=1e-5)
    two = [[f"{kern}I", 1]]
    one_f32 = two + [["EfEEv", 2]]  # the instance with float32 cotangents fits twice
    runs = [dict(params=params, calls=c, workgroups_per_cu=w) for w in (two, one_f32)
            for c in (["adjoint", "adjoint_f32"], ["adjoint_f32", "adjoint"])]

    def groups(run, logs):
        return {c: next(n for k, n in launches(lines) if k == kern) for c, lines in zip(run["calls"], logs[1:])}

    a, b, c, d = (groups(r, logs) for r, logs in zip(runs, record(runs)))
    assert a == b and c == d
    assert c["adjoint"] == a["adjoint"] and c["adjoint_f32"] > a["adjoint_f32"]
