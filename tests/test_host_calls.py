"""What the entry points ask of the HIP runtime, recorded on the CPU (see hip_calls.py)."""

import os
from types import SimpleNamespace

import pytest

from hip_calls import launches, record

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_04197_amd", "libdvbm.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libdvbm.so not built")


def test_adjoint_steps_only_launch():
    """On a new handle already the first adjoint step makes no runtime call besides its launches (header:
    dvbm_adjoint_step_noalloc, for callers that cannot allocate); a step asks about its kernel once."""
    cases = [dict(nx=64, ny=48, split=split, storage=st, dt=1e-5, bc_x=bx, bc_y=by)
             for split in (1, 2) for st in ("f64", "f32", "f32_dev")
             for bx in ("periodic", "zero_gradient") for by in ("periodic", "zero_gradient")]
    first = [["noalloc", "adjoint_f32", "adjoint"], ["adjoint_f32", "adjoint"], ["adjoint", "noalloc"]]
    scenarios = [dict(params=p, calls=first[k % 3] + ["step", "noalloc", "step", "step_from"]) for k, p in enumerate(cases)]
    scenarios += [dict(params=dict(nx=64, ny=48, split=2, storage=st, dt=1e-5, kernel=k, bc_y=by), calls=["step", "step"])
                  for st in ("f64", "fp16_dev") for k, by in (("auto", "wall"), ("cell", "wall"), ("sweep", "periodic"),
                                                              ("cell", "periodic"), ("tile", "periodic"))]
    for sc, (_, *logs) in zip(scenarios, record(scenarios)):
        done = set()
        for name, lines in zip(sc["calls"], logs):
            asked = [x for x in lines if not x.startswith("launch ")]
            assert launches(lines) and (not asked or (name == "step" and name not in done and len(asked) == 3)), (sc, name, lines)
            done.add(name)


@pytest.mark.parametrize("storage", ("f64", "f32"))
def test_adjoint_ranges_serve_both_cotangent_types(storage):
    """The adjoint's row ranges do not depend on which cotangent type is called first, nor on an answer of the runtime
    about one type's kernel (one workgroup per compute unit by its LDS); dvbm_init loads no kernel to ask."""
    params = dict(nx=256, ny=4096, split=2, storage=storage, dt=1e-5)
    runs = [dict(params=params, calls=c, workgroups_per_cu=w) for w in ([], [["k_adjoint", 2]], [["EfEEv", 2]])
            for c in (["adjoint", "adjoint_f32"], ["adjoint_f32", "adjoint"])]
    logs = record(runs)
    assert {x for run in logs for x in map(tuple, map(launches, run[1:]))} == {(("k_adjoint", 5 * 51),)}
    assert not any(line.startswith("hipOccupancy") for run in logs for line in run[0])


# workgroups a compute unit holds of the step kernels (256 compute units, as the recorder answers)
FITS = [["planes", 2], ["planesILi2ENS_8StoreF64E", 1]]


KERNELS = (  # the kernel AUTO launches
    # about the column sweep's lines, and the largest distributions
    (2, "f64", 900, 1000, "planes"), (2, "f64", 1024, 1024, "sweep"), (1, "f64", 4096, 4096, "planes"),
    (2, "f32", 900, 900, "planes"), (2, "f32_dev", 1000, 900, "planes"), (2, "f32", 2160, 402, "sweep"),
    (2, "f32", 1000, 920, "sweep"), (1, "f32_dev", 1400, 1000, "planes"), (1, "f32_dev", 1440, 1041, "sweep"),
    (1, "f32", 1440, 1041, "planes"), (1, "f32_dev", 1500, 1000, "planes"), (1, "f32", 1500, 1050, "sweep"), (2, "bf16_dev", 1024, 1024, "planes"), (2, "fp16_dev", 1200, 1000, "sweep"),
    (1, "bf16_dev", 2048, 2047, "planes"), (1, "fp16_dev", 2048, 2048, "sweep"), (2, "f32", 6528, 6528, ""),
    # narrow grids of 32-bit storage, with the sweep's groups of four strips full or not
    (2, "f32", 480, 1666, "sweep"), (2, "f32_dev", 192, 4096, "sweep"), (2, "f32", 72, 11000, "planes"),
    (1, "f32_dev", 480, 2145, "sweep"), (1, "f32", 192, 4096, "planes"), (1, "f32", 256, 4096, "planes"),
    # a second strip of at most four columns
    (2, "bf16_dev", 64, 4096, ""), (1, "fp16_dev", 61, 4096, ""), (2, "f32", 64, 11000, ""),
    (2, "bf16_dev", 61, 2000, ""), (2, "bf16_dev", 64, 2052, "planes"), (1, "bf16_dev", 64, 2048, "planes"),
    (2, "f32_dev", 64, 1024, ""), (2, "f32_dev", 64, 1025, "planes"), (1, "f32", 61, 2000, ""), (1, "f32", 64, 1000, "planes"),
    (2, "bf16_dev", 64, 1400, "planes"), (2, "bf16_dev", 60, 4096, "planes"), (2, "bf16_dev", 65, 4096, "planes"),
    (2, "f32", 64, 4096, "planes"), (1, "f32", 64, 11000, "planes"), (2, "f64", 64, 11000, "planes"))

GROUPS = (  # workgroups of the plane-group kernel
    (2, "f64", 64, 64, 2 * 64), (2, "f32", 256, 256, 5 * 51), (2, "f32", 512, 512, 9 * 56),  # one round
    (1, "bf16_dev", 15400, 16, 257 * 2), (2, "f64", 8000, 32, 134 * 3), (2, "f64", 8000, 16, 134),  # few ranges
    (1, "f64", 30000, 33, 500), (1, "f32", 1024, 1024, 18 * 28),  # one round of more than 32 rows
    (1, "f64", 1024, 1024, 18 * 85), (2, "bf16_dev", 25000, 40, 417 * 3), (2, "f64", 61500, 4, 1025),  # several rounds
)


@pytest.fixture(scope="module")
def first_steps():
    """The launches of a step, by (split, storage, nx, ny)."""
    grids = sorted({c[:4] for c in KERNELS + GROUPS})
    runs = [dict(params=dict(split=c[0], storage=c[1], nx=c[2], ny=c[3], dt=1e-5), calls=["step"], workgroups_per_cu=FITS)
            for c in grids]
    return {c: launches(logs[1]) for c, logs in zip(grids, record(runs))}


@pytest.mark.parametrize("case", KERNELS, ids=lambda c: "-".join(map(str, c)))
def test_auto_takes_the_kernel_that_is_faster(first_steps, case):
    assert [k for k, _ in first_steps[case[:4]]] == ["k_collide_advect" + ("_" + case[4] if case[4] else "")]


@pytest.mark.parametrize("case", KERNELS + GROUPS, ids=lambda c: "-".join(map(str, c)))
def test_bench_names_the_kernel_the_library_launches(first_steps, case):
    import bench
    split, storage, nx, ny = case[:4]
    assert [bench.launched_step_kernel(storage, SimpleNamespace(nx=nx, ny=ny), split)] == [k for k, _ in first_steps[case[:4]]]


@pytest.mark.parametrize("case", GROUPS, ids=lambda c: "-".join(map(str, c)))
def test_row_ranges_of_the_plane_groups(first_steps, case):
    assert first_steps[case[:4]] == [("k_collide_advect_planes", case[4])]


@pytest.mark.parametrize("call", ("adjoint", "adjoint_f32"))
def test_relaxation_part_of_the_deviation_adjoint(call):
    """Plane waves, one workgroup per 64 cells, up to 16384 cells; one thread per cell in at most 1024 blocks beyond."""
    grids = {(4, 5): ("k_adjoint_relax", 1), (128, 128): ("k_adjoint_relax", 256),
             (113, 145): ("k_adjoint_relax_cells", 65), (2048, 1024): ("k_adjoint_relax_cells", 1024)}
    runs = [dict(params=dict(split=2, storage="f32_dev", nx=nx, ny=ny, dt=1e-5), calls=[call]) for nx, ny in grids]
    for want, logs in zip(grids.values(), record(runs)):
        assert [launches(logs[1])[0], launches(logs[1])[1][0]] == [want, "k_adjoint_flux"]
