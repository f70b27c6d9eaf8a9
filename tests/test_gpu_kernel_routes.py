"""Step kernels on the routes and shapes where nothing else compares them: walls on the per-cell kernel, one range of
rows between two walls, and both distributions of the 16-bit plane groups value by value."""

import pytest
import torch

from oracle import dvbm_oracle as O
from paper_2510_04197_amd import velocity_set
from synth import smooth_random
from test_gpu_parity import oracle_cfg, oracle_state, rel, solver

pytestmark = pytest.mark.gpu

WALLS = dict(bc_y="wall", wall_T=(0.95, 1.1), wall_ux=(0.0, 0.3))
# half a unit in the last place, relative to the value (normal numbers)
HALF_ULP = {"bf16_dev": 2.0 ** -8, "fp16_dev": 2.0 ** -11}


def stored16(x, storage):
    """float64 values rounded once to the storage format (a cast of torch's rounds to float32 on the way)."""
    bits, emin = (7, -126) if storage == "bf16_dev" else (10, -14)
    ulp = torch.ldexp(torch.ones_like(x), (torch.frexp(x).exponent - 1).clamp(min=emin) - bits)
    return torch.round(x / ulp) * ulp


def check_steps(s, p, storage, n):
    """n steps against the oracle; relative L2 over each distribution (the tolerances of the wall tests)."""
    cfg = oracle_cfg(p)
    f0, g0 = oracle_state(s)
    s.step(n)
    f, g = oracle_state(s)
    s.close()
    fo, go = O.run(f0, g0, cfg, p.dt, n)
    tol, tol_inc = (1e-12, 1e-9) if storage == "f64" else (1e-5, 1e-3)
    assert rel(f, fo) < tol and rel(g, go) < tol
    assert rel(f - f0, fo - f0) < tol_inc and rel(g - g0, go - g0) < tol_inc


def check_stored(s, p, storage, monkeypatch):
    """One step in 16-bit deviations: every stored deviation of f and g within its rounding of the oracle's, plus 4e-6
    for the float32 arithmetic (its terms are at most about 12 per weight, each rounded a few times by 2^-24).  A
    wall's ghost rows are held in the storage format, so the oracle's are rounded to it too."""
    T = torch.bfloat16 if storage == "bf16_dev" else torch.float16
    cfg = oracle_cfg(p)
    split, nx, ny, Q = p.split, p.nx, p.ny, s.Q
    v, w = (torch.tensor(a) for a in velocity_set(split))
    w = w.view(1, Q, 1, 1)
    Cv = 1.0 / (p.gamma - 1.0)
    rest = torch.stack([torch.ones(Q, dtype=torch.float64),
                        Cv + 0.5 * ((v * v).sum(1) - 2.0) if split == 1 else torch.full((Q,), Cv - 1.0, dtype=torch.float64)])
    rest = rest.view(2, Q, 1, 1)
    ghosts = O.wall_ghosts

    def stored_ghosts(f, g, c):
        return tuple(tuple(w[0] * (rest[d] + stored16(X / w[0] - rest[d], storage)) for X in rows)
                     for d, rows in enumerate(ghosts(f, g, c)))

    monkeypatch.setattr(O, "wall_ghosts", stored_ghosts)
    X0 = s.store_populations().cpu()
    s.step(1)
    got = s.state_buffer.view(T).view(2, ny, Q, (nx + 63) // 64 * 64)[..., :nx].permute(0, 2, 1, 3).cpu().double()
    s.close()
    want = torch.stack(O.step(X0[0], X0[1], cfg, p.dt)) / w - rest
    excess = (got - want).abs() - HALF_ULP[storage] * want.abs() - 4e-6
    assert torch.isfinite(got).all()
    for d in range(2):
        worst = excess[d].max(-1).values.max(0).values  # by row
        assert float(worst.max()) <= 0.0, (d, int(worst.argmax()), float(worst.max()))
    moved = (want - (X0 / w - rest)).abs().amax((1, 2, 3))
    assert float(moved.min()) > 100 * 4e-6  # a distribution left as it was would fail


def make(nx, ny, **kw):
    wl = smooth_random(nx, ny, seed=37, amp_T=0.05)
    s, p = solver(wl, tau_ref=0.02, cfl=0.1, **kw)
    p.dt = s.dt
    return s, p


@pytest.mark.parametrize("split", (1, 2))
@pytest.mark.parametrize("Pr", (0.5, 1.0, 2.0))
@pytest.mark.parametrize("bc_x", ("periodic", "zero_gradient"))
@pytest.mark.parametrize("storage", ("f64", "f32", "f32_dev"))
def test_walls_on_the_per_cell_kernel(split, Pr, bc_x, storage):
    # ghost rows formed by their own kernel: a ragged block in both directions
    s, p = make(11, 9, split=split, storage=storage, Pr=Pr, bc_x=bc_x, kernel="cell", **WALLS)
    check_steps(s, p, storage, 6)


@pytest.mark.parametrize("split", (1, 2))
@pytest.mark.parametrize("storage", ("bf16_dev", "fp16_dev"))
def test_walls_on_the_per_cell_kernel_16bit(monkeypatch, split, storage):
    s, p = make(70, 13, split=split, storage=storage, Pr=0.6, kernel="cell", **WALLS)
    check_stored(s, p, storage, monkeypatch)


@pytest.mark.parametrize("split", (1, 2))
@pytest.mark.parametrize("ny", (4, 5, 9))
@pytest.mark.parametrize("storage", ("f64", "f32_dev"))
def test_one_range_between_two_walls(split, ny, storage):
    # more strips (1025) than workgroups run at a time: a range takes whole columns and forms the ghost rows of both
    s, p = make(61500, ny, split=split, storage=storage, Pr=0.6, **WALLS)
    check_steps(s, p, storage, 2)


@pytest.mark.parametrize("nx,ny", ((4, 4), (59, 5), (64, 9), (61, 40), (121, 13), (130, 2051), (20, 9000), (61500, 4)))
@pytest.mark.parametrize("bc", ("periodic", "zero_gradient", "wall"))
@pytest.mark.parametrize("split", (1, 2))
@pytest.mark.parametrize("storage", ("bf16_dev", "fp16_dev"))
def test_plane_groups_16bit_value_by_value(monkeypatch, nx, ny, bc, split, storage):
    kw = WALLS if bc == "wall" else dict(bc_x=bc, bc_y=bc)
    s, p = make(nx, ny, split=split, storage=storage, Pr=0.6, **kw)
    check_stored(s, p, storage, monkeypatch)


@pytest.mark.parametrize("storage", ("f64", "f32", "f32_dev"))
def test_first_adjoint_call_of_a_handle_without_a_work_array(storage):
    # each call on a handle of its own: nothing is left for the first adjoint step to set up
    out = []
    for entry in ("adjoint_step_noalloc", "adjoint_step"):
        s, _ = make(117, 17, split=2, storage=storage, Pr=0.71)
        lam1 = torch.randn((2, s.Q, 17, 117), dtype=torch.float64, generator=torch.Generator().manual_seed(4)).cuda()
        lam, d = s.new_cotangent(), torch.zeros(2, dtype=torch.float64, device="cuda")
        getattr(s, entry)(s.state_buffer, lam1, lam, d)
        torch.cuda.synchronize()
        s.close()
        out.append((lam.cpu(), d.cpu()))
    assert float(out[0][0].abs().max()) > 0 and float(out[0][1].abs().min()) > 0
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


def test_walls_above_2_GiB_of_a_distribution():
    """6528 x 6528 between walls in float32 deviations, 3.97 GiB a distribution: the plane groups (AUTO) against the
    per-cell kernel, every stored deviation.  Both round the same terms (at most about 12 per weight, a few roundings of
    2^-24 each), in another order."""
    out = []
    for kernel in ("auto", "cell"):
        s, p = make(6528, 6528, split=2, storage="f32_dev", Pr=0.6, kernel=kernel, **WALLS)
        before = s.state_buffer.view(torch.float32).clone()
        s.step(1)
        out.append(s.state_buffer.view(torch.float32).clone())
        s.close()
        del s
    worst = moved = 0.0
    for a, b, x in zip(*(t.split(1 << 28) for t in (*out, before))):
        worst = max(worst, float((a - b).abs().max()))
        moved = max(moved, float((a - x).abs().max()))
    assert moved > 1e-2 and worst <= 2 * 4e-6
    torch.cuda.empty_cache()
