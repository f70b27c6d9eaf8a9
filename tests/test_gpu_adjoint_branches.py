"""Every cell of the adjoint step in the float32 storages, whose states meet the limiter's kinks.

Neighbours of a float32 state are often stored equal, exactly on the kink a b = 0 of the limiter, where the oracle's
reverse mode takes a subgradient of its own.  The reference here is reverse mode through the oracle's step with face
values whose branch follows the stored values: the derivative is zero at a b = 0, and equal arguments take the first
of beta |a|, |a + b| / 2, beta |b|.  Float32 values (whose differences are exact in the adjoint's float64) are compared
everywhere.  Of float32 deviations the derivative at a kink rests on how the decoded neighbours were rounded, so the
cells that a face at a kink reads are left out there.  The arithmetic is float64 on both sides: the tolerances are
those of the float64 adjoint tests (1e-11 relative L2, 1e-10 for the parameters)."""

import numpy as np
import pytest
import torch

from oracle import dvbm_oracle as O
from paper_2510_04197_amd import Solver, make_params, velocity_set
from synth import smooth_random
from test_gpu_adjoint import check_step_adjoint, oracle_cfg, rel

pytestmark = pytest.mark.gpu
DEV = "cuda"


def branch_faces(stored):
    """Face values of the oracle with the limiter's branch chosen on stored values: ``stored`` lists triples of a
    population tensor, the values its branches follow, and a mask that collects the cells read by faces at a kink."""

    def faces(X, vel, axis, bc, beta, ghosts=None):
        D, kinked = next((d, m) for x, d, m in stored if x is X)
        n = X.shape[axis]
        k = torch.arange(n + 1)
        cell = [O.neighbour(n, k + off, bc) for off in (-2, -1, 0, 1)]

        def face(c, u, m, mine):  # upwind cell c, the one behind it u, the one across the face m
            at = lambda A, j: A.index_select(axis, cell[j])  # noqa: E731
            a, b = at(X, c) - at(X, u), at(X, m) - at(X, c)
            da, db = at(D, c) - at(D, u), at(D, m) - at(D, c)
            t1, t2, t3 = beta * da.abs(), 0.5 * (da + db).abs(), beta * db.abs()
            inc = torch.where((t1 <= t2) & (t1 <= t3), 0.5 * beta * a, torch.where(t2 <= t3, 0.25 * (a + b), 0.5 * beta * b))
            # (copies of an edge cell hand their shares back to it, whatever the derivative at their kink)
            own = [(cell[j] != cell[c]).reshape((-1,) + (1,) * (X.dim() - 1 - axis)) for j in (u, m)]
            kink = (((da == 0) & own[0]) | ((db == 0) & own[1])) & mine
            for j in (c, u, m):
                kinked.index_add_(axis, cell[j], kink.float())
            return at(X, c) + torch.where(da * db > 0, inc, torch.zeros_like(inc))

        shape = (-1,) + (1,) * (X.dim() - 1)
        up, down = (vel > 1e-12).reshape(shape), (vel < -1e-12).reshape(shape)
        return torch.where((vel >= 0).reshape(shape), face(1, 0, 2, up), face(2, 3, 1, down))

    return faces


def step_adjoint_on_stored(monkeypatch, nx, ny, split, bc, storage, grain=0.0, Pr=0.71, seed=21):
    """lam0, its reference, the cells that faces at a kink read (all [2, Q, ny, nx]), the parameter derivatives and the
    reference's, of one adjoint step at a perturbed state.  ``grain`` > 0 rounds the stored values to multiples of it,
    per weight, which makes many neighbours equal."""
    print(f"[adjoint branches] {nx}x{ny} split={split} Pr={Pr} bc={bc} {storage} grain={grain}", flush=True)
    wl = smooth_random(nx, ny, seed=seed)
    p = make_params(nx, ny, dx=wl.dx, dy=wl.dy, split=split, storage=storage, Pr=Pr, tau_ref=0.02, bc_x=bc[0],
                    bc_y=bc[1], dt=3e-3, R=1.1, T_ref=0.9, gamma=1.3)
    s = Solver(p, wl.rho, wl.ux, wl.uy, wl.T, device=DEV)
    cfg = oracle_cfg(p)
    Q, pitch = s.Q, (nx + 63) // 64 * 64
    rng = np.random.default_rng(1)

    def buffer():  # stored values [2, Q, ny, nx], a view of the state
        return s.state_buffer.view(torch.float32).view(2, ny, Q, pitch)[..., :nx].permute(0, 2, 1, 3)

    X = torch.stack(O.initial_state(wl.rho, wl.ux, wl.uy, wl.T, cfg))
    s.load_populations(X * (1 + 0.01 * torch.tensor(rng.standard_normal(tuple(X.shape)))))
    if grain > 0:
        unit = grain * torch.tensor(velocity_set(split)[1], device=DEV).float().view(1, Q, 1, 1)
        buffer().copy_((buffer() / unit).round() * unit)
    X = s.store_populations().cpu()
    D = buffer().cpu().double()
    lam1 = torch.tensor(rng.standard_normal(tuple(X.shape)))
    lam0 = s.new_cotangent()
    dpar = torch.zeros(2, dtype=torch.float64, device=DEV)
    s.adjoint_step(s.state_buffer, lam1.to(DEV), lam0, dpar)
    torch.cuda.synchronize()
    s.close()
    fr, gr = (X[d].clone().requires_grad_() for d in range(2))
    tau, prt = (torch.tensor(v, dtype=torch.float64, requires_grad=True) for v in (0.02, Pr))
    kinked = torch.zeros(X.shape)
    monkeypatch.setattr(O, "face_values", branch_faces([(fr, D[0], kinked[0]), (gr, D[1], kinked[1])]))
    fn, gn = O.step(fr, gr, cfg, 3e-3, tau, prt)
    ((lam1[0] * fn).sum() + (lam1[1] * gn).sum()).backward()
    return (lam0.cpu(), torch.stack([fr.grad, gr.grad]), kinked > 0, dpar.tolist(), (float(tau.grad), float(prt.grad)))


OPEN = ("zero_gradient", "zero_gradient")
PERIODIC = ("periodic", "periodic")


@pytest.mark.parametrize("split", (1, 2))
@pytest.mark.parametrize("nx,ny,bc,grain", ((131, 127, PERIODIC, 0.0), (70, 13, PERIODIC, 2.0 ** -9),
                                            (61, 23, OPEN, 2.0 ** -6), (59, 6, OPEN, 0.0), (60, 4, PERIODIC, 0.0),
                                            (63, 7, OPEN, 0.0), (64, 300, PERIODIC, 0.0), (121, 40, OPEN, 0.0),
                                            (20, 3000, OPEN, 0.0), (61500, 4, PERIODIC, 0.0)))
def test_adjoint_of_float32_values_on_every_cell(monkeypatch, split, nx, ny, bc, grain):
    # states of coarse values (many faces at a kink); strips of 60 columns with one owned column or none to spare,
    # the one-wrap width of 64, one row per range, unequal ranges, 1025 strips (two launches)
    lam0, ref, _, got, want = step_adjoint_on_stored(monkeypatch, nx, ny, split, bc, "f32", grain)
    check_step_adjoint((rel(lam0, ref), got, want))


@pytest.mark.parametrize("split", (1, 2))
@pytest.mark.parametrize("nx,ny,bc", ((131, 127, PERIODIC), (61, 23, OPEN), (333, 250, ("zero_gradient", "periodic")),
                                      (128, 128, PERIODIC), (113, 145, OPEN)))
def test_adjoint_of_float32_deviations_away_from_kinks(monkeypatch, split, nx, ny, bc):
    # the relaxation part by plane waves (up to 16384 cells) and by one thread per cell
    lam0, ref, kinked, got, want = step_adjoint_on_stored(monkeypatch, nx, ny, split, bc, "f32_dev")
    assert float(kinked.float().mean()) < 0.01
    ok = ~kinked
    check_step_adjoint((rel(lam0[ok], ref[ok]), got, want))
