"""The implicit stage by its residuals.  Past 64 radial points the forward
error against the oracle grows with the operators' condition numbers, and its
bar with it; the residuals of the equations, relative to the sizes of their
terms row by row, do not.  For sampled modes the state and pressure put into the
equations in extended precision (operators from the FP64 weights on the context's
own grid):

  H+- X+- = f+- - (D1 p -+ (m/r) p), H X_z = f_z - i kappa p, P p = div f on the
  inner rows, H_T T = f_T, and div X = 0 at the walls.

Bar: eight times what the oracle's own solution leaves, pivoted dense LU in
FP64 (the largest over the step sizes; in units of 2^-52 of the terms 1 for the
temperature, 2 to 200 for the others, where p0 and X0 cancel against the
influence responses), and at least 8 units.  On the host the same equations by
elimination without pivoting leave 0.3 to 3.1 times as much, so eight is three
bits past the method's own rounding or less."""
import sys

import numpy as np
import pytest
import torch

import oracle as O
from synthetic import direction

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52
DTS = (1e-3, 1e-4, 1e-5)
C = 0.5


def _ld(a):
    a = a.numpy()
    return a.astype(np.clongdouble if np.iscomplexobj(a) else np.longdouble)


def _residuals(p, r, modes, u, nn, nq, dt, X, P):
    """Largest residual over scale of each equation, over the modes."""
    D1, D2 = (_ld(d) for d in O.fd_matrices(p, r))
    r = _ld(r)
    n, c, idt = p.N_r, np.longdouble(C), 1 / np.longdouble(dt)
    base, eye, inner, ab = D2 + D1 / r[:, None], np.eye(n), slice(1, n - 1), np.abs
    worst = {}

    def keep(name, res, scale, rows):
        worst[name] = max(worst.get(name, 0.0), float((ab(res) / scale)[rows].max()))

    for b, (m, kk) in enumerate(modes):
        kap = np.longdouble(kk - p.K) * np.longdouble(p.kz)
        L = {q: base - np.diag(np.longdouble(q * q) / r ** 2 + kap * kap) for q in (m + 1, m - 1, m)}
        field = lambda a, f: _ld(a[f, :, b])
        comb = lambda a: (field(a, 0) + 1j * field(a, 1), field(a, 0) - 1j * field(a, 1), field(a, 2))

        def right(A, x, a, bq):
            return (idt * x + (1 - c) * (A @ x) + c * bq + (1 - c) * a,
                    idt * ab(x) + (1 - c) * (ab(A) @ ab(x)) + c * ab(bq) + (1 - c) * ab(a))

        x = comb(X)
        pr = _ld(P[:, b])
        f, fs = zip(*(right(L[q], *v) for q, v in zip((m + 1, m - 1, m), zip(comb(u), comb(nn), comb(nq)))))
        dp, mr = D1 @ pr, m * pr / r
        grad = (dp - mr, dp + mr, 1j * kap * pr)
        gs = (ab(D1) @ ab(pr) + ab(mr),) * 2 + (ab(kap * pr),)
        for name, q, xx, ff, fsc, g, gsc in zip("+-z", (m + 1, m - 1, m), x, f, fs, grad, gs):
            H = idt * eye - c * L[q]
            keep(name, H @ xx - (ff - g), ab(H) @ ab(xx) + fsc + gsc, inner)

        def div(a, D, up, down, ik):
            return 0.5 * (D @ a[0] + up / r * a[0] + D @ a[1] + down / r * a[1]) + ik * a[2]

        one, size = (D1, 1 + m, 1 - m, 1j * kap), (ab(D1), 1 + m, ab(1 - m), ab(kap))
        keep("p", L[m] @ pr - div(f, *one), ab(L[m]) @ ab(pr) + div(fs, *size), inner)
        keep("wall", div(x, *one), div([ab(v) for v in x], *size), [0, -1])
        if p.heated:
            A = L[m] / np.longdouble(p.Pr)
            H = idt * eye - c * A
            ff, fsc = right(A, field(u, 3), field(nn, 3), field(nq, 3))
            T = field(X, 3)
            keep("T", H @ T - ff, ab(H) @ ab(T) + fsc, inner)
    return worst


@pytest.mark.parametrize("N_r", [9, 16, 17, 33, 64, 65, 96, 97, 127, 128, 130, 144, 159, 160])
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_stage_residuals(N_r, Ra):
    print("stage residuals", N_r, Ra, flush=True)
    sys.stdout.flush()
    import paper_1908_00587_amd as nsc
    grid = (N_r, 6, 11)
    args = (0.6, 80.0, 10.0, Ra, 0.7) + grid + (4.0,)
    p = O.Params(*args)
    u = O.base_state(p) + 1e-2 * direction(p.F, *grid, 31)
    nn, nq = 10 * direction(p.F, *grid, 32), 10 * direction(p.F, *grid, 33)
    K = p.K
    modes = [(1, K), (1, 0), (2, K + 3), (3, K - 1), (5, 0), (5, 10)]
    m, kk = (torch.tensor(v) for v in zip(*modes))
    at = [a[:, :, m, kk] for a in (u, nn, nq)]
    ctx = nsc.Context(*args)
    got, ref = {}, {}
    for dt in DTS:
        ctx.set_timestep(dt=dt, c=C)
        x, pr = (t.cpu() for t in ctx.radial_solve(u.cuda(), nn.cuda(), nq.cuda(), pressure=True))
        assert float(x[:3, [0, -1]][:, :, m, kk].abs().max()) == 0.0  # no slip
        X, P = O.radial_solve_modes(p, m, kk, *at, dt, C)
        for out, a, b in ((got, x[:, :, m, kk], pr[:, m, kk]), (ref, X, P)):
            for k, v in _residuals(p, ctx.grid(), modes, *at, dt, a, b).items():
                out[k] = max(out.get(k, 0.0), v / EPS)
    print("  " + ", ".join(f"{k} {got[k]:.1f} ({ref[k]:.1f})" for k in got), flush=True)
    for k in got:
        assert got[k] < max(8.0, 8.0 * ref[k]), k
