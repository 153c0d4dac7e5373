"""beta for p <= 16 is computed to float64 accuracy.

Two beta steps with the same lambda, tau and noise s but different b: the noise
cancels, and what is left is Q (beta_1 - beta_2) = b_1 - b_2, up to rounding
(u = 2^-53), held against extended precision.

Q close to singular: factorisation and two triangular solves have |Q'- Q| <= (3 p + 1) u |U^T||U| for
each beta; Q's own diagonal, the sum of the two right-hand sides and the rounding
of beta add at most 7 u, and (|U^T||U|)_ij <= sqrt(Q_ii Q_jj).

Diagonal Q (columns that share no row): beta_j = b_j / q_j + s_j / sqrt(q_j) by a
few correctly rounded operations.  Rounding q_j, the square root and up to two
divisions by it move b_j / q_j by at most 3 u, the sum adds u / 2 of beta, and the
noise is the same number both times; a reciprocal square root from the hardware
estimate and one Newton step is off by up to 38 u."""
import numpy as np
import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


L = np.longdouble
U = 2.0 ** -53


def sampler(torch, hsp, X, rng):
    y = (rng.random(len(X)) < 0.5).astype(np.uint8)
    return hsp.Sampler(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), seed=11, debug_store_z=True)


def two_steps(hsp, s, lam, tau):
    """(b, beta) of two beta steps that differ in b alone."""
    out = []
    for start in (-0.5, 0.5):
        s.set_state(beta=np.full(len(lam), start), lam_m2=lam, nu_m1=np.ones(len(lam)), tau_m2=tau, xi_m1=1.0, sweep=4)
        s.step(hsp.HSP_STEP_Z)
        b = s.debug()[2]
        s.step(hsp.HSP_STEP_BETA)
        out += [b, s.state()["beta"]]
    return out


@pytest.mark.parametrize("p", [2, 3, 7, 15, 16])
@pytest.mark.parametrize("spread", [1.0, 1e-5])
def test_residual_of_the_solve(p, spread):
    torch, hsp = need_gpu()
    rng = np.random.default_rng(100 * p)
    N = 400
    X = (rng.standard_normal((N, 1)) + spread * rng.standard_normal((N, p))).astype(np.float32)
    s = sampler(torch, hsp, X, rng)
    lam, tau = rng.gamma(2.0, 1.0, p), 1e-9
    b1, x1, b2, x2 = two_steps(hsp, s, lam, tau)
    Q = s.gram().astype(L) + np.diag(L(tau) * lam.astype(L))
    s.close()
    res = np.abs(Q @ (x1.astype(L) - x2.astype(L)) - (b1.astype(L) - b2.astype(L)))
    d = np.sqrt(np.diag(Q))
    assert np.max(np.abs(b1 - b2)) > 1.0
    assert np.all(res <= (3 * p + 8) * U * d * np.sum(d * (np.abs(x1) + np.abs(x2))))


def test_diagonal_q():
    torch, hsp = need_gpu()
    rng = np.random.default_rng(3)
    p, rows = 16, 40
    X = np.zeros((p * rows, p), np.float32)
    for j in range(p):
        X[j * rows:(j + 1) * rows, j] = rng.standard_normal(rows)
    s = sampler(torch, hsp, X, rng)
    G = s.gram()
    assert np.count_nonzero(G - np.diag(np.diag(G))) == 0
    for _ in range(40):
        lam, tau = rng.gamma(2.0, 10.0, p), float(rng.gamma(2.0, 1.0))
        b1, x1, b2, x2 = two_steps(hsp, s, lam, tau)
        q = np.diag(G).astype(L) + L(tau) * lam.astype(L)
        err = np.abs((x1.astype(L) - x2.astype(L)) - (b1.astype(L) - b2.astype(L)) / q)
        assert np.all(err <= U * (3 * (np.abs(b1) + np.abs(b2)) / q + (np.abs(x1) + np.abs(x2))))
    s.close()


@pytest.mark.parametrize("p", [2, 5, 16])
def test_infinite_precision_pins_beta_to_zero(p):
    """tau^-2 lambda^-2 that overflows is an infinite pivot, not a failed one."""
    torch, hsp = need_gpu()
    rng = np.random.default_rng(p)
    s = sampler(torch, hsp, rng.standard_normal((300, p)).astype(np.float32), rng)
    s.set_state(beta=np.zeros(p), lam_m2=np.full(p, 1e300), nu_m1=np.ones(p), tau_m2=1e100, xi_m1=1.0, sweep=2)
    s.step(hsp.HSP_STEP_Z | hsp.HSP_STEP_BETA)
    s.sync()
    assert np.all(s.state()["beta"] == 0.0)
    s.close()
