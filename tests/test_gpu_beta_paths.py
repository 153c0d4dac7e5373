"""The ways beta is solved, at the sizes where one takes over from another: one
block (p <= 16), substitution with few tiles (up to six 64-wide tiles), L^-1 and
two products from seven, substitution again beyond 24 (the updates in runs).
One sweep of a lone chain, and three more of which the last is compared, against
one float64 oracle sweep each from the chain's own state.  Bars: lambda, tau,
nu, xi are float64 from the same state (1e-10 leaves room for sums in another
order); a relative change of 1e-5 of X^T z (float32 sums), propagated through
Q^-1, bounds beta."""
import numpy as np
import pytest

from gpu_util import b_scale, dataset, need_gpu, random_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,p", [(700, 2), (1000, 3), (2000, 15), (5003, 16), (900, 17), (1501, 64), (1501, 65),
                                 (2003, 128), (2003, 193), (1700, 384), (1700, 385), (1900, 448), (2300, 1537),
                                 (2300, 2113)])
def test_one_sweep_matches_the_oracle(orc, N, p):
    torch, hsp = need_gpu()
    d = dataset(N, p, 900 + p)
    s = hsp.Sampler(torch.from_numpy(d.X).cuda(), torch.from_numpy(d.y).cuda(), seed=77, debug_store_z=True,
                    record_lambda=True)
    G = orc.gram(d.X)
    st = random_state(p, p, 0.2)
    s.set_state(**st, sweep=5)
    for n in (1, 3):
        s.sweep(n - 1)
        before = s.state()
        s.sweep(1)
        after = s.state()
        z, _, _ = s.debug()
        ch = orc.Chain(p)
        ch.beta, ch.lam_m2, ch.nu_m1 = before["beta"].copy(), before["lam_m2"].copy(), before["nu_m1"].copy()
        ch.tau_m2, ch.xi_m1, ch.sweep = before["tau_m2"], before["xi_m1"], before["sweep"]
        zo, _, _ = ch.sweep_once(d.X, d.y, G, seed=77, want_z=True)
        flips = int(np.sum(np.abs(z - zo) > 1e-3))
        assert flips <= max(1, N // 100000)
        for key in ("lam_m2", "nu_m1"):
            np.testing.assert_allclose(after[key], getattr(ch, key), rtol=1e-10)
        assert after["tau_m2"] == pytest.approx(ch.tau_m2, rel=1e-10)
        assert after["xi_m1"] == pytest.approx(ch.xi_m1, rel=1e-10)
        if flips == 0:
            Qi = np.abs(np.linalg.inv(G + ch.tau_m2 * np.diag(ch.lam_m2)))
            tol = Qi @ (1e-5 * b_scale(d.X, zo)) + 1e-10 * np.abs(ch.beta)
            assert np.all(np.abs(after["beta"] - ch.beta) <= tol)
    beta, tau, lam, n = s.draws()
    assert n == 4 and np.array_equal(beta[-1], after["beta"]) and np.array_equal(lam[-1], after["lam_m2"])
    assert tau[-1] == after["tau_m2"]
