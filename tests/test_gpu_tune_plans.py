"""The autotuner times the plan that a state has anyway, so that it cannot end
with a slower one: also for short passes over wide rows and beyond p = 4096,
whose built-in unit (one tile) is none that it would try by itself."""
import pytest

from gpu_util import dataset, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,p,xt", [(2000, 10, "f32"), (30000, 100, "f32"), (3000, 1700, "f32"), (2500, 1200, "bf16"),
                                    (1500, 4200, "bf16")])
def test_the_states_own_plan_is_timed_first(N, p, xt):
    torch, hsp = need_gpu()
    d = dataset(N, p, p)
    s = hsp.Sampler(torch.from_numpy(d.X).cuda(), torch.from_numpy(d.y).cuda(), seed=2, x_type=xt)
    plans = hsp.hsp_tune_candidates(s.h)
    gp, _, pct, unit, _ = s.plan()
    assert plans[0] == (gp, pct, unit)
    assert len(plans) == len(set(plans)) > 1
    assert s.plan()[:4] == (gp, s.plan()[1], pct, unit)
    s.close()
