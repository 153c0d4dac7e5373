"""A batched sweep's launches side by side (a captured graph) and one after
another (launched directly) draw the same, bit for bit: a batch with a
multi-chain pass beside packs of other chains, forced either way through the
autotuner's cache file.  Sweeps, states and draws alternate, so that the graph is
replayed with other work in between."""
import re

import numpy as np
import pytest

from gpu_util import dataset, need_gpu

pytestmark = pytest.mark.gpu

SETS = [((3001, 40, 71), "f32", 1), ((2500, 300, 72), "f32", 2), ((1800, 12, 73), "f32", 1), ((6000, 200, 74), "bf16", 5),
        ((900, 100, 75), "bf16", 1)]


@pytest.mark.parametrize("pre", [0, 8])
def test_graph_draws_what_direct_launches_draw(tmp_path, monkeypatch, pre):
    torch, hsp = need_gpu()
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("HSP_TUNE_CACHE", str(path))
    ds = [(dataset(*shape), xt) for shape, xt, _ in SETS]
    data = [(torch.from_numpy(d.X).cuda(), torch.from_numpy(d.y).cuda(), xt) for d, xt in ds]

    def run():
        b = hsp.Batch(data, [c for *_, c in SETS], seed=8, max_draws=32, autotune=True)
        out = []
        for n in (1, 3, 2, 5):
            b.sweep(n)
            out += [c.draws()[0] for c in b.chains] + [c.state()["lam_m2"] for c in b.chains]
        plan = b.plan()[3]
        b.close()
        return plan, out

    plan, _ = run()
    assert plan.endswith("(measured)")
    text = path.read_text()
    results = []
    for ov in (0, 1):
        path.write_text(re.sub(r"\bov=\d+", f"ov={ov}", re.sub(r"\bpre=\d+", f"pre={pre}", text)))
        plan, out = run()
        assert plan.endswith("(cache)") and f"ov={ov} " in plan and f"pre={pre} " in plan
        results.append(out)
    for x, y in zip(*results):
        assert np.array_equal(x, y)
