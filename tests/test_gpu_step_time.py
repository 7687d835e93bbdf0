"""The tuner's ms_per_step is what a step of a solve takes, not what the split
it chose takes in launches by tile class, and it sets no flag without effect."""
import pytest
import torch

from workloads import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tb", [1, 2])
def test_tuner_reports_the_step_of_a_solve(tb, tmp_path, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_03352_amd import autotune
    from paper_2505_03352_amd.plan import advance_many, plan_for
    monkeypatch.setenv("YEEOPT_AUTOTUNE_CACHE", str(tmp_path / "autotune.json"))
    dev = configs.micro(n_steps=2000, nx=150, ny=100, nz=80)
    p = plan_for(dev, time_blocking=tb)
    print(f"[gpu] tuner's step time tb={tb}", flush=True)
    rec = autotune.tune(p, 3, shared=[(10, 0)], pair_shared=[(10, 128)])
    assert not rec["flags"] & 1024
    advance_many([p], [3], 400, chunk=400, use_graph=False)
    e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    e0.record()
    advance_many([p], [3], 800, chunk=800, use_graph=False)
    e1.record()
    e1.synchronize()
    step = e0.elapsed_time(e1) / 800
    print(f"[gpu] step {step:.4f} ms, reported {rec['ms_per_step']:.4f}", flush=True)
    # the launches alone against whole steps: apart by the gaps between them
    assert 0.6 * step < rec["ms_per_step"] < 1.4 * step
    assert min(t["split_ms"] for t in rec["timings"].values()) == pytest.approx(rec["split_ms"], abs=1e-4)
    p.close()

    # a record without the split's own time is one that reported it as the step's
    key = autotune.shape_key(p, 3)
    d = autotune._load()
    assert key in d
    del d[key]["split_ms"]
    autotune._store(d)
    q = plan_for(dev, time_blocking=tb)
    assert not autotune.tune(q, 3, shared=[(10, 0)], pair_shared=[(10, 128)])["cached"]
    assert autotune.tune(q, 3)["cached"]
    q.close()
