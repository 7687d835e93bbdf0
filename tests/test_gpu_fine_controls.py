"""The parametrization where controls are as many as sub-pixels and more (the
filter's x pass is then made per sub-pixel, not per control row), against the
FP64 oracle.  Tolerances as in test_gpu_parity's chain tests: kappa 1e-5 of its
largest value, the transpose 1e-4 relative L2."""
import numpy as np
import pytest
import torch

from oracle import chain
from workloads import configs

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_built")]


@pytest.mark.parametrize("extra", [0, 1, 37])
@pytest.mark.parametrize("md,nd,mc,r", [(6, 4, 3, 1.5), (3, 5, 90, 2.6)])
def test_fine_controls_match_oracle(md, nd, mc, r, extra):
    from paper_2505_03352_amd.plan import plan_for
    dev = configs.micro(n_steps=40, md=md, nd=nd, mc=4, nc=4)
    S = dev.supersample
    dev.mc, dev.nc, dev.filter_r = mc, S * nd + extra, r
    rng = np.random.default_rng(extra)
    dev.C = rng.uniform(0.0, 1.0, (dev.nc, dev.mc)).astype(np.float32).astype(np.float64)
    print(f"[gpu] {md}x{nd} pixels of {S}, controls {dev.mc}x{dev.nc} r={r}", flush=True)
    ops = chain.make_ops(dev)
    kref, st = chain.kappa(dev, ops=ops)
    p = plan_for(dev)
    kap = p.get_kappa().cpu().numpy()
    x0, y0, z0, bx, by, bz = dev.dft_box()
    g3 = rng.standard_normal((3, bz, by, bx))
    gC = p.chain_vjp(torch.as_tensor(g3, dtype=torch.float32)).cpu().numpy()
    p.close()
    gref = chain.vjp(dev, st, dev.beta, *chain.zsum(dev, g3), ops)
    assert np.abs(kap - kref).max() <= 1e-5 * np.abs(kref).max()
    assert np.linalg.norm(gC - gref) <= 1e-4 * np.linalg.norm(gref)
