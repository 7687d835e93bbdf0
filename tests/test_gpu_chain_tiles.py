"""The tiled disc sums, the filter's transposed weights and the grey count at
the sizes where they can go wrong, through the C ABI against the FP64 oracle:
canvases of exactly one tile, one row or column over and ragged; discs of one
tap, of rows too short for the shared reads, of fractional radius and of the
largest radius the library takes; controls coarser than the pixels.

Tolerances as in test_gpu_morph: kappa 5e-5 of its largest value, the
transpose 1e-4 relative L2 (sums of up to 3209 FP32 terms of one sign err by
at most about sqrt(3209) 2^-24 = 3.4e-6, then the chain's own factors); the
grey fraction by one sub-pixel per thousand."""
import numpy as np
import pytest
import torch

from oracle import chain
from oracle import optimize as O
from workloads import configs

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_built")]


@pytest.mark.parametrize("md,nd,mc,nc,ops,d", [
    (12, 12, 12, 12, "ed", 0.4),     # 64 x 64 canvas, one tap
    (12, 13, 5, 13, "de", 0.5),      # five taps, rows of one and three
    (13, 11, 13, 4, "ed", 0.75),     # 68 x 60, radius 1.5
    (16, 16, 7, 9, "e", 2.3),
    (13, 16, 13, 16, "de", 16.0),    # the largest disc, wider than the design's margin
])
def test_chain_matches_oracle_at_tile_edges(md, nd, mc, nc, ops, d):
    from paper_2505_03352_amd.plan import plan_for
    dev = configs.micro(n_steps=40, nx=40, ny=40, md=md, nd=nd, mc=mc, nc=nc, filter_r=1.5)
    dev.morph_ops, dev.morph_d, dev.morph_alpha = ops, d, 20.0
    print(f"[gpu] chain {md}x{nd} controls {mc}x{nc} {ops} d={d}", flush=True)
    o = chain.make_ops(dev)
    kref, st = chain.kappa(dev, ops=o)
    p = plan_for(dev)
    kap = p.get_kappa().cpu().numpy()
    x0, y0, z0, bx, by, bz = dev.dft_box()
    g3 = np.random.default_rng(1).standard_normal((3, bz, by, bx))
    gC = p.chain_vjp(torch.as_tensor(g3, dtype=torch.float32)).cpu().numpy()
    u = float(p.unbinarity()[0])
    p.close()
    gref = chain.vjp(dev, st, dev.beta, *chain.zsum(dev, g3), o)
    assert np.abs(kap - kref).max() <= 5e-5 * np.abs(kref).max()
    assert np.linalg.norm(gC - gref) <= 1e-4 * np.linalg.norm(gref)
    assert abs(u - O.unbinarity(O.design_rho(dev, st))) < 1e-3
