"""Plan creation with a filter as wide as its controls stays linear in the
filter's taps."""
import time


def test_plan_creation_with_a_wide_filter():
    from paper_2505_03352_amd.plan import FreqSpec, Plan
    from workloads import Plane
    grid = dict(nx=420, ny=420, nz=8, dx=4e-8, dy=4e-8, dz=4e-8, courant=0.4, npml=(0,) * 6)
    design = dict(i0=8, j0=8, md=400, nd=400, k_lo=3, k_hi=4, mc=600, nc=600, filter_r=300.0, supersample=10,
                  eps_core=12.0, eps_clad=2.0, sobel_delta=1e-6)
    best = 1e9
    for _ in range(2):
        t = time.perf_counter()
        Plan(grid, design, 10, [FreqSpec(1e15, 1.0, 1, 5)], [Plane(0, 4, 0, 0, 420, 8)], [], device="cpu").close()
        best = min(best, time.perf_counter() - t)
    # 2 x 4000 sub-pixels of 600 taps: 0.15 s; every control against every tap of
    # its sub-pixels was 2.6 s
    print(f"plan creation {best:.3f} s")
    assert best < 1.2
