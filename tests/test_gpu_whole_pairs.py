"""Two steps per launch over the whole grid (launch parts 6 and 7) against
single steps, bitwise, at the sizes where its tiles can go wrong: strips of
60 columns, blocks of 12 rows, slabs of unequal and no width, source and port
planes at strip edges, the two-term ports' five component planes, and grids
large enough to take the tiles clear of the slabs in a launch of their own."""
import numpy as np
import pytest
import torch

from workloads import Plane

gpu = pytest.mark.gpu


def _plan(nx, ny, nz, npml, tb, device, src_x, port_x, two_term=False, steps=23, nf=1):
    from paper_2505_03352_amd.plan import FreqSpec, Plan
    grid = dict(nx=nx, ny=ny, nz=nz, dx=40e-9, dy=36e-9, dz=45e-9, courant=0.4, npml=npml, pml_kappa_max=1.5,
                pml_a_max=0.1)
    design = dict(i0=nx // 2, j0=ny // 2, md=1, nd=1, k_lo=nz // 2, k_hi=nz // 2, mc=1, nc=1, filter_r=1.0,
                  supersample=2, eps_core=12.11, eps_clad=2.085, sobel_delta=1e-6)
    y0, z0, n0, n1 = npml[2], npml[4], ny - npml[2] - npml[3], nz - npml[4] - npml[5]
    src, port = Plane(0, src_x, y0, z0, n0, n1), Plane(0, port_x, y0 + 1, z0, n0 - 1, n1)
    dt = 0.4 * 36e-9 / 299792458.0
    f = [FreqSpec(2 * np.pi / (19.0 + q) / dt, 5.0, steps - 5, 5 - q % 2) for q in range(nf)]
    return Plan(grid, design, steps, f, [src], [port], device=device, two_term=two_term, time_blocking=tb)


CASES = [
    # nx, ny, nz, npml, source x, port x, two-term, wavelengths
    (60, 24, 12, (5, 5, 4, 4, 3, 3), 6, 50, False, 1),
    (61, 25, 13, (5, 5, 4, 4, 3, 3), 7, 54, True, 1),
    (119, 37, 21, (8, 6, 3, 12, 0, 4), 58, 61, False, 1),
    (121, 36, 16, (0, 9, 0, 5, 2, 0), 59, 60, True, 1),
    (182, 62, 40, (10, 10, 10, 10, 8, 8), 60, 120, False, 1),
    (420, 330, 14, (6, 6, 6, 6, 4, 4), 40, 380, False, 16),
]


@pytest.mark.parametrize("nx,ny,nz,npml,sx,px,two,nf", CASES)
def test_whole_grid_tiles_own_every_cell_once(nx, ny, nz, npml, sx, px, two, nf):
    p = _plan(nx, ny, nz, npml, 2, "cpu", sx, px, two, nf=nf)
    p.set_tiling(4, 10, 512)
    cov = np.zeros((nz, ny, nx), np.int16)
    for part in (6, 7):
        for x0, x1, y0, y1, z0, z1, _ in p.tile_table(part):
            cov[z0:z1, y0:y1, x0:x1] += 1
    assert cov.min() == 1 and cov.max() == 1
    p.close()


@pytest.mark.parametrize("planes", ["y", "wide"])
def test_plans_the_whole_grid_kernel_cannot_take(planes):
    """A plane normal to y, or slabs of more rows than its LDS holds: no such
    tiles, and the pairs go through the two-step region as before."""
    from paper_2505_03352_amd.plan import FreqSpec, Plan
    npml = (6,) * 6 if planes == "y" else (6, 6, 13, 6, 6, 6)
    grid = dict(nx=150, ny=60, nz=40, dx=40e-9, dy=40e-9, dz=40e-9, courant=0.5, npml=npml)
    design = dict(i0=70, j0=30, md=4, nd=4, k_lo=18, k_hi=20, mc=2, nc=2, filter_r=1.0, supersample=2,
                  eps_core=12.11, eps_clad=2.085, sobel_delta=1e-6)
    pl = Plane(1, 20, 12, 11, 16, 12) if planes == "y" else Plane(0, 16, 14, 11, 16, 12)
    p = Plan(grid, design, 50, [FreqSpec(1e15, 0.0, 40, 8)], [pl], [], device="cpu", time_blocking=2)
    p.set_tiling(4, 10, 512)
    assert len(p.tile_table(6)) == len(p.tile_table(7)) == 0 and len(p.tile_table(2)) > 0
    p.close()


@gpu
@pytest.mark.parametrize("nx,ny,nz,npml,sx,px,two,nf", CASES)
def test_whole_grid_pairs_bitwise_equal_single_steps(nx, ny, nz, npml, sx, px, two, nf):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_03352_amd.plan import advance_many
    rng = np.random.default_rng(nx)
    kap = torch.as_tensor(1.0 / rng.uniform(2.0, 12.0, (3, nz, ny, nx)), dtype=torch.float32)
    out = {}
    for tb, fl in ((2, 0), (1, 0), (2, 512)):    # (2, 0): single steps
        print(f"[gpu] whole pairs {nx}x{ny}x{nz} tb={tb} flags={fl}", flush=True)
        p = _plan(nx, ny, nz, npml, tb, "cuda", sx, px, two, nf=nf)
        p.bind()
        p.set_background(kap, torch.zeros(p.canvas_shape))
        r = np.random.default_rng(3)
        for put, pl in ((lambda e, h: p.set_source_mode(0, h), p.src_planes[0]),
                        (lambda e, h: p.set_port_mode(0, e, h), p.port_planes[0])):
            e, h = (r.standard_normal((2, pl.n1, pl.n0)) + 1j * r.standard_normal((2, pl.n1, pl.n0))
                    for _ in range(2))
            put(e, h)
        p.set_tiling(4, 10, fl)
        p.reset(3)
        gen = torch.Generator(device="cuda").manual_seed(5)
        for q in range(p.n_rhs):
            p.set_fields(q, *(torch.randn(p.shape, generator=gen, device="cuda") for _ in range(2)))
        pairs = tb == 1 or fl == 512
        assert (len(p.tile_table(7)) > 0) == pairs
        assert (len(p.tile_table(6)) > 0) == (pairs and nf == 16)
        # graphs of pairs, plain pairs, and odd counts whose last step goes alone;
        # the run's last steps are in the DFT window
        advance_many([p], [3], 10, chunk=5, use_graph=True)
        advance_many([p], [3], 7, chunk=7, use_graph=False)
        some = range(0, p.n_rhs, max(1, p.n_rhs // 4))
        got = [x for q in some for x in p.get_fields(q)]
        advance_many([p], [3], 6, chunk=6, use_graph=True)
        p.finalize(3)
        got += [p.get_dft(q, region) for q in some for region in (0, 1)]
        out[tb, fl] = [x.cpu().numpy() for x in got]
        p.close()
    assert all(np.abs(a).max() > 0 for a in out[2, 0])
    for k in ((1, 0), (2, 512)):
        for a, b in zip(out[2, 0], out[k]):
            assert np.array_equal(a, b), k
