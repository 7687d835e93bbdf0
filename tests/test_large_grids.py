"""Grids at the interface's own limits: what it admits is taken, and stepped as
a short grid of the same cross-section is."""
import numpy as np
import pytest
import torch

from workloads import Plane


def _plan(nx, ny, nz, npml, device="cpu", steps=40, tb=1):
    from paper_2505_03352_amd.plan import FreqSpec, Plan
    grid = dict(nx=nx, ny=ny, nz=nz, dx=40e-9, dy=40e-9, dz=40e-9, courant=0.5, npml=npml, pml_kappa_max=1.5,
                pml_a_max=0.1)
    design = dict(i0=nx // 2, j0=ny // 2, md=1, nd=1, k_lo=nz // 2, k_hi=nz // 2, mc=1, nc=1, filter_r=1.0,
                  supersample=2, eps_core=12.11, eps_clad=2.085, sobel_delta=1e-6)
    f = FreqSpec(2 * np.pi / 31.0 / (0.5 * 40e-9 / 299792458.0), 5.0, steps - 5, 5)
    pl = Plane(2, nz // 2, npml[0], npml[2], nx - npml[0] - npml[1], ny - npml[2] - npml[3])
    return Plan(grid, design, steps, [f], [pl], [], device=device, time_blocking=tb)


# y-slabs of most of a grid whose rows fill half of a strip: under 2 GiB of CPML
# memories as the interface counts them, over 4 GiB in strips
WIDE_SLABS = (30, 84, 32400, (0, 0, 34, 34, 0, 0))


@pytest.mark.parametrize("nx,ny,nz,npml", [WIDE_SLABS, (62, 84, 16200, (0, 0, 34, 34, 0, 0)),
                                           (22, 1300, 2000, (8, 8, 0, 0, 0, 0))])
@pytest.mark.parametrize("tb", [1, 2])
def test_cpml_memories_below_the_stated_limit_are_taken(nx, ny, nz, npml, tb):
    rowp = (nx + 2 + 31) // 32 * 32
    w = [npml[2 * a] + npml[2 * a + 1] for a in range(3)]
    counted = 4 * 6 * tb * (nz * ny * w[0] + nz * w[1] * rowp + w[2] * ny * rowp)
    assert 24 * rowp * (ny + 2) * (nz + 2) < 2**31
    if counted < 2**31:
        _plan(nx, ny, nz, npml, tb=tb).close()
        return
    from paper_2505_03352_amd import _abi
    with pytest.raises(_abi.YeeOptError) as e:
        _plan(nx, ny, nz, npml, tb=tb)
    assert e.value.status == _abi.YO_EUNSUPPORTED


# planes past 2^15, in strips of both kinds of tile (with and without slabs in x
# and y) and in one that is narrower
TALL = [(64, 8, 40000, (0, 0, 0, 0, 5, 5)), (20, 30, 33000, (3, 3, 4, 4, 0, 6))]


@pytest.mark.parametrize("nx,ny,nz,npml", TALL)
@pytest.mark.parametrize("tb,flags", [(1, 0), (2, 512), (2, 512 | 2048 | 128)])
def test_tiles_of_a_tall_grid_own_every_cell_once(nx, ny, nz, npml, tb, flags):
    p = _plan(nx, ny, nz, npml, tb=tb)
    p.set_tiling(4, 40, flags)
    for parts in ((0, 1), (2, 3, 4, 5), (6, 7)):
        t = np.concatenate([p.tile_table(q) for q in parts])
        if parts[0] == 2 and not len(p.tile_table(2)):
            continue
        cov = np.zeros((nz, ny, nx), np.int8)
        for x0, x1, y0, y1, z0, z1, _ in t:
            cov[z0:z1, y0:y1, x0:x1] += 1
        assert cov.min() == 1 and cov.max() == 1, parts
    p.close()


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny,nz,npml", [WIDE_SLABS] + TALL)
def test_a_tall_grid_steps_as_a_short_one(nx, ny, nz, npml):
    """Random fields in the lowest or highest 60 planes, bitwise those of a grid
    of 120 planes after 16 steps (which carry them 32 planes at most)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gen = torch.Generator(device="cuda").manual_seed(7)
    block = [torch.randn((3, 60, ny, nx), generator=gen, device="cuda") for _ in range(2)]
    for top in (False, True):
        out = []
        for z in (nz, 120):
            print(f"[gpu] {nx}x{ny}x{z} npml {npml} top={top}", flush=True)
            p = _plan(nx, ny, z, npml, "cuda")
            p.bind()
            p.set_background(torch.full(p.shape, 0.25, device="cuda"), torch.zeros(p.canvas_shape))
            at = slice(z - 60, z) if top else slice(0, 60)
            full = []
            for b in block:
                full.append(torch.zeros(p.shape, device="cuda"))
                full[-1][:, at] = b
            p.reset(1)
            p.set_fields(0, *full)
            del full
            p.advance(1, 10)
            p.advance(1, 5)
            p.advance(1, 1)
            at = slice(z - 100, z) if top else slice(0, 100)
            out.append([x[:, at].cpu().numpy() for x in p.get_fields(0)])
            p.close()
            del p
            torch.cuda.empty_cache()
        assert np.abs(out[0][0]).max() > 0
        for a, b in zip(*out):
            assert np.array_equal(a, b)
