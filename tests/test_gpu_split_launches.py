"""The launches by tile class, which step a plan whose single-step launches are
timed, against the whole-grid launches of the same steps, bitwise."""
import numpy as np
import pytest
import torch

from workloads import Plane

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu_available():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_03352_amd import _abi
    _abi.lib()


GRIDS = {
    "wide": (187, 43, 35, (6, 6, 5, 7, 4, 6)),      # strips of 60, 60, 60 and 7
    "cut": (66, 31, 23, (5, 3, 4, 0, 0, 5)),        # a strip cut at the slabs, faces without layers
}


def _plan(name, tb, tiling):
    from paper_2505_03352_amd.plan import FreqSpec, Plan
    nx, ny, nz, npml = GRIDS[name]
    grid = dict(nx=nx, ny=ny, nz=nz, dx=40e-9, dy=36e-9, dz=45e-9, courant=0.4, npml=npml, pml_kappa_max=1.5,
                pml_a_max=0.1)
    design = dict(i0=nx // 2, j0=ny // 2, md=1, nd=1, k_lo=nz // 2, k_hi=nz // 2, mc=1, nc=1, filter_r=1.0,
                  supersample=2, eps_core=12.11, eps_clad=2.085, sobel_delta=1e-6)
    dt = 0.4 * 36e-9 / 299792458.0
    planes = [Plane(0, i, npml[2] + 1, npml[4] + 1, ny - npml[2] - npml[3] - 2, nz - npml[4] - npml[5] - 3)
              for i in (npml[0] + 2, nx - npml[1] - 4)]
    p = Plan(grid, design, 40, [FreqSpec(2 * np.pi / 19.0 / dt, 5.0, 35, 5)], planes[:1], planes[1:], device="cuda",
             time_blocking=tb)
    p.bind()
    rng = np.random.default_rng(2)
    kap = 1.0 / rng.uniform(2.0, 12.0, p.shape)
    kap[:, 2::3] = kap[:, 2::3, :1, :1]
    p.set_background(torch.as_tensor(kap, dtype=torch.float32), torch.zeros(p.canvas_shape))
    e, h = (rng.standard_normal((2, planes[0].n1, planes[0].n0)) + 1j * rng.standard_normal((2, planes[0].n1, planes[0].n0))
            for _ in range(2))
    p.set_source_mode(0, h)
    p.set_port_mode(0, e, h)
    p.set_tiling(*tiling)
    p.reset(3)
    gen = torch.Generator(device="cuda").manual_seed(3)
    for q in range(p.n_rhs):
        p.set_fields(q, *(torch.randn(p.shape, generator=gen, device="cuda") for _ in range(2)))
    return p


def _fields(p):
    return [x.cpu().numpy() for q in range(p.n_rhs) for x in p.get_fields(q)]


_whole = {}


def whole_grid(name):
    if name not in _whole:
        p = _plan(name, 1, (4, 16, 0))
        p.advance(3, 13)
        _whole[name] = _fields(p)
        p.close()
        assert all(np.abs(x).max() > 0 for x in _whole[name])
    return _whole[name]


def _check(name, tb, tiling, part):
    print(f"[gpu] split launches {name} tb={tb} tiling={tiling} timed part {part}", flush=True)
    p = _plan(name, tb, tiling)
    p.set_timing(part, 100)
    p.advance(3, 7)
    p.advance(3, 6)
    got = _fields(p)
    ms, n = p.timing(part)
    assert n == (13 if len(p.tile_table(part)) else 0) and (ms > 0) == (n > 0)
    p.close()
    for a, b in zip(got, whole_grid(name)):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("part", [0, 1])
@pytest.mark.parametrize("name", sorted(GRIDS))
@pytest.mark.parametrize("flags", [512, 512 | 128, 512 | 256 | 1 | 64, 512 | 2048 | 128 | 8, 512 | 8192 | 4096 | 2])
def test_single_step_launches_are_timed_in_plans_that_ask_for_pairs(name, flags, part):
    _check(name, 2, (4, 10, flags), part)


# every interior choice (16 cooperative, 32 no prefetch) and shell choice (4
# cooperative, 8 code by class, 64 no prefetch, 16384 six rows) with the cuts
# along x (1, 128, 256), waves per block (2) and chunk lengths from 4 to 63
VARIANTS = [(16, 0), (8, 1), (4, 2), (48, 3), (16, 4), (16, 13), (8, 70), (4, 23), (16, 45), (8, 122), (16, 77), (8, 53),
            (16, 16384 | 73), (10, 16384 | 2), (16, 128), (16, 201), (8, 178), (16, 129), (4, 232), (16, 329), (16, 456),
            (8, 256), (16, 304), (63, 256 | 16 | 2), (5, 256 | 48 | 4 | 8), (7, 16 | 32 | 4 | 64 | 2), (10, 4 | 8 | 64),
            (10, 8 | 64), (16, 16384 | 8), (8, 16384 | 64 | 2), (4, 16384 | 8 | 64 | 1)]


@pytest.mark.parametrize("tb", [1, 2])
@pytest.mark.parametrize("zc,flags", VARIANTS)
@pytest.mark.parametrize("name", sorted(GRIDS))
def test_every_single_step_variant_gives_the_whole_grid_fields(name, zc, flags, tb):
    _check(name, tb, (4, zc, flags), 1)


def _buffers(p):
    """The state buffers of right-hand side 0 as the library lays them out:
    [buffer][strip of 60 cells: 64 floats of each of 6 components], rows of
    planes of ny + 1 from row -1 on."""
    nx, ny, nz = (p.grid[k] for k in ("nx", "ny", "nz"))
    ns = -(-nx // 60)
    rows = nz * (ny + 1) + 1
    off = (-p.workspace.data_ptr()) % 256
    raw = p.workspace[off:off + 3 * rows * ns * 6 * 64 * 4].view(torch.float32).cpu().numpy()
    raw = raw.reshape(3, rows, ns, 6, 64)[:, 1:].reshape(3, nz, ny + 1, ns, 6, 64)[:, :, :ny, :, :, 2:62]
    return raw.transpose(0, 4, 1, 2, 3, 5).reshape(3, 6, nz, ny, ns * 60)[..., :nx]


@pytest.mark.parametrize("start", [3, 4])
@pytest.mark.parametrize("zc,flags", [(16, 512), (5, 512 | 2), (10, 512 | 4096), (8, 512 | 8192 | 2),
                                      (10, 512 | 8192 | 4096), (10, 512 | 2048 | 128), (4, 512 | 2048 | 128 | 2)])
@pytest.mark.parametrize("name", sorted(GRIDS))
def test_two_step_launches_of_the_regions_write_the_state_two_steps_on(name, zc, flags, start):
    """Launch parts 2 and 4 (timed, not stepped): each of their cells in the
    buffer two steps on, and the two-step region's outermost layer in the next."""
    print(f"[gpu] two-step region {name} tiling=(4,{zc},{flags}) after step {start}", flush=True)
    p = _plan(name, 2, (4, zc, flags))
    p.advance(3, start)
    parts = [q for q in (2, 4) if len(p.tile_table(q))]
    assert 2 in parts
    for q in parts:
        assert p.time_kernel(q, 1)[0] > 0
    torch.cuda.synchronize()
    got = _buffers(p)
    want = {}
    for n in (1, 2):
        p.advance(3, 1)
        want[n] = torch.cat(p.get_fields(0)).cpu().numpy()
    tiles = {q: p.tile_table(q) for q in parts}
    p.close()
    lo = [tiles[2][:, 2 * a].min() for a in range(3)]
    hi = [tiles[2][:, 2 * a + 1].max() for a in range(3)]
    for q in parts:
        for x0, x1, y0, y1, z0, z1, _ in tiles[q]:
            box = np.s_[:, z0:z1, y0:y1, x0:x1]
            assert np.array_equal(got[(start + 2) % 3][box], want[2][box])
    box = np.s_[:, lo[2]:hi[2], lo[1]:hi[1], lo[0]:hi[0]]
    rim = np.ones([hi[a] - lo[a] for a in (2, 1, 0)], bool)
    rim[1:-1, 1:-1, 1:-1] = False
    assert np.array_equal(got[(start + 1) % 3][box][:, rim], want[1][box][:, rim])
