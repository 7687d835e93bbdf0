"""The static workspace's limit does not move with the library's own layout: the
tallest grid of a cross-section that it admits, next to 32 MiB.  (Without a device
an admitted plan gets as far as asking for one.)"""
import ctypes as ct

import pytest

from paper_2505_03352_amd import _abi
from paper_2505_03352_amd.plan import FreqSpec, Plan
from workloads import Plane


def _status(nx, ny, nz, w, n_src, n_ports, n_freq, tb, two_term, **controls):
    grid = dict(nx=nx, ny=ny, nz=nz, dx=1e-8, dy=1e-8, dz=1e-8, courant=0.4, npml=(w, w, w, w, 0, 0))
    design = dict(i0=nx // 2, j0=ny // 2, md=2, nd=2, k_lo=nz // 2, k_hi=nz // 2, mc=5, nc=4, filter_r=1.5,
                  supersample=4, eps_core=12.0, eps_clad=2.0, sobel_delta=1e-6)
    design.update(controls)
    f = [FreqSpec(1e15 * (1 + 0.01 * q), 1.0, 1, 5) for q in range(n_freq)]
    pl = [Plane(0, nx // 2 - 3, w, 0, ny - 2 * w, nz)] * (n_src + n_ports)
    p = Plan(grid, design, 8, f, pl[:n_src], pl[n_src:], device="cpu", two_term=two_term, time_blocking=tb)
    st = _abi.lib().yo_bind_static_workspace(p.handle, ct.c_void_p())
    p.close()
    return st


@pytest.mark.parametrize("nz,case", [
    (123, (61, 30, 5, 1, 1, 1, 1, False)),       # strips of 64 floats, half of them pads
    (123, (30, 40, 4, 1, 1, 1, 2, False)),
    (66, (90, 20, 0, 1, 2, 1, 2, True)),
    (65, (56, 56, 8, 1, 1, 1, 1, False)),
    (30, (24, 60, 6, 2, 2, 2, 1, True)),
])
def test_tallest_grid_admitted(nz, case):
    nx, ny, rest = case[0], case[1], case[2:]
    assert _status(nx, ny, nz, *rest) != _abi.YO_EWORKSPACE
    assert _status(nx, ny, nz + 1, *rest) == _abi.YO_EWORKSPACE


def test_controls_finer_than_sub_pixels_need_no_rows_of_their_own():
    """400 sub-pixel columns of 30000 control rows would be 48 MB of filtered rows,
    900 of them 108 MB; sixteen sub-pixel rows read a few of them."""
    for md in (100, 225):
        assert _status(240, 12, 8, 0, 1, 1, 1, 1, False, i0=5, j0=4, md=md, nd=4, mc=1, nc=30000) != _abi.YO_EWORKSPACE
