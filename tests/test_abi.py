"""Host-side checks of the C-ABI library (no GPU compute calls)."""
import ctypes as C
import os
import re

import numpy as np
import pytest

from paper_2403_15768_amd import lbm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_functions():
    src = open(os.path.join(ROOT, "include", "lbm.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(lbm_[a-z_]+)\s*\(", src)))


def test_library_exports_every_declared_symbol():
    lib = lbm.load()
    names = header_functions()
    assert len(names) >= 20
    for n in names:
        assert hasattr(lib, n), n
    assert sorted(lbm.EXPORTS) == names


def test_footprint_host_logic():
    p = lbm.make_params(lbm.D3Q19, lbm.DUCT, 256, 128, 64, tau=0.7, precision="f32")
    nb = lbm.footprint(p)
    pops = 2 * 19 * 256 * 128 * 64 * 4
    assert pops <= nb < pops * 1.05
    p64 = lbm.make_params(lbm.D3Q19, lbm.DUCT, 256, 128, 64, tau=0.7, precision="f64")
    assert lbm.footprint(p64) > 1.9 * nb
    # x-lines up to 128 cells stored back to back; longer ones padded to
    # whole 128-byte lines (nx = 200 -> 224 floats, 256 halves); a duct also
    # reserves its electron and phonon lines: (2 nz + 2 ny) shells x nx x 14
    # doubles (two buffers of 6 rows, two velocities)
    def electrons(nx, ny, nz):
        return (2 * nz + 2 * ny) * nx * 14 * 8
    p = lbm.make_params(lbm.D3Q19, lbm.DUCT, 37, 5, 4, tau=0.7, precision="f32")
    pops = 2 * 19 * 37 * 20 * 4
    assert pops + electrons(37, 5, 4) <= lbm.footprint(p) < pops * 1.2 + electrons(37, 5, 4)
    for prec, nxp, size in (("f32", 224, 4), ("f16s", 256, 2)):
        p = lbm.make_params(lbm.D3Q19, lbm.DUCT, 200, 5, 4, tau=0.7, precision=prec)
        pops = 2 * 19 * nxp * 20 * size
        assert pops <= lbm.footprint(p) < pops * 1.2 + electrons(200, 5, 4)


@pytest.mark.parametrize("kw", [
    dict(tau=0.5), dict(tau=float("nan")), dict(nx=0), dict(lattice=27),
    dict(lattice=9, nz=2), dict(lattice=9, geometry=lbm.DUCT, nz=1),
    dict(geometry=lbm.TUBE, tube_radius=0.0), dict(wall_velocity_top=0.1, geometry=lbm.TUBE,
                                                  tube_radius=3.0),
    dict(force=(float("inf"), 0, 0)), dict(precision=7),
])
def test_footprint_rejects_bad_parameters(kw):
    base = dict(lattice=lbm.D3Q19, geometry=lbm.DUCT, nx=8, ny=8, nz=8, tau=0.7)
    base.update(kw)
    p = lbm.make_params(**base)
    lib = lbm.load()
    n = C.c_size_t()
    assert lib.lbm_footprint(C.byref(p), C.byref(n)) == -1


def test_tube_footprint_counts_box():
    p = lbm.make_params(lbm.D3Q19, lbm.TUBE, 512, 72, 72, tau=0.8, tube_radius=32,
                        tube_cy=35.5, tube_cz=35.5)
    assert lbm.footprint(p) >= 2 * 19 * 512 * 72 * 72 * 4


def test_masked_footprint_host_logic():
    # walls that vary along x: the plan reserves the class table of the
    # (x, y) plane and the partner tables; a mask is required, an all-solid
    # mask and a moving wall are refused
    nx, ny, nz = 40, 12, 3
    solid = np.zeros((ny, nx), dtype=bool)
    solid[:2, 10:20] = True
    p = lbm.make_params(lbm.D3Q19, lbm.MASKED, nx, ny, nz, tau=0.8, precision="f32", solid=solid)
    pops = 2 * 19 * nx * ny * nz * 4
    nb = lbm.footprint(p)
    assert pops + nx * ny * 4 <= nb < pops * 1.3 + 200_000
    p2 = lbm.make_params(lbm.D2Q9, lbm.MASKED, nx, ny, 1, tau=0.8, precision="f64", solid=solid)
    assert lbm.footprint(p2) >= 2 * 9 * nx * ny * 8
    lib = lbm.load()
    n = C.c_size_t()
    for bad in (dict(solid=None), dict(solid=np.ones((ny, nx))),
                dict(solid=solid, wall_velocity_top=1e-3)):
        q = lbm.make_params(lbm.D3Q19, lbm.MASKED, nx, ny, nz, tau=0.8, precision="f32", **bad)
        assert lib.lbm_footprint(C.byref(q), C.byref(n)) == -1
    with pytest.raises(ValueError):
        lbm.make_params(lbm.D3Q19, lbm.MASKED, nx, ny, nz, tau=0.8, solid=np.zeros((nx, ny)))


def test_an_empty_sweep_needs_no_gpu():
    from paper_2403_15768_amd import permeability

    assert permeability.sweep([], [1.0]) == []
    assert permeability.sweep([], [], tau=0.1) == []  # parameters of no tube


def test_bench_prices_the_pair_kernel_by_what_it_moves():
    # one read and one write of 19 doubles per cell for two steps
    import bench

    assert bench.step_bytes("f64", True) == 152 and bench.step_bytes("f64", False) == 304
    assert bench.step_bytes("f32", False) == 152 and bench.step_bytes("f16s", False) == 76
    assert all(os.path.exists(os.path.join(ROOT, p)) for p in bench.KERNEL_SOURCES)
    assert "lbm_plan.h" in " ".join(bench.KERNEL_SOURCES)  # the tiles decide the traffic
