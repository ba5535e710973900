"""GPU: the electron and phonon lines stepped with the water in one launch
against lines and water in two (a workgroup that holds only part of an x-line),
bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbm():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2403_15768_amd import lbm as mod

    mod.load()
    return mod


def channel(lbm, q, geo, nx, ny, nz, precision, phonons, kT):
    ch = lbm.Channel(q, geo, nx, ny, nz, tau=0.71, force=(1e-5, 0.0, 0.0), precision=precision)
    ch.set_friction(np.random.default_rng(nx + ny).uniform(0.0, 0.3, ch.wall_count))
    if kT:
        ch.set_thermal(kT, 1, 5)
    ch.set_electrons(0.9, 1.0, 0.05, 1e-5)
    if phonons:
        ch.set_phonons(0.7, 1.3, 0.02, 0.08)
    return ch


# corners, columns with two and four shells (one or two rows), D2Q9, padded
# and ragged lines, the longest line of one workgroup
@pytest.mark.parametrize("q,geo,nx,ny,nz", [
    (19, "duct", 100, 5, 4), (19, "duct", 70, 2, 2), (19, "duct", 200, 12, 9),
    (19, "slab", 130, 7, 6), (19, "slab", 90, 2, 1), (9, "slab", 66, 9, 1), (9, "slab", 500, 1, 1),
    (9, "slab", 512, 3, 1),
])
@pytest.mark.parametrize("precision,phonons,kT", [("f64", True, 0.0), ("f32", False, 0.0),
                                                  ("f32", True, 1e-6), ("f16s", True, 0.0)])
def test_one_launch_equals_two(lbm, q, geo, nx, ny, nz, precision, phonons, kT):
    print("lines", q, geo, nx, ny, nz, precision, phonons, kT, flush=True)
    kind = lbm.DUCT if geo == "duct" else lbm.SLAB
    A, B = (channel(lbm, q, kind, nx, ny, nz, precision, phonons, kT) for _ in range(2))
    B.set_block(64)  # several workgroups per x-line
    for n in (3, 64 + 9):
        A.step(n)
        B.step(n)
        for a, b in zip(A.electrons(), B.electrons()):
            assert np.array_equal(np.asarray(a), np.asarray(b))
        assert np.array_equal(A.get_state()[0], B.get_state()[0])
    assert np.isfinite(A.flux()) and A.flux() == B.flux()
