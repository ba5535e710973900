"""GPU: the tubes of a permeability sweep, run together on streams of their own,
against the same tubes run one by one."""
import math

import numpy as np
import pytest

from paper_2403_15768_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mods():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2403_15768_amd import lbm, permeability

    lbm.load()
    return torch, lbm, permeability


def alone(lbm, perm, sp, R, scale):
    ch = lbm.Channel(**perm._tube_spec(R, 8, 0.8, 1e-6, "f64"))
    lam = math.inf
    if scale is not None:
        ch.set_friction_spectral(sp, np.full(ch.wall_count, scale * sp.omega0))
        lam = float(ch.get_friction()[0])
    n = ch.run_to_steady(rel_tol=1e-5, check_every=100)
    return lam, ch.flux(), int(n)


# one tube and its reference, and more of both than run at a time; the caller
# on a stream of its own with work pending on memory that the arenas may reuse
@pytest.mark.parametrize("radii,scales", [([4], [1.0]), ([3, 5], [0.6, 1.0, 1.6])])
def test_sweep_equals_tubes_one_by_one(mods, radii, scales):
    torch, lbm, perm = mods
    print("sweep", radii, scales, flush=True)
    sp = inputs.draw_spectral(inputs.rng_for("tube", 3), nq=32, nw=64)
    with torch.cuda.stream(torch.cuda.Stream()):
        for _ in range(8):
            junk = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
            junk.fill_(255)
            del junk
        got = perm.sweep(radii, scales, spectral=sp, nx=8, rel_tol=1e-5, check_every=100)
    want = []
    for R in radii:
        q0 = alone(lbm, perm, sp, R, None)[1]
        want += [(R, s, q0, *alone(lbm, perm, sp, R, s)) for s in scales]
    assert [(r.radius, r.omega_scale, r.flux_noslip, r.lam, r.flux, r.steps) for r in got] == want


def test_a_failing_tube_raises(mods):
    torch, lbm, perm = mods
    print("sweep, no steady state", flush=True)
    with pytest.raises(lbm.LBMError):
        perm.sweep([3, 4], [1.0], nx=4, rel_tol=1e-12, check_every=10, max_steps=20)
    assert len(perm.sweep([3], [1.0], nx=4, rel_tol=1e-3, check_every=50)) == 1


def test_no_tube_is_started_after_a_failure(mods):
    # four run at a time; the fourth fails while the first three wait, so a
    # fifth could only start after the failure
    torch, lbm, perm = mods
    import threading

    print("sweep, tasks behind a failed one", flush=True)
    late, ran = threading.Event(), []

    def waits(stream):
        late.wait(0.5)

    def fails(stream):
        raise ValueError("fourth")

    def behind(k):
        def task(stream):
            ran.append(k)
            late.set()
        return task

    with pytest.raises(ValueError, match="fourth"):
        perm._together([waits] * 3 + [fails] + [behind(k) for k in range(8)], 0)
    assert ran == []
