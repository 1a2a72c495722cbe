"""Thin lattices advance several updates per launch (windows of whole cross-sections); the
stored populations must be those of single updates bit for bit.

Cases sit where windows can go wrong: lattices of one window and of several, a
last window cut short, windows at either end with every kind of end, one plane,
one cell across, cross-sections that leave threads idle, 16-bit storage with
scaled codes (an equilibrium end enters it rounded only every second update), odd
levels and odd counts.  Setting the launch shape of the update (to its default)
keeps a lattice on single updates, which gives the reference.
"""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

BCS = {"periodic": W.BC_PERIODIC, "walls": W.BC_WALL, "ends": W.BC_DIRICHLET, "noslip": W.BC_NOSLIP}


def _case(dims, bc):
    c = W.smooth_random_case(*dims, seed=31) if min(dims) > 1 else W.random_case(*dims, seed=31, amp=0.3)
    prm = dict(c.params, bc_x=BCS[bc], wall_u=[[0.0, 0.1, -0.05], [0.0, 0.2, 0.1]], wall_T=[0.0, 1.1])
    if bc == "ends":
        prm["Q_left"] = W.uniform_state(1.1, (0.1, 0.0, 0.0), 1.05, prm["gamma"])
        prm["Q_right"] = W.uniform_state(0.9, (0.05, 0.02, 0.0), 0.97, prm["gamma"])
    return prm, c.Q0


@pytest.mark.parametrize("bc", sorted(BCS))
@pytest.mark.parametrize("dims", [(1, 4, 3), (16, 4, 4), (17, 4, 4), (61, 4, 4), (257, 1, 1), (300, 3, 2), (50, 5, 7)])
@pytest.mark.parametrize("storage,scale", [(W.STORAGE_FP32, 0.0), (W.STORAGE_FP16, 0.0), (W.STORAGE_BF16, 0.25)])
def test_windows_equal_single_updates(bc, dims, storage, scale):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_13437_amd as cnsf
    prm, Q = _case(dims, bc)
    prm.update(storage=storage, storage_scale=[scale] * 14)
    print(f"case {dims} {bc} storage {storage} scale {scale}", flush=True)
    a, b = cnsf.Lattice(prm), cnsf.Lattice(prm)
    for L in (a, b):
        L.set_state(Q)
    a.set_launch(*a.get_launch())
    for n in (4, 1, 6, 33, 70):
        a.step(n)
        b.step(n)
        assert a.info()[:2] == b.info()[:2]
        assert torch.equal(a.buf, b.buf), n
    a.close()
    b.close()


# one window and several, with threads left idle: 245, 253, 252, 253 and 255 of 256 at work
IDLE = [(7, 5, 7), (23, 11, 1), (40, 9, 1), (60, 11, 1), (700, 5, 3)]


@pytest.mark.parametrize("bc", sorted(BCS))
@pytest.mark.parametrize("dims", IDLE)
@pytest.mark.parametrize("storage,scale", [(W.STORAGE_FP32, 0.0), (W.STORAGE_FP16, 0.25), (W.STORAGE_BF16, 0.0)])
def test_windows_with_idle_threads_equal_single_updates(bc, dims, storage, scale):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_13437_amd as cnsf
    prm, Q = _case(dims, bc)
    prm.update(storage=storage, storage_scale=[scale] * 14, visc_law=W.VISC_POWER, visc_param=0.76)
    print(f"case {dims} {bc} storage {storage} scale {scale}", flush=True)
    a, b = cnsf.Lattice(prm), cnsf.Lattice(prm)
    for L in (a, b):
        L.set_state(Q)
    a.set_launch(*a.get_launch())
    for n in (70, 9, 34, 65):
        a.step(n)
        b.step(n)
        assert a.info()[:2] == b.info()[:2]
        assert torch.equal(a.buf, b.buf), n
    a.close()
    b.close()


@pytest.mark.parametrize("bc", sorted(BCS))
@pytest.mark.parametrize("scale", [0.25, 0.3])
@pytest.mark.parametrize("dims", [(16, 4, 4), (90, 4, 3)])
def test_scaled_codes_keep_the_sign_of_zero(dims, scale, bc):
    """Updates leave a few negative zeros among scaled FP16 codes (small negative deviations that
    underflow); a window stores them as it found them."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_13437_amd as cnsf
    prm, Q = _case(dims, bc)
    prm.update(storage=W.STORAGE_FP16, storage_scale=[scale] * 14)
    print(f"case {dims} {bc} scale {scale}", flush=True)
    a, b = cnsf.Lattice(prm), cnsf.Lattice(prm)
    for L in (a, b):
        L.set_state(Q)
    zeros = 0
    for n in (70, 16, 32, 64):
        b.step(n)
        for _ in range(n):
            a.step(1)
        zeros += int((a.buf.view(torch.int16) == -32768).sum())
        assert torch.equal(a.buf, b.buf), n
    print(f"  {zeros} negative zeros", flush=True)
    a.close()
    b.close()
