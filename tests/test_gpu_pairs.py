"""Multi-step calls that advance two updates per pass over memory, against single updates.

The paired passes must leave every stored population bit for bit as single
updates do.  Cases sit where the cut of the lattice can go wrong: one tile and
several along x and y with ragged last tiles, one and several blocks along z,
a second array of the lattice's size and slabs shifted through a workspace
(whose first and last planes cross the periodic end by their own route), an
odd level at entry and every remainder of the step count.  Setting the launch
shape of the update (to its default) keeps a lattice on single updates, which
gives the reference; a drop of the free device memory shows that the other
lattice did allocate the workspace of the paired passes.
"""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _cnsf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_13437_amd as cnsf
    cnsf.library()
    return cnsf


def _state(prm, seed):
    """Random positive state on the device (every cell its own sensor decision)."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    sh = (prm["nz"], prm["ny"], prm["nx"])
    r = lambda a: a * (2 * torch.rand(sh, generator=g, device="cuda", dtype=torch.float64) - 1)
    rho, p = 1.0 + r(0.4), 1.0 + r(0.4)
    u = [r(0.3) for _ in range(3)]
    Q = torch.empty((14,) + sh, device="cuda", dtype=torch.float64)
    Q[0] = rho
    for a in range(3):
        Q[1 + a] = rho * u[a]
    Q[4] = p / (prm["gamma"] - 1.0) + 0.5 * rho * (u[0] ** 2 + u[1] ** 2 + u[2] ** 2)
    for k in range(5, 14):
        Q[k] = r(0.01)
    return Q


# nx, ny, nz, storage, storage scale, steps per call
CASES = [
    (64, 64, 64, W.STORAGE_FP32, 0.0, (1, 5, 4, 7, 40, 9)),   # one tile along x, second array
    (80, 79, 80, W.STORAGE_FP32, 0.0, (4, 2, 18)),            # whole rows of three, one row in the last tile
    (96, 95, 100, W.STORAGE_FP32, 0.0, (4, 6)),           # the longest whole rows
    (150, 147, 150, W.STORAGE_FP32, 0.0, (5, 4, 14)),     # tiles of 64, 64 and 22 columns, ragged rows
    (128, 128, 127, W.STORAGE_FP16, 0.0, (4, 3, 9)),      # 16-bit links
    (128, 128, 128, W.STORAGE_BF16, 0.0, (8,)),
    (128, 126, 128, W.STORAGE_FP16, 0.5, (5, 4, 9)),         # scaled codes, two rows in the last tile
    (192, 192, 192, W.STORAGE_FP32, 0.0, (4, 1, 10)),     # slabs through a workspace
    (256, 254, 192, W.STORAGE_FP32, 0.0, (4, 5)),         # slabs of whole slot groups, two rows in the last tile
    (320, 256, 256, W.STORAGE_FP16, 0.0, (4, 6)),         # 16-bit, second array
    (384, 340, 340, W.STORAGE_FP16, 0.0, (4, 6, 8)),         # 16-bit slabs (from 8 GiB on)
    (448, 440, 424, W.STORAGE_FP32, 0.0, (4,)),           # non-temporal stores (from 32 GB on)
]


@pytest.mark.parametrize("nx,ny,nz,storage,scale,calls", CASES)
def test_paired_passes_equal_single_updates(nx, ny, nz, storage, scale, calls):
    import torch
    cnsf = _cnsf()
    prm = dict(W.random_params(nx, ny, nz, seed=3), storage=storage, storage_scale=[scale] * 14)
    print(f"case {nx}x{ny}x{nz} storage {storage} scale {scale} calls {calls}", flush=True)
    Q = _state(prm, 17)
    a, b = cnsf.Lattice(prm), cnsf.Lattice(prm)
    a.set_state(Q)
    b.set_state(Q)
    del Q
    a.set_launch(*a.get_launch())
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for n in calls:
        b.step(n)
    torch.cuda.synchronize()
    taken = free0 - torch.cuda.mem_get_info()[0]
    for n in calls:
        a.step(n)
    assert taken >= a.nbytes // 32, f"single updates ran: {taken} bytes taken"
    assert a.info()[:2] == b.info()[:2]
    assert torch.equal(a.buf, b.buf)
    assert bool(torch.isfinite(b.moments(device=True)).all())
    a.close()
    b.close()


# nx, ny, nz, storage, viscosity law and its parameter, steps per call: the power law of the run driver and the
# bench, and constant viscosity (the cases above have Sutherland's law)
LAWS = [
    (96, 96, 96, W.STORAGE_FP32, W.VISC_POWER, 0.76, (5, 8, 6)),
    (128, 128, 128, W.STORAGE_FP16, W.VISC_POWER, 0.76, (9, 8)),
    (128, 126, 128, W.STORAGE_BF16, W.VISC_POWER, 1.3, (8, 9)),
    (192, 192, 192, W.STORAGE_FP32, W.VISC_POWER, 0.76, (4, 5)),
    (128, 96, 97, W.STORAGE_FP32, W.VISC_CONST, 0.0, (7, 8)),
]


@pytest.mark.parametrize("nx,ny,nz,storage,law,param,calls", LAWS)
def test_paired_passes_of_other_viscosity_laws(nx, ny, nz, storage, law, param, calls):
    import torch
    cnsf = _cnsf()
    prm = dict(W.random_params(nx, ny, nz, seed=4), storage=storage, visc_law=law, visc_param=param)
    print(f"case {nx}x{ny}x{nz} storage {storage} law {law} calls {calls}", flush=True)
    Q = _state(prm, 23)
    a, b = cnsf.Lattice(prm), cnsf.Lattice(prm)
    a.set_state(Q)
    b.set_state(Q)
    del Q
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for n in calls:
        b.step(n)
    torch.cuda.synchronize()
    taken = free0 - torch.cuda.mem_get_info()[0]
    for _ in range(sum(calls)):
        a.step(1)
    assert taken >= a.nbytes // 32, f"single updates ran: {taken} bytes taken"
    assert torch.equal(a.buf, b.buf)
    assert bool(torch.isfinite(b.moments(device=True)).all())
    a.close()
    b.close()


def test_paired_passes_give_their_workspace_back():
    import torch
    cnsf = _cnsf()
    prm = W.random_params(128, 128, 128)
    Q = _state(prm, 5)
    torch.cuda.synchronize()
    free = []
    for _ in range(3):
        L = cnsf.Lattice(prm)
        L.set_state(Q)
        L.step(8)
        L.close()
        del L
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
    assert abs(free[2] - free[1]) < 64 << 20


@pytest.mark.parametrize("kind", ["pairs", "windows", "batch"])
def test_first_steps_beside_a_capture_on_another_stream(kind):
    """The workspaces of multi-step calls are allocated by the first call; a capture that
    runs on another stream meanwhile must survive that, and the steps come out the same."""
    import torch
    cnsf = _cnsf()
    print(f"case {kind}", flush=True)
    c = W.sod(256, 4, 4) if kind == "windows" else W.smooth_random_case(64, 64, 64)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        if kind == "batch":
            a, b = cnsf.Batch([c.params] * 32), cnsf.Batch([c.params] * 32)
            for B in (a, b):
                for j in range(32):
                    B.set_state(j, c.Q0)
        else:
            a, b = cnsf.Lattice(c.params), cnsf.Lattice(c.params)
            a.set_state(c.Q0)
            b.set_state(c.Q0)
    x = torch.zeros(64, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        x += 1.0
        b.step(66, b.MODE_GRAPH) if kind == "batch" else b.step(66)
        x += 1.0
    for _ in range(66):
        a.step(1, a.MODE_LAUNCH) if kind == "batch" else a.step(1)
    for _ in range(2):
        g.replay()
    torch.cuda.synchronize()
    assert float(x[0]) == 4.0
    assert torch.equal(a.buf, b.buf)
    del g
    a.close()
    b.close()


@pytest.mark.parametrize("kind", ["pairs", "windows", "batch"])
def test_workspace_is_made_beside_a_capture_on_another_stream(kind):
    """As above, with lattices whose workspace shows in the free memory: it is made while the other
    stream captures."""
    import torch
    cnsf = _cnsf()
    print(f"case {kind}", flush=True)
    dims = (60000, 2, 1) if kind == "windows" else (64, 64, 64)
    c = W.smooth_random_case(*dims)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        if kind == "batch":
            b = cnsf.Batch([c.params] * 32)
            for j in range(32):
                b.set_state(j, c.Q0)
        else:
            b = cnsf.Lattice(c.params)
            b.set_state(c.Q0)
    x = torch.zeros(64, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        x += 1.0
        free0 = torch.cuda.mem_get_info()[0]      # the capture's start gave torch's cached memory back
        b.step(66, b.MODE_GRAPH) if kind == "batch" else b.step(66)
        free1 = torch.cuda.mem_get_info()[0]
        x += 1.0
    torch.cuda.synchronize()
    assert free0 - free1 >= b.nbytes // 2
    g.replay()
    torch.cuda.synchronize()
    assert float(x[0]) == 2.0
    del g
    b.close()
