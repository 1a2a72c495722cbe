"""Lattices of few cells, and FP16 ones within the last-level cache, are launched in shapes
of their own; a lattice whose caller sets the default shape is not.  Populations must be
the same bit for bit, the diagnostics' sums up to the order of their FP64 additions.

Cells on both sides of every line of the rule, ragged counts, each end type and storage
type, all-cell and walled lattices, odd levels at entry.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

F32, F16, B16 = W.STORAGE_FP32, W.STORAGE_FP16, W.STORAGE_BF16
CASES = [
    (1, 1, 1, F32, 0), (7, 5, 3, F16, 3), (63, 1, 1, B16, 1), (40, 39, 41, F32, 2),
    (64, 48, 32, F16, 0), (97, 32, 32, F16, 0), (96, 32, 32, B16, 3), (97, 32, 32, F32, 1),   # 96 x 1024 cells
    (64, 64, 48, F16, 1), (65, 64, 48, F16, 3), (64, 64, 64, F16, 0), (65, 64, 64, F16, 0),   # three and four blocks per CU
    (128, 100, 101, F16, 1), (128, 102, 101, F16, 1),                                         # 256 MB
]


@pytest.mark.parametrize("nx,ny,nz,storage,bc", CASES)
def test_own_shape_equals_default_shape(nx, ny, nz, storage, bc):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_13437_amd as cnsf
    print(f"case {nx}x{ny}x{nz} storage {storage} ends {bc}", flush=True)
    c = W.smooth_random_case(nx, ny, nz)
    end = W.uniform_state(1.0, (0.0, 0.0, 0.0), 1.0, c.params["gamma"])
    prm = dict(c.params, storage=storage, bc_x=bc, wall_u=[[0.0, 0.1, -0.05], [0.0, 0.2, 0.1]], wall_T=[0.0, 1.1],
               Q_left=end, Q_right=end)
    a, b = cnsf.Lattice(prm), cnsf.Lattice(prm)
    for L in (a, b):
        L.set_state(c.Q0)
    b.set_launch(*b.get_launch())
    assert a.get_launch() == b.get_launch()
    for n in (1, 3, 2):
        a.step(n)
        b.step(n)
        assert torch.equal(a.buf, b.buf)
        da, db = a.step_diagnostics(1), b.step_diagnostics(1)
        assert torch.equal(a.buf, b.buf)
        size = abs(da["mass"]) + abs(da["energy"])   # of the sums' absolute terms
        for k in da:
            assert np.allclose(da[k], db[k], rtol=0.0, atol=1e-12 * size), (k, da[k], db[k])
    a.close()
    b.close()


def test_readouts_of_many_lattices_share_pinned_pages():
    """More lattices alive than one page of totals has places, destroyed and made again in
    another order, read out from several threads: each gets its own sums."""
    import threading
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_13437_amd as cnsf
    c = W.smooth_random_case(9, 5, 4)
    made = {}

    def make(j):
        made[j] = cnsf.Lattice(c.params)
        made[j].set_state(c.Q0 * np.where(np.arange(14) < 5, 1.0 + j, 0.0)[:, None, None, None])

    def read(js):
        for j in js:
            for _ in range(3):
                got.setdefault(j, []).append(made[j].diagnostics(spectral=False)["mass"])

    for j in range(150):
        make(j)
    got = {}
    read(range(150))
    for j in list(range(0, 150, 2)) + [149, 1]:
        made.pop(j).close()
    for j in range(0, 60, 2):
        make(j)
    got.clear()
    parts = [list(made)[k::4] for k in range(4)]
    threads = [threading.Thread(target=read, args=(p,)) for p in parts]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    mass = float(c.Q0[0].sum())
    assert len(got) == len(made)
    for j, m in got.items():
        assert np.allclose(m, (1.0 + j) * mass, rtol=1e-5, atol=0.0), j
    for L in made.values():
        L.close()


@pytest.mark.parametrize("nx,ny,nz,storage,bc", CASES)
def test_own_shape_equals_shape_of_large_lattices(nx, ny, nz, storage, bc):
    """The shape by size against the one that large lattices of the storage type run in."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_13437_amd as cnsf
    print(f"case {nx}x{ny}x{nz} storage {storage} ends {bc}", flush=True)
    c = W.smooth_random_case(nx, ny, nz)
    end = W.uniform_state(1.0, (0.0, 0.0, 0.0), 1.0, c.params["gamma"])
    prm = dict(c.params, storage=storage, bc_x=bc, wall_u=[[0.0, 0.1, -0.05], [0.0, 0.2, 0.1]], wall_T=[0.0, 1.1],
               Q_left=end, Q_right=end)
    a, b = cnsf.Lattice(prm), cnsf.Lattice(prm)
    for L in (a, b):
        L.set_state(c.Q0)
    large = (256, 512, 0, 0) if storage == F16 else (256, 256, 0, 1)
    b.set_launch(*large)
    assert b.get_launch() == large
    for n in (1, 3, 2):
        a.step(n)
        b.step(n)
        assert torch.equal(a.buf, b.buf)
        a.step_diagnostics(1)
        b.step_diagnostics(1)
        assert torch.equal(a.buf, b.buf)
    a.close()
    b.close()
