"""Graph-mode batches advance two updates per pass over memory where that is faster; every
member's stored populations must be those of one launch per step bit for bit.

Members of different tiles (whole rows of 32 to 96 cells, 64-cell tiles with a
ragged last one), ragged rows, flat and tall ones, a few cells wide, in both population layouts, at
odd levels and every remainder of four; a drop of the free memory shows that the
second array was allocated.
"""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

DIMS = [(96, 96, 96), (64, 64, 64), (80, 79, 77), (48, 50, 96), (32, 32, 32), (130, 66, 40), (96, 96, 70), (128, 128, 64),
        (64, 200, 33), (128, 96, 96), (5, 4, 64), (3, 70, 20), (40, 2, 9), (7, 1, 4), (1, 30, 12)]


@pytest.mark.parametrize("storage,scale,spacing", [(W.STORAGE_FP32, 0.0, 0), (W.STORAGE_FP16, 0.0, 1 << 28),
                                                   (W.STORAGE_BF16, 0.5, 0)])
def test_paired_batch_equals_single_updates(storage, scale, spacing):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_13437_amd as cnsf
    prms = [dict(W.random_params(*d, seed=j), storage=storage, storage_scale=[scale if j % 2 else 0.0] * 14)
            for j, d in enumerate(DIMS * 3)]
    print(f"case {len(prms)} members storage {storage} scale {scale} spacing {spacing}", flush=True)
    a, b = cnsf.Batch(prms, spacing=spacing), cnsf.Batch(prms, spacing=spacing)
    for j, d in enumerate(DIMS * 3):
        g = torch.Generator(device="cuda").manual_seed(j)
        r = lambda s: s * (2 * torch.rand(d[::-1], generator=g, device="cuda", dtype=torch.float64) - 1)
        Q = torch.zeros((14,) + d[::-1], device="cuda", dtype=torch.float64)
        Q[0] = 1.0 + r(0.4)
        for k in range(1, 4):
            Q[k] = Q[0] * r(0.3)
        Q[4] = (1.0 + r(0.4)) / 0.4 + 0.5 * (Q[1] ** 2 + Q[2] ** 2 + Q[3] ** 2) / Q[0]
        for B in (a, b):
            cnsf.cnsf_batch_set_state(B.h, j, Q.data_ptr(), cnsf.CNSF_DEVICE)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for n in (4, 1, 7, 10, 22):
        b.step(n, b.MODE_GRAPH)
    torch.cuda.synchronize()
    taken = free0 - torch.cuda.mem_get_info()[0]
    for n in (4, 1, 7, 10, 22):
        a.step(n, a.MODE_LAUNCH)
    assert taken >= cnsf.cnsf_batch_required_bytes(b.ps) // 2, f"single updates ran: {taken} bytes taken"
    assert torch.equal(a.buf, b.buf)
    a.close()
    b.close()


@pytest.mark.parametrize("pairs", [None, 0, 1])
def test_autotune_keeps_the_state_and_honours_its_cache(tmp_path, pairs):
    """A cached entry says whether paired steps were the faster ones; without a cache the
    trials restore the state, at an odd level too."""
    import json
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_13437_amd as cnsf
    prms = [W.random_params(64, 64, 64, seed=j) for j in range(32)]
    Q = W.smooth_random_case(64, 64, 64).Q0
    a, b = cnsf.Batch(prms), cnsf.Batch(prms)
    for B in (a, b):
        for j in range(len(prms)):
            B.set_state(j, Q)
        B.step(3, B.MODE_LAUNCH)
    cache = tmp_path / "tuned.json"
    if pairs is not None:
        first = cnsf.Batch(prms)
        first.autotune(str(cache), steps_per_trial=4)
        first.close()
        entries = json.loads(cache.read_text())
        for v in entries.values():
            v["pairs"] = pairs
        cache.write_text(json.dumps(entries))
    torch.cuda.synchronize()
    b.autotune(str(cache) if pairs is not None else None, steps_per_trial=4)
    assert torch.equal(a.buf, b.buf)
    free0 = torch.cuda.mem_get_info()[0]
    a.step(9, a.MODE_LAUNCH)
    b.step(9, b.MODE_GRAPH)
    torch.cuda.synchronize()
    taken = free0 - torch.cuda.mem_get_info()[0]
    if pairs is not None:
        assert (taken >= b.nbytes // 2) == bool(pairs)
    assert torch.equal(a.buf, b.buf)
    a.close()
    b.close()
