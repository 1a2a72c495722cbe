"""Line transforms of the spectral readouts at the edges of their tiles.

Lengths of 1 to 128 (powers of two) or 1024 points go through FP64 matrix
products over sixteen lines at a time; longer ones through the LDS or register
transforms or a direct sum.  White-noise states put energy in every mode, so
each coefficient, fold and pad shows in eps_s, eps_d and the spectrum, against
the oracle's numpy.fft on the same state.

Tolerance: a derivative is a sum of n/2 products in FP64, so its rounding is below
n 2^-53 times the sum of |coefficient| |value|, which for noise exceeds the
result by about sqrt(n): below 1e-12 of the result at the lengths used.  1e-11
leaves a factor of ten for the oracle's own rounding.
"""
import pytest

import workloads as W
from oracle import diagnostics as odiag

pytestmark = pytest.mark.gpu


def _lattice(dims, amp=0.5):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_13437_amd as cnsf
    cnsf.library()
    case = W.random_case(*dims, seed=21, amp=amp)
    print(f"case {case.name}", flush=True)
    L = cnsf.Lattice(case.params)
    L.set_state(case.Q0)
    return L, case


# (nx, ny, nz): shortest lines, either side of whole tiles and k-steps, odd and even, few and many
# lines, more than 64 KiB of LDS (from 441 points), the longest product and the first direct sum,
# one axis on another route than the others
DERIV = [(1, 2, 3), (4, 5, 6), (15, 16, 17), (31, 32, 33), (34, 7, 64), (63, 66, 9), (97, 128, 5), (129, 3, 31),
         (5, 192, 18), (441, 3, 2), (2, 600, 3), (3, 2, 1023), (1025, 2, 2), (2, 256, 7), (6, 9, 1024)]


@pytest.mark.parametrize("dims", DERIV)
def test_spectral_derivatives_by_matrix_products(dims):
    L, case = _lattice(dims)
    o = odiag.diagnostics(L.moments(), case.params)
    d = L.diagnostics(spectral=True)
    s = L.step_diagnostics(1, spectral=True)       # the sums into partials of their own
    for got in (d, s):
        for k in ("eps_s", "eps_d"):
            assert abs(got[k] - o[k]) <= 1e-11 * max(abs(o["eps_s"]), abs(o["eps_d"])), (k, got[k], o[k])
    L.close()


# the last length of the general transform, the shortest product, tile edges, LDS above 64 KiB
@pytest.mark.parametrize("n", [5, 6, 7, 16, 31, 33, 64, 97, 236])
def test_shell_spectrum_by_matrix_products(n):
    L, case = _lattice((n, n, n))
    E = L.spectrum()
    o = odiag.shell_spectrum(L.moments(), case.params)
    assert E.shape == o.shape
    assert abs(E - o).max() <= 1e-11 * o.max()
    L.close()
