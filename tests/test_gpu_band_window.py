"""The macro band solver at every width of its window, against the oracle's driver.

A plate of nx elements in width has the bandwidth 2 nx + 5 and a window of
(bw + 15) / 16 + 1 tile rows of 16; the factor kernel is compiled for each of 2 to
10.  The plates below have first and last bandwidths of such a range (15 | 17, ..,
111 | 113) and lengths for which the window is never full, full once, and moves on.
"""
import pytest

from paper_1908_08292_amd import fehmm
from tests.test_gpu_macro import need_gpu, run_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(1, 1), (5, 9), (6, 3), (13, 2), (14, 1), (24, 2), (29, 3), (30, 1), (38, 2),
                                   (46, 1), (53, 2), (54, 2), (61, 1), (62, 2)])
def test_band_window(nx, ny):
    need_gpu()
    print(f"case macro {nx}x{ny}, RVE 4x4", flush=True)
    # the same Newton iterations and displacements within 1e-8 of the oracle's
    run_pair(nx, ny, 4, 0.3, 1, 1.05, fehmm.BC_UNIAXIAL, fehmm.NESTED)
