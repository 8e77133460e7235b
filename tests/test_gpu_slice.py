"""The fused slice kernel at the edges of its segments, blocks and tube lengths (needs an MI355X).

The W-step shares a row between S lanes of up to 6, 9, 12 or 16 columns each; tubes of up to
32 entries are one thread's, longer ones four or eight lanes'.  Every size runs against the FP64
oracle with the tolerances of the parity tests (FP32 rounding over eight iterations), through
the iteration, the results (W and Z) and the stationarity measures.
"""
import pytest

from tests.gpu_helpers import gpu_run, make_inputs, oracle, oracle_run
from tests.test_gpu_parity import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,n3,r,rho2", [
    (3, 12, 5, 2, 1e-2),     # one lane per row of 12 columns
    (3, 13, 5, 2, 1e-2),     # two lanes of 7 and 6
    (4, 31, 1, 2, 0.7),      # eight lanes, the last of three columns; a single frequency
    (2, 100, 28, 2, 0.7),    # sixteen lanes, four of them one column longer; strong coupling
    (2, 96, 112, 2, 0.7),    # eight full lanes of 12; eight lanes per tube
    (2, 97, 84, 2, 1e-2),    # a last wavefront with one tube
    (3, 288, 20, 3, 0.7),    # 32 lanes per row: scans across the 16-lane groups
    (2, 600, 6, 2, 0.7),     # 64 lanes per row, uneven
    (2, 769, 4, 2, 1e-2),    # 64 lanes of 13 and 12 columns
    (2, 1024, 3, 2, 0.7),    # the longest row: 64 full lanes of 16
    (257, 24, 40, 2, 1e-2),  # more rows than compute units; four lanes per tube
    (256, 10, 32, 2, 1e-2),
    (5, 9, 56, 3, 0.0),      # rho2 = 0: every map is constant
])
def test_slice_kernel_edges(n1, n2, n3, r, rho2):
    d = make_inputs(n1, n2, n3, r, p=0.4, seed=n1 + n2 + n3, weekly=True, sigma_od=1.0, noise=0.02)
    print(f"{n1}x{n2}x{n3} r{r} rho2 {rho2}", flush=True)
    g = gpu_run(d, r, 8, rho2=rho2)
    st, info = oracle_run(d, r, 8, rho2=rho2, history=True)
    _compare(g, st, info, label=f"{n1}x{n2}x{n3} r{r} rho2 {rho2}")
    s = g["ctx"].stationarity()
    so = oracle.stationarity(info["problem"], st)
    assert abs(s[0] - so["factor"]) <= 1e-3 * so["factor"] + 1e-7, (s, so)
    assert s[1] < 1e-5 and s[2] == 0.0
