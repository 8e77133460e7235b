"""The FP64 tube transforms and the W-step of the three-launch slice path (needs an MI355X).

Tubes go through mixed-radix passes in LDS, two real tubes per complex sequence, or through
direct sums where n3 is short, or a prime or twice one with few tubes.  Every size runs against
the FP64 oracle with the tolerances of the parity tests, through the factor transforms, the
iteration, the results and the stationarity measures.
"""
import pytest

from tests.gpu_helpers import gpu_run, make_inputs, oracle, oracle_run
from tests.test_gpu_parity import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,n3,r,rho2", [
    (2, 1, 98, 1, 1e-2),     # one tube per OD row: its partner is empty
    (3, 5, 22, 2, 0.7),      # direct sums: short
    (3, 6, 30, 2, 1e-2),     # direct sums: below the line of small radices
    (3, 5, 67, 2, 1e-2),     # direct sums: prime
    (5, 103, 67, 2, 0.7),    # the same length as a pass: 260 pairs; W-step segments with a short last one
    (3, 5, 183, 2, 0.7),     # a pass of radix 61
    (3, 5, 134, 2, 1e-2),    # direct sums: twice a prime, few tubes
    (21, 27, 134, 2, 1e-2),  # the same length in passes: 294 pairs
    (3, 16, 90, 2, 0.7),     # a full W-step segment of 16, several pairs per block
    (4, 17, 125, 2, 1e-2),
    (2, 32, 121, 2, 0.7),
    (3, 33, 256, 2, 0.7),    # three W-step segments of 11 in four; a full block of tubes
    (2, 7, 257, 2, 1e-2),    # prime; two W-step blocks per OD row, the second with one row
    (2, 3, 1000, 2, 0.7),    # roots beside the sequence in the factor transforms
    (2, 3, 1331, 2, 1e-2),   # three passes of radix 11
    (3, 4, 2187, 2, 0.7),    # seven passes of radix 3
    (2, 3, 2046, 2, 0.7),    # the longest pairs of few even tubes
    (2, 3, 2048, 2, 1e-2),   # sequences of half the length
    (20, 27, 2048, 2, 0.7),  # pairs again: 280
    (3, 5, 4094, 2, 0.7),    # passes of radix 23 and 89
    (2, 2, 8064, 2, 1e-2),
    (2, 3, 8191, 2, 1e-2),   # the largest prime: direct sums
    (2, 3, 8192, 2, 0.7),    # the longest tube
])
def test_tube_transform_edges(n1, n2, n3, r, rho2):
    d = make_inputs(n1, n2, n3, r, p=0.4, seed=n1 + n2 + n3, weekly=True, sigma_od=1.0, noise=0.02)
    print(f"{n1}x{n2}x{n3} r{r} rho2 {rho2}", flush=True)
    g = gpu_run(d, r, 8, rho2=rho2, want=("W", "Z", "X", "Y"))
    st, info = oracle_run(d, r, 8, rho2=rho2, history=True)
    _compare(g, st, info, label=f"{n1}x{n2}x{n3} r{r} rho2 {rho2}")
    s = g["ctx"].stationarity()
    so = oracle.stationarity(info["problem"], st)
    assert abs(s[0] - so["factor"]) <= 1e-3 * so["factor"] + 1e-7, (s, so)
    assert s[1] < 1e-5 and s[2] == 0.0
