"""Tubes with a large prime factor on both sides of the choice between direct sums and passes
(needs an MI355X): every size against the FP64 oracle with the tolerances of the parity tests,
through the factor transforms, the iteration, the results and the objective's gradient."""
import pytest

from tests.gpu_helpers import gpu_run, make_inputs, oracle_run
from tests.test_gpu_parity import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,n3,r", [
    (64, 64, 67, 2),     # a prime, many tubes: one pass of 67, four pairs per block
    (17, 9, 67, 2),      # the same length, few tubes: direct sums
    (46, 12, 419, 2),    # a prime, 276 pairs: direct sums
    (24, 25, 1021, 2),   # a prime past the roots' LDS, one tube without a partner: a pass
    (65, 7, 1481, 2),    # direct sums over many blocks
    (2, 3, 7115, 2),     # 5 x 1423, few tubes: direct sums
    (9, 16, 5105, 2),    # 5 x 1021, more tubes: two passes in more than 64 KB of LDS
    (2, 3, 2042, 2),     # twice a prime, few tubes: direct sums
    (24, 32, 2042, 2),   # more: passes of pairs
    (3, 5, 4084, 2),     # 4 x 1021, few tubes: direct sums
    (20, 5, 4084, 2),    # more: sequences of half the length
])
def test_prime_tubes_on_both_sides_of_the_rule(n1, n2, n3, r):
    d = make_inputs(n1, n2, n3, r, p=0.4, seed=n1 + n2 + n3, weekly=True, sigma_od=1.0, noise=0.02)
    print(f"{n1}x{n2}x{n3} r{r}", flush=True)
    g = gpu_run(d, r, 4, rho2=0.7, want=("W", "Z", "X", "Y"))
    st, info = oracle_run(d, r, 4, rho2=0.7, history=True)
    _compare(g, st, info, label=f"{n1}x{n2}x{n3} r{r}")
    g["ctx"].close()
