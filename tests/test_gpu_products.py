"""The products of the iteration at the edges of their tiles (needs an MI355X), each run against
the FP64 oracle with the tolerances of the parity tests."""
import numpy as np
import pytest

from tests.gpu_helpers import gpu_run, make_inputs, oracle_run, rel
from tests.test_gpu_parity import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,n3,r,rho1,eta", [
    (22, 48, 3, 8, 1e-2, 1.0),     # one block of 32 rows less the halo, one pass of 48 columns
    (23, 49, 3, 9, 1e-2, 0.7),     # a second block, a second wavefront column with one column
    (32, 97, 4, 16, 0.0, 1.0),     # no halo: exactly 32 rows; three wavefront columns
    (40, 300, 3, 8, 0.1, 0.8),     # halo 22: 64-row blocks; a pass of four wavefront columns, then another
    (20, 1000, 2, 5, 1e-2, 1.0),   # 32-row blocks, three passes of eight wavefront columns
    (55, 17, 80, 7, 1e-2, 1.0),    # a tube length outside the fused set, one row past a 64-row block's 54
    (70, 60, 5, 17, 1e-2, 0.7),    # r > 16: the right-hand side, two wavefront columns
    (45, 200, 4, 32, 0.3, 1.0),    # the largest rank, four wavefront columns and a second pass
    (1200, 10, 56, 3, 1e-2, 1.0),  # enough blocks for 64 rows each
])
@pytest.mark.parametrize("precision", ["fp32", "mixed"])
def test_x_update_edges(n1, n2, n3, r, rho1, eta, precision):
    d = make_inputs(n1, n2, n3, r, p=0.5, seed=n1 + n2 + r, sigma_od=1.0, noise=0.02)
    print(f"{n1}x{n2}x{n3} r{r} rho1 {rho1} eta {eta} {precision}", flush=True)
    iters = 6 if precision == "fp32" else 1
    g = gpu_run(d, r, iters, rho1=rho1, eta=eta, precision=precision)
    st, info = oracle_run(d, r, iters, rho1=rho1, eta=eta, history=True)
    if precision == "fp32":
        _compare(g, st, info, label=f"{n1}x{n2}x{n3} r{r}")
    else:
        # one iteration from BF16 W~ (relative rounding up to 2^-8 per entry): W is a smoothed
        # product of sums over it
        _compare(g, st, None, label=f"{n1}x{n2}x{n3} r{r} mixed", tol=2.0**-7, tol_max=2.0**-5, tol_row=2.0**-5)


@pytest.mark.parametrize("n1,n2,n3,r", [
    (1, 3, 4, 1),        # one row: no difference
    (7, 9, 5, 2),        # inside one run of eight rows
    (8, 17, 4, 8),       # exactly one run; a column past a 16-column group
    (9, 33, 3, 7),       # one row in the second run, an odd rank: a last 1 x 1 pivot
    (65, 16, 4, 15),     # nine runs over eight wavefronts
    (130, 40, 6, 16),    # the largest rank of one tile
    (66, 50, 4, 17),     # two tiles, one column in the second
    (80, 64, 3, 32),     # two full tiles
    (12, 12, 512, 8),    # two wavefronts per block (many frequencies of few rows)
    (64, 20, 510, 9),    # its last row count and first frequency count
    (65, 20, 510, 9),    # one row more: eight wavefronts
])
@pytest.mark.parametrize("pinv_mode", [0, 1])
def test_gram_and_product_edges(n1, n2, n3, r, pinv_mode):
    """X~^* W~ and G_X in one launch, with the pivot sweep (pinv_mode 0) and the eigen route (1)."""
    d = make_inputs(n1, n2, n3, r, p=0.7, seed=n1 + n2 + n3 + r, sigma_od=1.0, noise=0.02)
    print(f"{n1}x{n2}x{n3} r{r} pinv_mode {pinv_mode}", flush=True)
    g = gpu_run(d, r, 4, pinv_mode=pinv_mode)
    st, info = oracle_run(d, r, 4, history=True)
    _compare(g, st, info, label=f"{n1}x{n2}x{n3} r{r}")


@pytest.mark.parametrize("n1,n2,n3,r", [
    (63, 31, 5, 3),      # one block per frequency, its last column missing; odd rows
    (64, 32, 6, 8),      # one full block
    (65, 33, 7, 9),      # a row and a column over; odd rows
    (1, 1, 4, 1),
    (130, 66, 3, 17),    # even rows whose last block holds two columns
    (40, 96, 1, 32),     # the largest rank
])
@pytest.mark.parametrize("precision", ["fp32", "mixed"])
def test_factor_product_edges(n1, n2, n3, r, precision):
    """Z = X * Y of the initial factors.  A term of the product is rounded by 2^-24 in FP32 and
    by 2^-16 where the factors are split into BF16 parts; the sums and the two transforms of
    either add less than 8 such roundings in norm."""
    rng = np.random.default_rng(n1 + n2 + n3 + r)
    d = make_inputs(n1, n2, n3, r, p=0.5, seed=n1 + n2, weekly=True, sigma_od=1.0, noise=0.02)
    d["X0"] = rng.normal(size=(n1, r, n3)).astype(np.float32)
    print(f"{n1}x{n2}x{n3} r{r} {precision}", flush=True)
    g = gpu_run(d, r, 0, precision=precision, want=("Z",))
    ref = np.einsum("irk,rjk->ijk", np.fft.fft(d["X0"].astype(float)), np.fft.fft(d["Y0"].astype(float)))
    assert rel(g["Z"], np.fft.ifft(ref).real) <= 8 * (2.0**-24 if precision == "fp32" else 2.0**-16)
    g["ctx"].close()
