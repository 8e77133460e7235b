"""Many rows, few columns and large ranks: G_X in row groups, X-update blocks whose column tiles
outnumber the columns of W~, and inverses hosted by slice blocks of short rows (needs an MI355X)."""
import numpy as np
import pytest

from tests.gpu_helpers import gpu_run, make_inputs, oracle_run
from tests.test_gpu_parity import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,n3,r,pinv_mode", [
    (383, 24, 5, 17, 0),     # one block per Gram: less than four groups
    (384, 24, 5, 17, 0),     # four groups of 96 rows
    (389, 33, 3, 32, 0),     # a short last group, the largest rank
    (1001, 20, 7, 18, 1),    # ten groups before the eigen route
    (1999, 12, 34, 9, 1),    # 18 frequencies, up to r = 16: one block ...
    (2000, 12, 34, 9, 1),    # ... and groups from 2000 rows on by the eigen route
    (600, 20, 126, 20, 0),   # 64 frequencies: four groups each
    (600, 20, 128, 20, 0),   # 65: one block each
    (1999, 6, 5, 4, 0),      # up to r = 16 one block ...
    (2000, 6, 5, 4, 0),      # ... and groups from 2000 rows on
    (2049, 18, 3, 18, 0),    # idle wavefronts in slice blocks of more than 2048 rows
    (2049, 14, 4, 13, 0),
    (2049, 12, 4, 12, 0),
    (40, 9, 6, 9, 0),        # two column tiles, one run of columns
    (40, 33, 7, 32, 0),      # four
])
def test_tall_and_wide_rank(n1, n2, n3, r, pinv_mode):
    d = make_inputs(n1, n2, n3, r, p=0.7, seed=n1 + n2 + n3 + r, sigma_od=1.0, noise=0.02)
    print(f"{n1}x{n2}x{n3} r{r} pinv_mode {pinv_mode}", flush=True)
    g = gpu_run(d, r, 3, pinv_mode=pinv_mode, eta=0.9)
    st, info = oracle_run(d, r, 3, eta=0.9, history=True)
    _compare(g, st, info, label=f"{n1}x{n2}x{n3} r{r}")
    s = g["ctx"].stationarity()
    assert s[1] < 1e-5 and s[2] == 0.0


def test_stage_timing_with_row_groups_leaves_the_iterate_unchanged():
    """The partial Grams lie in Z~'s buffer: any order of timed stages goes on to the same bits."""
    d = make_inputs(500, 24, 6, 20, p=0.6, seed=7)
    a = gpu_run(d, 20, 9)
    c = gpu_run(d, 20, 4)["ctx"]
    for st in (4, 0, 4, 1, 5, 6):
        assert c.time_stage(st, reps=2) > 0.0
    c.step(5)
    assert np.array_equal(c.result()["W"].cpu().numpy(), a["W"].astype(np.float32))
    assert c.objective() == a["ctx"].objective()
