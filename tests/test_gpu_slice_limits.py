"""The largest slices that the fused kernel takes, by tube length (needs an MI355X): the launch asks
for up to 160 KB of LDS there.  Against the FP64 oracle with the tolerances of the parity tests,
through the iteration, the results and the stationarity measures."""
import pytest

from tests.gpu_helpers import gpu_run, make_inputs, oracle, oracle_run
from tests.test_gpu_parity import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n2,n3", [(264, 128), (301, 112), (349, 96), (395, 84), (508, 64), (574, 56), (657, 48),
                                   (770, 40), (931, 32), (1024, 28)])
def test_largest_fused_slices(n2, n3):
    d = make_inputs(2, n2, n3, 2, p=0.4, seed=n2 + n3, weekly=True, sigma_od=1.0, noise=0.02)
    print(f"2x{n2}x{n3}", flush=True)
    g = gpu_run(d, 2, 4)
    assert g["ctx"].tuning()[0] != 3   # not the three-launch path
    st, info = oracle_run(d, 2, 4, history=True)
    _compare(g, st, info, label=f"2x{n2}x{n3}")
    s = g["ctx"].stationarity()
    so = oracle.stationarity(info["problem"], st)
    assert abs(s[0] - so["factor"]) <= 1e-3 * so["factor"] + 1e-7, (s, so)
    assert s[1] < 1e-5 and s[2] == 0.0
