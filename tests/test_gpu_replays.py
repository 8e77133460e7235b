"""Graph replays of the three-launch slice path and its long tubes (needs an MI355X)."""
import numpy as np
import pytest

from tests.gpu_helpers import make_inputs, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,n3,r", [
    (5, 6, 90, 2),       # several pairs per block
    (9, 8, 67, 2),       # direct sums
    (2, 3, 2048, 2),     # sequences of half the length
    (3, 5, 4094, 2),     # the same with passes of radix 23 and 89
    (2, 3, 4725, 2),     # pairs in more than 64 KB of LDS: the limit is raised during capture
    (150, 2, 4100, 2),   # the same at an even length: too many tubes for halves
    (2, 2, 8192, 2),     # the longest
])
@pytest.mark.parametrize("precision", ["fp32", "mixed"])
def test_replays_of_the_three_launch_path(n1, n2, n3, r, precision):
    """53 iterations in two calls (ten eager, two replays, three eager; two replays), with the
    caller's own work and reads between them, against 53 calls of one: the same bits."""
    import torch
    from paper_2005_09838_amd import Completion
    d = make_inputs(n1, n2, n3, r, p=0.4, seed=n1 + n2 + n3, weekly=True, sigma_od=1.0, noise=0.02)
    print(f"{n1}x{n2}x{n3} r{r} {precision}", flush=True)
    mk = lambda: Completion(to_dev(d["G"]), to_dev(d["omega"]), r, X0=to_dev(d["X0"]), Y0=to_dev(d["Y0"]),
                            precision=precision)
    a, b = mk(), mk()
    a.step(33)
    assert np.isfinite(a.objective())
    junk = torch.rand(1 << 20, device="cuda:0").cumsum(0)
    w33 = a.result()["W"]
    a.step(20)
    for _ in range(33):
        b.step(1)
    assert torch.equal(b.result()["W"], w33)
    for _ in range(20):
        b.step(1)
    ra, rb = a.result(Z=True, X=True, Y=True), b.result(Z=True, X=True, Y=True)
    assert all(torch.equal(ra[k], rb[k]) for k in ra)
    assert a.objective() == b.objective() and a.iterations == b.iterations == 53
    assert bool(torch.isfinite(junk).all())
    a.close()
    b.close()


@pytest.mark.parametrize("n1,n2,n3,r,iters", [(300, 14, 5, 3, 33), (529, 96, 112, 16, 30)])
def test_two_replays_against_the_oracle(n1, n2, n3, r, iters):
    """Ten eager iterations and two replays of ten (and the rest eager) in one call."""
    from tests.gpu_helpers import gpu_run, oracle, oracle_run
    from tests.test_gpu_parity import _compare
    d = make_inputs(n1, n2, n3, r, p=0.4, seed=3005, weekly=True, sigma_od=1.0, noise=0.02)
    g = gpu_run(d, r, iters)
    st, info = oracle_run(d, r, iters)
    info["f0"] = [oracle.objective(info["problem"], st)]
    _compare(g, st, info, label=f"{n1}x{n2}x{n3} r{r}, {iters} iterations")
