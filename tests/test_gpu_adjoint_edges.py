"""One iteration's reverse pass at the edges of its row and column solves (needs an MI355X).

The W-step adjoint splits a row into segments of up to 9, 12 or 16 columns, the H_rho1 solves a
column into 64 entries at a time.  Against the FP64 oracle, with the tolerance of the
one-iteration test at the differentiation shape.
"""
import numpy as np
import pytest

from oracle import adjoint as AD
from tests.gpu_helpers import make_inputs, oracle, to_dev
from tests.test_gpu_adjoint import _from_complex_dev, _maxrel, _stored, _to_complex_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,n3,r,rho2", [
    (1, 9, 5, 1, 0.7),       # a single row of H_rho1; one segment of 9
    (64, 10, 12, 2, 0.7),    # one full chunk of a column; a segment of 10
    (65, 16, 9, 2, 0.7),     # a second chunk of one entry; one full segment of 16
    (130, 17, 6, 3, 1e-2),   # two segments, uneven
    (5, 130, 28, 2, 0.7),    # sixteen segments, the last ones short
    (4, 300, 20, 2, 0.7),    # 32 segments of 10: the last two without columns
    (6, 1024, 3, 2, 0.7),    # 64 full segments
    (7, 40, 70, 2, 0.0),     # the three-launch slice path's packed order; no coupling
    (300, 3, 1, 2, 1e-2),    # a single frequency, short rows
])
def test_one_iteration_adjoint_edges(n1, n2, n3, r, rho2):
    import torch
    from paper_2005_09838_amd import Completion, binding as B
    d = make_inputs(n1, n2, n3, r, p=0.4, seed=n1 + n2 + n3, weekly=True, sigma_od=1.0, noise=0.02)
    nb = n3 // 2 + 1
    rng = np.random.default_rng(n1 * n2 + n3)
    print(f"{n1}x{n2}x{n3} r{r} rho2 {rho2}", flush=True)
    c = Completion(to_dev(d["G"]), to_dev(d["omega"]), r, rho1=0.3, rho2=rho2, X0=to_dev(d["X0"]), Y0=to_dev(d["Y0"]))
    s0 = c.get_state()
    c.step(1)
    s1 = c.get_state()
    xb = oracle.dft3(rng.normal(size=(n1, r, n3)))
    yb = oracle.dft3(rng.normal(size=(r, n2, n3)))
    wb = rng.normal(size=(n1, n2, n3))
    xt_bar = _to_complex_dev(_stored(xb, (2, 1, 0)))
    yt_bar = _to_complex_dev(_stored(yb, (2, 0, 1)))
    w_bar = torch.from_numpy(wb.copy()).to("cuda:0")
    th = torch.zeros(3, dtype=torch.float64, device="cuda:0")
    ws, nbytes = c.adjoint_workspace()
    B.tctf_adjoint_step(c.ctx, s0, s1, xt_bar, yt_bar, w_bar, th, ws, nbytes)
    prob = oracle.Problem(d["G"], d["omega"], r, 1e-2, 0.3, rho2, 1.0)
    st0 = oracle.initial_state(prob, d["X0"], d["Y0"])
    st1 = oracle.iterate(prob, st0)
    tb = AD.ThetaBar()
    ox, oy, ow = AD.iterate_adjoint(prob, st0, st1, xb, yb, wb, tb)
    gx, gy = _from_complex_dev(xt_bar, (nb, r, n1)), _from_complex_dev(yt_bar, (nb, r, n2))
    ot, gt = tb.as_array(), th.cpu().numpy()
    # X0 = 0 and eta = 1: X~_bar is 0
    ex = float(np.abs(gx - _stored(ox, (2, 1, 0))).max())
    ey, ew = _maxrel(gy, _stored(oy, (2, 0, 1))), _maxrel(w_bar.cpu().numpy(), ow)
    et = np.abs(gt - ot) / np.maximum(np.abs(ot), 1e-3 * np.abs(ot).max())
    print(f"X~ {ex:.2e} Y~ {ey:.2e} W {ew:.2e} theta {et}", flush=True)
    assert ex <= 1e-12 and ey <= 1e-5 and ew <= 1e-5 and np.all(et <= 1e-5), (ex, ey, ew, et)
    c.close()
