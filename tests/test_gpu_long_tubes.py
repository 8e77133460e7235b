"""Long tubes in FP64 and with BF16 spectra (needs an MI355X): the reverse pass and the transforms
of the initial factors' adjoints against the oracle on the same stored iterates, and the first W~ of
mixed precision against the transform of W."""
import numpy as np
import pytest

from oracle import adjoint as AD
from tests.gpu_helpers import make_inputs, oracle, to_dev
from tests.test_gpu_adjoint import _from_complex_dev, _maxrel, _stored, _to_complex_dev

pytestmark = pytest.mark.gpu

LENGTHS = [
    (3, 4, 257, 2),      # direct sums
    (3, 4, 2046, 2),     # the longest pairs of few even tubes
    (3, 4, 2048, 2),     # sequences of half the length
    (2, 3, 4094, 2),     # the same with passes of radix 23 and 89
    (2, 3, 4725, 2),     # pairs in more than 64 KB of LDS
    (2, 3, 8192, 2),     # the longest
]


def _iterate(blob, n1, n2, n3, r):
    """The oracle's state at a checkpoint's FP32 iterate."""
    nb = n3 // 2 + 1
    b = blob.cpu().numpy()[72:]
    nx, ny = 8 * nb * r * n1, 8 * nb * r * n2

    def full(half):   # [nb] first -> all n3 frequencies last
        half = np.moveaxis(half.astype(complex), 0, 2)
        return np.concatenate([half, np.conj(half[:, :, 1:(n3 + 1) // 2][:, :, ::-1])], axis=2)

    x = b[:nx].view(np.complex64).reshape(nb, r, n1)
    y = b[nx:nx + ny].view(np.complex64).reshape(nb, r, n2)
    w = b[nx + ny:nx + ny + 8 * n1 * nb * n2].view(np.complex64).reshape(n1, nb, n2)
    wt = full(np.moveaxis(w, 1, 0))
    return oracle.State(full(np.swapaxes(x, 1, 2)), full(y), oracle.idft3(wt).real, wt)


@pytest.mark.parametrize("n1,n2,n3,r", LENGTHS)
def test_reverse_pass_at_long_tubes(n1, n2, n3, r):
    """1e-12 for the FP64 transforms back to X0 and Y0 alone, and the tolerance of the one-iteration
    test at the differentiation shape, from the stored iterates: at r near n1 the least Gram
    eigenvalue of thousands of frequencies amplifies the forward's own FP32 rounding past it."""
    import torch
    from paper_2005_09838_amd import Completion, binding as B
    d = make_inputs(n1, n2, n3, r, p=0.4, seed=n1 + n2 + n3, weekly=True, sigma_od=1.0, noise=0.02)
    nb = n3 // 2 + 1
    rng = np.random.default_rng(n1 * n2 + n3)
    print(f"{n1}x{n2}x{n3} r{r}", flush=True)
    c = Completion(to_dev(d["G"]), to_dev(d["omega"]), r, rho1=0.3, rho2=0.7, X0=to_dev(d["X0"]), Y0=to_dev(d["Y0"]))
    s0 = c.get_state()
    c.step(1)
    s1 = c.get_state()
    xb = oracle.dft3(rng.normal(size=(n1, r, n3)))
    yb = oracle.dft3(rng.normal(size=(r, n2, n3)))
    wb = rng.normal(size=(n1, n2, n3))
    xt_bar = _to_complex_dev(_stored(xb, (2, 1, 0)))
    yt_bar = _to_complex_dev(_stored(yb, (2, 0, 1)))
    x0_bar = torch.empty((n1, r, n3), dtype=torch.float64, device="cuda:0")
    y0_bar = torch.empty((r, n2, n3), dtype=torch.float64, device="cuda:0")
    B.tctf_adjoint_initial(c.ctx, xt_bar, yt_bar, x0_bar, y0_bar)
    # sum over all frequencies of Re(X_b exp(-2 pi i b l / n3))
    assert _maxrel(x0_bar.cpu().numpy(), np.fft.fft(xb, axis=2).real) <= 1e-12
    assert _maxrel(y0_bar.cpu().numpy(), np.fft.fft(yb, axis=2).real) <= 1e-12
    w_bar = torch.from_numpy(wb.copy()).to("cuda:0")
    th = torch.zeros(3, dtype=torch.float64, device="cuda:0")
    ws, nbytes = c.adjoint_workspace()
    B.tctf_adjoint_step(c.ctx, s0, s1, xt_bar, yt_bar, w_bar, th, ws, nbytes)
    prob = oracle.Problem(d["G"], d["omega"], r, 1e-2, 0.3, 0.7, 1.0)
    st0, st1 = _iterate(s0, n1, n2, n3, r), _iterate(s1, n1, n2, n3, r)
    tb = AD.ThetaBar()
    ox, oy, ow = AD.iterate_adjoint(prob, st0, st1, xb, yb, wb, tb)
    gx, gy = _from_complex_dev(xt_bar, (nb, r, n1)), _from_complex_dev(yt_bar, (nb, r, n2))
    ot, gt = tb.as_array(), th.cpu().numpy()
    # X0 = 0 and eta = 1: X~_bar is 0
    ex = float(np.abs(gx - _stored(ox, (2, 1, 0))).max()) / max(1.0, float(np.abs(xb).max()))
    ey, ew = _maxrel(gy, _stored(oy, (2, 0, 1))), _maxrel(w_bar.cpu().numpy(), ow)
    et = np.abs(gt - ot) / np.maximum(np.abs(ot), 1e-3 * np.abs(ot).max())
    print(f"X~ {ex:.2e} Y~ {ey:.2e} W {ew:.2e} theta {et}", flush=True)
    assert ex <= 1e-12 and ey <= 1e-5 and ew <= 1e-5 and np.all(et <= 1e-5), (ex, ey, ew, et)
    c.close()


@pytest.mark.parametrize("n1,n2,n3,r", LENGTHS)
def test_first_bf16_spectrum_at_long_tubes(n1, n2, n3, r):
    """W~ of P_Omega(G): every stored part lies within one BF16 step (2^-7 of it) of the FP64
    transform, and FP32 rounding of the value before it (2^-23 of the largest entry)."""
    from paper_2005_09838_amd import Completion
    d = make_inputs(n1, n2, n3, r, p=0.4, seed=n1 + n2 + n3, weekly=True, sigma_od=1.0, noise=0.02)
    print(f"{n1}x{n2}x{n3} r{r}", flush=True)
    nb = n3 // 2 + 1
    c = Completion(to_dev(d["G"]), to_dev(d["omega"]), r, X0=to_dev(d["X0"]), Y0=to_dev(d["Y0"]), precision="mixed")
    blob = c.get_state().cpu().numpy()
    at = 72 + 8 * nb * r * (n1 + n2)
    words = blob[at:at + 4 * n1 * nb * n2].view(np.uint32).reshape(n1, nb, n2)
    re = (words << 16).view(np.float32).astype(float)
    im = (words & 0xffff0000).view(np.float32).astype(float)
    ref = np.transpose(oracle.dft3(np.where(d["omega"] > 0, d["G"], 0.0))[:, :, :nb], (0, 2, 1))
    for got, exact in ((re, ref.real), (im, ref.imag)):
        err = np.abs(got - exact) - 2.0**-7 * np.abs(exact)
        assert err.max() <= 2.0**-23 * np.abs(ref).max(), (err.max(), np.abs(ref).max())
    c.close()
