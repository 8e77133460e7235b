"""The X-update of mixed precision from the context's own stored operands (needs an MI355X).

One iteration with full-rank Grams and eta = 1 gives X~ = H_rho1^{-1} W~ Y~^* G_Y^{-1}.  W~ is taken
in BF16 as it is stored and Y~ as a high and a low BF16 part, which keep it to 2^-18; the sums are
FP32 over at most 48 columns (below 2^-20).  G_Y^{-1} of a normal Y0 at these sizes amplifies by
less than 8, so X~ is within 2^-14 of the FP64 result from the same operands, in norm; one row, with
fewer terms to average, within 2^-13.  Without the low parts the error would be near 2^-9."""
import numpy as np
import pytest

from tests.gpu_helpers import make_inputs, to_dev

pytestmark = pytest.mark.gpu


def _state(blob, n1, n2, n3, r):
    nb = n3 // 2 + 1
    b = blob.cpu().numpy()[72:]
    nx, ny = 8 * nb * r * n1, 8 * nb * r * n2
    x = b[:nx].view(np.complex64).reshape(nb, r, n1).astype(complex)
    y = b[nx:nx + ny].view(np.complex64).reshape(nb, r, n2).astype(complex)
    w = b[nx + ny:nx + ny + 4 * n1 * nb * n2].view(np.uint32).reshape(n1, nb, n2)
    wt = (w << 16).view(np.float32).astype(float) + 1j * (w & 0xffff0000).view(np.float32).astype(float)
    return x, y, wt


@pytest.mark.parametrize("n1,n2,n3,r,rho1", [
    (22, 48, 3, 8, 1e-2),    # one pass of 48 columns
    (23, 49, 3, 7, 1e-2),    # a second wavefront column with one column
    (32, 97, 4, 16, 0.0),    # three wavefront columns
    (40, 300, 3, 8, 0.1),    # two passes
    (20, 1000, 2, 5, 1e-2),  # three passes of eight wavefront columns
    (55, 17, 80, 3, 1e-2),
    (70, 90, 5, 17, 1e-2),   # the right-hand side and the separate solve
    (45, 200, 4, 32, 0.3),
    (1200, 10, 56, 2, 1e-2), # 64-row blocks
])
def test_mixed_x_update_from_stored_operands(n1, n2, n3, r, rho1):
    from paper_2005_09838_amd import Completion
    d = make_inputs(n1, n2, n3, r, p=0.5, seed=n1 + n2 + r, sigma_od=1.0, noise=0.02)
    print(f"{n1}x{n2}x{n3} r{r} rho1 {rho1}", flush=True)
    c = Completion(to_dev(d["G"]), to_dev(d["omega"]), r, rho1=rho1, X0=to_dev(d["X0"]), Y0=to_dev(d["Y0"]),
                   precision="mixed")
    _, y, wt = _state(c.get_state(), n1, n2, n3, r)
    c.step(1)
    x1, _, _ = _state(c.get_state(), n1, n2, n3, r)
    diff = np.eye(n1)[1:] - np.eye(n1)[:-1]
    h = np.eye(n1) + rho1 * diff.T @ diff
    for b in range(n3 // 2 + 1):
        yh = y[b].conj().T
        ref = np.linalg.solve(h, wt[:, b] @ yh @ np.linalg.inv(y[b] @ yh))   # n1 x r
        if b == 0 or 2 * b == n3:
            ref = ref.real
        err = x1[b].T - ref
        assert np.linalg.norm(err) <= 2.0**-14 * np.linalg.norm(ref), b
        rows, size = np.linalg.norm(err, axis=1), np.linalg.norm(ref, axis=1)
        assert np.all(rows <= 2.0**-13 * np.maximum(size, np.sqrt(np.mean(size**2)))), b
    c.close()
