"""Packing of G and the checkpoint copies at the edges of their segments and alignments (needs an
MI355X)."""
import numpy as np
import pytest

from tests.gpu_helpers import make_inputs, oracle_run, rel, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,n3", [
    (3, 16, 5),      # one full segment
    (2, 17, 28),     # two, uneven
    (2, 290, 7),     # 32 segments of 10: the last three without columns
    (2, 1024, 3),    # 64 full segments
    (2, 33, 70),     # G's own order
])
@pytest.mark.parametrize("p", [0.0, 0.03, 1.0])
def test_pack_edges(n1, n2, n3, p):
    """Rows with runs across several segments, without an observed entry and fully observed: the
    W-step at strong coupling against the oracle (FP32 tolerance of the parity tests), and a
    non-finite observed entry in the last column is refused."""
    import torch
    from paper_2005_09838_amd import Completion, binding as B
    d = make_inputs(n1, n2, n3, 2, p=p, seed=n1 + n2 + n3, weekly=True, sigma_od=1.0, noise=0.02)
    print(f"{n1}x{n2}x{n3} p {p}", flush=True)
    c = Completion(to_dev(d["G"]), to_dev(d["omega"]), 2, rho2=0.9, X0=to_dev(d["X0"]), Y0=to_dev(d["Y0"]))
    c.step(2)
    W = c.result(W=True)["W"].cpu().numpy()
    st, _ = oracle_run(d, 2, 2, rho2=0.9)
    assert rel(W, st.w) <= 1e-5
    c.close()
    if p > 0:
        g, om = d["G"].copy(), d["omega"].copy()
        g[-1, -1, -1], om[-1, -1, -1] = np.inf, 1
        with pytest.raises(B.TctfError) as e:
            Completion(to_dev(g), to_dev(om), 2, Y0=to_dev(d["Y0"]))
        assert e.value.status == B.TCTF_E_NONFINITE


@pytest.mark.parametrize("shift", [0, 8, 4, 2])
def test_state_copies_at_any_alignment(shift):
    """Bytes equal to those of an aligned blob, and a bitwise equal continuation from them."""
    import torch
    from paper_2005_09838_amd import Completion, binding as B
    d = make_inputs(7, 9, 5, 2, p=0.4, seed=3, weekly=True, sigma_od=1.0, noise=0.02)   # nb = 3: odd words
    c = Completion(to_dev(d["G"]), to_dev(d["omega"]), 2, X0=to_dev(d["X0"]), Y0=to_dev(d["Y0"]))
    c.step(3)
    ref = c.get_state()
    n = ref.numel()
    buf = torch.full((n + 64,), 0x5a, dtype=torch.uint8, device="cuda:0")
    B.tctf_get_state(c.ctx, buf.data_ptr() + shift, n)
    used = shift + int(B.tctf_state_bytes(c.ctx))
    assert torch.equal(buf[shift:used], ref)
    assert bool((buf[:shift] == 0x5a).all()) and bool((buf[used:] == 0x5a).all())
    c.step(2)
    w = c.result(W=True)["W"]
    B.tctf_set_state(c.ctx, buf.data_ptr() + shift, n)
    c.step(2)
    assert torch.equal(c.result(W=True)["W"], w)
    c.close()
