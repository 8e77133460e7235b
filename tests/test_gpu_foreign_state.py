"""Checkpoint blobs of another problem (needs an MI355X): refused, with the context untouched."""
import pytest

from tests.gpu_helpers import make_inputs, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("word", range(7))    # magic (two words), n1, n2, n3, r, precision
@pytest.mark.parametrize("shift", [0, 4, 2])  # one launch, one launch with narrow words, copy calls
def test_a_foreign_blob_leaves_the_context_alone(word, shift):
    import torch
    from paper_2005_09838_amd import Completion, binding as B
    d = make_inputs(7, 9, 5, 2, p=0.4, seed=3, weekly=True, sigma_od=1.0, noise=0.02)
    c = Completion(to_dev(d["G"]), to_dev(d["omega"]), 2, X0=to_dev(d["X0"]), Y0=to_dev(d["Y0"]))
    blob = c.get_state()
    c.step(3)
    before = c.get_state()
    n = blob.numel()
    buf = torch.zeros(n + 64, dtype=torch.uint8, device="cuda:0")
    buf[shift:shift + n] = blob
    buf[shift + 4 * word] ^= 1
    with pytest.raises(B.TctfError) as e:
        B.tctf_set_state(c.ctx, buf.data_ptr() + shift, n)
    assert e.value.status == B.TCTF_E_STATE
    assert c.iterations == 3 and torch.equal(c.get_state(), before)
    c.step(2)
    w = c.result()["W"]
    c.set_state(before)
    c.step(2)
    assert torch.equal(c.result()["W"], w)
    buf[shift + 4 * word] ^= 1   # and the right one is taken
    B.tctf_set_state(c.ctx, buf.data_ptr() + shift, n)
    assert c.iterations == 0 and torch.equal(c.get_state(), blob)
    c.close()
