"""Observed values that are not finite, on every slice path (needs an MI355X)."""
import numpy as np
import pytest

from tests.gpu_helpers import make_inputs, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,n3", [
    (3, 16, 5),     # fused, one thread per tube
    (2, 20, 56),    # fused, lanes share a tube
    (2, 17, 70),    # three launches: the pivot table is read from memory
])
@pytest.mark.parametrize("bits", [0x7fffffff, 0xffffffff, 0x7f800001, 0x7fc00000, 0x7f800000])
def test_observed_nan_of_any_payload_is_refused(n1, n2, n3, bits):
    """A NaN's payload is no index into the pivot table: the kernels that create launches before
    it reads the flag stay inside the table, and a context made next to it is right."""
    from paper_2005_09838_amd import Completion, binding as B
    d = make_inputs(n1, n2, n3, 2, p=0.5, seed=n2, weekly=True, sigma_od=1.0, noise=0.02)
    g, om = d["G"].copy(), d["omega"].copy()
    for at in ((0, 0, 0), (-1, -1, -1), (0, n2 // 2, n3 - 1)):
        g[at], om[at] = np.array(bits, np.uint32).view(np.float32), 1
    print(f"{n1}x{n2}x{n3} {bits:08x}", flush=True)
    with pytest.raises(B.TctfError) as e:
        Completion(to_dev(g), to_dev(om), 2, Y0=to_dev(d["Y0"]))
    assert e.value.status == B.TCTF_E_NONFINITE
    c = Completion(to_dev(d["G"]), to_dev(d["omega"]), 2, Y0=to_dev(d["Y0"]))
    c.step(1)
    obs = d["omega"].astype(bool)
    assert np.array_equal(c.result()["W"].cpu().numpy()[obs], d["G"][obs])
    c.close()
