"""Contexts whose launches are the same kernels at different LDS sizes, in turn and from two threads
(needs an MI355X): each gives the bits that it gives alone."""
import threading

import pytest

from tests.gpu_helpers import make_inputs, to_dev

pytestmark = pytest.mark.gpu


def _make(n1, n2, n3, r, precision="fp32", stream=None):
    from paper_2005_09838_amd import Completion
    d = make_inputs(n1, n2, n3, r, p=0.4, seed=n1 + n2 + n3, weekly=True, sigma_od=1.0, noise=0.02)
    return Completion(to_dev(d["G"]), to_dev(d["omega"]), r, X0=to_dev(d["X0"]), Y0=to_dev(d["Y0"]), precision=precision,
                      stream=stream)


PAIRS = [
    ((2, 349, 96, 2), (2, 300, 96, 2)),      # slices of 157 and 135 KB
    ((3, 3, 8191 - 2, 2), (3, 3, 4725, 2)),  # tubes of 128 and 74 KB (8189 is prime: direct sums)
    ((3, 3, 7875, 2), (3, 3, 4725, 2)),      # tubes of 123 and 74 KB
    ((40, 300, 4, 32), (40, 180, 4, 32)),    # X-update and Gram blocks of rank 32
]


@pytest.mark.parametrize("big,small", PAIRS)
def test_interleaved_sizes(big, small):
    import torch
    print(f"{big} {small}", flush=True)
    alone = []
    for shape in (big, small):
        c = _make(*shape)
        c.step(13)
        alone.append(c.result()["W"])
        c.close()
    a, b = _make(*big), _make(*small)   # the smaller size is set up last
    for _ in range(13):
        a.step(1)
        b.step(1)
    assert torch.equal(a.result()["W"], alone[0]) and torch.equal(b.result()["W"], alone[1])
    a.close()
    b.close()


@pytest.mark.parametrize("big,small", PAIRS)
def test_sizes_from_two_threads(big, small):
    import torch
    print(f"{big} {small}", flush=True)
    alone, ctx, out, errors = [], [], [None, None], []
    for shape in (big, small):
        c = _make(*shape)
        c.step(33)
        alone.append(c.result()["W"])
        c.close()
        s = torch.cuda.Stream()
        torch.cuda.synchronize()
        ctx.append(_make(*shape, stream=s))

    def run(k):
        try:
            for n in (1, 1, 1, 30):
                ctx[k].step(n)
            out[k] = ctx[k].result()["W"]
        except Exception as e:  # pragma: no cover
            errors.append(e)

    threads = [threading.Thread(target=run, args=(k,)) for k in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    torch.cuda.synchronize()
    assert not errors, errors
    assert torch.equal(out[0], alone[0]) and torch.equal(out[1], alone[1])
    for c in ctx:
        c.close()
