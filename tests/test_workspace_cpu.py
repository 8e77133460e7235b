"""Workspace sizes, computed on the host."""
import pytest


@pytest.mark.parametrize("n1,n2,n3,r", [(144, 288, 28, 8), (529, 96, 112, 16), (300, 64, 32, 4)])
def test_the_three_launch_path_holds_two_spatial_tensors(n1, n2, n3, r):
    """An autotuned context of a fused size also holds the three-launch path's buffers: spatial Z
    and W, and beside them only partial sums, roots and the Y-step's further Gram partials (columns
    blocks of 8)."""
    from paper_2005_09838_amd import binding as B
    more = (B.tctf_workspace_bytes(B.make_params(n1, n2, n3, r, autotune=True)) -
            B.tctf_workspace_bytes(B.make_params(n1, n2, n3, r)))
    nb, tensor = n3 // 2 + 1, 4 * n1 * n2 * n3
    grams = nb * -(-n2 // 8) * r * r * 16
    # at most one block per OD row and four rows of it in the W-step; roots; rounding to 256 bytes
    small = 24 * n1 * -(-n3 // 4) + 16 * n3 + 8 * 256
    assert 2 * tensor <= more <= 2 * tensor + grams + small
