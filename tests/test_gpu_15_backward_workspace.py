"""What the backward's workspace holds per slice (a question to the library that needs a device: which kernels run follows from its LDS), from its size at two large batches: the gradient rows and dL/dp of the k assignments, dL/dg of
the expert tiles (two or three bf16 terms), and the ReLU pattern (256 bits) only where two kernels hand it over -- where one kernel does both
halves of the router's backward it stays in registers."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ds,E,terms,one_kernel", [(24, 16, 3, True), (24, 64, 3, True), (48, 16, 3, True), (48, 64, 3, True), (64, 32, 2, True),
                                                   (64, 64, 2, True), (96, 32, 2, True), (96, 33, 2, False), (128, 32, 2, False),
                                                   (128, 64, 2, False), (192, 32, 3, False)])
def test_bytes_per_slice(ds, E, terms, one_kernel):
    from paper_2510_04286_amd import binding as B
    k, n0, n1 = 2, 1 << 20, 3 << 20   # (beyond the sizes at which partial sums and capacity sums grow with the batch)
    size = [B.lib().slicemoe_backward_workspace_bytes(B.make_config(n, ds, 1, k, E, 4 * ds)) for n in (n0, n1)]
    assert (size[1] - size[0]) == (n1 - n0) * (k * (4 * ds + 4) + terms * 2 * 32 * ((E + 31) // 32) + (0 if one_kernel else 32))
