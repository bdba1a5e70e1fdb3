"""The scratch of lordba_backward must not grow past the library's own array (lordba_backward_noalloc) on shapes that fitted it: the
sizes of some shapes close to the limit, on the host (no GPU)."""
import pytest

from paper_2605_24058_amd import binding


# (T, d_in, d_out, r): long batches at ranks above 32 whose token ranges, dealt in pieces of 32 rows, would need more than the array
@pytest.mark.parametrize("shape", [(4141, 128, 1664, 48), (4141, 128, 5504, 48), (4141, 128, 8704, 48), (4019, 512, 512, 64), (2048, 4096, 4096, 64), (8192, 13824, 5120, 16)])
def test_fits_the_librarys_own_array(shape):
    assert binding.lordba_backward_workspace_bytes(*shape) <= binding.BACKWARD_NOALLOC_MAX_BYTES
