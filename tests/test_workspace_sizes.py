"""Workspace sizes are part of the interface: programs keep a workspace of a stored size, and lordba_backward_noalloc refuses the shapes beyond
its array (no GPU: the sizes are computed, and the size check comes before anything else)."""
import ctypes

import pytest

from paper_2605_24058_amd import binding

SIZES = {
    "lordba_backward_workspace_bytes": {(1, 512, 384, 16): 122944, (2048, 4096, 4096, 16): 3145984, (8192, 13824, 5120, 16): 7831744,
                                        (300, 1000, 3001, 12): 721024, (8927, 4672, 2656, 26): 16778240},
    "lordba_backward_multi_workspace_bytes": {(2048, 5120, 5120, 32, 2): 9962240, (1500, 2208, 2016, 16, 3): 5801088, (70, 1024, 768, 32, 3): 360576},
    "lordba_ptq_workspace_bytes": {(4096, 4096, 16, 16): 4278272, (10, 14613, 15, 29): 8460800, (512, 300, 3, 4): 72448, (700, 1025, 16, 32): 1143552},
}


@pytest.mark.parametrize("name,shape", [(n, s) for n in SIZES for s in SIZES[n]], ids=str)
def test_sizes_are_what_they_were(name, shape):
    assert getattr(binding, name)(*shape) == SIZES[name][shape]


def test_a_shape_just_beyond_the_array_is_refused():
    T, d_in, d_out, r = 8927, 4672, 2656, 26   # 1024 bytes beyond it
    assert binding.lordba_backward_workspace_bytes(T, d_in, d_out, r) == binding.BACKWARD_NOALLOC_MAX_BYTES + 1024
    lib = binding.load_library()
    p = [0x10000000 + i * 0x1000000 for i in range(17)]   # (never touched)
    st = lib.lordba_backward_noalloc(*p[:10], ctypes.c_float(100.0), None, 0, *p[10:17], T, d_in, d_out, r, None)
    assert st == 9
