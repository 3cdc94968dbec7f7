"""Host-side check of the adjoint's choice between kept states and checkpoints."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def keeps():
    from paper_2002_12717_amd import binding
    fn = binding.load().adj_keeps_states
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.c_int64, ctypes.c_size_t, ctypes.c_size_t, ctypes.c_size_t]
    return fn


def test_kept_states_follow_the_free_memory(keeps):
    state, total = 64 ** 4 * 16, 288 << 30                 # the 8x8 cluster on an empty device
    assert keeps(12, state, total, total)
    assert keeps(32, state, total, total)
    assert not keeps(33, state, total, total)              # more than 128 stage states
    need = (4 * 32 + 6) * state                            # every buffer of the gradient
    assert keeps(32, state, 4 * need, total)
    assert not keeps(32, state, 4 * need - 4, total)       # another program holds the rest
    assert not keeps(32, state, 8 << 30, total)            # checkpoints (7.5 GB) still fit
    assert keeps(12, state, total, 96 << 30)               # 12 GiB, an eighth of the device
    assert not keeps(12, state, total, (96 << 30) - 8)
    assert not keeps(1, state, 0, total)
    assert not keeps(0, state, total, total)
    assert not keeps(1 << 62, state, total, total)
