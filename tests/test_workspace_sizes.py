"""Workspace queries against the receive buffers of the kernels that run all rounds in one launch (host only): one
workgroup is one wave of 64 lanes per party and, for every ordered pair of parties, keeps `rows` words per lane, whether
or not the lane has an element of its own."""
import os

import pytest

LANES, WORD = 64, 8
PAIRS = {2: 2, 3: 6}


@pytest.fixture(scope="module")
def lib():
    from paper_2209_13643_amd import mpc
    if not os.path.exists(mpc.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    return mpc.lib()


def buffers(parties, elements, words_per_lane):
    """Bytes of the receive buffers of `elements` elements at one element per lane (up to 66 elements: every call here
    is far below the sizes where a workgroup takes a second tile)."""
    return (elements + LANES - 1) // LANES * PAIRS[parties] * words_per_lane * LANES * WORD


@pytest.mark.parametrize("n_out", list(range(1, 67)))
def test_maxpool_backward_query_holds_the_receive_buffers(lib, n_out):
    # two rows of two words per lane (the pair of first-level products)
    assert lib.mpc_maxpool_backward_workspace_bytes(1, 2, 2, n_out) >= buffers(2, n_out, 4)
    assert lib.mpc_maxpool3_backward_workspace_bytes(1, 2, 2, n_out) >= buffers(3, n_out, 4)


@pytest.mark.parametrize("n", list(range(1, 67)))
def test_other_queries_hold_the_receive_buffers(lib, n):
    assert lib.mpc_relu_workspace_bytes(n) >= buffers(2, n, 4) and lib.mpc_relu3_workspace_bytes(n) >= buffers(3, n, 4)
    assert lib.mpc_relu_msb_workspace_bytes(n) >= buffers(2, n, 4) and lib.mpc_relu3_msb_workspace_bytes(n) >= buffers(3, n, 4)
    assert lib.mpc_mul_workspace_bytes(n) >= buffers(2, n, 2) and lib.mpc_mul3_workspace_bytes(n) >= buffers(3, n, 2)
    # four rows of the first level's pairs
    for q in (lib.mpc_maxpool_workspace_bytes, lib.mpc_maxpool_msb_workspace_bytes):
        assert q(1, 2, 2, n) >= buffers(2, n, 8)
    for q in (lib.mpc_maxpool3_workspace_bytes, lib.mpc_maxpool3_msb_workspace_bytes):
        assert q(1, 2, 2, n) >= buffers(3, n, 8)
