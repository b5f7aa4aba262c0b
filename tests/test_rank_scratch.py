"""The workspace holds scratch for the sorting ranks only where ranks are
sorted: more than 16384 members."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2512_15187_amd as pid
import synth


def _bytes(n, variant):
    lib = pid.load_library()
    e = pid.pid_ensemble(n, 64, 64, pid.PID_F32, 0, 0x1000, None)
    out = ctypes.c_size_t(0)
    assert lib.pid_workspace_size(ctypes.byref(e), None, variant, 0, ctypes.byref(out)) == pid.PID_OK
    return out.value


@pytest.mark.parametrize("n", [2048, 2049, 16384, 16385])
def test_scratch_bytes(n):
    """pid_both's workspace is that of pid_all_pairs and its own extras: two
    depth arrays, 512 bytes, and beyond 16384 members the rank scratch of both
    (a key, an index and a count per member, in tiles of 2048)."""
    tiles = -(-n // 2048) * 2048
    scratch = -(-(tiles * 12 + n * 4) // 256) * 256 if n > 16384 else 0
    extras = -(-n * 8 * 2 // 256) * 256 + 512 + 2 * scratch
    assert _bytes(n, 2) - -(-_bytes(n, 0) // 256) * 256 == extras


@pytest.mark.gpu
@pytest.mark.parametrize("n", [16384, 16385, 18432, 18433])
def test_ranks_on_both_sides(n):
    """Depth calls just below and above the first sorted size: exact ranks,
    with many ties (binary masks of few points)."""
    B = synth.random_binary(n, 24, n)
    r = pid.pid_mean(B.to("cuda:0"))
    rank, order = oracle.rank_order(oracle.binary_pid_mean(B.numpy())["depth"])
    assert np.array_equal(r["rank"].cpu().numpy(), rank)
    assert np.array_equal(r["order"].cpu().numpy(), order)
