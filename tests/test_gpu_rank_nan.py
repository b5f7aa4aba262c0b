"""Ranks of large ensembles with depths that are not numbers: the values are
unspecified, the order is still a permutation, and numbers keep the order of
the definition among themselves."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_15187_amd as pid

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(rank, order, depth):
    n = depth.size
    rank, order = rank.cpu().numpy(), order.cpu().numpy()
    assert np.array_equal(np.sort(rank), np.arange(n))
    assert np.array_equal(order[rank], np.arange(n))
    num = ~np.isnan(depth)
    kept = order[num[order]]                       # the numbers, as ranked
    _, o = oracle.rank_order(depth[num])
    assert np.array_equal(kept, np.flatnonzero(num)[o])


@pytest.mark.parametrize("n", [2049, 4096, 16384, 16385])
def test_rank_entry_point(n):
    rng = np.random.Generator(np.random.PCG64(n))
    d = rng.integers(0, 600, size=n) / 600.0
    d[rng.integers(0, n, size=n // 7)] = np.nan
    d[rng.integers(0, n, size=5)] = np.inf
    d[rng.integers(0, n, size=5)] = -0.0
    _check(*pid.pid_rank(torch.from_numpy(d).to(DEV)), d)


@pytest.mark.parametrize("n", [2049, 16384, 16385])
def test_depth_call(n):
    U = torch.full((n, 8), 0.25, device=DEV)
    U[::3] = 0.5
    U[5, 2] = float("inf")
    r = pid.pid_mean(U)
    assert bool(r["depth"].isnan().any())
    _check(r["rank"], r["order"], r["depth"].cpu().numpy())
