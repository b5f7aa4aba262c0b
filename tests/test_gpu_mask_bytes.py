"""PID-mean of U8 masks whose set points hold any nonzero byte (masks drawn as
0/255, labels): a nonzero byte counts as 1, as in pid_pack_bits, in the one-pass
and the two-pass kernels, inside and at the ragged end of rows of any address."""
import pytest
import torch

import paper_2512_15187_amd as pid

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("n,m", [(5, 7), (50, 2048 * 2 + 37), (200, 2048 + 31), (200, 4096)])
def test_nonzero_bytes(n, m, off):
    g = torch.Generator(device=DEV)
    g.manual_seed(n + m)
    V = torch.randint(0, 256, (n, m + 4), generator=g, device=DEV, dtype=torch.uint8)
    V *= torch.randint(0, 2, (n, m + 4), generator=g, device=DEV, dtype=torch.uint8)
    U = V[:, off:off + m]
    B = (U != 0).to(torch.uint8)
    r, e, p = pid.pid_mean(U), pid.pid_mean(B), pid.pid_mean(pid.pid_pack_bits(U))
    assert torch.equal(e["mass"], B.to(torch.float64).sum(1))
    for k in ("mass", "in_in", "in_out", "depth", "rank", "order"):
        assert torch.equal(r[k], e[k]) and torch.equal(p[k], e[k]), k
