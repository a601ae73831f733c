"""The bf16 Gram pass on the matrix cores (seven tasks and more): buckets at
the edges of its tiles and chunks against float64 sums, and non-finite,
subnormal and huge values staying in their own rows."""

import numpy as np
import pytest
import torch

from tests.parity import assert_gram

pytestmark = pytest.mark.gpu

# a wavefront's tile is 512 elements of every row, a chunk 32,768
LENS = [511, 512, 513, 1, 0, 8, 7, 9, 31, 2047, 2049, 4 * 2048 + 32, 32_767, 32_768, 32_769, 3 * 32_768 + 600]


def _gram64(x, offs):
    x = x.double()
    return torch.stack([x[:, a:b] @ x[:, a:b].t().contiguous() for a, b in zip(offs, offs[1:])]).cpu().numpy()


@pytest.mark.parametrize("K", [6, 7, 8, 9, 13, 16])
def test_tile_edges(gpu_lib, K):
    """K = 6 is the other side of the line from which the matrix cores are used."""
    offs = np.concatenate([[0], np.cumsum(LENS)]).astype(np.int64)
    print(f"case gram mfma K={K}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K)
    x = torch.randn((K, int(offs[-1])), generator=gen, device="cuda")
    x = (x * torch.logspace(-3, 3, K, device="cuda")[:, None] + 0.3 * x[:1]).bfloat16()
    G = gpu_lib.gram(x, torch.from_numpy(offs).cuda())
    # 256 fp32 additions and a few more at 2^-24 each: 2e-5 at the very most
    got, want = G.cpu().numpy(), _gram64(x, offs)
    d = np.sqrt(np.einsum("bii->bi", want))
    assert np.all(np.abs(got - want) <= 2e-5 * d[:, :, None] * d[:, None, :])
    assert_gram(got, want, "bf16", f"K={K}")
    assert np.array_equal(got, got.transpose(0, 2, 1))


@pytest.mark.parametrize("K", [7, 8, 11, 16])
def test_special_values_stay_in_their_rows(gpu_lib, K):
    n = 3 * 2048 + 5
    offs = np.array([0, 2048, 2048 + 2053, n], dtype=np.int64)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(100 + K)
    x = torch.randn((K, n), generator=gen, device="cuda")
    x[1] *= 1e-39  # subnormal
    x[2] *= 1e35
    x = x.bfloat16()
    x[3, 5] = float("inf")
    x[4, 3000] = float("nan")
    G = gpu_lib.gram(x, torch.from_numpy(offs).cuda()).cpu().numpy()
    want = _gram64(x, offs)
    bad = np.zeros(G.shape, dtype=bool)
    bad[0, 3], bad[0, :, 3], bad[1, 4], bad[1, :, 4] = True, True, True, True
    assert not np.isfinite(G[bad]).any()
    bad[:, 2, 2] = True  # squares of 1e35 exceed fp32
    ok = ~bad
    assert np.isfinite(G[ok]).all()
    d = np.sqrt(np.abs(np.einsum("bii->bi", np.where(np.isfinite(want), want, 1.0))))
    # (products of two subnormal values are below fp32's range)
    assert np.all(np.abs(G[ok] - want[ok]) <= (2e-5 * d[:, :, None] * d[:, None, :] + 1e-42)[ok])
