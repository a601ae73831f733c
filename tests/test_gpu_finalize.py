"""The Gram finalize at the line where chunk slots are first added in groups
(512 chunks in a call), and the resolve call's finalize that also solves,
against float64 sums of the same bytes."""

import numpy as np
import pytest
import torch

import oracle
from tests.parity import assert_gram, assert_weights

pytestmark = pytest.mark.gpu

CHUNK = {(2, "f32"): 16384, (16, "bf16"): 32768}  # elements of a Gram chunk


def _gram64(x, offs):
    G = []
    for lo, hi in zip(offs, offs[1:]):
        r = x[:, lo:hi].double()
        G.append(r @ r.t().contiguous())
    return torch.stack(G).cpu().numpy()


@pytest.mark.parametrize("past", [-1, 0, 1])
@pytest.mark.parametrize("K,dtype", [(2, "f32"), (16, "bf16")])
def test_grouped_and_direct_sums(gpu_lib, K, dtype, past):
    """Buckets of no, one, 63 to 65 and about 300 chunks, one a chunk and an
    element long, at N just below, at and just above 512 chunks."""
    C = CHUNK[K, dtype]
    lens = [1, 0, 63 * C, 64 * C, 64 * C + 1, C + 1, 0, 20 * C - 2]
    lens.append(512 * C + past - sum(lens))
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    print(f"case finalize K={K} {dtype} N={offs[-1]}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(60 + K)
    x = torch.randn((K, int(offs[-1])), generator=gen, device="cuda")
    x = (x + x[0]).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    want = _gram64(x, offs)
    o = torch.from_numpy(offs).cuda()
    G = gpu_lib.gram(x, o)
    # the tolerance of assert_gram covers 128 fp32 additions of a lane and 6 of the butterfly
    assert_gram(G.cpu().numpy(), want, dtype, f"K={K} past={past}")
    method = "mgda" if K == 2 else "pcgrad"
    G2 = torch.empty_like(G)
    W = torch.empty((len(lens), K), device="cuda")
    gpu_lib.set_resolve_path(gpu_lib.PATH_TWO_PASS)
    try:
        gpu_lib.resolve(x, o, method, gram_out=G2, weights=W)
    finally:
        gpu_lib.set_resolve_path(0)
    assert torch.equal(G, G2)
    w, _ = oracle.solve(G.cpu().numpy(), method, 20)
    assert_weights(W.cpu().numpy().astype(np.float64), w, "weights(iso)", f"K={K} past={past}")
