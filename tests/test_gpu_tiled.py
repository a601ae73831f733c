"""The refill kernel's tiled form, which the device selects when the buckets'
sizes differ too much for the pipelined one: results against
float64 sums of the same bytes, and the word that says which form ran."""

import numpy as np
import pytest
import torch

import oracle
from tests.parity import assert_gram, assert_weights

pytestmark = pytest.mark.gpu

TILED_WORD = 1  # uint32 index in the workspace's header


def _uneven(n, count, seed):
    """One bucket of about two thirds of the elements, empty ones, one-element ones, and ragged others."""
    rng = np.random.default_rng(seed)
    lens = [int(x) for x in np.exp(rng.uniform(0, np.log(n / (4 * count)), size=count - 4))]
    lens = lens[: count // 2] + [0, 1, n - sum(lens) - 2, 1] + lens[count // 2:]
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)


# (K, dtype, out, method, elements, buckets)
CASES = [
    (2, "f32", "f32", "mgda", 30_000_000, 64),
    (3, "bf16", "bf16", "cagrad", 40_000_008, 40),
    (4, "bf16", "f32", "cagrad", 48_000_000, 100),
    (7, "bf16", "bf16", "mgda", 30_000_000, 100),
    (10, "f32", "bf16", "pcgrad", 20_000_000, 60),
    (10, "bf16", "bf16", "mean", 20_000_000, 150),
]


@pytest.mark.parametrize("K,dtype,out,method,n,count", CASES)
def test_uneven_buckets(gpu_lib, K, dtype, out, method, n, count):
    print(f"case tiled K={K} {dtype}->{out} {method} n={n} B={count}", flush=True)
    dts = {"f32": torch.float32, "bf16": torch.bfloat16}
    offs = _uneven(n, count, K)
    B = len(offs) - 1
    gen = torch.Generator(device="cuda")
    gen.manual_seed(90 + K)
    x = torch.randn((K, n), generator=gen, device="cuda")
    x[1] -= 0.5 * x[0]
    x = x.to(dts[dtype])
    o = torch.from_numpy(offs).cuda()
    gpu_lib.set_resolve_path(0)
    assert gpu_lib.resolve_path(x, B + 1, method, 20, out_dtype=dts[out]) == gpu_lib.PATH_REFILL
    ws = torch.empty(gpu_lib.workspace_size(K, n, B, dts[dtype]), dtype=torch.uint8, device="cuda")
    G = torch.empty((B, K, K), dtype=torch.float64, device="cuda")
    W = torch.empty((B, K), device="cuda")
    A = torch.empty((B, K), dtype=torch.float64, device="cuda")
    res = [gpu_lib.resolve(x, o, method, gram_out=G, weights=W, aux=A, workspace=ws, out_dtype=dts[out])
           for _ in range(2)]
    assert gpu_lib.read_device_error(ws) == 0
    assert int(ws[:8].view(torch.int32)[TILED_WORD]) == 1
    assert torch.equal(res[0].view(torch.uint8), res[1].view(torch.uint8))
    want = torch.stack([x[:, lo:hi].double() @ x[:, lo:hi].double().t().contiguous()
                        for lo, hi in zip(offs, offs[1:])])
    assert_gram(G.cpu().numpy(), want.cpu().numpy(), dtype, "gram")
    w, _ = oracle.solve(G.cpu().numpy(), method, 20)
    assert_weights(W.cpu().numpy().astype(np.float64), w, "weights(iso)", f"K={K}")
    # the update is the streaming combine's, bit for bit
    assert torch.equal(gpu_lib.combine(x, o, W, out_dtype=dts[out]).view(torch.uint8), res[0].view(torch.uint8))


@pytest.mark.parametrize("count,uneven", [(48, 0), (100, 1)])
def test_form_follows_the_offsets(gpu_lib, count, uneven):
    """Equal buckets keep the pipelined form; the same number of ragged ones, or an offsets error, does not set it."""
    K, n = 4, 48_000_000
    x = torch.ones((K, n), dtype=torch.bfloat16, device="cuda")
    even = np.linspace(0, n, count + 1).astype(np.int64)
    offs = _uneven(n, count, 4) if uneven else even
    ws = torch.empty(gpu_lib.workspace_size(K, n, count, torch.bfloat16), dtype=torch.uint8, device="cuda")
    gpu_lib.set_resolve_path(0)
    gpu_lib.resolve(x, torch.from_numpy(offs).cuda(), "cagrad", workspace=ws)
    assert int(ws[:8].view(torch.int32)[TILED_WORD]) == uneven
    offs[1], offs[2] = offs[2] + 1, offs[1]
    gpu_lib.resolve(x, torch.from_numpy(offs).cuda(), "cagrad", workspace=ws)
    assert gpu_lib.read_device_error(ws) & gpu_lib.DEVERR_OFFSETS
    assert int(ws[:8].view(torch.int32)[TILED_WORD]) == 0


@pytest.mark.parametrize("K,dtype", [(2, "f32"), (3, "bf16")])
def test_one_large_bucket_of_many_keeps_the_pipelined_form(gpu_lib, K, dtype):
    """2.4 GiB in 40 buckets, one of a third of it: the others' groups end early,
    but the pipelined form still reads less."""
    item = 4 if dtype == "f32" else 2
    n = 2500 * (1 << 20) // (K * item) // 8 * 8
    w = np.ones(40)
    w[13] = 20
    offs = (np.concatenate([[0], np.cumsum(w)]) / w.sum() * n).astype(np.int64)
    offs[-1] = n
    x = torch.ones((K, n), dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
    gpu_lib.set_resolve_path(0)
    print(f"case tiled or not K={K} {dtype} n={n}", flush=True)
    assert gpu_lib.resolve_path(x, 41, "cagrad", 20) == gpu_lib.PATH_REFILL
    ws = torch.empty(gpu_lib.workspace_size(K, n, 40, x.dtype), dtype=torch.uint8, device="cuda")
    gpu_lib.resolve(x, torch.from_numpy(offs).cuda(), "cagrad", workspace=ws)
    assert gpu_lib.read_device_error(ws) == 0
    assert int(ws[:8].view(torch.int32)[TILED_WORD]) == 0
    # the host's byte count takes the same form: some bytes are read once
    assert gpu_lib.resolve_traffic(K, offs, dtype, gpu_lib.PATH_REFILL, method="cagrad") < (2 * K + 1) * item * n
