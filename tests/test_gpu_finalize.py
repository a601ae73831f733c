"""The Gram finalize at the line where chunk slots are first added in groups
(512 chunks in a bucket, fewer with many tasks), the resolve call's finalize that also solves, and the
schedule that a streaming pass makes for itself, against float64 sums of the
same bytes."""

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
    """Buckets of no, one, 63 to 65 chunks, one a chunk and an element long, and
    one of just below, at and just above the line from which a bucket's slots are
    first added in groups (64 for each thread of a pair: 512 chunks at most, with
    16 tasks 192)."""
    C = CHUNK[K, dtype]
    lens = [1, 0, 63 * C, 64 * C, 64 * C + 1, C + 1, 0, 20 * C - 2, ({2: 512, 16: 192}[K] + past) * C - 2, 513 * C]
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


@pytest.mark.parametrize("K,dtype", [(2, "f32"), (16, "bf16")])
def test_a_buckets_matrix_does_not_depend_on_the_others(gpu_lib, K, dtype):
    """The order of a bucket's sum is its own: bit for bit the same matrix in a
    call of that bucket and in one that has a bucket of 600 chunks as well."""
    C = CHUNK[K, dtype]
    n = 100 * C + 777
    print(f"case finalize alone and in a long call K={K} {dtype}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(70 + K)
    x = torch.randn((K, n + 600 * C), generator=gen, device="cuda")
    x = x.to(torch.float32 if dtype == "f32" else torch.bfloat16)
    both = gpu_lib.gram(x, torch.tensor([0, n, n + 600 * C], device="cuda"))
    alone = gpu_lib.gram([r[:n] for r in x], torch.tensor([0, n], device="cuda"))
    assert torch.equal(both[0], alone[0])


@pytest.mark.parametrize("K,dtype", [(2, "f32"), (10, "bf16"), (16, "f32")])
def test_sums_by_one_wavefront(gpu_lib, K, dtype):
    """Thousands of short buckets (and no, one and 100 chunks in some), whose
    slots one wavefront a bucket adds: bit for bit the matrices, and weights,
    that the buckets get in calls of few, by the whole workgroup."""
    C = 32768 if dtype == "bf16" else 16384
    rng = np.random.default_rng(K)
    lens = rng.integers(0, 300, size=4096)
    lens[[7, 8, 4095]] = 0, 100 * C + 5, 3 * C
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    print(f"case finalize by a wavefront K={K} {dtype} N={offs[-1]}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(75 + K)
    x = torch.randn((K, int(offs[-1])), generator=gen, device="cuda")
    x = x.to(torch.float32 if dtype == "f32" else torch.bfloat16)
    method = "mgda" if K < 16 else "pcgrad"
    o = torch.from_numpy(offs).cuda()

    def call(o):
        G = torch.empty((len(o) - 1, K, K), dtype=torch.float64, device="cuda")
        W = torch.empty((len(o) - 1, K), device="cuda")
        gpu_lib.set_resolve_path(gpu_lib.PATH_TWO_PASS)
        try:
            gpu_lib.resolve(x, o, method, gram_out=G, weights=W)
        finally:
            gpu_lib.set_resolve_path(0)
        assert torch.equal(G, gpu_lib.gram(x, o))
        return G, W

    G, W = call(o)
    assert_gram(G.cpu().numpy(), _gram64(x, offs), dtype, f"K={K}")
    for b in (0, 7, 8, 4000, 4095):  # the bucket, and all before and all after it as one
        cut = torch.tensor([0, offs[b], offs[b + 1], offs[-1]], device="cuda")
        G3, W3 = call(cut)
        assert torch.equal(G3[1], G[b]) and torch.equal(W3[1], W[b]), f"bucket {b}"


@pytest.mark.parametrize("more", [0, 600])
@pytest.mark.parametrize("K,dtype", [(3, "f32"), (10, "bf16")])
def test_a_chunks_parts(gpu_lib, K, dtype, more):
    """Buckets that end around the half of a chunk, where the combine's last
    part of it begins, with `more` one-element buckets among them (so that the
    pass finds its parts in LDS or in the workspace): every element once."""
    C = 32768 if dtype == "bf16" else 16384
    lens = [C // 2 - 1, C // 2, C // 2 + 1, C - 1, C, C + 1, 0, 1] + [1] * more
    lens += [3 * C // 2 - 1, 3 * C // 2, 3 * C // 2 + 1, 2 * C, 0, 5 * C // 2, 7]
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n, B = int(offs[-1]), len(lens)
    print(f"case combine parts K={K} {dtype} B={B} N={n}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(80 + K)
    x = torch.randn((K, n), generator=gen, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
    w = torch.randn((B, K), generator=gen, device="cuda")
    o = torch.from_numpy(offs).cuda()
    out = torch.full((n,), float("nan"), device="cuda")
    gpu_lib.combine(x, o, w, out=out)
    terms = w.double()[torch.repeat_interleave(torch.arange(B, device="cuda"), torch.tensor(lens, device="cuda"))].t()
    terms = terms * x.double()
    # an fp32 FMA chain of K terms
    assert bool(((out.double() - terms.sum(0)).abs() <= K * 2.0 ** -24 * terms.abs().sum(0) + 1e-30).all())
    two_pass = torch.full((n,), float("nan"), device="cuda")
    W = torch.empty((B, K), device="cuda")
    gpu_lib.set_resolve_path(gpu_lib.PATH_TWO_PASS)
    try:
        gpu_lib.resolve(x, o, "mgda", out=two_pass, weights=W)
    finally:
        gpu_lib.set_resolve_path(0)
    assert torch.equal(two_pass, gpu_lib.combine(x, o, W, out_dtype=torch.float32))


@pytest.mark.parametrize("B", [1, 256, 257, 511, 512, 1025])
@pytest.mark.parametrize("K,dtype", [(2, "f32"), (8, "bf16")])
def test_schedule_by_the_pass_or_its_own_kernel(gpu_lib, K, dtype, B):
    """Bucket counts at the edges of a workgroup's scan and of the line (511)
    up to which a streaming pass makes its own schedule; also with offsets
    that it has to reject."""
    rng = np.random.default_rng(B)
    lens = rng.integers(0, 3_000, size=B)
    lens[B // 2] += 40_000
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(offs[-1])
    print(f"case schedule K={K} {dtype} B={B} N={n}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(B)
    x = torch.randn((K, n), generator=gen, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
    o = torch.from_numpy(offs).cuda()
    ws = torch.empty(gpu_lib.workspace_size(K, n, B, x.dtype), dtype=torch.uint8, device="cuda")
    G = gpu_lib.gram(x, o, workspace=ws)
    assert_gram(G.cpu().numpy(), _gram64(x, offs), dtype, f"B={B}")
    w = torch.randn((B, K), generator=gen, device="cuda")
    out = gpu_lib.combine(x, o, w, out_dtype=torch.float32, workspace=ws)
    per = torch.repeat_interleave(torch.arange(B, device="cuda"), torch.from_numpy(lens).cuda())
    want = (w.double()[per].t() * x.double()).sum(0)
    scale = (w.double()[per].t() * x.double()).abs().sum(0)
    # an fp32 FMA chain of K terms
    assert bool(((out.double() - want).abs() <= K * 2.0 ** -24 * scale + 1e-30).all())
    if B > 2:
        bad = o.clone()
        bad[1] = bad[2] + 1
        keep = torch.full((n,), 7.0, device="cuda")
        gpu_lib.combine(x, bad, w, out=keep, workspace=ws)
        assert gpu_lib.read_device_error(ws) == gpu_lib.DEVERR_OFFSETS and bool((keep == 7.0).all())
        assert bool(torch.isnan(gpu_lib.gram(x, bad, workspace=ws)).all())
        assert gpu_lib.read_device_error(ws) == gpu_lib.DEVERR_OFFSETS
        gpu_lib.gram(x, o, workspace=ws)
        assert gpu_lib.read_device_error(ws) == 0
