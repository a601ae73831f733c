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


def _tiled_call(gpu_lib, K=4, n=48_000_000, count=100, seed=4):
    """Offsets that select the tiled form for CAGrad on bf16 rows, a workspace and outputs."""
    offs = _uneven(n, count, seed)
    B = len(offs) - 1
    ws = torch.empty(gpu_lib.workspace_size(K, n, B, torch.bfloat16), dtype=torch.uint8, device="cuda")
    G = torch.empty((B, K, K), dtype=torch.float64, device="cuda")
    W = torch.empty((B, K), device="cuda")
    gpu_lib.set_resolve_path(0)
    return offs, torch.from_numpy(offs).cuda(), ws, G, W


def _rows(K, n, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    x = torch.randn((K, n), generator=gen, device="cuda")
    x[1] -= 0.5 * x[0]
    return x.bfloat16()


def _assert_tiled(gpu_lib, ws, err=0):
    assert gpu_lib.read_device_error(ws) == err
    assert int(ws[:8].view(torch.int32)[TILED_WORD]) == 1


def test_wait_timeout_forced_from_host(gpu_lib):
    """A one-poll wait limit: solvers that poll while the first window is still
    being read give up at once, as do data workgroups whose weights are not there.
    The call completes, says so, and leaves NaN: in the matrix and weights of a
    bucket whose solver gave up and in all of its update, and nowhere an update
    that is not the one of the weights it returns; the next call on the same
    workspace is clean."""
    K, n = 4, 48_000_000
    offs, o, ws, G, W = _tiled_call(gpu_lib)
    x = _rows(K, n, 31)
    print("case tiled timeout", flush=True)
    try:
        gpu_lib.set_wait_limit(1)
        out = gpu_lib.resolve(x, o, "cagrad", gram_out=G, weights=W, workspace=ws)
        _assert_tiled(gpu_lib, ws, gpu_lib.DEVERR_TIMEOUT)
        with pytest.raises(gpu_lib.BkmooError, match="bounded wait"):
            gpu_lib.resolve(x, o, "cagrad", workspace=ws, check_error=True)
    finally:
        gpu_lib.set_wait_limit(1 << 22)
    gave_up = torch.isnan(W).any(1)
    large = int(np.argmax(np.diff(offs)))  # read for most of the call: its solver has given up long before
    assert bool(gave_up[large])
    assert torch.equal(gave_up, torch.isnan(W).all(1)) and torch.equal(gave_up, torch.isnan(G).all(2).all(1))
    per = torch.repeat_interleave(gave_up, torch.from_numpy(np.diff(offs)).cuda())
    assert bool(torch.isnan(out[per]).all())
    finite = ~torch.isnan(out)
    again = gpu_lib.resolve(x, o, "cagrad", gram_out=G, weights=W, workspace=ws)
    _assert_tiled(gpu_lib, ws)
    assert not bool(torch.isnan(again).any()) and not bool(torch.isnan(W).any())
    assert torch.equal(out[finite], again[finite])


@pytest.mark.parametrize("phase", [1, 5])
def test_rows_at_a_common_odd_phase(gpu_lib, phase):
    """Rows and output that all start `phase` elements past a 16-byte boundary
    take the same path and form; the matrices are those of float64 sums, the
    update the streaming combine's, and nothing beside it is written."""
    K, n = 4, 48_000_000
    offs, o, ws, G, W = _tiled_call(gpu_lib)
    buf = torch.empty((K, n + 16), dtype=torch.bfloat16, device="cuda")  # 16-byte rows: n + 16 = 0 (mod 8)
    rows = [buf[i, phase: phase + n] for i in range(K)]
    x = _rows(K, n, 32 + phase)
    for i in range(K):
        rows[i].copy_(x[i])
    assert {r.data_ptr() % 16 for r in rows} == {2 * phase}
    print(f"case tiled phase {phase}", flush=True)
    room = torch.full((n + 16,), 7.0, dtype=torch.bfloat16, device="cuda")
    out = room[phase: phase + n]
    gpu_lib.resolve(rows, o, "cagrad", out=out, gram_out=G, weights=W, workspace=ws)
    _assert_tiled(gpu_lib, ws)
    want = torch.stack([x[:, lo:hi].double() @ x[:, lo:hi].double().t().contiguous() for lo, hi in zip(offs, offs[1:])])
    assert_gram(G.cpu().numpy(), want.cpu().numpy(), "bf16", "gram")
    w, _ = oracle.solve(G.cpu().numpy(), "cagrad", 20)
    assert_weights(W.cpu().numpy().astype(np.float64), w, "weights(iso)", f"phase {phase}")
    assert torch.equal(out.view(torch.int16), gpu_lib.combine(x, o, W).view(torch.int16))
    assert bool((room[:phase] == 7.0).all()) and bool((room[phase + n:] == 7.0).all())


@pytest.mark.parametrize("row", [0, 3])
def test_in_place_update(gpu_lib, row):
    """The update over one of the rows: a window is written after the next one
    has been read, each chunk by the workgroup that read it."""
    K, n = 4, 48_000_000
    offs, o, ws, G, W = _tiled_call(gpu_lib, seed=5)
    x = _rows(K, n, 40)
    print(f"case tiled in place of row {row}", flush=True)
    want = gpu_lib.resolve(x, o, "cagrad", gram_out=G, weights=W, workspace=ws)
    _assert_tiled(gpu_lib, ws)
    others = x.clone()
    G2 = torch.empty_like(G)
    gpu_lib.resolve(x, o, "cagrad", out=x[row], gram_out=G2, workspace=ws)
    _assert_tiled(gpu_lib, ws)
    assert torch.equal(G, G2)
    assert torch.equal(x[row].view(torch.int16), want.view(torch.int16))
    for i in range(K):
        assert i == row or torch.equal(x[i].view(torch.int16), others[i].view(torch.int16))
