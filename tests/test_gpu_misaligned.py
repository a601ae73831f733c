"""Rows and outputs at any element alignment: 128-bit loads of rows that do
not share a 16-byte phase, and an output whose stores are aligned elsewhere
than the rows.  The update of the same values is the same bits wherever they
lie, nothing beside the output is written, and the Gram matrices are those of
float64 sums."""

import numpy as np
import pytest
import torch

from tests.parity import assert_gram

pytestmark = pytest.mark.gpu

DTS = {"f32": torch.float32, "bf16": torch.bfloat16}
LENS = [33_000, 1, 0, 7, 16, 70_001, 5]  # chunk ends, and buckets shorter than a vector


MARK = -77.0  # of the elements around a view


def _at_phase(t, phase):
    """The same values, `phase` elements past a 16-byte boundary, and what they
    are a view of: 32 elements more on either side, all MARK."""
    buf = torch.full((t.numel() + 80,), MARK, dtype=t.dtype, device=t.device)
    view = buf[32 + phase: 32 + phase + t.numel()]
    view.copy_(t)
    assert view.data_ptr() % 16 == phase * t.element_size() % 16
    return view, buf


def _assert_untouched_around(view, buf, what):
    at = (view.data_ptr() - buf.data_ptr()) // buf.element_size()
    assert bool((buf[:at] == MARK).all()) and bool((buf[at + view.numel():] == MARK).all()), what


@pytest.mark.parametrize("rows", ["one phase", "mixed"])
@pytest.mark.parametrize("dtype,out", [("f32", "f32"), ("f32", "bf16"), ("bf16", "f32"), ("bf16", "bf16")])
@pytest.mark.parametrize("K", [2, 4, 9, 16])
def test_any_alignment(gpu_lib, K, dtype, out, rows):
    n = sum(LENS)
    per = 16 // DTS[dtype].itemsize
    offs = torch.from_numpy(np.concatenate([[0], np.cumsum(LENS)]).astype(np.int64)).cuda()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K)
    x = torch.randn((K, n), generator=gen, device="cuda")
    x = (x + 0.5 * x[:1]).to(DTS[dtype])
    aligned = [_at_phase(x[i], 0)[0] for i in range(K)]
    w = torch.randn((len(LENS), K), generator=gen, device="cuda")
    want = gpu_lib.combine(aligned, offs, w, out_dtype=DTS[out])
    xd = x.double()
    gram = torch.stack([xd[:, a:b] @ xd[:, a:b].t().contiguous() for a, b in zip(offs[:-1], offs[1:])])
    for shift in range(per):
        print(f"case alignment K={K} {dtype}->{out} {rows} {shift}", flush=True)
        placed = [_at_phase(x[i], shift if rows == "one phase" else (shift + 3 * i) % per) for i in range(K)]
        got = [view for view, _ in placed]
        assert_gram(gpu_lib.gram(got, offs).cpu().numpy(), gram.cpu().numpy(), dtype, f"{rows} {shift}")
        for op in (0, 1, 3):
            y, room = _at_phase(torch.full((n,), 9.0, dtype=DTS[out], device="cuda"), op)
            gpu_lib.combine(got, offs, w, out=y)
            assert torch.equal(y.view(torch.uint8), want.view(torch.uint8)), f"{rows} {shift} out {op}"
            _assert_untouched_around(y, room, f"{rows} {shift} out {op}")
        if out == dtype:  # in place of one row
            gpu_lib.combine(got, offs, w, out=got[K // 2])
            assert torch.equal(got[K // 2].view(torch.uint8), want.view(torch.uint8)), f"{rows} {shift} in place"
        for i, (view, room) in enumerate(placed):
            _assert_untouched_around(view, room, f"{rows} {shift} row {i}")
            assert (out == dtype and i == K // 2) or torch.equal(view.view(torch.uint8), x[i].view(torch.uint8))
