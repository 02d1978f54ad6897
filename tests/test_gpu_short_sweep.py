"""Sweeps of few matrices in one launch of row groups: the ends of the range of sizes that takes it."""
import numpy as np
import pytest
import torch

from gpu_util import needs_gpu, stream, zeros_u8

from paper_2608_12114_amd import wsr

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("fmt,M", [(wsr.WSR_F16, (1 << 26) + 5), (wsr.WSR_Q4, (1 << 26) + 5), (wsr.WSR_I8, (1 << 26) + 5),
                                   (wsr.WSR_BF16, 1 << 24), (wsr.WSR_BF16, (1 << 24) + 1)])
def test_more_empty_rows_than_a_grid_of_row_groups_holds(fmt, M):
    """Empty rows (K = 0) take next to nothing of the weight stream, so a table of many looks short; every
    output is the empty sum all the same (a launch holds fewer than 2^32 threads)."""
    y = torch.full((M + 1,), 7.0, dtype=torch.float32, device="cuda")
    any16 = zeros_u8(64)
    mats = wsr.make_mats([dict(fmt=fmt, M=M, K=0, w=any16, scales=zeros_u8(2 * M) if fmt == wsr.WSR_I8 else any16, x=any16, y=y,
                               y_tok_stride=4 * M)])
    ws = zeros_u8(wsr.wsr_sweep_workspace_bytes(mats))
    wsr.wsr_decode_sweep(mats, 1, ws, ws.numel(), stream())
    torch.cuda.synchronize()
    assert y[M].item() == 7.0
    assert not y[:M].any().item()


@pytest.mark.parametrize("fmt,M,K", [(wsr.WSR_BF16, 768, 4104), (wsr.WSR_BF16, 769, 4104), (wsr.WSR_F16, 512, 4096),
                                     (wsr.WSR_F16, 3, 28680), (wsr.WSR_I8, 4096, 4112), (wsr.WSR_I8, 4097, 4112),
                                     (wsr.WSR_I8, 4096, 4096), (wsr.WSR_I8, 5, 28672), (wsr.WSR_I8, 1, 5136), (wsr.WSR_Q4, 7, 28672), (wsr.WSR_Q4, 4096, 8224),
                                     (wsr.WSR_Q4, 4097, 8224),
                                     (wsr.WSR_Q4, 4099, 544)])
def test_blocks_of_one_wave_and_of_four(fmt, M, K):
    """Both sides of the rule that gives long rows of few waves a block for each, alone and beside short rows:
    the GEMV's bits."""
    nb = {wsr.WSR_Q4: K // 2, wsr.WSR_I8: K}.get(fmt, 2 * K)
    g = torch.Generator(device="cuda").manual_seed(M + K)
    w = torch.randint(0, 60, (M * nb,), dtype=torch.uint8, device="cuda", generator=g)
    s = torch.randint(0x2800, 0x2C00, (M * max(1, K // 32),), dtype=torch.int16, device="cuda", generator=g)
    x = torch.randn(K, device="cuda", generator=g).to(torch.bfloat16 if fmt == wsr.WSR_BF16 else torch.float16)
    want = torch.full((2, M), float("nan"), dtype=torch.float32, device="cuda")
    y = torch.full((3, M + 1), float("nan"), dtype=torch.float32, device="cuda")

    def gemv(M, K, out):
        if fmt in (wsr.WSR_F16, wsr.WSR_BF16):
            wsr.wsr_gemv_f16(w, x, out, M, K, fmt, stream())
        else:
            (wsr.wsr_gemv_q4 if fmt == wsr.WSR_Q4 else wsr.wsr_gemv_i8)(w, s, x, out, M, K, stream())

    rec = dict(fmt=fmt, M=M, K=K, w=w, scales=s, x=x)
    gemv(M, K, want[0])
    gemv(M, 64, want[1])
    for records in ([dict(rec, y=y[0])], [dict(rec, K=64, y=y[1]), dict(rec, y=y[2])]):
        mats = wsr.make_mats(records)
        ws = zeros_u8(wsr.wsr_sweep_workspace_bytes(mats))
        wsr.wsr_decode_sweep(mats, 1, ws, ws.numel(), stream())
    torch.cuda.synchronize()
    assert torch.isnan(y[:, M]).all()
    for i, j in ((0, 0), (1, 1), (2, 0)):
        assert torch.equal(y[i, :M].view(torch.int32), want[j].view(torch.int32)), i
