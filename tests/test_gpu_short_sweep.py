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
