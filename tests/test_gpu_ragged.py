"""Single-token rows that are no whole number of a kernel's steps, through the GEMVs, the sweep of few
matrices (one launch of row groups), of many (spans) and of a mixed table (tiles): all bit for bit the
same, and within 2e-3 of the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from synth import device as dv
from synth import workloads as wl
from gpu_util import TOL, f32_bits, needs_gpu, rel_l2, stream, zeros_u8

from paper_2608_12114_amd import wsr

pytestmark = [pytest.mark.gpu, needs_gpu]
FMT = {wl.F16: wsr.WSR_F16, wl.BF16: wsr.WSR_BF16, wl.Q4: wsr.WSR_Q4, wl.I8: wsr.WSR_I8}
UNIT = {wl.F16: 8, wl.BF16: 8, wl.Q4: 32, wl.I8: 16}


def matrix(fmt, M, K, seed):
    xfmt = wl.BF16 if fmt == wl.BF16 else wl.F16
    x = synth.normal16(K, wl.X_SIGMA, xfmt, seed=seed, stream=803)
    if fmt == wl.Q4:
        return (synth.q4_codes(M, K, seed=seed, stream=801), synth.q4_scales(M, K, seed=seed, stream=802)), x
    if fmt == wl.I8:
        return (synth.i8_codes(M, K, seed=seed, stream=801), synth.i8_scales(M, seed=seed, stream=802)), x
    return (synth.normal16((M, K), wl.W_SIGMA, fmt, seed=seed, stream=801), None), x


def spec(fmt, M, K, w, s, x, y):
    return dict(fmt=FMT[fmt], M=M, K=K, w=w, scales=s, x=x, x_tok_stride=0, y=y, y_tok_stride=4 * M)


def sweep(specs):
    mats = wsr.make_mats(specs)
    ws = zeros_u8(wsr.wsr_sweep_workspace_bytes(mats))
    wsr.wsr_decode_sweep(mats, 1, ws, ws.numel(), stream())


@pytest.mark.parametrize("fmt", [wl.F16, wl.BF16, wl.Q4, wl.I8])
@pytest.mark.parametrize("chunks", [1, 63, 64, 65, 127, 129, 257, 300])
def test_every_route(fmt, chunks):
    K = UNIT[fmt] * chunks
    ora = oracle.get()
    for M in (1, 5, 8, 33):
        (W, S), xh = matrix(fmt, M, K, seed=M + chunks)
        want = ora.gemv(dict(fmt=fmt, w=W, s=S), xh) if fmt in (wl.Q4, wl.I8) else ora.gemv16(W, xh, fmt)
        w, s, x = dv.to_device(W), (None if S is None else dv.to_device(S)), dv.to_device(xh)
        ys = torch.full((14, M + 1), float("nan"), dtype=torch.float32, device="cuda")
        g = ys[0]
        if fmt == wl.Q4:
            wsr.wsr_gemv_q4(w, s, x, g, M, K, stream())
        elif fmt == wl.I8:
            wsr.wsr_gemv_i8(w, s, x, g, M, K, stream())
        else:
            wsr.wsr_gemv_f16(w, x, g, M, K, FMT[fmt], stream())
        sweep([spec(fmt, M, K, w, s, x, ys[1]), spec(fmt, M, K, w, s, x, ys[2])])              # few matrices
        sweep([spec(fmt, M, K, w, s, x, ys[3 + i]) for i in range(9)])                         # spans
        other = wl.BF16 if fmt != wl.BF16 else wl.F16
        z = torch.zeros(8, dtype=torch.int16, device="cuda")
        yz = torch.zeros(1, dtype=torch.float32, device="cuda")
        sweep([spec(fmt, M, K, w, s, x, ys[12]), spec(other, 1, 8, z, None, z, yz), spec(fmt, M, K, w, s, x, ys[13])])
        got = ys.cpu().numpy()
        assert np.isnan(got[:, M]).all()
        assert rel_l2(got[0, :M], want) <= TOL, (M, K)
        for i in range(1, 14):
            assert np.array_equal(f32_bits(got[i, :M]), f32_bits(got[0, :M])), (M, K, i)


def test_last_block_of_a_q4_row_with_an_infinite_scale():
    """Lanes past a ragged row's end load its last block again: an infinite scale there must count once,
    giving the infinity the oracle has and no NaN."""
    M, K = 24, 32 * 70
    W, S = synth.q4_codes(M, K, seed=3, stream=801), synth.q4_scales(M, K, seed=3, stream=802)
    S = S.copy()
    S[::2, -1] = 0x7C00
    xh = synth.normal16(K, wl.X_SIGMA, wl.F16, seed=3, stream=803)
    w, s, x = dv.to_device(W), dv.to_device(S), dv.to_device(xh)
    y = torch.zeros((2, M), dtype=torch.float32, device="cuda")
    wsr.wsr_gemv_q4(w, s, x, y[0], M, K, stream())
    sweep([spec(wl.Q4, M, K, w, s, x, y[1])])
    got = y.cpu().numpy()
    assert np.isinf(got[:, ::2]).all() and np.isfinite(got[:, 1::2]).all()
    assert np.array_equal(f32_bits(got[0]), f32_bits(got[1]))


# 16-bit streams: over spans with the table in the arguments (136 matrices of 67 MB) and in the workspace
# (300, 1,023), and from 64 GiB on (1,024) over claimed tiles, whose counters each token leaves at zero for
# the next one.  Record i begins i rows into one buffer of weights and 8 i elements into one of
# activations, so that no two give the same outputs.
@pytest.mark.parametrize("fmt", [wl.F16, wl.BF16])
@pytest.mark.parametrize("n", [136, 300, 1023, 1024, 1040])
def test_long_16bit_stream(fmt, n):
    M, K, T = 4099, 8192, 2
    assert (n >= 1024) == (n * M * K * 2 >= 64 << 30)
    w = dv.to_device(synth.normal16((M + n, K), wl.W_SIGMA, fmt, seed=n, stream=801))
    x = dv.to_device(synth.normal16((T, K + 8 * n), wl.X_SIGMA, fmt, seed=n, stream=803))
    ys = torch.full((n, T, M + 1), float("nan"), dtype=torch.float32, device="cuda")
    one = torch.full((n, T, M), float("nan"), dtype=torch.float32, device="cuda")
    specs = [dict(fmt=FMT[fmt], M=M, K=K, w=w[i:], scales=None, x=x[0, 8 * i:], x_tok_stride=2 * (K + 8 * n), y=ys[i],
                  y_tok_stride=4 * (M + 1)) for i in range(n)]
    mats = wsr.make_mats(specs)
    ws = zeros_u8(wsr.wsr_sweep_workspace_bytes(mats))
    wsr.wsr_decode_sweep(mats, T, ws, ws.numel(), stream())
    for i in range(n):
        for t in range(T):
            wsr.wsr_gemv_f16(w[i:], x[t, 8 * i:], one[i, t], M, K, FMT[fmt], stream())
    torch.cuda.synchronize()
    assert torch.equal(ys[..., :M].contiguous().view(torch.int32), one.view(torch.int32))
    assert torch.isnan(ys[..., M]).all() and not torch.equal(one[0], one[1])
