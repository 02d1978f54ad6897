"""Multi-column GEMVs at the edges of their kernels: columns between the powers of two the quads hold,
rows around a round, chunks around a quarter, a step and the steps LDS holds, both kernels, unaligned
strides, non-finite and subnormal 16-bit values.  Every column must equal the single-column GEMV bit
for bit (the contract of include/wsr.h), which the oracle tests hold to 2e-3."""
import numpy as np
import pytest
import torch

import synth
from synth import device as dv
from synth import workloads as wl
from gpu_util import f32_bits, needs_gpu, stream, zeros_u8

from paper_2608_12114_amd import wsr

pytestmark = [pytest.mark.gpu, needs_gpu]
FMT = {wl.F16: wsr.WSR_F16, wl.BF16: wsr.WSR_BF16, wl.Q4: wsr.WSR_Q4, wl.I8: wsr.WSR_I8}


def matrix(fmt, M, K, seed):
    if fmt == wl.Q4:
        return dv.to_device(synth.q4_codes(M, K, seed=seed, stream=701)), dv.to_device(synth.q4_scales(M, K, seed=seed, stream=702))
    if fmt == wl.I8:
        return dv.to_device(synth.i8_codes(M, K, seed=seed, stream=701)), dv.to_device(synth.i8_scales(M, seed=seed, stream=702))
    return dv.to_device(synth.normal16((M, K), wl.W_SIGMA, fmt, seed=seed, stream=701)), None


def batched(fmt, W, S, X, M, K, tokens, batch, gap=0):
    """y (tokens, M + gap) of one matrix through the batched sweep; X holds (tokens, K)."""
    y = torch.full((tokens, M + gap), float("nan"), dtype=torch.float32, device="cuda")
    mats = wsr.make_mats([dict(fmt=FMT[fmt], M=M, K=K, w=W, scales=S, x=X, x_tok_stride=2 * X.stride(0), y=y,
                               y_tok_stride=4 * (M + gap))])
    ws = zeros_u8(wsr.wsr_sweep_workspace_bytes(mats))
    wsr.wsr_decode_sweep_batched(mats, tokens, batch, ws, ws.numel(), stream())
    return y.cpu().numpy()


def compare(fmt, M, K, T, gap=3):
    W, S = matrix(fmt, M, K, seed=M + K)
    X = dv.to_device(synth.normal16((T, K + 8), wl.X_SIGMA, wl.BF16 if fmt == wl.BF16 else wl.F16, seed=K, stream=703))
    one = batched(fmt, W, S, X, M, K, T, 1, gap)
    many = batched(fmt, W, S, X, M, K, T, T, gap)
    assert np.isnan(many[:, M:]).all()
    assert np.array_equal(f32_bits(one[:, :M]), f32_bits(many[:, :M])), (fmt, M, K, T)


# K at the ends of a quarter (16 chunks), of a step (64) and past the steps that stay in LDS
STEP = {wl.F16: 512, wl.BF16: 512, wl.Q4: 2048, wl.I8: 1024}
UNIT = {wl.F16: 8, wl.BF16: 8, wl.Q4: 32, wl.I8: 16}


@pytest.mark.parametrize("fmt,T", [(f, T) for f in (wl.F16, wl.BF16, wl.Q4, wl.I8) for T in (2, 4, 8, 16)
                                   if T <= 8 or f in (wl.F16, wl.BF16)])
@pytest.mark.parametrize("chunks", [1, 15, 17, 63, 64, 65, 200])
def test_short_streams(fmt, T, chunks):
    """Few rounds (the split kernel): rows at and around a round of 8 and of 16."""
    for M in (1, 7, 16, 33):
        compare(fmt, M, UNIT[fmt] * chunks, T)


@pytest.mark.parametrize("fmt,T,steps", [(wl.Q4, 2, 1), (wl.Q4, 4, 5), (wl.Q4, 8, 2), (wl.Q4, 8, 3), (wl.I8, 4, 8),
                                         (wl.I8, 4, 9), (wl.I8, 8, 4), (wl.I8, 8, 5), (wl.BF16, 8, 10), (wl.BF16, 8, 11),
                                         (wl.F16, 16, 5), (wl.F16, 16, 6), (wl.F16, 16, 1)])
def test_long_streams(fmt, T, steps):
    """Enough rounds for the kernel that shares activations through LDS: rows that stay there whole and
    rows one step too long, with a last step of 64, 1 and 33 chunks, and a ragged last round."""
    for last in (64, 1, 33):
        compare(fmt, 32 * 400 + 5, STEP[fmt] * (steps - 1) + UNIT[fmt] * last, T)


@pytest.mark.parametrize("fmt,T,M", [(wl.F16, 2, 16387), (wl.BF16, 2, 16383), (wl.I8, 2, 32 * 512 + 3), (wl.I8, 2, 32 * 511)])
def test_two_columns(fmt, T, M):
    """Both sides of the rows from which two columns stay with the vector ALUs, through the GEMV and the
    sweep, against single columns."""
    for K in (STEP[fmt] + UNIT[fmt], 3 * UNIT[fmt]):
        compare(fmt, M, K, T)
        W, S = matrix(fmt, M, K, seed=M)
        X = dv.to_device(synth.normal16((T, K), wl.X_SIGMA, wl.BF16 if fmt == wl.BF16 else wl.F16, seed=K, stream=703))
        one = batched(fmt, W, S, X, M, K, T, 1)
        y = torch.full((T, M + 2), float("nan"), dtype=torch.float32, device="cuda")
        if fmt == wl.I8:
            wsr.wsr_gemv_i8_cols(W, S, X, 2 * K, y, 4 * (M + 2), M, K, T, stream())
        else:
            wsr.wsr_gemv_f16_cols(W, X, 2 * K, y, 4 * (M + 2), M, K, T, FMT[fmt], stream())
        y = y.cpu().numpy()
        assert np.array_equal(f32_bits(one), f32_bits(y[:, :M])) and np.isnan(y[:, M:]).all()


@pytest.mark.parametrize("n", [8, 9, 32, 33, 40, 288, 289])
def test_one_pass_over_matrices_sharing_activations(n):
    """Runs of matrices with one activation, with another and with another length in one table, as many
    as each size of the launch arguments holds and one more; batch 8, 13 tokens (passes of 8, 4 and
    1)."""
    specs, outs = [], []
    shapes = ([(700, 512), (100, 512), (300, 2048), (50, 544)] * 73)[:n]
    xs = {K: dv.to_device(synth.normal16((13, K), wl.X_SIGMA, wl.F16, seed=K, stream=704)) for K in (512, 2048, 544)}
    for i, (M, K) in enumerate(shapes):
        W, S = matrix(wl.Q4, M, K, seed=i)
        outs.append(torch.full((13, M), float("nan"), dtype=torch.float32, device="cuda"))
        specs.append(dict(fmt=wsr.WSR_Q4, M=M, K=K, w=W, scales=S, x=xs[K], x_tok_stride=2 * K, y=outs[-1], y_tok_stride=4 * M))
    mats = wsr.make_mats(specs)
    ws = zeros_u8(wsr.wsr_sweep_workspace_bytes(mats))
    wsr.wsr_decode_sweep(mats, 13, ws, ws.numel(), stream())
    want = [f32_bits(y.cpu().numpy()) for y in outs]
    for y in outs:
        y.fill_(float("nan"))
    wsr.wsr_decode_sweep_batched(mats, 13, 8, ws, ws.numel(), stream())
    for a, y in zip(want, outs):
        assert np.array_equal(a, f32_bits(y.cpu().numpy()))


@pytest.mark.parametrize("fmt", [wl.F16, wl.BF16])
@pytest.mark.parametrize("T,M", [(4, 40), (16, 40), (16, 32 * 300)])
def test_values_at_the_ends_of_16_bit_formats(fmt, T, M):
    """Weights and activations with infinities, subnormals, the largest finite value and zeros of both
    signs: where the single-column result is a number or an infinity the column has its bits, where it
    is NaN so is the column."""
    K = 1096
    rng = np.random.default_rng(5)
    inf, big = (0x7C00, 0x7BFF) if fmt == wl.F16 else (0x7F80, 0x7F7F)
    vals = np.array([0, 0x8000, 1, 0x8001, big, big | 0x8000, inf, inf | 0x8000], dtype=np.uint16)
    Wh = synth.normal16((M, K), wl.W_SIGMA, fmt, seed=9, stream=705)
    Xh = synth.normal16((T, K), wl.X_SIGMA, fmt, seed=9, stream=706)
    for row in range(M):                                 # a few special weights in most rows
        Wh[row, rng.integers(0, K, size=row % 4)] = rng.choice(vals, size=row % 4)
    for t in range(0, T, 2):
        Xh[t, rng.integers(0, K, size=2)] = rng.choice(vals[:6], size=2)
    Xh[1, rng.integers(0, K)] = inf
    W, X = dv.to_device(Wh), dv.to_device(Xh)
    one = batched(fmt, W, None, X, M, K, T, 1)
    many = batched(fmt, W, None, X, M, K, T, T)
    nan = np.isnan(one)
    assert np.array_equal(nan, np.isnan(many)) and nan.any() and not nan.all()
    assert np.array_equal(f32_bits(one)[~nan], f32_bits(many)[~nan])
