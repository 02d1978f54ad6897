"""Multi-column GEMVs at the edges of their kernels: columns between the powers of two the quads hold,
rows around a round, chunks around a quarter, a step and the steps LDS holds, both kernels, unaligned
strides, rows of 256 MiB, non-finite and subnormal values.  Every column must equal the single-column GEMV bit
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
    """Enough rounds of 32 rows (384 to 512; over 704 for int8 with four columns) for the kernel that shares
    activations through LDS: rows that stay there whole and rows one step too long, with a last step
    of 64, 1 and 33 chunks, and a ragged last round."""
    rounds = 710 if fmt == wl.I8 and T <= 4 else 400
    for last in (64, 1, 33):
        compare(fmt, 32 * rounds + 5, STEP[fmt] * (steps - 1) + UNIT[fmt] * last, T)


@pytest.mark.parametrize("fmt,T,rounds,steps", [(wl.Q4, 4, 768, 1), (wl.Q4, 4, 769, 1), (wl.Q4, 8, 600, 3), (wl.Q4, 8, 600, 4),
                                                (wl.I8, 4, 704, 2), (wl.I8, 8, 600, 7), (wl.I8, 8, 600, 8), (wl.BF16, 8, 576, 1),
                                                (wl.F16, 8, 577, 1), (wl.I8, 2, 512, 2), (wl.I8, 2, 513, 2), (wl.I8, 4, 512, 1), (wl.Q4, 2, 384, 1), (wl.Q4, 2, 385, 1)])
def test_both_sides_of_the_rule_between_the_kernels(fmt, T, rounds, steps):
    compare(fmt, 32 * rounds - 3, STEP[fmt] * steps - UNIT[fmt] * 5, T)


@pytest.mark.parametrize("T", [2, 4, 8])
def test_mixed_table_of_long_and_short_rows(T):
    """A table of several formats, 1,200 rounds for at most 512 workgroups, so that each goes through two or
    three matrices: rows longer than LDS holds (a ring of two steps) and short ones (kept whole) in
    turn, of one format and of another, all with the same activations."""
    LONG, SHORT, M = 32 * 321, 544, 33                       # LONG: 21, 6 and 11 steps of 16-bit, q4, int8 rows
    X = dv.to_device(synth.normal16((T, LONG), wl.X_SIGMA, wl.F16, seed=12, stream=707))
    made = {(f, K): matrix(f, M, K, seed=K) for f in (wl.F16, wl.Q4, wl.I8) for K in (LONG, SHORT)}
    order = [(wl.F16, LONG), (wl.F16, SHORT), (wl.Q4, SHORT), (wl.Q4, LONG), (wl.I8, SHORT), (wl.F16, SHORT), (wl.I8, LONG),
             (wl.I8, SHORT), (wl.Q4, SHORT), (wl.F16, LONG), (wl.I8, LONG), (wl.Q4, LONG)] * 50
    y = torch.full((2, len(order), T, M + 1), float("nan"), dtype=torch.float32, device="cuda")
    for i, batch in enumerate((1, T)):
        mats = wsr.make_mats([dict(fmt=FMT[f], M=M, K=K, w=made[f, K][0], scales=made[f, K][1], x=X, x_tok_stride=2 * LONG,
                                   y=y[i, m], y_tok_stride=4 * (M + 1)) for m, (f, K) in enumerate(order)])
        ws = zeros_u8(wsr.wsr_sweep_workspace_bytes(mats))
        wsr.wsr_decode_sweep_batched(mats, T, batch, ws, ws.numel(), stream())
    torch.cuda.synchronize()
    assert torch.isnan(y[..., M]).all() and not torch.isnan(y[..., :M]).any()
    assert torch.equal(y[0, ..., :M].contiguous().view(torch.int32), y[1, ..., :M].contiguous().view(torch.int32))


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


@pytest.mark.parametrize("fmt,T", [(f, T) for f in (wl.F16, wl.BF16, wl.Q4, wl.I8) for T in (2, 4, 8, 16)
                                   if T <= 8 or f in (wl.F16, wl.BF16)])
@pytest.mark.parametrize("n", [5, 20])
def test_rows_of_very_unequal_lengths(fmt, T, n):
    """Tables whose rows are weighed by their steps, among them empty rows and a matrix of no rows; rounds for
    both kernels."""
    shapes = ([(700, UNIT[fmt] * 2), (33, STEP[fmt] * 9 + UNIT[fmt]), (0, 64), (45, 0), (20000, UNIT[fmt] * 5)] * 4)[:n]
    xfmt = wl.BF16 if fmt == wl.BF16 else wl.F16
    X = dv.to_device(synth.normal16((T, STEP[fmt] * 10), wl.X_SIGMA, xfmt, seed=33, stream=710))
    z = zeros_u8(256)
    made = {mk: matrix(fmt, *mk, seed=34) if mk[0] * mk[1] else (z, zeros_u8(2 * 256)) for mk in set(shapes)}
    made = {mk: (w, dv.to_device(synth.i8_scales(mk[0], seed=34, stream=702)) if fmt == wl.I8 and mk[0] else s)
            for mk, (w, s) in made.items()}
    outs = [[torch.full((T, M + 1), float("nan"), dtype=torch.float32, device="cuda") for M, _ in shapes] for _ in range(2)]
    for y, batch in zip(outs, (1, T)):
        mats = wsr.make_mats([dict(fmt=FMT[fmt], M=M, K=K, w=made[M, K][0], scales=made[M, K][1], x=X, x_tok_stride=2 * X.shape[1],
                                   y=y[i], y_tok_stride=4 * (M + 1)) for i, (M, K) in enumerate(shapes)])
        ws = zeros_u8(wsr.wsr_sweep_workspace_bytes(mats))
        wsr.wsr_decode_sweep_batched(mats, T, batch, ws, ws.numel(), stream())
    torch.cuda.synchronize()
    for (M, K), a, b in zip(shapes, *outs):
        assert torch.isnan(b[:, M]).all() and not torch.isnan(b[:, :M]).any()
        assert torch.equal(a[:, :M].contiguous().view(torch.int32), b[:, :M].contiguous().view(torch.int32)), (M, K)


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


def same_bits(fmt, W, S, Xh, M, K, T):
    X = dv.to_device(Xh)
    one, many = (batched(fmt, W, S, X, M, K, T, b) for b in (1, T))
    nan = np.isnan(one)
    assert np.array_equal(nan, np.isnan(many))
    assert np.array_equal(f32_bits(one)[~nan], f32_bits(many)[~nan])
    return one


@pytest.mark.parametrize("fmt", [wl.F16, wl.BF16])
@pytest.mark.parametrize("T,M", [(2, 40), (4, 40), (8, 40), (16, 40), (8, 32 * 400), (16, 32 * 400)])
def test_products_of_subnormal_values_alone(fmt, T, M):
    """Rows whose only weights are subnormal, against ordinary activations, the largest finite ones and
    subnormal ones: the outputs are those products and their sums alone, so that a matrix instruction
    that took a subnormal operand, product or sum for zero, or rounded it another way, would show."""
    K = 264
    rng = np.random.default_rng(17)
    sub = np.concatenate([np.arange(1, 128), 0x8000 + np.arange(1, 128)]).astype(np.uint16)   # subnormal in both formats
    Wh = np.zeros((M, K), np.uint16)
    for row in range(M):
        n = (1, 2, 5, K)[row % 4]
        Wh[row, rng.choice(K, n, replace=False)] = rng.choice(sub, n)
    big = 0x7BFF if fmt == wl.F16 else 0x7F7F
    Xh = synth.normal16((T, K), wl.X_SIGMA, fmt, seed=18, stream=708)
    Xh[1] = rng.choice(np.array([big, big | 0x8000, big - 1, 0x3C00, 0x3F80], np.uint16), K)
    if T > 2:
        Xh[2] = rng.choice(sub, K)
        Xh[3] = rng.choice(np.array([0x0080, 0x8080, 0x0400, 0x8400, 0x1000], np.uint16), K)   # the smallest normal ones
    one = same_bits(fmt, dv.to_device(Wh), None, Xh, M, K, T)
    assert np.isfinite(one).all() and one[0].any() and one[1].any()


@pytest.mark.parametrize("fmt", [wl.F16, wl.BF16])
@pytest.mark.parametrize("T,M", [(4, 40), (16, 32 * 400)])
def test_small_results(fmt, T, M):
    """Small weights against small activations: products and sums down to the smallest results of the
    format's products, fp32 subnormals among them for bf16."""
    K = 264
    rng = np.random.default_rng(19)
    lo, hi = (0x0001, 0x1000) if fmt == wl.F16 else (0x0001, 0x2800)
    Wh = (rng.integers(lo, hi, (M, K)) | rng.choice([0, 0x8000], (M, K))).astype(np.uint16)
    Xh = (rng.integers(lo, hi, (T, K)) | rng.choice([0, 0x8000], (T, K))).astype(np.uint16)
    same_bits(fmt, dv.to_device(Wh), None, Xh, M, K, T)


@pytest.mark.parametrize("fmt", [wl.Q4, wl.I8])
@pytest.mark.parametrize("T,M", [(2, 40), (4, 40), (8, 40), (4, 32 * 710), (8, 32 * 400)])
def test_activations_that_are_not_finite(fmt, T, M):
    """An infinity or NaN among the activations of one token makes that token's outputs NaN (an infinity meets
    the decoders' offset terms too), single and in a column, and touches no other token; activations at
    the ends of fp16 keep their bits."""
    K = 1120
    W, S = matrix(fmt, M, K, seed=23)
    Xh = synth.normal16((T, K), wl.X_SIGMA, wl.F16, seed=23, stream=709)
    Xh[0, [3, 700]] = 0x7BFF, 0x0001
    Xh[1, 1119] = 0x7C00
    if T > 2:
        Xh[2, 64] = 0x7E00
        Xh[3, [0, 555]] = 0xFC00, 0x7C00
    one = same_bits(fmt, W, S, Xh, M, K, T)
    assert np.isnan(one[1:4]).all() and np.isfinite(one[0]).all() and np.isfinite(one[4:]).all()


@pytest.mark.parametrize("fmt,M,K", [(wl.F16, 3, 1 << 27), (wl.BF16, 2, (1 << 27) - 8), (wl.Q4, 5, (1 << 29) + 32), (wl.I8, 5, 1 << 28),
                                     (wl.I8, 2, (1 << 28) - 16)])
def test_rows_of_256_mib(fmt, M, K):
    """Rows at the limit of the kernels' 32-bit offsets (2^24 chunks) and one chunk below: columns equal the
    single column bit for bit, through the GEMV and the sweep, alone and beside a short matrix, and the
    products of the few activations that are not zero, at both ends of the row among them."""
    T, n = 2, 200
    nb, sb = {wl.Q4: K // 2, wl.I8: K}.get(fmt, 2 * K), {wl.Q4: K // 16, wl.I8: 2}.get(fmt, 0)
    g = torch.Generator(device="cuda").manual_seed(29)
    w = torch.randint(0, 60, (M * nb,), dtype=torch.uint8, device="cuda", generator=g)          # 16-bit: finite, up to 1.2
    s = torch.full((max(8, M * sb // 2),), 0x2C00, dtype=torch.int16, device="cuda")            # fp16 1 / 16
    at = torch.cat([torch.tensor([0, 1, K // 2, K - 2, K - 1], device="cuda"), torch.randint(0, K, (n,), device="cuda", generator=g)])
    x = torch.zeros((T, K), dtype=torch.bfloat16 if fmt == wl.BF16 else torch.float16, device="cuda")
    x[:, at] = torch.randn((T, n + 5), device="cuda", generator=g).to(x.dtype)
    pos = at.unique()
    if fmt in (wl.F16, wl.BF16):
        wd = w.view(x.dtype).view(M, K)[:, pos].double()
    elif fmt == wl.I8:
        wd = w.view(torch.int8).view(M, K)[:, pos].double() / 16
    else:
        q = (w.view(M, K // 2)[:, pos // 2] >> (4 * (pos % 2)).to(torch.uint8)) & 15
        wd = ((q ^ 8).double() - 8) / 16
    want = x[:, pos].double() @ wd.t()
    y = torch.full((4, T, M), float("nan"), dtype=torch.float32, device="cuda")
    small = torch.zeros((2, T, 4), dtype=torch.float32, device="cuda")
    rec = dict(fmt=FMT[fmt], M=M, K=K, w=w, scales=s if sb else None, x=x, x_tok_stride=2 * K, y_tok_stride=4 * M)
    short = dict(rec, M=4, K=64, x_tok_stride=2 * K, y_tok_stride=16)
    for i, (batch, records) in enumerate(((1, [dict(rec, y=y[0])]), (T, [dict(rec, y=y[1])]),
                                          (T, [dict(short, y=small[0]), dict(rec, y=y[2]), dict(short, y=small[1])]))):
        mats = wsr.make_mats(records)
        ws = zeros_u8(wsr.wsr_sweep_workspace_bytes(mats))
        wsr.wsr_decode_sweep_batched(mats, T, batch, ws, ws.numel(), stream())
    cols = y[3]
    if fmt in (wl.F16, wl.BF16):
        wsr.wsr_gemv_f16_cols(w, x, 2 * K, cols, 4 * M, M, K, T, FMT[fmt], stream())
    else:
        (wsr.wsr_gemv_q4_cols if fmt == wl.Q4 else wsr.wsr_gemv_i8_cols)(w, s, x, 2 * K, cols, 4 * M, M, K, T, stream())
    torch.cuda.synchronize()
    for i in range(1, 4):
        assert torch.equal(y[i].view(torch.int32), y[0].view(torch.int32)), i
    # sums of at most 205 exact products in fp32, and of the decoders' offset terms (q4 8, int8 128 times an activation)
    bound = 205 * 2.0 ** -24 * (x[:, pos].double().abs() @ (wd.abs() + {wl.Q4: 0.5, wl.I8: 8.0}.get(fmt, 0.0)).t())
    assert ((y[0].double() - want).abs() <= bound).all()
    del w, x
    torch.cuda.empty_cache()
