"""The matrix-core sweep whose workgroups split every row's steps over four waves (16-bit, int8): rows of
fewer steps than waves (some waves have none), of uneven shares, with a ragged last step and of 16 KiB
(128 steps: each row group begins at a step of its own), over several row groups with a ragged last
one, several matrices in one call and the outputs' bounds."""
import numpy as np
import pytest
import torch

import oracle
import synth
from synth import device as dv
from synth import workloads as wl
from gpu_util import f32_bits, needs_gpu, rel_l2, stream, zeros_u8
from test_gpu_mma import CODE, TOL, host_matrix, run_mma

from paper_2608_12114_amd import wsr

pytestmark = [pytest.mark.gpu, needs_gpu]

STEP = {wl.F16: 64, wl.BF16: 64, wl.I8: 128}      # weights of a 128-byte step


@pytest.mark.parametrize("fmt", [wl.F16, wl.BF16, wl.I8])
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 7, 9, 128, 256])
@pytest.mark.parametrize("ragged", [0, 16], ids=["whole", "ragged"])
def test_split_steps(fmt, steps, ragged):
    M, T, K = 150, 5, steps * STEP[fmt] + ragged
    W, S = host_matrix(fmt, M, K, seed=31)
    X = synth.normal16((T + 1, K), wl.X_SIGMA, wl.BF16 if fmt == wl.BF16 else wl.F16, seed=31, stream=631)
    y = run_mma(fmt, W, S, X, M, K, T, y_rows=M + 3)
    assert np.isnan(y[:, M:]).all() and np.isnan(y[T:]).all()
    ora = oracle.get()
    for t in range(T):
        want = ora.gemv(dict(fmt=fmt, w=W, s=S), X[t]) if fmt == wl.I8 else ora.gemv16(W, X[t], fmt)
        assert rel_l2(y[t, :M], want) <= TOL, (fmt, K, t)


def mma_table(entries, T):
    """Outputs of one call over [(fmt, M, K, w, s, x)], each (T, M)."""
    ys = [torch.full((T, M), float("nan"), dtype=torch.float32, device="cuda") for _, M, *_ in entries]
    mats = wsr.make_mats([dict(fmt=CODE[f], M=M, K=K, w=w, scales=s, x=x, x_tok_stride=2 * K, y=y, y_tok_stride=4 * M)
                          for (f, M, K, w, s, x), y in zip(entries, ys)])
    ws = zeros_u8(wsr.wsr_sweep_workspace_bytes(mats))
    wsr.wsr_decode_sweep_mma(mats, T, ws, ws.numel(), stream())
    return [f32_bits(y.cpu().numpy()) for y in ys]


@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 7, 9, 30, 128])
@pytest.mark.parametrize("ragged", [0, 16, -48], ids=["whole", "longer", "shorter"])
def test_outputs_do_not_depend_on_the_rest_of_the_table(steps, ragged):
    """A matrix's outputs are the same bits alone, and in a table that holds other formats too, where one
    wave takes the rows that four share when all are of one format."""
    T, entries = 5, []
    for i, fmt in enumerate((wl.F16, wl.I8, wl.Q4, wl.BF16)):
        M, K = 150 + 7 * i, {wl.Q4: 256}.get(fmt, STEP.get(fmt)) * steps + (32 if fmt == wl.Q4 and ragged else ragged)
        W, S = host_matrix(fmt, M, K, seed=37 + i)
        X = synth.normal16((T, K), wl.X_SIGMA, wl.BF16 if fmt == wl.BF16 else wl.F16, seed=37 + i, stream=632)
        entries.append((fmt, M, K, dv.to_device(W), None if S is None else dv.to_device(S), dv.to_device(X)))
    for e, got in zip(entries, mma_table(entries, T)):
        assert np.array_equal(got, mma_table([e], T)[0]), (e[0], e[2])


@pytest.mark.parametrize("fmt", [wl.BF16, wl.I8])
def test_rows_of_16_kib_do_not_depend_on_their_workgroup(fmt):
    """Row groups in the spans' main part and in the tail (581 groups of 64 rows leave one), and the same rows
    as matrices of their own: the same bits, since the step a row begins at depends on the row alone (and
    repeats every 32 groups)."""
    T, K, M = 5, STEP[fmt] * 128, 2048 * 18 + 300
    g = torch.Generator(device="cuda").manual_seed(11)
    W = torch.randn((M, K), device="cuda", generator=g)
    W = (W * 40).to(torch.int8) if fmt == wl.I8 else W.to(torch.bfloat16)
    S = torch.rand(M, device="cuda", generator=g).to(torch.float16) if fmt == wl.I8 else None
    X = torch.randn((T, K), device="cuda", generator=g).to(torch.float16 if fmt == wl.I8 else torch.bfloat16)
    whole = mma_table([(fmt, M, K, W, S, X)], T)[0]
    for r0, n in ((0, 150), (2048 * 9, 64), (2048 * 17, M - 2048 * 17), (2048 * 18, 300)):
        part = mma_table([(fmt, n, K, W[r0:r0 + n], None if S is None else S[r0:r0 + n], X)], T)[0]
        assert np.array_equal(part, whole[:, r0:r0 + n]), r0
    del W, X
    torch.cuda.empty_cache()


@pytest.mark.parametrize("fmts", [(wl.F16,), (wl.BF16,), (wl.I8,), (wl.Q4,), (wl.Q4, wl.F16, wl.I8)], ids=str)
def test_empty_rows_give_empty_sums(fmts):
    """K = 0: every output is 0, in tables of one format and of several."""
    any16 = torch.ones(4096, dtype=torch.uint8, device="cuda")
    entries = [(fmt, M, 0, any16, any16 if fmt in (wl.Q4, wl.I8) else None, any16) for fmt in fmts for M in (1, 64, 150)]
    for y in mma_table(entries, 3):
        assert not y.any()


@pytest.mark.parametrize("fmt,K", [(wl.I8, 96), (wl.I8, 512), (wl.I8, 2048), (wl.F16, 48), (wl.BF16, 512), (wl.BF16, 520)])
def test_long_streams_of_short_rows(fmt, K):
    """Streams of 40 MiB and more whose rows all hold few steps go one wave per workgroup: the bits of the
    same rows in a short stream, which four waves share."""
    T, row = 5, K if fmt == wl.I8 else 2 * K
    M = (41 << 20) // 3 // row // 64 * 64 + 70
    g = torch.Generator(device="cuda").manual_seed(K)
    W = torch.randn((3 * M, K), device="cuda", generator=g)
    W = (W * 40).to(torch.int8) if fmt == wl.I8 else W.to(torch.bfloat16 if fmt == wl.BF16 else torch.float16)
    S = torch.rand(3 * M, device="cuda", generator=g).to(torch.float16) if fmt == wl.I8 else None
    X = torch.randn((T, K), device="cuda", generator=g).to(torch.bfloat16 if fmt == wl.BF16 else torch.float16)
    part = lambda r0, n: (fmt, n, K, W[r0:r0 + n], None if S is None else S[r0:r0 + n], X)  # noqa: E731
    long = mma_table([part(i * M, M) for i in range(3)], T)
    for i in range(3):
        assert np.array_equal(long[i][:, :200], mma_table([part(i * M, 200)], T)[0])
        assert np.array_equal(long[i][:, M - 134:], mma_table([part(i * M + M - 134, 134)], T)[0])
