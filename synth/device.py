"""Device plumbing for the synthetic inputs: generate on the host, stream into GPU memory.

PyTorch is used here only as an allocator and copy engine (device tensors, pinned staging buffers).
Nothing here computes anything of the method; it places the generated bytes where the kernels read
them and keeps enough bookkeeping to regenerate any row on the host for the oracle.
"""
from __future__ import annotations

import ctypes

import numpy as np
import torch

import synth
from synth import workloads as wl

_TORCH_DT = {np.dtype(np.uint16): torch.int16, np.dtype(np.uint8): torch.uint8,
             np.dtype(np.float32): torch.float32, np.dtype(np.float64): torch.float64}
WSR_FMT = {wl.F16: 1, wl.BF16: 2, wl.Q4: 3, wl.I8: 4}


def to_device(arr: np.ndarray, device="cuda") -> torch.Tensor:
    """Same bytes, same shape, on the device (uint16 travels as int16)."""
    a = np.ascontiguousarray(arr)
    t = torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a)
    return t.to(device)


def to_host(t: torch.Tensor, dtype) -> np.ndarray:
    return t.detach().cpu().numpy().view(dtype)


# ---- the same generator on the GPU (libsynth_dev.so) --------------------------------------------

_dev = None
_dev_tables = {}


def dev_lib() -> ctypes.CDLL:
    global _dev
    if _dev is None:
        L = ctypes.CDLL(synth.DEV_LIB_PATH)
        vp, i64, u64, i32, dbl = ctypes.c_void_p, ctypes.c_int64, ctypes.c_uint64, ctypes.c_int, ctypes.c_double
        L.synth_dev_normal16.argtypes = [vp, i64, u64, u64, u64, vp, vp, vp]
        L.synth_dev_uniform16.argtypes = [vp, i64, u64, u64, u64, dbl, dbl, i32, vp]
        L.synth_dev_q4.argtypes = [vp, i64, u64, u64, u64, vp]
        L.synth_dev_grid_f32.argtypes = [vp, i64, u64, u64, u64, vp]
        L.synth_dev_i8.argtypes = [vp, i64, u64, u64, u64, vp]
        for f in ("synth_dev_normal16", "synth_dev_uniform16", "synth_dev_q4", "synth_dev_grid_f32",
                  "synth_dev_i8"):
            getattr(L, f).restype = ctypes.c_int
        _dev = L
    return _dev


def _dev_table(fmt, sigma):
    key = (fmt, float(sigma))
    if key not in _dev_tables:
        q, alias = synth.table_arrays(fmt, sigma)
        _dev_tables[key] = (torch.from_numpy(q.view(np.int64).copy()).cuda(),
                            torch.from_numpy(alias.view(np.int16).copy()).cuda())
    return _dev_tables[key]


def _s():
    return torch.cuda.current_stream().cuda_stream


def _ok(rc):
    if rc != 0:
        raise RuntimeError(f"device generator launch failed (hipError {rc})")


def gen_normal16(t: torch.Tensor, sigma, fmt, seed, stream, e0=0):
    """Fill t (2-byte elements, on the GPU) with the same codes synth.normal16 draws on the host."""
    q, alias = _dev_table(fmt, sigma)
    _ok(dev_lib().synth_dev_normal16(t.data_ptr(), t.numel(), seed, stream, e0, q.data_ptr(),
                                     alias.data_ptr(), _s()))
    return t


def gen_uniform16(t: torch.Tensor, lo, hi, fmt, seed, stream, e0=0):
    _ok(dev_lib().synth_dev_uniform16(t.data_ptr(), t.numel(), seed, stream, e0, float(lo), float(hi),
                                      synth._FMT[fmt], _s()))
    return t


def gen_q4(t: torch.Tensor, seed, stream, e0=0):
    """Fill t (bytes) with packed int4 codes of elements e0, e0 + 1, ... (two per byte)."""
    _ok(dev_lib().synth_dev_q4(t.data_ptr(), t.numel(), seed, stream, e0, _s()))
    return t


def gen_i8(t: torch.Tensor, seed, stream, e0=0):
    """Fill t (bytes) with signed int8 codes of elements e0, e0 + 1, ..."""
    _ok(dev_lib().synth_dev_i8(t.data_ptr(), t.numel(), seed, stream, e0, _s()))
    return t


def gen_grid_f32(t: torch.Tensor, seed, stream, e0=0):
    _ok(dev_lib().synth_dev_grid_f32(t.data_ptr(), t.numel(), seed, stream, e0, _s()))
    return t


class Stager:
    """Double-buffered host->device upload through pinned staging memory.

    fill(view) writes into a pinned numpy view; the copy to `dst` is asynchronous on a copy stream,
    and the next fill goes to the other buffer once its previous copy has finished."""

    def __init__(self, nbytes: int = 256 << 20):
        self.nbytes = nbytes
        self.bufs = [torch.empty(nbytes, dtype=torch.uint8, pin_memory=True) for _ in range(2)]
        self.events = [None, None]
        self.i = 0
        self.stream = torch.cuda.Stream()

    def put(self, dst: torch.Tensor, fill, nbytes: int, dst_offset: int = 0):
        """Copy `nbytes` produced by fill(np.ndarray[uint8]) into dst's bytes at dst_offset."""
        dst_b = dst.view(torch.uint8).view(-1)
        done = 0
        while done < nbytes:
            n = min(self.nbytes, nbytes - done)
            k = self.i
            if self.events[k] is not None:
                self.events[k].synchronize()
            view = self.bufs[k][:n].numpy()
            fill(view, done, n)
            with torch.cuda.stream(self.stream):
                dst_b[dst_offset + done: dst_offset + done + n].copy_(self.bufs[k][:n], non_blocking=True)
                ev = torch.cuda.Event()
                ev.record(self.stream)
            self.events[k] = ev
            self.i ^= 1
            done += n

    def finish(self):
        self.stream.synchronize()


def _fill_normal16(fmt, sigma, seed, stream, threads):
    def fill(view, off, n):
        assert off % 2 == 0 and n % 2 == 0
        synth.normal16(n // 2, sigma, fmt, seed=seed, stream=stream, e0=off // 2,
                       out=view.view(np.uint16), threads=threads)
    return fill


def _fill_q4(seed, stream, threads):
    def fill(view, off, n):
        synth.lib().synth_q4(view.ctypes.data, n, seed, stream, 2 * off, threads)
    return fill


def _fill_scales(seed, stream, threads):
    def fill(view, off, n):
        synth.uniform16(n // 2, wl.Q4_SCALE_LO, wl.Q4_SCALE_HI, wl.F16, seed=seed, stream=stream,
                        e0=off // 2, out=view.view(np.uint16), threads=threads)
    return fill


def _fill_i8(seed, stream, threads):
    def fill(view, off, n):
        synth.lib().synth_i8(view.ctypes.data, n, seed, stream, off, threads)
    return fill


def _fill_i8_scales(seed, stream, threads):
    def fill(view, off, n):
        synth.uniform16(n // 2, synth.I8_SCALE_LO, synth.I8_SCALE_HI, wl.F16, seed=seed, stream=stream,
                        e0=off // 2, out=view.view(np.uint16), threads=threads)
    return fill


class SweepInputs:
    """Device-resident inputs and outputs of a decode sweep.

    mats: list of synth.workloads.Mat (sweep order); fmts: storage format per matrix; activations
    are one vector per (layer, slot, token), in the matrix's activation format (fp16 for q4)."""

    def __init__(self, mats, fmts, tokens: int, seed: int = wl.SEED, threads: int | None = None,
                 stager: Stager | None = None, w_sigma: float = wl.W_SIGMA, gen: str = "device",
                 arena: bool = False):
        """arena: every weight and scale tensor is a view into one device buffer (each at a 2 MiB
        boundary), as an engine that loads a whole checkpoint into one allocation would hold it;
        otherwise each tensor is an allocation of its own."""
        self.mats, self.fmts, self.tokens, self.seed = list(mats), list(fmts), tokens, seed
        self.w_sigma = w_sigma
        threads = threads or synth.default_threads()
        st = None
        if gen == "host":
            st = stager or Stager()
        self.w, self.s, self.y = [], [], []
        self.x = {}
        empty = torch.empty
        if arena:
            align = 2 << 20
            nbytes = []
            for m, fmt in zip(self.mats, self.fmts):
                if fmt == wl.Q4:
                    nbytes += [m.M * m.K // 2, m.M * (m.K // 32) * 2]
                elif fmt == wl.I8:
                    nbytes += [m.M * m.K, m.M * 2]
                else:
                    nbytes += [m.M * m.K * 2]
            total = sum(-(-n // align) * align for n in nbytes)
            room = torch.empty(total + align, dtype=torch.uint8, device="cuda")   # the allocator may hand out part of a block
            self.arena = room[-room.data_ptr() % align:][:total]
            cursor = [0]

            def empty(n, dtype, device):
                nb = n * torch.empty((), dtype=dtype).element_size()
                v = self.arena[cursor[0]:cursor[0] + nb].view(dtype)
                cursor[0] += -(-nb // align) * align
                return v
        for m, fmt in zip(self.mats, self.fmts):
            ws, ss = wl.w_stream(m.index), wl.s_stream(m.index)
            if fmt == wl.Q4:
                w = empty(m.M * m.K // 2, dtype=torch.uint8, device="cuda")
                s = empty(m.M * (m.K // 32), dtype=torch.int16, device="cuda")
                if st is None:
                    gen_q4(w, seed, ws)
                    gen_uniform16(s, wl.Q4_SCALE_LO, wl.Q4_SCALE_HI, wl.F16, seed, ss)
                else:
                    st.put(w, _fill_q4(seed, ws, threads), w.numel())
                    st.put(s, _fill_scales(seed, ss, threads), s.numel() * 2)
            elif fmt == wl.I8:
                w = empty(m.M * m.K, dtype=torch.int8, device="cuda")
                s = empty(m.M, dtype=torch.int16, device="cuda")
                if st is None:
                    gen_i8(w, seed, ws)
                    gen_uniform16(s, synth.I8_SCALE_LO, synth.I8_SCALE_HI, wl.F16, seed, ss)
                else:
                    st.put(w, _fill_i8(seed, ws, threads), w.numel())
                    st.put(s, _fill_i8_scales(seed, ss, threads), s.numel() * 2)
            else:
                w = empty(m.M * m.K, dtype=torch.int16, device="cuda")
                s = None
                if st is None:
                    gen_normal16(w, w_sigma, fmt, seed, ws)
                else:
                    st.put(w, _fill_normal16(fmt, w_sigma, seed, ws, threads), w.numel() * 2)
            self.w.append(w)
            self.s.append(s)
            key = (m.layer, m.slot)
            if key not in self.x:
                xfmt = self.x_fmt(fmt)
                xs = torch.empty((tokens, m.K), dtype=torch.int16, device="cuda")
                gen_normal16(xs, wl.X_SIGMA, xfmt, seed, wl.x_stream(m.layer, wl.X_SLOTS[m.slot]))
                self.x[key] = (xs, xfmt)
            self.y.append(torch.zeros((tokens, m.M), dtype=torch.float32, device="cuda"))
        if st is not None:
            st.finish()
        torch.cuda.synchronize()

    @staticmethod
    def x_fmt(fmt):
        return wl.F16 if fmt in (wl.Q4, wl.I8) else fmt

    def weight_bytes(self) -> int:
        return sum(wl.matrix_bytes(m.M, m.K, f) for m, f in zip(self.mats, self.fmts))

    def specs(self, chained: bool = False):
        """Keyword dicts for wsr.make_mats; chained marks each activation-slot boundary of a layer
        as depending on earlier outputs (q|k|v, o, gate|up, down, head)."""
        out, prev = [], None
        for i, (m, fmt) in enumerate(zip(self.mats, self.fmts)):
            xt, _ = self.x[(m.layer, m.slot)]
            flags = 1 if (chained and prev is not None and (m.layer, m.slot) != prev) else 0
            prev = (m.layer, m.slot)
            out.append(dict(fmt=WSR_FMT[fmt], flags=flags, M=m.M, K=m.K, w=self.w[i],
                            scales=self.s[i], x=xt, x_tok_stride=m.K * 2, y=self.y[i],
                            y_tok_stride=m.M * 4))
        return out

    # -- host regeneration (for the oracle) --
    def host_weights(self, i: int, row0: int = 0, nrows: int | None = None):
        m, fmt = self.mats[i], self.fmts[i]
        nrows = m.M - row0 if nrows is None else nrows
        if fmt == wl.Q4:
            return (synth.q4_codes(nrows, m.K, seed=self.seed, stream=wl.w_stream(m.index), row0=row0),
                    synth.q4_scales(nrows, m.K, seed=self.seed, stream=wl.s_stream(m.index), row0=row0))
        if fmt == wl.I8:
            return (synth.i8_codes(nrows, m.K, seed=self.seed, stream=wl.w_stream(m.index), row0=row0),
                    synth.i8_scales(nrows, seed=self.seed, stream=wl.s_stream(m.index), row0=row0))
        return synth.normal16((nrows, m.K), self.w_sigma, fmt, seed=self.seed,
                              stream=wl.w_stream(m.index), e0=row0 * m.K)

    def host_x(self, i: int, t: int):
        m, fmt = self.mats[i], self.fmts[i]
        return synth.normal16(m.K, wl.X_SIGMA, self.x_fmt(fmt), seed=self.seed,
                              stream=wl.x_stream(m.layer, wl.X_SLOTS[m.slot]), e0=t * m.K)

    def dev_y(self, i: int, t: int) -> np.ndarray:
        return self.y[i][t].cpu().numpy()


def small_model(layers=2, d=256, ffn=512, vocab=1024, n_q=4, n_kv=1, head_dim=64):
    return wl.ModelShape("small", layers, d, n_q, n_kv, head_dim, ffn, vocab)
