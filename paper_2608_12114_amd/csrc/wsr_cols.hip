/*
 * wsr_cols.hip - multi-column GEMV and batched decode sweep, every column bit for bit the single-column
 * result: kernels and launcher.
 *
 *  k_cols    long streams: activations shared by a workgroup through LDS
 *  k_split   short streams: the waves of a workgroup split their rows' chunks
 */
#include <hip/hip_runtime.h>

#include <algorithm>

#include "wsr_cols.h"

namespace wsr {

/* A table by value: the kernel's arguments, or (N = 0) pointers to the table in device memory.  q4 and int8
   passes take up to COLS_TABLE_ARG_MAX matrices by value, in the sizes of the single-token sweep: the
   upload before them costs 2 to 3 us (us a pass at 8 columns, uploaded and by value: nine q4 4096 x
   4096 37.1 and 34.2, 28 int8 1024 x 1024 14.8 and 11.6, twelve int8 12288 x 7168 221 and 220, the
   8B q4 model 1,107 and 1,104). */
constexpr int COLS_TABLE_ARG = 8, COLS_TABLE_ARG_MID = 32, COLS_TABLE_ARG_MAX = 288;
int cols_table_by_value(int fmt_all) {
    return fmt_all == FMT_Q4 || fmt_all == FMT_I8 ? COLS_TABLE_ARG_MAX : COLS_TABLE_ARG;
}
template <int N>
struct ColsTable {
    DevMat m_[N];
    int64_t cost_[N];
    __device__ const DevMat* m() const { return m_; }
    __device__ const int64_t* cost() const { return cost_; }
};
static_assert(sizeof(ColsTable<COLS_TABLE_ARG_MAX>) + 64 <= 32000, "the by-value table must stay within the checked argument size");
template <>
struct ColsTable<0> {
    const DevMat* __restrict__ m_;
    const int64_t* __restrict__ cost_;
    __device__ const DevMat* m() const { return m_; }
    __device__ const int64_t* cost() const { return cost_; }
};

template <int FMT, int TQ>
constexpr int cols_lds_bytes() {
    if constexpr (FMT == 0) {
        constexpr int a = ColsLds<FMT_F16, TQ>::STEP * ColsLds<FMT_F16, TQ>::SLABS;
        if constexpr (TQ <= 2) {
            constexpr int b = ColsLds<FMT_Q4, TQ>::STEP * ColsLds<FMT_Q4, TQ>::SLABS;
            constexpr int c = ColsLds<FMT_I8, TQ>::STEP * ColsLds<FMT_I8, TQ>::SLABS;
            return std::max(a, std::max(b, c));
        } else {
            return a;
        }
    } else {
        return ColsLds<FMT, TQ>::STEP * ColsLds<FMT, TQ>::SLABS;
    }
}

template <int FMT, int TQ, int WAVES, int N>
__global__ __launch_bounds__(WAVE * WAVES) __attribute__((amdgpu_waves_per_eu(FMT == 0 ? 2 : WAVES / 2)))
void k_cols(int nmat, int32_t token, int64_t total, int64_t span, int ntok, ColsTable<N> tb) {
    __shared__ __align__(16) char lds[cols_lds_bytes<FMT, TQ>()];
    const int64_t lo = (int64_t)blockIdx.x * span, hi = std::min<int64_t>(total, lo + span);
    if (lo < hi)
        stream_range_cols<FMT, TQ, WAVES>(tb.m(), tb.cost(), nmat, lo, hi, token, ntok, threadIdx.x & (WAVE - 1),
                                          wave_in_block(), lds);
}

template <int FMT, int TQ, int RG, int N>
__global__ __launch_bounds__(4 * WAVE) __attribute__((amdgpu_waves_per_eu(2)))
void k_split(int nmat, int32_t token, int64_t total, int64_t span, int ntok, ColsTable<N> tb) {
    __shared__ __align__(16) char lds[split_lds_bytes<FMT, TQ, RG>()];
    const int64_t lo = (int64_t)blockIdx.x * span, hi = std::min<int64_t>(total, lo + span);
    if (lo < hi)
        stream_range_split<FMT, TQ, RG>(tb.m(), tb.cost(), nmat, lo, hi, token, ntok, threadIdx.x & (WAVE - 1),
                                    wave_in_block(), lds);
}

/* Rounds of `rows` rows that the table's matrices hold. */
static int64_t rounds_of(const DevMat* m, int nmat, int64_t rows) {
    int64_t n = 0;
    for (int i = 0; i < nmat; ++i) n += (m[i].M + rows - 1) / rows;
    return std::max<int64_t>(n, 1);
}

/* Whether a pass takes k_split.  k_cols needs its rounds of 32 rows to fill the 512 workgroups the
   chip holds: with fewer, and so with parts of the chip idle, the split form's smaller rounds win
   (in us, k_split against k_cols and against the vector-ALU form before both: q4 at 8 columns
   4096 x 4096 7.6, 11.6, 11.9; 4096 x 14336 15.2, 29.4, 35.1; 28672 x 4096 (896 rounds) 39.1, 25.2,
   77.7; int8 at 4 columns 12288 x 7168 (384 rounds) 18.5, 22.5, 23.3, at 8 columns 25.7, 24.5, 37.1;
   bf16 8192 x 8192 (256 rounds) at 8 columns 27.9, 34.1, 34.7, at 16 35.2, 36.5, 38.9).  16-bit
   weights with at most four columns, whose activations are half their weights' size or less, stay
   with the split form on long streams too (four layers and the head of the 70B model in bf16 at 2
   columns: 1.37, 1.46, 1.47 ms per pass, at 4 1.38, 1.46, 1.51). */
static bool cols_split(int fmt, int T, int64_t rounds32) {
    const bool w16 = fmt == FMT_F16 || fmt == FMT_BF16;
    if (w16 && T <= 4) return true;
    return rounds32 < (T > 8 ? 256 : fmt == FMT_I8 && T <= 4 ? 512 : 384);
}

bool cols_takes_split(const DevMat* htab, int nmat, int fmt_all, int T) {
    return cols_split(fmt_all, T, rounds_of(htab, nmat, COLS_ROUND));
}

/* Bytes per workgroup: k_cols keeps its activations over a span, and longer spans balance worse
   (8B q4 at 8 columns: 1.12, 1.11, 1.21 ms with 1, 2, 4 MiB; the 72B model in int8 at 4 columns 0.78
   ms with 1 or 2, 0.76 with 4); k_split's workgroups are smaller. */
constexpr int64_t COLS_SPAN = 2 << 20, COLS_SPAN_I8 = 4 << 20, SPLIT_SPAN = 1 << 20, SPLIT_SPAN_I8 = 512 << 10;
constexpr int64_t COLS_BLOCKS = 512, SPLIT_BLOCKS = 1024;    /* least, where there are that many rounds */

/* Workgroups and bytes of the stream for each: `want` of them at most, and no more than there are rounds
   of `rows` rows, since an empty one still waits for its LDS (1024 x 4096 q4 at 8 columns: 23 us with
   2,048 workgroups for its 128 rounds of 8 rows, 6.1 us with 128). */
static hipError_t cols_grid(const DevMat* htab, int nmat, int64_t total, int64_t rows, int64_t want, dim3& g,
                            int64_t* span) {
    const int64_t rounds = rounds_of(htab, nmat, rows), each = (rounds + want - 1) / want;
    const int64_t blocks = (rounds + each - 1) / each;          /* the same number of rounds for each */
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    g = dim3((unsigned)blocks);
    *span = (total + blocks - 1) / blocks;
    return hipSuccess;
}

template <int FMT, int TQ, int RG, int N>
static hipError_t launch_split(const ColsTable<N>& tb, const DevMat* htab, int nmat, int64_t total, int32_t token, int T,
                               hipStream_t s) {
    const int64_t bytes = FMT == FMT_I8 ? SPLIT_SPAN_I8 : SPLIT_SPAN;
    dim3 g;
    int64_t span = 0;
    const hipError_t e = cols_grid(htab, nmat, total, 4 * RG, std::max<int64_t>(SPLIT_BLOCKS, (total + bytes - 1) / bytes), g,
                                   &span);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_split<FMT, TQ, RG, N>), g, dim3(4 * WAVE), 0, s, nmat, token, total, span, T, tb);
    return hipGetLastError();
}

template <int FMT, int TQ, int N>
static hipError_t launch_table(const ColsTable<N>& tb, const DevMat* htab, int nmat, int64_t total, int32_t token, int T,
                               hipStream_t s) {
    if constexpr (FMT != 0) {
        if (cols_split(FMT, T, rounds_of(htab, nmat, COLS_ROUND))) {
            constexpr int RG = split_rg<FMT>();
            /* us, with two and with four groups per round: q4 at 8 columns 1024 x 4096 6.1 and 7.2, 4096 x
               4096 8.8 and 7.4 */
            if constexpr (N == COLS_TABLE_ARG && RG > SPLIT_RG_FEW)
                if (rounds_of(htab, nmat, 4 * RG) <= 128)
                    return launch_split<FMT, TQ, SPLIT_RG_FEW, N>(tb, htab, nmat, total, token, T, s);
            return launch_split<FMT, TQ, RG, N>(tb, htab, nmat, total, token, T, s);
        }
    }
    if constexpr (FMT == 0 || FMT == FMT_Q4 || FMT == FMT_I8 || TQ > 1) {    /* 16-bit, TQ = 1: always split */
        constexpr int WAVES = cols_waves<FMT, TQ>();
        /* a whole number of workgroups for each that the chip holds at once */
        const int64_t bytes = COLS_BLOCKS * (FMT == FMT_I8 ? COLS_SPAN_I8 : COLS_SPAN);
        dim3 g;
        int64_t span = 0;
        const hipError_t e = cols_grid(htab, nmat, total, COLS_ROUND,
                                       COLS_BLOCKS * std::max<int64_t>(1, (total + bytes / 2) / bytes), g, &span);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_cols<FMT, TQ, WAVES, N>), g, dim3(WAVE * WAVES), 0, s, nmat, token, total, span, T, tb);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

template <int FMT, int TQ, int N>
static hipError_t launch_arg(const DevMat* htab, int nmat, int64_t total, int32_t token, int T, hipStream_t s) {
    ColsTable<N> tb;
    for (int i = 0; i < nmat; ++i) {
        tb.m_[i] = htab[i];
        tb.cost_[i] = htab[i].cost0;
    }
    return launch_table<FMT, TQ, N>(tb, htab, nmat, total, token, T, s);
}

template <int FMT, int TQ>
static hipError_t launch_q(const DevMat* tab, const int64_t* cost, const DevMat* htab, int nmat, int64_t total,
                           int32_t token, int T, hipStream_t s) {
    if (nmat <= COLS_TABLE_ARG) return launch_arg<FMT, TQ, COLS_TABLE_ARG>(htab, nmat, total, token, T, s);
    if constexpr (FMT == FMT_Q4 || FMT == FMT_I8) {
        if (nmat <= COLS_TABLE_ARG_MID) return launch_arg<FMT, TQ, COLS_TABLE_ARG_MID>(htab, nmat, total, token, T, s);
        if (nmat <= COLS_TABLE_ARG_MAX) return launch_arg<FMT, TQ, COLS_TABLE_ARG_MAX>(htab, nmat, total, token, T, s);
    }
    return launch_table<FMT, TQ, 0>({tab, cost}, htab, nmat, total, token, T, s);
}

template <int FMT>
static hipError_t launch_f(const DevMat* tab, const int64_t* cost, const DevMat* htab, int nmat, int64_t total,
                           int32_t token, int T, hipStream_t s) {
    if (T >= 2 && T <= 4) return launch_q<FMT, 1>(tab, cost, htab, nmat, total, token, T, s);
    if (T > 4 && T <= 8) return launch_q<FMT, 2>(tab, cost, htab, nmat, total, token, T, s);
    if constexpr (FMT != FMT_Q4 && FMT != FMT_I8)
        if (T > 8 && T <= 16) return launch_q<FMT, 4>(tab, cost, htab, nmat, total, token, T, s);
    return hipErrorInvalidValue;
}

hipError_t launch_cols(const DevMat* tab, const int64_t* cost, const DevMat* htab, int nmat, int64_t total, int fmt_all,
                       int32_t token, int T, hipStream_t s) {
    if (nmat == 0 || total == 0) return hipSuccess;
    switch (fmt_all) {
        case FMT_F16: return launch_f<FMT_F16>(tab, cost, htab, nmat, total, token, T, s);
        case FMT_BF16: return launch_f<FMT_BF16>(tab, cost, htab, nmat, total, token, T, s);
        case FMT_Q4: return launch_f<FMT_Q4>(tab, cost, htab, nmat, total, token, T, s);
        case FMT_I8: return launch_f<FMT_I8>(tab, cost, htab, nmat, total, token, T, s);
        default: return launch_f<0>(tab, cost, htab, nmat, total, token, T, s);
    }
}

}  // namespace wsr
