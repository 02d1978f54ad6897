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
   chip holds: with fewer, and so with parts of the chip idle, the split form's smaller rounds win.  us,
   k_split and k_cols, at K = 4096 / 14336 (16 columns: / 7168):
     rounds            192                    256                    384                    448                    512
     q4   2 columns   7.6 8.4 / 15.4 19.0    7.7 8.6 / 16.5 19.6    9.9 11.0 / 23.1 26.8   11.9 11.1 / 27.5 27.4  13.4 11.2 / 28.4 28.2
     q4   8 columns  10.4 11.3 / 22.6 29.5  10.6 11.6 / 23.8 29.6  14.4 15.7 / 34.0 41.0  17.0 15.8 / 41.3 41.9  17.4 16.1 / 43.1 43.5
     int8 4 columns   9.1 11.3 / 20.1 27.2  10.7 12.7 / 21.5 28.3  13.5 15.0 / 31.7 35.4  15.4 15.8 / 39.2 37.0  16.1 17.5 / 40.9 39.4
     int8 8 columns  10.5 11.6 / 24.5 27.7  11.9 12.8 / 26.6 30.6  16.1 16.5 / 39.0 42.7  19.2 17.4 / 48.0 45.3  21.5 19.1 / 52.9 48.6
     bf16 8 columns  13.4 17.3 / 36.1 44.1  17.6 21.7 / 47.9 47.6  21.2 28.3 / 67.6 69.2  26.1 29.4 / 87.6 76.5  27.3 34.3 / 91.0 88.1
     bf16 16 columns 16.4 18.6 / 25.7 25.7  23.9 22.6 / 37.4 26.9  27.8 28.9 / 46.4 39.1  40.4 29.1 / 68.1 41.1  41.6 37.5 / 70.5 44.3
   Just above 512 rounds k_cols runs a second round of workgroups that is mostly empty, and the split form
   wins again up to about one and a half where rows are long or columns few (K = 4096 / 16384):
     rounds            576                    704                    768                    832
     q4   2 columns    15  16 /  49  52       16  16 /  49  53       16  16 /  52  53       19  17 /  63  54
     q4   8 columns    23  22 /  67  84       24  22 /  69  84       24  22 /  69  85       29  23 /  85  85
     int8 4 columns    20  22 /  73  73       20  23 /  74  77       21  24 /  77  78       25  25 /  92  80
     int8 8 columns    23  23 /  81  86       24  24 /  86  89       25  25 /  85  92       32  26 / 106  92
     bf16 8 columns    30  41 / 105 137       38  41 / 140 155       39  40 / 144 140       50  41 / 195 150
   16-bit weights with at most four columns, whose activations are half their weights' size or less, stay
   with the split form on long streams too (four layers and the head of the 70B model in bf16 at 2
   columns: 1.37, 1.46 ms per pass, at 4 1.38, 1.46).
   Tables of several formats always take k_cols, which replaced claimed tiles on the vector ALUs (us a
   pass at 2, 4 and 8 columns, before and now: four layers each in q4, int8 and f16, 4096 and 14336
   wide, 885 -> 523, 1,074 -> 541, 1,826 -> 632; two of each 2048 and 5632 wide, and a head, 176 -> 91,
   201 -> 92, 300 -> 125). */
static bool cols_split(int fmt, int T, int64_t rounds32, int64_t steps) {   /* steps of the longest row */
    const bool w16 = fmt == FMT_F16 || fmt == FMT_BF16, i8 = fmt == FMT_I8;
    if (w16 && T <= 4) return true;
    if (T > 8) return rounds32 < 256;
    if (rounds32 <= 512) return rounds32 <= (i8 && T <= 4 ? 512 : 384);
    return rounds32 <= (w16 ? 576 : i8 && T <= 4 ? 704 : 768) && (w16 || T <= 4 || steps >= (i8 ? 8 : 4));
}
static int64_t longest_steps(const DevMat* m, int nmat) {
    int64_t nc = 0;
    for (int i = 0; i < nmat; ++i) nc = std::max(nc, m[i].nc);
    return (nc + WAVE - 1) / WAVE;
}

bool cols_takes_split(const DevMat* htab, int nmat, int fmt_all, int T) {
    const int64_t rounds = rounds_of(htab, nmat, COLS_ROUND);
    if (fmt_all == FMT_I8 && T == 2) return rounds <= 512;      /* above, two columns stay with the vector ALUs
                                                                   (640 rounds of 8,192: 28.9 us, split 33.1) */
    return cols_split(fmt_all, T, rounds, longest_steps(htab, nmat));
}

/* Bytes per workgroup: k_cols keeps its activations over a span, and longer spans balance worse
   (8B q4 at 8 columns: 1.12, 1.11, 1.21 ms with 1, 2, 4 MiB; the 72B model in int8 at 4 columns 0.78
   ms with 1 or 2, 0.76 with 4); k_split's workgroups are smaller. */
constexpr int64_t COLS_SPAN = 2 << 20, COLS_SPAN_I8 = 4 << 20, SPLIT_SPAN = 1 << 20, SPLIT_SPAN_I8 = 512 << 10;
constexpr int64_t COLS_BLOCKS = 512, SPLIT_BLOCKS = 1024;    /* least, where there are that many rounds */

/* Workgroups and bytes of the stream for each: `want` of them at most, and no more than there are rounds
   of `rows` rows, since an empty one still waits for its LDS (1024 x 4096 q4 at 8 columns: 23 us with
   2,048 workgroups for its 128 rounds of 8 rows, 6.1 us with 128). */
static hipError_t cols_grid(const DevMat* htab, int nmat, int64_t cost, int64_t rows, int64_t want, dim3& g,
                            int64_t* span) {
    const int64_t rounds = rounds_of(htab, nmat, rows), each = (rounds + want - 1) / want;
    const int64_t blocks = (rounds + each - 1) / each;          /* the same number of rounds for each */
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    g = dim3((unsigned)blocks);
    *span = (cost + blocks - 1) / blocks;
    return hipSuccess;
}

template <int FMT, int TQ, int RG, int N>
static hipError_t launch_split(const ColsTable<N>& tb, const DevMat* htab, int nmat, int64_t total, int64_t cost, int32_t token,
                               int T, hipStream_t s) {
    const int64_t bytes = FMT == FMT_I8 ? SPLIT_SPAN_I8 : SPLIT_SPAN;
    dim3 g;
    int64_t span = 0;
    const hipError_t e = cols_grid(htab, nmat, cost, 4 * RG, std::max<int64_t>(SPLIT_BLOCKS, (total + bytes - 1) / bytes), g,
                                   &span);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_split<FMT, TQ, RG, N>), g, dim3(4 * WAVE), 0, s, nmat, token, cost, span, T, tb);
    return hipGetLastError();
}

template <int FMT, int TQ, int N>
static hipError_t launch_table(const ColsTable<N>& tb, const DevMat* htab, int nmat, int64_t total, int64_t cost, int32_t token,
                               int T, hipStream_t s) {
    if constexpr (FMT != 0) {
        if (cols_split(FMT, T, rounds_of(htab, nmat, COLS_ROUND), longest_steps(htab, nmat))) {
            constexpr int RG = split_rg<FMT>();
            /* us, with two and with four groups per round: q4 at 8 columns 1024 x 4096 6.1 and 7.2, 4096 x
               4096 8.8 and 7.4 */
            if constexpr (N == COLS_TABLE_ARG && RG > SPLIT_RG_FEW)
                if (rounds_of(htab, nmat, 4 * RG) <= 128)
                    return launch_split<FMT, TQ, SPLIT_RG_FEW, N>(tb, htab, nmat, total, cost, token, T, s);
            return launch_split<FMT, TQ, RG, N>(tb, htab, nmat, total, cost, token, T, s);
        }
    }
    if constexpr (FMT == 0 || FMT == FMT_Q4 || FMT == FMT_I8 || TQ > 1) {    /* 16-bit, TQ = 1: always split */
        constexpr int WAVES = cols_waves<FMT, TQ>();
        /* a whole number of workgroups for each that the chip holds at once */
        const int64_t bytes = COLS_BLOCKS * (FMT == FMT_I8 ? COLS_SPAN_I8 : COLS_SPAN);
        dim3 g;
        int64_t span = 0;
        const hipError_t e = cols_grid(htab, nmat, cost, COLS_ROUND,
                                       COLS_BLOCKS * std::max<int64_t>(1, (total + bytes / 2) / bytes), g, &span);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_cols<FMT, TQ, WAVES, N>), g, dim3(WAVE * WAVES), 0, s, nmat, token, cost, span, T, tb);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

/* Whether the rows of a table by value are weighed by their steps (of 64 chunks, and one more for the join
   and the start) instead of their bytes: where the shortest are a few chunks long, equal bytes give some
   workgroups hundreds of rounds of short rows, each with its own latency (us a pass, by bytes and by
   steps: q4 at 4 columns 115 x 512, 2000 x 64 and 609 x 11008 62 and 9.2; f16 at 4 892 x 8192, 5000 x 64,
   20000 x 256 and 7272 x 28672 314 and 107; bf16 at 2 6777 x 88, 60000 x 7000 and 4655 x 7352 516 and 180).
   Long rows stream at their bytes: where the lengths differ by up to four, as in a model's layers,
   weighing by steps costs up to a third (layers of 2,048 and 5,632 in q4 at 8 columns 53.5 and 67.7, int8
   8B layers at 4 148.5 and 172.6). */
constexpr int64_t COLS_STEPS_FROM = 4;
static bool cols_by_steps(const DevMat* htab, int nmat) {
    int64_t lo = INT64_MAX, hi = 0;
    for (int i = 0; i < nmat; ++i) {
        if (htab[i].M == 0) continue;
        lo = std::min(lo, htab[i].nc);
        hi = std::max(hi, htab[i].nc);
    }
    return COLS_STEPS_FROM * lo < hi;
}

template <int FMT, int TQ, int N>
static hipError_t launch_arg(const DevMat* htab, int nmat, int64_t total, int32_t token, int T, hipStream_t s) {
    ColsTable<N> tb;
    const bool steps = cols_by_steps(htab, nmat);
    int64_t cost = 0;
    for (int i = 0; i < nmat; ++i) {
        tb.m_[i] = htab[i];
        if (steps) {
            tb.m_[i].cost0 = cost;
            tb.m_[i].row_bytes = (htab[i].nc + WAVE - 1) / WAVE + 1;
            cost += tb.m_[i].row_bytes * htab[i].M;
        }
        tb.cost_[i] = tb.m_[i].cost0;
    }
    return launch_table<FMT, TQ, N>(tb, htab, nmat, total, steps ? cost : total, token, T, s);
}

template <int FMT, int TQ>
static hipError_t launch_q(const DevMat* tab, const int64_t* cost, const DevMat* htab, int nmat, int64_t total,
                           int32_t token, int T, hipStream_t s) {
    if (nmat <= COLS_TABLE_ARG) return launch_arg<FMT, TQ, COLS_TABLE_ARG>(htab, nmat, total, token, T, s);
    if constexpr (FMT == FMT_Q4 || FMT == FMT_I8) {
        if (nmat <= COLS_TABLE_ARG_MID) return launch_arg<FMT, TQ, COLS_TABLE_ARG_MID>(htab, nmat, total, token, T, s);
        if (nmat <= COLS_TABLE_ARG_MAX) return launch_arg<FMT, TQ, COLS_TABLE_ARG_MAX>(htab, nmat, total, token, T, s);
    }
    return launch_table<FMT, TQ, 0>({tab, cost}, htab, nmat, total, total, token, T, s);
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
