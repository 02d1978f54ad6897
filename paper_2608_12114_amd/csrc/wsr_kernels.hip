/*
 * wsr_kernels.hip - HIP kernels of the weight-streaming read path for gfx950 and their launchers.
 *
 *  k_probe_part / k_probe_final   pure-read reference: fp32 buffer -> fp64 sum (paper Sec. 3.1, 3.3)
 *  k_gemv      single-token GEMV, fp32 accumulate: fp16 / bf16 weights (Sec. 3.1), 4-bit blocks and int8
 *              rows decoded in registers; k_gemv_small the same for the smallest matrices
 *  k_sweep     one decode token: every matrix of a table in one persistent launch (Sec. 6.2)
 *  k_put_table writes the sweep's matrix table into the caller's workspace from kernel arguments
 *              and clears the sweep's tile counters, so a sweep needs no host copy or host
 *              synchronisation (C3, Table 1)
 *
 * Streaming layout.  HBM3E serves long sequential runs best.  Each probe block walks its own
 * contiguous region.  The sweeps give each wave an equal contiguous span of the weight stream, and far
 * more blocks than the chip holds, so that retiring blocks are replaced up to the end.  16-bit streams
 * of 64 GiB or more and mixed tables hand out tiles of the stream (64 KiB to 2 MiB) in order from a
 * counter, so the waves in flight work on one moving front of memory and finish together.
 */
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "wsr_device.h"

namespace wsr {

constexpr int BLOCK = 256;
constexpr int WAVES_PER_BLOCK = BLOCK / WAVE;

/* ======================================= probe ================================================ */

constexpr int PROBE_UNROLL = 4;            /* 16-byte loads in flight per thread               */
constexpr int PROBE_ACC = 4;               /* independent fp64 accumulators per thread          */
constexpr int64_t PROBE_MAX_GRID = 512;    /* two blocks per CU: few, long sequential streams   */

int64_t probe_grid(int64_t n) {
    const int64_t n4 = n / 4;
    const int64_t per_block = (int64_t)BLOCK * PROBE_UNROLL * 4;
    const int64_t g = (n4 + per_block - 1) / per_block;
    return std::max<int64_t>(1, std::min(g, PROBE_MAX_GRID));
}

/* Elements are reinterpreted through __uint_as_float: applying __builtin_bit_cast to an element of
   an ext_vector_type value makes this compiler read element 0 for every component. */
__device__ __forceinline__ double sum4(u32x4 v, double acc) {
    acc += (double)__uint_as_float(v.x);
    acc += (double)__uint_as_float(v.y);
    acc += (double)__uint_as_float(v.z);
    acc += (double)__uint_as_float(v.w);
    return acc;
}

/* Sum over a block's threads, in a fixed order: valid in thread 0. */
__device__ __forceinline__ double block_sum(double v, double* red) {
    v = wave_sum(v);
    if ((threadIdx.x & (WAVE - 1)) == 0) red[threadIdx.x / WAVE] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < WAVES_PER_BLOCK; ++i) s += red[i];
    return s;
}

/* Block b sums 16-byte groups [b * chunk, (b + 1) * chunk): per step its 256 threads read 16 KiB of
   consecutive memory, thread t taking groups t, t + 256, t + 512, t + 768 into accumulators 0..3. */
__global__ __launch_bounds__(BLOCK) void k_probe_part(const u32x4* __restrict__ buf, int64_t n4,
                                                      double* __restrict__ part) {
    __shared__ double red[WAVES_PER_BLOCK];
    g_u32x4* b = as_global<g_u32x4*>(buf);
    const int64_t chunk = (n4 + gridDim.x - 1) / gridDim.x;
    const int64_t beg = (int64_t)blockIdx.x * chunk;
    const int64_t end = std::min<int64_t>(n4, beg + chunk);
    double acc[PROBE_ACC];
#pragma unroll
    for (int a = 0; a < PROBE_ACC; ++a) acc[a] = 0.0;
    int64_t i = beg + threadIdx.x;
    for (; i + (PROBE_UNROLL - 1) * BLOCK < end; i += PROBE_UNROLL * BLOCK) {
        u32x4 v[PROBE_UNROLL];
#pragma unroll
        for (int j = 0; j < PROBE_UNROLL; ++j) v[j] = load_once(b + i + j * BLOCK);
#pragma unroll
        for (int j = 0; j < PROBE_UNROLL; ++j) acc[j % PROBE_ACC] = sum4(v[j], acc[j % PROBE_ACC]);
    }
    for (; i < end; i += BLOCK) acc[0] = sum4(load_once(b + i), acc[0]);
    double t = 0.0;
#pragma unroll
    for (int a = 0; a < PROBE_ACC; ++a) t += acc[a];
    t = block_sum(t, red);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

/* One block: the partials in index order, then the n % 4 trailing elements. */
__global__ __launch_bounds__(BLOCK) void k_probe_final(const double* __restrict__ part, int G,
                                                       const float* __restrict__ tail, int ntail,
                                                       double* __restrict__ out) {
    __shared__ double red[WAVES_PER_BLOCK];
    double a = 0.0;
    for (int j = threadIdx.x; j < G; j += BLOCK) a += part[j];
    double s = block_sum(a, red);
    if (threadIdx.x == 0) {
        for (int j = 0; j < ntail; ++j) s += (double)tail[j];
        *out = s;
    }
}

hipError_t launch_probe(const float* buf, int64_t n, double* sum_dev, void* ws, hipStream_t s) {
    const int64_t g = probe_grid(n);
    const int64_t n4 = n / 4;
    double* part = static_cast<double*>(ws);
    hipLaunchKernelGGL(k_probe_part, dim3((unsigned)g), dim3(BLOCK), 0, s,
                       reinterpret_cast<const u32x4*>(buf), n4, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_probe_final, dim3(1), dim3(BLOCK), 0, s, part, (int)g, buf + 4 * n4,
                       (int)(n % 4), sum_dev);
    return hipGetLastError();
}

/* ======================================= GEMVs ================================================ */

/* One group of ROWS rows of a matrix, by one wave. */
template <int FMT, int R, int U>
struct Gemv16 {
    static constexpr int ROWS = R;
    static __device__ __forceinline__ void run(const DevMat& d, int64_t r0, int lane) {
        rows16<FMT, R, U>(d, r0, std::min<int64_t>(r0 + R, d.M), 0, lane);
    }
};
template <int R, int U>
struct GemvQ4 {
    static constexpr int ROWS = R;
    static __device__ __forceinline__ void run(const DevMat& d, int64_t r0, int lane) {
        rows_q4<R, U>(d, r0, std::min<int64_t>(r0 + R, d.M), 0, lane);
    }
};
/* The full and the partial group take separate branches rather than a clamp of the row end: the clamp's
   select was miscompiled (the pre-emit peephole dropped the instruction that set the select's
   condition, so the end became r0 + R past the last row). */
struct GemvI8 {
    static constexpr int ROWS = I8_GEMV_R;
    static __device__ __forceinline__ void run(const DevMat& d, int64_t r0, int lane) {
        if (d.M - r0 >= ROWS) rows_i8<ROWS>(d, r0, r0 + ROWS, 0, lane);
        else rows_i8<1>(d, r0, d.M, 0, lane);
    }
};
template <typename G>
__device__ __forceinline__ void gemv_wave(const DevMat& d) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t r0 = ((int64_t)blockIdx.x * WAVES_PER_BLOCK + wave_in_block()) * G::ROWS;
    if (r0 < d.M) G::run(d, r0, lane);
}

/* The matrix as single arguments, which the command processor puts into registers before the first
   instruction (the build asks for 16 of them): a launch among others takes 0.2 to 0.25 us less
   than with one structure, which is read from the argument memory (us, this and that: f16 4096 x 4096
   6.35 and 6.57, q4 4.00 and 4.20, int8 12288 x 7168 14.80 and 15.07).  The addresses go as integers:
   the runtime looks up the allocation of every pointer argument (3.26 us of host time per call against
   3.33, as one structure 3.15). */
template <typename G>
__global__ __launch_bounds__(BLOCK) void k_gemv(uint64_t w, uint64_t s, uint64_t x, uint64_t y, int64_t M, int64_t nc) {
    DevMat d{};
    d.w = reinterpret_cast<const void*>(w);
    d.s = reinterpret_cast<const void*>(s);
    d.x = reinterpret_cast<const void*>(x);
    d.y = reinterpret_cast<float*>(y);
    d.M = M;
    d.nc = nc;
    gemv_wave<G>(d);
}
/* The matrix as one structure: where the GPU is done before the host has enqueued the next call, the
   cheaper call is the faster one. */
template <typename G>
__global__ __launch_bounds__(BLOCK) void k_gemv_small(DevMat d) { gemv_wave<G>(d); }

/* Calls that the host bounds: those the GPU takes less than about 2.8 us for, with rows of one or two
   steps of a wave.  us a call back to back, as a structure and as single arguments: bf16 256 x 4096 2.95 and
   3.09, 768 x 4096 3.00 and 3.13, 512 x 2048 2.92 and 3.08, 2048 x 512 2.96 and 3.11, but 1536 x
   2048 3.38 and 3.09, 32 x 8192 3.30 and 3.13; q4 2048 x 2048 2.94 and 3.07, 256 x 4096 3.12 and
   3.09 to 3.18 and 3.27, but 8192 x 512 3.52 and 3.28, 1024 x 4096 3.83 and 3.58; int8 2048 x 1024
   2.96 and 3.09, 256 x 2048 2.96 and 3.12, but 1024 x 2048 3.54 and 3.27. */
static bool gemv_small(const DevMat& m) {
    const int64_t bytes = m.M * m.row_bytes;
    if (m.fmt == FMT_F16 || m.fmt == FMT_BF16) return m.nc <= 512 && (m.M <= 1024 || bytes <= (2 << 20));
    return m.nc <= 128 && bytes <= (m.nc <= 64 ? 2 << 20 : 1 << 20);
}

/* Rows [r0, M) of a matrix of the single-column kernels' layout. */
static DevMat rows_from(const DevMat& m, int64_t r0) {
    DevMat d = m;
    d.w = static_cast<const char*>(m.w) + r0 * m.nc * 16;
    if (m.s) d.s = static_cast<const char*>(m.s) + r0 * (m.fmt == FMT_Q4 ? m.nc * 2 : 2);
    d.y = m.y + r0;
    d.M = m.M - r0;
    return d;
}

/* A launch holds fewer than 2^32 threads: matrices of more rows than the waves of 2^23 blocks take go in
   several (16-bit ones from 2^25 rows on). */
constexpr int64_t GEMV_BLOCKS = int64_t{1} << 23;
template <typename G>
static hipError_t launch_rows(const DevMat& m, hipStream_t s) {
    constexpr int64_t each = WAVES_PER_BLOCK * G::ROWS;
    for (int64_t r0 = 0; r0 < m.M; r0 += GEMV_BLOCKS * each) {
        DevMat d = r0 ? rows_from(m, r0) : m;
        d.M = std::min<int64_t>(d.M, GEMV_BLOCKS * each);
        const dim3 grid((unsigned)((d.M + each - 1) / each));
        if (gemv_small(d))
            hipLaunchKernelGGL((k_gemv_small<G>), grid, dim3(BLOCK), 0, s, d);
        else
            hipLaunchKernelGGL((k_gemv<G>), grid, dim3(BLOCK), 0, s, reinterpret_cast<uint64_t>(d.w),
                               reinterpret_cast<uint64_t>(d.s), reinterpret_cast<uint64_t>(d.x),
                               reinterpret_cast<uint64_t>(d.y), d.M, d.nc);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

/* Two columns of a 16-bit matrix on the vector ALUs, four rows per wave. */
constexpr int PAIR16_R = 4;
template <int FMT>
__global__ __launch_bounds__(BLOCK) void k_gemv16_pair(DevMat d) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t r0 = ((int64_t)blockIdx.x * WAVES_PER_BLOCK + wave_in_block()) * PAIR16_R;
    if (r0 >= d.M) return;
    rows16_cols<FMT, PAIR16_R, 4, 2>(d, r0, std::min<int64_t>(r0 + PAIR16_R, d.M), 0, lane);
}

static hipError_t launch_gemv16_pair(const DevMat& m, hipStream_t s) {
    const int64_t rows = WAVES_PER_BLOCK * PAIR16_R, blocks = (m.M + rows - 1) / rows;
    if (m.fmt == FMT_F16)
        hipLaunchKernelGGL(k_gemv16_pair<FMT_F16>, dim3((unsigned)blocks), dim3(BLOCK), 0, s, m);
    else
        hipLaunchKernelGGL(k_gemv16_pair<FMT_BF16>, dim3((unsigned)blocks), dim3(BLOCK), 0, s, m);
    return hipGetLastError();
}

/* Where a matrix has rows for four waves per SIMD, two columns cost the vector ALUs little and whole
   rows per wave, with no sums to join, win over the matrix-core form (us, this and that: 20,000 x
   1,024 f16 8.1 and 10.5, 20,000 x 4,096 27.4 and 29.2, 100,000 x 4,096 bf16 121 and 128; 8,192 x
   8,192 29.8 and 25.2). */
static bool gemv16_pair(const DevMat& m, int T) {
    return T == 2 && (m.fmt == FMT_F16 || m.fmt == FMT_BF16) && m.M >= 4 * 4 * 1024 &&
           m.M <= GEMV_BLOCKS * WAVES_PER_BLOCK * PAIR16_R;     /* more than a launch holds */
}

hipError_t launch_gemv_cols(const DevMat& m, int T, hipStream_t s) {
    if (gemv16_pair(m, T))
        return launch_gemv16_pair(m, s);
    if (T > 1 && m.nc <= COLS_MAX_NC) return launch_cols(nullptr, nullptr, &m, 1, m.M * m.row_bytes, m.fmt, 0, T, s);
    DevMat d = m;                                   /* one column, or rows too long: column by column */
    for (int t = 0; t < T; ++t) {
        const hipError_t e = launch_gemv(d, s);
        if (e != hipSuccess) return e;
        d.x = static_cast<const char*>(d.x) + m.x_stride;
        d.y = reinterpret_cast<float*>(reinterpret_cast<char*>(d.y) + m.y_stride);
    }
    return hipSuccess;
}

/* Rows of 128 KiB or more (K >= 65536 at 16 bits) go four to a wave when that still leaves a wave
   per SIMD: with one row per wave each row rereads the whole activation vector from L2, as many
   bytes as its weights.  Measured on 4096 rows: K = 65536 5.87 -> 6.47 TB/s, K = 140800 6.13 ->
   6.76 TB/s; at K <= 32768 four rows per wave were slower (the 1,024 waves cannot cover the
   latency), so shorter rows keep one per wave. */
static bool gemv16_long_rows(const DevMat& m) { return m.nc >= 8192 && m.M >= 4 * 1024; }

hipError_t launch_gemv(const DevMat& m, hipStream_t s) {
    if (m.M == 0) return hipSuccess;
    switch (m.fmt) {
        case FMT_F16:
            return gemv16_long_rows(m) ? launch_rows<Gemv16<FMT_F16, 4, 8>>(m, s)
                                       : launch_rows<Gemv16<FMT_F16, 1, 8>>(m, s);
        case FMT_BF16:
            return gemv16_long_rows(m) ? launch_rows<Gemv16<FMT_BF16, 4, 8>>(m, s)
                                       : launch_rows<Gemv16<FMT_BF16, 1, 8>>(m, s);
        case FMT_Q4:
            return m.nc >= 256 ? launch_rows<GemvQ4<2, 2>>(m, s)
                               : launch_rows<GemvQ4<4, 1>>(m, s);
        case FMT_I8:
            return launch_rows<GemvI8>(m, s);
        default:
            return hipErrorInvalidValue;
    }
}

/* ======================================= sweep ================================================ */

/* Matrices per table-upload launch.  The chunk travels as a by-value kernel argument (30.7 KB at
   320 entries; arguments of up to 32,000 bytes were checked to arrive intact on this stack), so one
   launch uploads the table of a 225-matrix model and the arguments are captured by value when a
   caller records the sweep into a graph. */
constexpr int TABLE_CHUNK = 320;
struct TableChunk {
    int32_t n;
    int32_t pad_[3];
    DevMat m[TABLE_CHUNK];
};
static_assert(sizeof(TableChunk) <= 31 * 1024, "table chunk must stay within the checked argument size");

__global__ __launch_bounds__(BLOCK) void k_put_table(DevMat* __restrict__ dst, int64_t* __restrict__ cost,
                                                     TableChunk c, unsigned* __restrict__ ctr) {
    for (int i = threadIdx.x; i < c.n; i += BLOCK) {
        dst[i] = c.m[i];
        cost[i] = c.m[i].cost0;
    }
    if (ctr && threadIdx.x < 2) ctr[threadIdx.x] = 0u;
}

hipError_t launch_put_table(DevMat* dst, int64_t* cost, const DevMat* src, int n, unsigned* ctr,
                            hipStream_t s) {
    for (int first = 0; first < n; first += TABLE_CHUNK) {
        TableChunk c{};
        c.n = std::min(TABLE_CHUNK, n - first);
        for (int i = 0; i < c.n; ++i) c.m[i] = src[first + i];
        hipLaunchKernelGGL(k_put_table, dim3(1), dim3(BLOCK), 0, s, dst + first, cost + first, c,
                           first == 0 ? ctr : nullptr);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

enum : int { SCHED_TILES = 0, SCHED_SPANS = 1 };

/* Tile size: about four tiles per wave, a power of two between 64 KiB and 2 MiB. */
int64_t sweep_tile(int64_t total, int64_t waves) {
    int64_t t = 64 << 10;
    while (t < (2 << 20) && t * waves * 4 < total) t <<= 1;
    return t;
}

/* The wave's index in the order of spans.  The hardware hands consecutive blocks to the 8 XCDs in
   turn, each with its own L2, so numbering spans by block index would have every XCD work on every
   part of the stream at once.  Block b, on XCD b % 8, instead takes place b / 8 among that XCD's
   blocks inside the XCD's own eighth of the spans: each L2 then holds one contiguous part of the
   stream, so the activations of a matrix are fetched into fewer L2s and the output lines that
   neighbouring waves share are written through one L2 (8B q4 token: 619 -> 612 us). */
constexpr unsigned XCDS = 8;
__device__ __forceinline__ int64_t span_wave() {
    const unsigned nb = gridDim.x, b = blockIdx.x, xcd = b % XCDS, per = nb / XCDS, rem = nb % XCDS;
    const unsigned place = xcd * per + (xcd < rem ? xcd : rem) + b / XCDS;
    return (int64_t)place * WAVES_PER_BLOCK + wave_in_block();
}

/* Wave w takes bytes [w span, (w + 1) span) of the stream, cut at its end; the launcher sets span to
   ceil(total / waves), so no division runs on the device. */
__device__ __forceinline__ void span_bounds(int64_t total, int64_t w, int64_t span, int64_t& lo, int64_t& hi) {
    lo = w * span;
    hi = std::min<int64_t>(total, lo + span);
}

/* Work distribution over the weight stream [0, total) of one token:
     SCHED_TILES   tiles of `tile` bytes, claimed in order from a counter;
     SCHED_SPANS   wave w takes [span w, span (w + 1)) (span = ceil(total / nw)); with many more blocks than the
                   chip holds at once, the hardware starts each block as an earlier one retires,
                   which balances the end of the token at no cost.
   The counters ctr[0] (next tile) and ctr[1] (waves done) start at zero and the last wave to
   finish puts them back to zero for the next launch. */
template <int FMT, int SCHED, int R16, int U16, int RQ, int UQ, int T = 1>
__global__ __launch_bounds__(BLOCK) void k_sweep(const DevMat* __restrict__ tab, const int64_t* __restrict__ cost,
                                                 int nmat, int64_t total, int64_t span, int64_t tile,
                                                 int32_t token, unsigned* __restrict__ ctr) {
    const int lane = threadIdx.x & (WAVE - 1);
    const unsigned nw = gridDim.x * WAVES_PER_BLOCK;
    int hint = 0;
    if constexpr (SCHED == SCHED_SPANS) {
        int64_t lo, hi;
        span_bounds(total, span_wave(), span, lo, hi);
        if (lo < hi) stream_range<FMT, R16, U16, RQ, UQ, T>(tab, cost, nmat, lo, hi, token, lane, hint);
    } else {
        /* Each wave claims its next tile before working on the current one, so the round trip of
           the claim overlaps the current tile's loads. */
        const int64_t ntiles = ceil_div(total, tile);
        unsigned claim = 0;
        if (lane == 0) claim = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (;;) {
            const unsigned t = __builtin_amdgcn_readfirstlane(claim);
            if ((int64_t)t >= ntiles) break;
            if (lane == 0) claim = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int64_t lo = (int64_t)t * tile;
            stream_range<FMT, R16, U16, RQ, UQ, T>(tab, cost, nmat, lo, std::min<int64_t>(total, lo + tile),
                                                     token, lane, hint);
        }
        if (lane == 0) {
            const unsigned e = __hip_atomic_fetch_add(ctr + 1, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            if (e == nw - 1) {
                __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(ctr + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

/* A table of up to N matrices carried by value in the arguments of a span-scheduled sweep launch.
   The waves read their matrix records and stream offsets straight from the argument memory through
   the scalar cache, so such a sweep needs neither a workspace nor the table upload launch before
   it, whose kernel boundary measured about 4 us per call against a 1 GB pass of about 150 us.  Two
   sizes: 32 entries (3.3 KB, about 1 us per launch cheaper than the large block on a 32-matrix
   pass) and TABLE_ARG_MAX (29,952 bytes; arguments of up to 32,000 bytes were checked to arrive
   intact). */
constexpr int TABLE_ARG_SMALL = 32, TABLE_ARG_MAX = 288;
template <int N>
struct TableArg {
    DevMat m[N];
    int64_t cost[N];
};
static_assert(sizeof(TableArg<TABLE_ARG_MAX>) + 32 <= 32000, "the by-value table must stay within the checked argument size");

template <int FMT, int R16, int U16, int N, int T>
__global__ __launch_bounds__(BLOCK) void k_sweep_arg(int nmat, int32_t token, int64_t total, int64_t span,
                                                     TableArg<N> tb) {
    const int lane = threadIdx.x & (WAVE - 1);
    int hint = 0;
    int64_t lo, hi;
    span_bounds(total, span_wave(), span, lo, hi);
    if (lo < hi) stream_range<FMT, R16, U16, 8, 1, T>(tb.m, tb.cost, nmat, lo, hi, token, lane, hint);
}

/* Short streams: up to SHORT_MATS matrices, one group of rows per wave, blocks given to the matrices in
   turn by the host (f1 .. f7: the first block of matrices 1 .. 7, in registers when the kernel starts;
   one read of the argument memory then brings the matrix).  Such a launch lasts a few us, most of it
   before the first load and after the last: the sweep's spans spend that on looking up their rows
   (bisection, division) and give each wave eight rows or more, this form starts at once and has
   more waves (a launch of the 8B model's q, k and v in q4: 6.4 -> 4.4 us). */
constexpr int SHORT_MATS = 8;
struct ShortTable {
    DevMat m[SHORT_MATS];
};

template <int FMT, int R, int U, int WAVES>
__device__ __forceinline__ void short_rows(const DevMat& d, int64_t r0, int64_t r1, int32_t token, int lane) {
    if constexpr (FMT == FMT_Q4) {
        rows_q4<R, U, 2>(d, r0, r1, token, lane);
    } else if constexpr (FMT == FMT_I8 && WAVES == 1) {
        if (d.nc % WAVE == 0) rows_i8_pipe<R, 1, I8_NB, false>(d, r0, r1, token, lane);
        else rows_i8_pipe<R, 1, I8_NB, true>(d, r0, r1, token, lane);
    } else if constexpr (FMT == FMT_I8) {
        rows_i8<R>(d, r0, r1, token, lane);
    } else {
        rows16<FMT, R, U>(d, r0, r1, token, lane);
    }
}

template <int FMT, int R, int U, int WAVES>
__global__ __launch_bounds__(WAVE * WAVES) void k_sweep_short(int f1, int f2, int f3, int f4, int f5, int f6, int f7,
                                                       int32_t token, ShortTable tb) {
    const int lane = threadIdx.x & (WAVE - 1), b = (int)blockIdx.x;
    const int m = (b >= f1) + (b >= f2) + (b >= f3) + (b >= f4) + (b >= f5) + (b >= f6) + (b >= f7);
    const int first = m == 0 ? 0 : m == 1 ? f1 : m == 2 ? f2 : m == 3 ? f3 : m == 4 ? f4 : m == 5 ? f5 : m == 6 ? f6 : f7;
    const DevMat& d = tb.m[m];
    const int64_t r0 = ((int64_t)(b - first) * WAVES + (WAVES == 1 ? 0 : wave_in_block())) * R;
    if (r0 >= d.M) return;
    if (d.M - r0 >= R) short_rows<FMT, R, U, WAVES>(d, r0, r0 + R, token, lane);
    else short_rows<FMT, 1, U, WAVES>(d, r0, d.M, token, lane);
}

template <int FMT, int R, int U, int WAVES>
static hipError_t launch_short_blocks(const DevMat* htab, int nmat, int32_t token, hipStream_t s) {
    ShortTable tb;
    int f[SHORT_MATS + 1];
    int64_t blocks = 0;
    for (int i = 0; i < SHORT_MATS; ++i) {
        f[i] = i < nmat ? (int)blocks : INT32_MAX;
        if (i >= nmat) continue;
        tb.m[i] = htab[i];
        blocks += (htab[i].M + WAVES * R - 1) / (WAVES * R);   /* at most SHORT_ROWS / 4 */
    }
    hipLaunchKernelGGL((k_sweep_short<FMT, R, U, WAVES>), dim3((unsigned)blocks), dim3(WAVE * WAVES), 0, s, f[1], f[2], f[3],
                       f[4], f[5], f[6], f[7], token, tb);
    return hipGetLastError();
}

/* Launches of few 16-bit or int8 waves over long rows are bound by the latency of a wave's own steps and by
   the loads a CU keeps in flight: their waves go to CUs of their own, in blocks of one, with longer
   steps (16-bit) or the pipelined loop (int8).  us, blocks of four and of one: bf16 64 x 28672 10.0 and
   7.7, 512 x 14336 6.5 and 6.3, 17 x 28672 beside 625 x 10496 11.2 and 8.8, but 768 x 14336 6.8 and 7.1,
   1024 x 14336 7.2 and 7.9, 8192 x 2048 6.7 and 7.2, and rows of 4,096 alike; int8 1024 x 14336 12.5
   and 6.6, 4096 x 8192 10.5 and 7.8, but 8192 x 14336 19.6 and 20.1, 8192 x 2064 6.0 and 6.5.  q4, two
   sets of loads in flight in any case, takes blocks of one (8192 x 8192 11.0 and 9.0, 28672 x 4096 14.6
   and 13.6; a 5,120-wide model's layers as a chain 335 and 309) but for long rows of at most a wave per
   SIMD: the 8B model as a chain, with 4096 x 14336 matrices in it, 1,131 and 1,135, and so 1,100. */
static bool short_few(const DevMat* htab, int nmat, int rows, int64_t nc_over, int64_t most_long, int64_t most) {
    int64_t waves = 0, of_long = 0;
    for (int i = 0; i < nmat; ++i) {
        const int64_t n = (htab[i].M + rows - 1) / rows;
        waves += n;
        if (htab[i].nc > nc_over) of_long += n;
    }
    return of_long > 0 && of_long <= most_long && waves <= most;
}

template <int FMT>
static hipError_t launch_short(const DevMat* htab, int nmat, int32_t token, hipStream_t s) {
    if constexpr (FMT == FMT_Q4)
        return short_few(htab, nmat, 4, 256, 1024, 1024) ? launch_short_blocks<FMT, 4, 1, WAVES_PER_BLOCK>(htab, nmat, token, s)
                                                         : launch_short_blocks<FMT, 4, 1, 1>(htab, nmat, token, s);
    else if constexpr (FMT == FMT_I8)
        return short_few(htab, nmat, 2, 256, 2048, 4096) ? launch_short_blocks<FMT, 2, 1, 1>(htab, nmat, token, s)
                                                   : launch_short_blocks<FMT, 2, 1, WAVES_PER_BLOCK>(htab, nmat, token, s);
    else
        return short_few(htab, nmat, 1, 512, 768, 2048) ? launch_short_blocks<FMT, 1, 8, 1>(htab, nmat, token, s)
                                                  : launch_short_blocks<FMT, 1, 4, WAVES_PER_BLOCK>(htab, nmat, token, s);
}

static int cu_count() {
    static int cache[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cache[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cache[dev] = n;
    }
    return cache[dev];
}

/* 16-bit weights in very long streams, and mixed tables: tiles, 4 rows x 4 KiB steps per wave, one
   block (4 waves) per CU.  q4: spans of about 48 KiB per wave, 8 rows x 1 block per lane per step (eight rows
   share each block's activation decode), two register sets in flight; the grid is sized so that
   blocks retire and are replaced throughout the token (21,500 blocks for 4.2 GB).  int8: spans of
   about SWEEP_SPAN_I8 bytes per wave with 8 rows x 1 chunk per lane per step and three register
   sets in flight; tiles with one block per CU reach about half the rate
   (one wave per SIMD cannot cover the latency at each row group's start). */
constexpr int SWEEP_BLOCKS_PER_CU_16 = 1;
constexpr int64_t SWEEP_SPAN_Q4 = 48 << 10;
/* 16-bit streams up to 64 GiB go over spans of about 48 KiB per wave, two rows x 8 KiB steps, instead
   of claimed tiles: with few tiles per wave the end of the launch is uneven, and the blocks that
   retire and are replaced balance it.  Measured over tiles and over spans: the 1 GiB pass of 32
   fp16 matrices of 4096 x 4096 4.47 and 6.8 TB/s, four 70B bf16 layers and head (9 GB) 6.25 and 7.1,
   ten layers (17 GB) 6.8 and 7.12, forty layers and head (70 GB) 7.14 and 7.15, but 78 layers
   (136 GB) 7.15 and 6.42: over streams that long the eight contiguous parts lie far apart, and tiles
   keep the waves on one moving front.  Spans of 24, 32, 64 and 96 KiB: 9 GB at 6.86, 6.87, 6.99 and
   7.01 TB/s. */
constexpr int64_t SWEEP_SPAN_16 = 48 << 10;
constexpr int64_t SWEEP16_TILES_FROM = int64_t{64} << 30;
constexpr int SPAN16_R = 2, SPAN16_U = 8;
constexpr int64_t SWEEP_SPAN_I8 = 32 << 10;

/* Grid of a span-scheduled sweep: about `target` bytes per wave, at least one wave per SIMD; *span
   receives the bytes per wave, ceil(total / waves). */
static hipError_t span_grid(int64_t total, int64_t target, dim3& g, int64_t* span) {
    const int64_t waves = std::max<int64_t>((int64_t)cu_count() * WAVES_PER_BLOCK, (total + target - 1) / target);
    const int64_t blocks = (waves + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    g = dim3((unsigned)blocks);
    const int64_t nw = blocks * WAVES_PER_BLOCK;
    *span = (total + nw - 1) / nw;
    return hipSuccess;
}

template <int N>
static void fill_table_arg(TableArg<N>& tb, const DevMat* htab, int nmat) {
    for (int i = 0; i < nmat; ++i) {
        tb.m[i] = htab[i];
        tb.cost[i] = htab[i].cost0;
    }
}

/* One span-scheduled launch: the table by value when the host table is given (nmat <= TABLE_ARG_MAX),
   else from the device table. */
template <int FMT, int T = 1>
static hipError_t launch_sweep_spans(int64_t target, hipStream_t s, const DevMat* tab, const int64_t* cost,
                                     const DevMat* htab, int nmat, int64_t total, int32_t token) {
    constexpr int R = (FMT == FMT_F16 || FMT == FMT_BF16) ? SPAN16_R : 4;
    constexpr int U = (FMT == FMT_F16 || FMT == FMT_BF16) ? SPAN16_U : 4;
    dim3 g;
    int64_t span = 0;
    const hipError_t e = span_grid(total, target, g, &span);
    if (e != hipSuccess) return e;
    if (htab && nmat <= TABLE_ARG_SMALL) {
        TableArg<TABLE_ARG_SMALL> tb;
        fill_table_arg(tb, htab, nmat);
        hipLaunchKernelGGL((k_sweep_arg<FMT, R, U, TABLE_ARG_SMALL, T>), g, dim3(BLOCK), 0, s, nmat, token, total, span, tb);
    } else if (htab) {
        TableArg<TABLE_ARG_MAX> tb;
        fill_table_arg(tb, htab, nmat);
        hipLaunchKernelGGL((k_sweep_arg<FMT, R, U, TABLE_ARG_MAX, T>), g, dim3(BLOCK), 0, s, nmat, token, total, span, tb);
    } else {
        hipLaunchKernelGGL((k_sweep<FMT, SCHED_SPANS, R, U, 8, 1, T>), g, dim3(BLOCK), 0, s, tab, cost, nmat, total, span,
                           (int64_t)0, token, nullptr);
    }
    return hipGetLastError();
}

/* Which single-token launches run over spans (those may take their table by value). */
static bool sweep_spans(int64_t total, int fmt_all) {
    return fmt_all == FMT_Q4 || fmt_all == FMT_I8 ||
           ((fmt_all == FMT_F16 || fmt_all == FMT_BF16) && total < SWEEP16_TILES_FROM);
}

/* Single-token launches of one format over few matrices and at most SHORT_BYTES take k_sweep_short.
   Measured as chains of launches, short form against spans (us): the 8B model's layer (14 to 66 MB a
   launch) q4 1,139 and 1,395 for 32 layers and the head, int8 46.5 and 52.3 for one layer, bf16 71.7
   and 77.4; the layer as one launch (122 to 436 MB) q4 24.5 and 24.7, int8 37.2 and 38.4, bf16 equal. */
constexpr int64_t SHORT_BYTES = 256 << 20;
/* Empty rows (K = 0) cost a byte of the stream or two and could be more than a grid holds: a launch has
   fewer than 2^32 threads, and a wave of this form takes as little as one row.  Rows that are not empty
   stay below the limit, at 16 bytes or more each. */
constexpr int64_t SHORT_ROWS = int64_t{1} << 24;
static bool sweep_short(const DevMat* htab, int nmat, int64_t total, int fmt_all) {
    if (nmat > SHORT_MATS || total > SHORT_BYTES || fmt_all == 0) return false;
    int64_t rows = 0;
    for (int i = 0; i < nmat; ++i) rows += htab[i].M;
    return rows <= SHORT_ROWS;
}

/* int8 with two columns in long streams: two packed dot products per code pair are no burden to the
   vector ALUs, and the two-column form of the sweep's loop streams best (per pass against the
   matrix-core form, which forms four columns whatever it is asked for: the 72B model 0.732 and 0.742
   ms, a 0.6 GB model of 2,048-wide layers 95 and 109 us). */
static bool sweep_i8_pair(const DevMat* htab, int nmat, int fmt_all, int T) {
    return T == 2 && fmt_all == FMT_I8 && !cols_takes_split(htab, nmat, fmt_all, T);
}

bool sweep_table_by_value(const DevMat* htab, int nmat, int64_t total, int fmt_all, int T) {
    if (T > 1 && !sweep_i8_pair(htab, nmat, fmt_all, T)) return nmat <= cols_table_by_value(fmt_all);
    return (T == 1 && sweep_short(htab, nmat, total, fmt_all)) || (nmat <= TABLE_ARG_MAX && sweep_spans(total, fmt_all));
}

hipError_t launch_sweep(const DevMat* tab, const int64_t* cost, const DevMat* htab, int nmat, int64_t total,
                        int fmt_all, int32_t token, int T, unsigned* ctr, hipStream_t s) {
    if (nmat == 0 || total == 0) return hipSuccess;
    if (T == 1 && sweep_short(htab, nmat, total, fmt_all)) {
        switch (fmt_all) {
            case FMT_Q4: return launch_short<FMT_Q4>(htab, nmat, token, s);
            case FMT_I8: return launch_short<FMT_I8>(htab, nmat, token, s);
            case FMT_F16: return launch_short<FMT_F16>(htab, nmat, token, s);
            default: return launch_short<FMT_BF16>(htab, nmat, token, s);
        }
    }
    const bool pair = sweep_i8_pair(htab, nmat, fmt_all, T);
    if (T > 1 && !pair) return launch_cols(tab, cost, htab, nmat, total, fmt_all, token, T, s);
    if (!sweep_table_by_value(htab, nmat, total, fmt_all, T)) htab = nullptr;
    if (pair) return launch_sweep_spans<FMT_I8, 2>(SWEEP_SPAN_I8, s, tab, cost, htab, nmat, total, token);
    if (fmt_all == FMT_Q4) return launch_sweep_spans<FMT_Q4>(SWEEP_SPAN_Q4, s, tab, cost, htab, nmat, total, token);
    if (fmt_all == FMT_I8) return launch_sweep_spans<FMT_I8>(SWEEP_SPAN_I8, s, tab, cost, htab, nmat, total, token);
    if (sweep_spans(total, fmt_all))
        return fmt_all == FMT_F16 ? launch_sweep_spans<FMT_F16>(SWEEP_SPAN_16, s, tab, cost, htab, nmat, total, token)
                                  : launch_sweep_spans<FMT_BF16>(SWEEP_SPAN_16, s, tab, cost, htab, nmat, total, token);
    /* 16-bit (or mixed-format) sweep over tiles */
    const dim3 grid((unsigned)(cu_count() * SWEEP_BLOCKS_PER_CU_16));
    const int64_t tile = sweep_tile(total, (int64_t)grid.x * WAVES_PER_BLOCK);
#define WSR_TILES(F)                                                                                               \
    hipLaunchKernelGGL((k_sweep<F, SCHED_TILES, 4, 4, 8, 1>), grid, dim3(BLOCK), 0, s, tab, cost, nmat, total, \
                       (int64_t)0, tile, token, ctr)
    switch (fmt_all) {
        case FMT_F16: WSR_TILES(FMT_F16); break;
        case FMT_BF16: WSR_TILES(FMT_BF16); break;
        default: WSR_TILES(0); break;
    }
#undef WSR_TILES
    return hipGetLastError();
}

/* ================================ allocation-free sweep scratch ================================ */

/* Each device holds its own copy of this array, at its own address, from the time the library's
   code is loaded on that device until the process ends.  Host code never passes the array's name
   to a kernel or a copy: that name is a host-side stand-in, not a device address.  It uses the
   address hipGetSymbolAddress reports for the current device, looked up once per device. */
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

hipError_t noalloc_scratch(void** ptr) {
    static std::mutex mu;
    static void* addr[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

}  // namespace wsr
