/*
 * wsr_mma.hip - the batched decode sweep on the matrix cores: kernel and launcher.
 *
 *  k_sweep_mma   up to 16 tokens of the sweep per pass over the weights, each workgroup taking the
 *                whole row groups that start in its span of the stream: one wave (q4 and mixed
 *                tables) or four that split every row's steps (16-bit and int8)
 */
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "wsr_mma.h"
#include "wsr_mma_launch.h"

namespace wsr {

constexpr int MMA_TILES = MMA_ROWS / 16, MMA_TAIL_TILES = MMA_TAIL_ROWS / 16;   /* 16-row tiles per row group */
constexpr int64_t SWEEP_SPAN_MMA = 64 << 10;  /* least bytes of the weight stream per workgroup        */

/* Waves of a workgroup, which split the steps of its rows.  What bounds a 16-bit or int8 pass is its
   end: a row group is never split over workgroups, and one wave reads a 64-row group of 56 KiB rows,
   3.6 MB, at 5 GB/s.  With the steps over four waves the groups in flight are a quarter as many and
   end four times sooner.  Measured per pass, against one wave with groups of 128 rows (16-bit, and
   int8 from 12 tokens): four 70B layers and head, bf16 1,608 -> 1,401 us at 16 tokens (6.41 TB/s) and
   1,582 -> 1,354 at 4; 72B int8 918 -> 855 and 778 -> 745; a 1.2 GB bf16 model of 2,048-wide layers
   258 -> 210; an 8B bf16 layer as a chain of four launches 289 -> 139.  With two waves 1,468, 918, 231 and
   169; with eight 1,405, 874, 227 and 143; four waves with groups of 128 rows, one wave per SIMD, 1,487,
   843, 230 and 216.  What it costs: int8 at 13 to 16 tokens reads the activations once per 64 rows where
   one wave read them once per 128, and equal matrices whose 128-row groups came out even over the
   CUs were faster so (at 16 tokens twelve of 12288 x 7168 181, now 190; 24 of 4096 x 14336 217, now 241;
   128256 x 8192 168 to 187, now 168 to 180); with other sizes and in models they were slower (32 of 4096
   x 4096 128, now 103; 48 of 4096 x 14336 527, now 477; 8B layers 435, now 366).  q4 rows are short (2 to
   8 KiB) and their passes bound by decoding: one wave, and one for mixed tables, which hold the q4
   loops (it sums 16-bit and int8 rows in the same parts, 0.5 % slower than in one: int8 and f16 8B
   layers 520 -> 522). */
/* Rows of two to four steps for each of the four waves leave little to split and still pay for the joins:
   streams of MMA_WHOLE_FROM bytes and more of such rows alone go one wave per workgroup, which sums the
   same parts.  us, four waves and one: int8 30 of 15536 x 96 39.3 and 25.6, of 15536 x 1024 105 and 82,
   24 of 2048 x 1024 (50 MB) 18.8 and 15.2, of 15536 x 2048 at 3 and 16 tokens 170 and 160, 193 and 192, of
   15536 x 3072 224 and 238; bf16 30 of 15536 x 512 94 and 80, of 15536 x 768 114 and 120; but 25 MB: int8
   24 of 2048 x 512 14.1 and 15.6, 100000 x 256 14.2 and 16.4; bf16 24 of 2048 x 256 11.5 and 12.5. */
constexpr int64_t MMA_WHOLE_FROM = 40 << 20;
static bool mma_splits(int fmt_all, int64_t max_row, int64_t total) {
    if (fmt_all != FMT_F16 && fmt_all != FMT_BF16 && fmt_all != FMT_I8) return false;
    return max_row > (fmt_all == FMT_I8 ? 2048 : 1024) || total < MMA_WHOLE_FROM;
}

/* Workgroups of KS waves, few so that one whose span holds no row group frees its slots
   at once.  Workgroups w < w1 split the stream's bytes [0, tail) into equal spans of whole row groups
   of MMA_ROWS rows; the others split [tail, total) into spans of 16-row groups.  The launcher sets a
   tail only where the main spans would leave the last round of workgroup slots at most a quarter full;
   then the last to finish hold a quarter of a group's work or less.  A matrix's rows from the first
   main-group boundary at or after byte `tail` on belong to the tail, the rows before it to the main
   spans. */
template <int FMT, int KS>
__global__ __launch_bounds__(WAVE * KS) __attribute__((amdgpu_waves_per_eu(FMT == FMT_Q4_WHOLE || (KS == 1 && FMT != 0 && FMT != FMT_Q4) ? 2 : 1)))
void k_sweep_mma(const DevMat* __restrict__ tab, const int64_t* __restrict__ cost, int nmat, int64_t total,
                 int64_t tail, int64_t w1, int32_t token0, int ntok) {
    constexpr int NT = MMA_TILES;
    const int lane = threadIdx.x & (WAVE - 1), wave = KS == 1 ? 0 : wave_in_block();
    const int64_t w = blockIdx.x;
    const bool main = w < w1;
    const int64_t base = main ? 0 : tail, len = main ? tail : total - tail;
    const int64_t nw = main ? w1 : (int64_t)gridDim.x - w1, k = main ? w : w - w1;
    const int64_t q = len / nw, r = len % nw;
    const int64_t lo = base + q * k + (int64_t)((uint64_t)r * (uint64_t)k / nw);
    const int64_t hi = base + q * (k + 1) + (int64_t)((uint64_t)r * (uint64_t)(k + 1) / nw);
    int hint = 0;
    if (lo >= hi) return;
    /* each wave's LDS ring: slots of 64 16-byte chunks (q4 20 KiB, int8 8 KiB, 16-bit 4 KiB;
       the kernel for mixed tables holds the largest); the tail's one-tile groups need no more */
    constexpr int F = mma_base_fmt(FMT);
    constexpr int RING = F == 0 ? mma_ring_slots<FMT_Q4, NT>() : mma_ring_slots<F, NT>();
    __shared__ u32x4 xlds[KS * RING * WAVE], joins[KS == 1 ? 1 : KS * NT * WAVE];
    u32x4* ring = xlds + wave * RING * WAVE;
    if (main)
        stream_range_mma<FMT, NT, KS>(tab, cost, nmat, lo, hi, 0, 16 * NT, token0, ntok, lane, wave, hint, ring,
                                      joins);
    else
        stream_range_mma<FMT, MMA_TAIL_TILES, KS>(tab, cost, nmat, lo, hi, tail, 16 * NT, token0, ntok, lane, wave,
                                                  hint, ring, joins);
}

template <int FMT, int KS>
static hipError_t occupancy_of(int& per_cu) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_sweep_mma<FMT, KS>, WAVE * KS, 0);
}

/* Workgroup slots of the device for the kernel of format fmt_all (its occupancy times the CU count),
   found once per device and format. */
static hipError_t mma_slots(int fmt_all, bool split, int64_t& slots) {
    static std::mutex mu;
    static int64_t cache[64][2][9] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const int f = (fmt_all >= 0 && fmt_all <= 4) || fmt_all == FMT_Q4_WHOLE ? fmt_all : 0;
    std::lock_guard<std::mutex> lock(mu);
    if (dev >= 0 && dev < 64 && cache[dev][split][f] > 0) {
        slots = cache[dev][split][f];
        return hipSuccess;
    }
    int cus = 0, per_cu = 0;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    switch (f) {
        case FMT_F16: e = split ? occupancy_of<FMT_F16, MMA_SPLIT>(per_cu) : occupancy_of<FMT_F16, 1>(per_cu); break;
        case FMT_BF16: e = split ? occupancy_of<FMT_BF16, MMA_SPLIT>(per_cu) : occupancy_of<FMT_BF16, 1>(per_cu); break;
        case FMT_I8: e = split ? occupancy_of<FMT_I8, MMA_SPLIT>(per_cu) : occupancy_of<FMT_I8, 1>(per_cu); break;
        default:   /* q4 too: by its own kernels, which hold two waves per SIMD, launches of little more than a
                      wave per SIMD would get no tail (us: 67529 x 8192 at 5 tokens 91, so 70; 81448 x 4608 at
                      12 54 and 47; 21 of 3808 x 4096 74 and 68; the 8B model alike) */
            e = occupancy_of<0, 1>(per_cu); break;
    }
    if (e != hipSuccess) return e;
    slots = (int64_t)cus * per_cu;
    if (dev >= 0 && dev < 64) cache[dev][split][f] = slots;
    return hipSuccess;
}

hipError_t launch_sweep_mma(const DevMat* tab, const int64_t* cost, int nmat, int64_t total, int64_t max_group,
                            int64_t max_tail_group, int64_t max_row, int fmt_all, int32_t token0, int ntok, hipStream_t s) {
    if (nmat == 0 || total == 0) return hipSuccess;
    if (ntok < 1 || ntok > MMA_TOKENS) return hipErrorInvalidValue;
    /* a workgroup's span holds at least the largest row group: a row group is never split, so a smaller
       span leaves most workgroups without one */
    const int64_t span = std::max(SWEEP_SPAN_MMA, max_group);
    const int64_t span_t = std::max(SWEEP_SPAN_MMA / 4, max_tail_group);
    const int64_t waves = (total + span - 1) / span;
    const bool split = mma_splits(fmt_all, max_row, total);
    int64_t slots = 0;
    const hipError_t e = mma_slots(fmt_all, split, slots);
    if (e != hipSuccess) return e;
    /* whole rounds of spans, and a tail only where the last round would be at most a quarter full
       (measured on int8 passes: 1/8 full 323 -> 265 us per pass with the tail; 1/2 full 356 -> 381) */
    int64_t tail = total, w1 = waves, w2 = 0;
    const int64_t rounds = slots > 0 ? waves / slots : 0, rest = slots > 0 ? waves % slots : 0;
    if (rounds >= 1 && rounds < 8 && rest > 0 && 4 * rest <= slots) {
        tail = rounds * slots * span;
        w1 = rounds * slots;
        w2 = (total - tail + span_t - 1) / span_t;
    }
    if (w1 + w2 > INT32_MAX) return hipErrorInvalidValue;
#define WSR_MMA(F, KS)                                                                                              \
    hipLaunchKernelGGL((k_sweep_mma<F, KS>), dim3((unsigned)(w1 + w2)), dim3(WAVE * KS), 0, s, tab, cost, nmat, total, \
                       tail, w1, token0, ntok)
#define WSR_MMA_SPLIT(F) \
    if (split) WSR_MMA(F, MMA_SPLIT); else WSR_MMA(F, 1)
    switch (fmt_all) {
        case FMT_F16: WSR_MMA_SPLIT(FMT_F16); break;
        case FMT_BF16: WSR_MMA_SPLIT(FMT_BF16); break;
        case FMT_Q4: WSR_MMA(FMT_Q4, 1); break;
        case FMT_I8: WSR_MMA_SPLIT(FMT_I8); break;
        case FMT_Q4_WHOLE: WSR_MMA(FMT_Q4_WHOLE, 1); break;
        default: WSR_MMA(0, 1); break;
    }
#undef WSR_MMA_SPLIT
#undef WSR_MMA
    return hipGetLastError();
}

}  // namespace wsr
