/*
 * wsr_cols.h - row loops of the multi-column GEMV and of the batched decode sweep: up to 4 TQ
 * activation columns per pass over the weights, every column's bits those of the single-column loops
 * of wsr_device.h.
 *
 * What bounded the vector-ALU form: one packed dot product per weight pair and column (8B q4 at 8
 * columns: 820 vector instructions per 4 KiB of codes, 86 % of the issue slots, 2.4 TB/s), and
 * activations taken from the caches by every wave (0.97 TB/s before they were shared through LDS).
 *
 * How the matrix cores give the same bits.  v_dot2 adds two exact products to its accumulator in
 * one rounding; v_mfma_f32_4x4x4 does the same for four products, so with two of its four weights
 * zero it returns what v_dot2 returns (compared on the device: 4 M random triples each at four
 * ratios of products to accumulator, fp16 with subnormal weights and bf16, every result equal).  One
 * instruction does it for 16 chunks x 4 rows x 4 columns: the matrix pipe takes half the time of
 * the dot products it replaces and the vector ALUs are left to decode and scale.
 * Operand layout (checked on the device): lane 4 b + j holds for block b the four activations of
 * column j (A), the four weights of row j (B), and of the result D the columns 0..3 of row j.
 *
 * Order of a sum.  The single-column loops keep 64 partial sums per row, one per chunk modulo 64, and
 * join them by a fixed tree.  Here partial sum 16 p + b lives in lane group b of accumulator p, so
 * the tree's first two levels are additions of registers and the other four are lane exchanges.
 */
#ifndef WSR_COLS_H
#define WSR_COLS_H

#include <type_traits>

#include "wsr_device.h"

namespace wsr {

typedef _Float16 ch4_t __attribute__((ext_vector_type(4)));
typedef short cs4_t __attribute__((ext_vector_type(4)));
typedef float cf4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int COLS_LDS = 80 << 10;                     /* half a CU's LDS: two workgroups per CU (three or
                                                          four for smaller steps: no faster)           */

/* XQ: 16-byte parts of activations per weight chunk and column; NP: weight pairs per chunk; OFF:
   whether a chunk has an offset term. */
template <int FMT> struct ColsFmt { static constexpr int XQ = 1, NP = 4; static constexpr bool OFF = false; };
template <> struct ColsFmt<FMT_Q4> { static constexpr int XQ = 4, NP = 16; static constexpr bool OFF = true; };
template <> struct ColsFmt<FMT_I8> { static constexpr int XQ = 2, NP = 8; static constexpr bool OFF = true; };

/* Groups of four rows per wave (RG) and waves per workgroup of rows_cols; two workgroups share a CU,
   so WAVES / 2 waves share a SIMD's registers.  Every combination takes 32 rows per round.  Two
   groups halve the LDS reads per weight, one group leaves registers for four waves per SIMD:
   measured on 100,000 x 7,168 int8 at 8 columns 157 against 168 us with one group and eight waves;
   on 200,000 x 4,096 q4 at 8 columns 120 against 152 us with two groups and four waves. */
template <int FMT, int TQ> constexpr int cols_rg() { return (FMT == FMT_I8 && TQ == 2) || TQ == 4 ? 1 : 2; }
template <int FMT, int TQ> constexpr int cols_waves() { return (FMT == FMT_I8 && TQ == 2) || TQ == 4 ? 8 : 4; }
constexpr int COLS_ROUND = 32;

/* LDS of one step (64 chunks per row): per quad of columns and quarter p of the step, XQ parts of
   1 KiB (lane 4 b + i: column i of the quad, chunk 16 p + b), then the offset terms, 16 bytes per
   chunk.  SLABS steps fit; a row of at most SLABS steps stays whole. */
template <int FMT, int TQ>
struct ColsLds {
    using F = ColsFmt<FMT>;
    static constexpr int QUAD = 4 * F::XQ * 1024 + (F::OFF ? 1024 : 0);
    static constexpr int STEP = TQ * QUAD;
    static constexpr int SLABS = COLS_LDS / STEP;
    static_assert(SLABS >= 2, "the ring needs two steps");
};

template <int FMT>
__device__ __forceinline__ cf4_t mfma4(u32x2 a, u32x2 b, cf4_t c) {
    if constexpr (FMT == FMT_BF16)
        return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(cs4_t, a), __builtin_bit_cast(cs4_t, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_4x4x4f16(__builtin_bit_cast(ch4_t, a), __builtin_bit_cast(ch4_t, b), c, 0, 0, 0);
}

/* One 16-byte part of a chunk's activations (as in memory) in the order the decoders produce weights:
   q4_prep and i8_prep, part by part. */
template <int FMT>
__device__ __forceinline__ u32x4 col_order(u32x4 x) {
    if constexpr (FMT == FMT_Q4)
        return u32x4{__builtin_amdgcn_perm(x.z, x.x, 0x05040100u), __builtin_amdgcn_perm(x.z, x.x, 0x07060302u),
                     __builtin_amdgcn_perm(x.w, x.y, 0x05040100u), __builtin_amdgcn_perm(x.w, x.y, 0x07060302u)};
    else if constexpr (FMT == FMT_I8)
        return u32x4{__builtin_amdgcn_perm(x.y, x.x, 0x05040100u), __builtin_amdgcn_perm(x.y, x.x, 0x07060302u),
                     __builtin_amdgcn_perm(x.w, x.z, 0x05040100u), __builtin_amdgcn_perm(x.w, x.z, 0x07060302u)};
    else
        return x;
}

/* A chunk's offset term from its ordered parts, summed as q4_prep and i8_prep sum it. */
template <int FMT, int XQ>
__device__ __forceinline__ float col_offset(const u32x4 (&x)[XQ]) {
    if constexpr (FMT == FMT_Q4) {
        float ce = 0.f, co = 0.f;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            ce = dot2<FMT_F16>(F16_OFS_EVEN, x[d].x, ce);
            co = dot2<FMT_F16>(F16_OFS_ODD, x[d].y, co);
            ce = dot2<FMT_F16>(F16_OFS_EVEN, x[d].z, ce);
            co = dot2<FMT_F16>(F16_OFS_ODD, x[d].w, co);
        }
        return __builtin_fmaf(co, 0.0625f, ce);
    } else {
        float off = 0.f;
#pragma unroll
        for (int d = 0; d < XQ; ++d) {
            off = dot2<FMT_F16>(F16_I8_OFS, x[d].x, off);
            off = dot2<FMT_F16>(F16_I8_OFS, x[d].y, off);
            off = dot2<FMT_F16>(F16_I8_OFS, x[d].z, off);
            off = dot2<FMT_F16>(F16_I8_OFS, x[d].w, off);
        }
        return off;
    }
}

/* Weight pair k of a chunk, decoded as q4_block_dot, i8_chunk_dot and dot8 take it. */
template <int FMT>
__device__ __forceinline__ uint32_t col_pair(const u32x4& w, int k) {
    if constexpr (FMT == FMT_Q4) {
        const uint32_t v = k % 4 < 2 ? w[k / 4] : w[k / 4] >> 8;
        return (v ^ Q4_SIGN) & (k % 2 ? Q4_HI : Q4_LO);
    } else if constexpr (FMT == FMT_I8) {
        return k % 2 ? (w[k / 2] >> 8 ^ 0x00800080u) & I8_LOHALF : (w[k / 2] ^ I8_SIGN) & I8_LOHALF;
    } else {
        return w[k];
    }
}

/* Totals over the 16 lane groups of E per-lane entries (lane 4 b + j: row j, partial sums of group
   b), with levels 2 to 5 of the tree of wave_sum_entries: b ^ 15, b ^ 7, b ^ 2, b ^ 1.  Every level's
   sums are the same for all groups the earlier levels joined, so b ^ 8 serves for b ^ 7 and b ^ 4
   for b ^ 1: each level then splits the list, while it has two entries, on a lane bit of its own.
   Afterwards lane l holds entries group_entry(l) and on (E / 16 of them, at least one). */
template <int E>
__device__ __forceinline__ void group_sum(float (&a)[E], int lane) {
    constexpr int ROW_ROR8 = 0x128;
    static_assert(E >= 2 && E <= 32 && (E & (E - 1)) == 0, "entries");
    const int far = (lane ^ 60) * 4;
    auto from_far = [&](float v) { return __int_as_float(__builtin_amdgcn_ds_bpermute(far, __float_as_int(v))); };
#pragma unroll
    for (int j = 0; j < E / 2; ++j) {
        const float send = lane & 4 ? a[j] : a[j + E / 2], keep = lane & 4 ? a[j + E / 2] : a[j];
        a[j] = keep + from_far(send);
    }
    if constexpr (E >= 4) {
#pragma unroll
        for (int j = 0; j < E / 4; ++j) a[j] = swap_add<0>(a[j], a[j + E / 4]);
    } else {
        a[0] = swap_add<0>(a[0], a[0]);
    }
    if constexpr (E >= 8) {
#pragma unroll
        for (int j = 0; j < E / 8; ++j) {
            const float send = lane & 8 ? a[j] : a[j + E / 8], keep = lane & 8 ? a[j + E / 8] : a[j];
            a[j] = keep + dpp_f32<ROW_ROR8>(send);
        }
    } else {
        a[0] += dpp_f32<ROW_ROR8>(a[0]);
    }
    if constexpr (E >= 16) {
#pragma unroll
        for (int j = 0; j < E / 16; ++j) a[j] = swap_add<1>(a[j], a[j + E / 16]);
    } else {
        a[0] = swap_add<1>(a[0], a[0]);
    }
}
template <int E>
__device__ __forceinline__ int group_entry(int lane) {
    int e = lane & 4 ? E / 2 : 0;
    if (E >= 4) e += lane & 32 ? E / 4 : 0;
    if (E >= 8) e += lane & 8 ? E / 8 : 0;
    if (E >= 16) e += lane & 16 ? E / 16 : 0;
    return e;
}
/* Of the lanes holding an entry, the one that stores it. */
template <int E>
__device__ __forceinline__ bool group_owner(int lane) {
    return (lane & ((E >= 16 ? 0 : 16) + (E >= 8 ? 0 : 8) + (E >= 4 ? 0 : 32))) == 0;
}

/* The four columns' sums of a quad where the vector ALUs add them up: four values on their own, not a
   run of registers. */
struct ColsSums {
    float v[4];
    __device__ __forceinline__ float& operator[](int i) { return v[i]; }
};

/* v, as a value of this place: what is computed from it is computed here, not kept in registers from
   before the loops around it (the compiler otherwise holds every address and index of the rarely
   run parts through the main loop, and spills). */
__device__ __forceinline__ int here_only(int v) {
    __asm__ volatile("" : "+v"(v));
    return v;
}

/* Forms v here: left alone, the compiler sinks the additions to the sums to the end of the unit and
   keeps every quarter's products in registers until then. */
__device__ __forceinline__ void here_now(float& v) { __asm__ volatile("" : "+v"(v)); }

/* What the LDS holds: the activations of one (x, stride, chunks, format). */
struct ColsHeld {
    const void* x = nullptr;
    int64_t stride = 0, nc = -1;
    int fmt = 0;
};

/* Rows [r0, r1) of matrix d for tokens token0 .. token0 + ntok - 1 (ntok <= 4 TQ), taken by the
   workgroup together: in each round every wave takes R = 4 RG rows.  The units (round, step of 64 chunks)
   run with the next unit's weights in flight: a quarter's registers take the next unit's quarter
   as soon as they are decoded.  Rows of at most SLABS steps find their activations in LDS for the
   whole call (and for the next matrix, if it reads the same ones); of longer rows LDS holds two
   steps in turn, the next one filled while the current one is multiplied, with a barrier per unit.
   Every wave runs the same units; rows past r1 repeat row r1 - 1 and are not stored, chunks past a
   row's end repeat its last one against zero activations (16-bit weights, which may not be finite,
   as zeros; q4 with a zero scale).  The caller keeps sixteen rows within 2^32 bytes (COLS_MAX_NC). */
template <int FMT, int TQ, int WAVES>
__device__ __forceinline__ void rows_cols(const DevMat& d, int64_t r0, int64_t r1, int32_t token0, int ntok, int lane_,
                                          int wave, char* lds, ColsHeld& held) {
    using F = ColsFmt<FMT>;
    using L = ColsLds<FMT, TQ>;
    constexpr int XQ = F::XQ, NP = F::NP, RG = COLS_ROUND / 4 / WAVES, R = 4 * RG, E = RG * 4 * TQ;
    constexpr bool W16 = FMT != FMT_Q4 && FMT != FMT_I8;
    const int lane = here_only(lane_), b = lane >> 2, j = lane & 3;
    const int nc = (int)d.nc;                                    /* chunks per row */
    const int64_t rb = (int64_t)nc * 16;                         /* code bytes per row */
    const int steps = (nc + WAVE - 1) / WAVE;
    const int rounds = (int)((r1 - r0 + WAVES * R - 1) / (WAVES * R));
    const int64_t n = (int64_t)rounds * steps;
    const char* x0 = static_cast<const char*>(d.x) + (int64_t)token0 * d.x_stride;
    char* y0 = reinterpret_cast<char*>(d.y) + (int64_t)token0 * d.y_stride;

    auto store = [&](int e, float v, int64_t i, int l) {         /* entry e of lane l: row 4 (e / 4 TQ) + l % 4 */
        const int64_t row = i + 4 * (e / (4 * TQ)) + (l & 3);
        const int t = e % (4 * TQ);
        if (row < r1 && t < ntok) {
            if constexpr (FMT == FMT_Q4) v = v * 16777216.0f;    /* undo 2^-24 (exact) */
            if constexpr (FMT == FMT_I8) v = v * 16777216.0f * f16_bits_to_f32(as_global<g_u16*>(d.s)[row]);
            as_global<g_f32*>(y0 + (int64_t)t * d.y_stride)[row] = v;
        }
    };
    if (nc == 0) {                                               /* empty sums */
        for (int64_t i = r0 + wave * R; i < r1; i += WAVES * R)
            for (int e = b; e < E; e += 16) store(e, 0.f, i, lane);
        return;
    }

    /* activations: item o is quarter o % 4 of quad o / 4 (of the steps' quads one after another).  The
       loads take 16-byte pieces in memory order, so that an instruction covers whole lines (with each
       lane at its own column and chunk, every line was asked for by four instructions, and waiting
       for those requests set the time of short calls: q4 4096 x 4096 at 8 columns 16.4 us). */
    constexpr int PIECES = 16 * XQ;                              /* of a column's quarter */
    auto fetch_x = [&](u32x4 (&raw)[XQ], int step, int o, int l) {
#pragma unroll
        for (int k = 0; k < XQ; ++k) {
            const int s = l + 64 * k, t = 4 * (o / 4 % TQ) + s / PIECES, c0 = step * WAVE + 16 * (o % 4);
            const bool in = c0 + s % PIECES / XQ < nc && t < ntok;
            g_u32x4* at = as_global<g_u32x4*>(x0 + (int64_t)t * d.x_stride) + ((int64_t)c0 * XQ + s % PIECES);
            raw[k] = in ? load_reused(at) : zero4();
        }
    };
    auto put_x = [&](const u32x4 (&raw)[XQ], int o, int l) {
        char* quad = lds + o / 4 * L::QUAD;
        u32x4* parts = reinterpret_cast<u32x4*>(quad) + o % 4 * (XQ * 64);
#pragma unroll
        for (int k = 0; k < XQ; ++k) {
            const int s = l + 64 * k;
            parts[s % XQ * 64 + s % PIECES / XQ * 4 + s / PIECES] = col_order<FMT>(raw[k]);
        }
        if constexpr (F::OFF) {                                  /* of this lane's chunk and column, now all there */
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
            u32x4 x[XQ];
#pragma unroll
            for (int k = 0; k < XQ; ++k) x[k] = parts[k * 64 + l];
            reinterpret_cast<float*>(quad + 4 * XQ * 1024 + o % 4 * 256)[l] = col_offset<FMT, XQ>(x);
        }
    };

    /* weights: a lane's part of the next unit */
    struct Raw {
        u32x4 w[RG][4];
        uint32_t s[RG][4];
    } raw;
    int gl = 0, kl = 0;                                          /* the unit being loaded */
    rsrc_t rw = buffer_of(d.w), rs = rw;                         /* the wave's first row of the round */
    uint32_t vr[RG], vs[RG];                                     /* the lane's rows from there */
    int last = 0;                                                /* last chunk of a row */
    auto aim = [&]() {                                           /* at a round's first step */
        const bool in = gl < rounds;
        const int64_t i = r0 + ((int64_t)gl * WAVES + wave) * R;
        const int64_t i0 = in && i < r1 ? i : r1 - 1;            /* past the last unit: all lanes one chunk */
        last = in ? nc - 1 : 0;
        rw = buffer_of(uniform_ptr(static_cast<const char*>(d.w) + i0 * rb));
        if constexpr (FMT == FMT_Q4) rs = buffer_of(uniform_ptr(static_cast<const char*>(d.s) + i0 * (2 * (int64_t)nc)));
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            const uint32_t row = (uint32_t)(in ? std::min<int64_t>(4 * g + j, r1 - 1 - i0) : 0);
            vr[g] = row * (uint32_t)rb;
            vs[g] = vr[g] / 8;
        }
    };
    auto load = [&](int g, int p) {
        const uint32_t c = (uint32_t)std::min(kl * WAVE + 16 * p + b, last);
        raw.w[g][p] = buf_once(rw, vr[g] + 16 * c, 0);
        if constexpr (FMT == FMT_Q4) raw.s[g][p] = buf_u16(rs, vs[g] + 2 * c, 0);
    };
    auto advance = [&]() {                                       /* after a unit's four quarters */
        if (++kl == steps) {
            kl = 0;
            ++gl;
            aim();
        }
    };
    aim();
#pragma unroll
    for (int p = 0; p < 4; ++p)                                  /* weights first: they come from farthest */
#pragma unroll
        for (int g = 0; g < RG; ++g) load(g, p);
    advance();

    const bool whole = steps <= L::SLABS;
    const bool here = whole && held.x == x0 && held.stride == d.x_stride && held.nc == nc && held.fmt == FMT;
    if (!here) {
        constexpr int AT = 8 / XQ;                               /* fetches in flight per wave */
        const int l = here_only(lane), items = (whole ? steps : 1) * TQ * 4;
        lds_barrier();                                           /* the previous matrix's reads are done */
        for (int o = wave; o < items; o += AT * WAVES) {
            u32x4 a[AT][XQ];
#pragma unroll
            for (int k = 0; k < AT; ++k)
                if (o + k * WAVES < items) fetch_x(a[k], (o + k * WAVES) / (4 * TQ), o + k * WAVES, l);
#pragma unroll
            for (int k = 0; k < AT; ++k)
                if (o + k * WAVES < items) put_x(a[k], o + k * WAVES, l);
        }
        held = whole ? ColsHeld{x0, d.x_stride, nc, FMT} : ColsHeld{};
        lds_barrier();
    }

    typename std::conditional<W16, cf4_t, ColsSums>::type acc[RG][TQ][4];
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int q = 0; q < TQ; ++q)
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[g][q][p][i] = 0.f;
    /* Weight operands: pair k alone in half k % 2 of its two registers, the other half zero.  The zeros
       are written once and stay; decoding writes the pairs only.  The empty asm at each use keeps the
       compiler from seeing that a half never changes: it would then hold the zeros apart and copy
       them beside every new pair. */
    constexpr int NB = NP < 8 ? NP : 8;
    u32x2 B[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) B[k] = u32x2{0u, 0u};

    int gc = 0, kc = 0;                                          /* the unit being multiplied */
    auto unit = [&](int slab, auto between) {                    /* between(p): run before quarter p */
        const u32x4* xl = reinterpret_cast<const u32x4*>(lds + slab * L::STEP) + lane;
        const cf4_t* ol = reinterpret_cast<const cf4_t*>(lds + slab * L::STEP + 4 * XQ * 1024) + b;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            between(p);
            const bool past = kc * WAVE + 16 * p + b >= nc;
            u32x4 x[TQ][XQ];                                     /* serve all the wave's rows */
#pragma unroll
            for (int q = 0; q < TQ; ++q) {
#pragma unroll
                for (int k = 0; k < XQ; ++k) x[q][k] = xl[q * (L::QUAD / 16) + (p * XQ + k) * 64];
            }
            /* pairs 2 m and 2 m + 1 of quad q's activations */
            auto xa = [&](int q, int m) {
                return m % 2 ? u32x2{x[q][m / 2].z, x[q][m / 2].w} : u32x2{x[q][m / 2].x, x[q][m / 2].y};
            };
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                if constexpr (W16)
                    if (past) raw.w[g][p] = zero4();
                const u32x4 w = raw.w[g][p];
                float sc = 0.f;
                if constexpr (FMT == FMT_Q4) sc = past ? 0.f : f16_bits_to_f32((uint16_t)raw.s[g][p]);
                load(g, p);
                auto pair = [&](int k) -> u32x2 {
                    B[k % NB][k % 2] = col_pair<FMT>(w, k);
                    __asm__("" : "+v"(B[k % NB]));
                    return B[k % NB];
                };
                if constexpr (FMT == FMT_Q4) {
                    cf4_t se[TQ], so[TQ];
#pragma unroll
                    for (int q = 0; q < TQ; ++q) se[q] = so[q] = cf4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int m = 0; m < 8; ++m) {
                        const u32x2 we = pair(2 * m), wo = pair(2 * m + 1);
#pragma unroll
                        for (int q = 0; q < TQ; ++q) {
                            se[q] = mfma4<FMT_F16>(xa(q, m), we, se[q]);
                            so[q] = mfma4<FMT_F16>(xa(q, m), wo, so[q]);
                        }
                    }
#pragma unroll
                    for (int q = 0; q < TQ; ++q) {
                        const cf4_t off = ol[q * (L::QUAD / 16) + p * 16];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            acc[g][q][p][i] = __builtin_fmaf(sc, __builtin_fmaf(so[q][i], 0.0625f, se[q][i]) - off[i],
                                                             acc[g][q][p][i]);
                            here_now(acc[g][q][p][i]);
                        }
                    }
                } else if constexpr (FMT == FMT_I8) {
                    cf4_t t[TQ];
#pragma unroll
                    for (int q = 0; q < TQ; ++q) t[q] = cf4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const u32x2 wk = pair(k);
#pragma unroll
                        for (int q = 0; q < TQ; ++q) t[q] = mfma4<FMT_F16>(xa(q, k / 2), wk, t[q]);
                    }
#pragma unroll
                    for (int q = 0; q < TQ; ++q) {
                        const cf4_t off = ol[q * (L::QUAD / 16) + p * 16];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            acc[g][q][p][i] += t[q][i] - off[i];
                            here_now(acc[g][q][p][i]);
                        }
                    }
                } else {                                         /* a non-finite activation meets no weight but its own */
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const u32x2 wk = pair(k);
#pragma unroll
                        for (int q = 0; q < TQ; ++q) {
                            const u32x2 a = k % 2 ? u32x2{0u, x[q][0][k]} : u32x2{x[q][0][k], 0u};
                            acc[g][q][p] = mfma4<FMT>(a, wk, acc[g][q][p]);
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        advance();
        if (kc + 1 == steps) {                                   /* a round's end: join, store, reset */
            const int64_t i0 = r0 + ((int64_t)gc * WAVES + wave) * R;
            const int l = here_only(lane);
            float s[E];
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int q = 0; q < TQ; ++q) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        s[(g * TQ + q) * 4 + i] = (acc[g][q][0][i] + acc[g][q][2][i]) + (acc[g][q][1][i] + acc[g][q][3][i]);
#pragma unroll
                    for (int p = 0; p < 4; ++p)
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[g][q][p][i] = 0.f;
                }
            group_sum<E>(s, l);
            const int e = group_entry<E>(l);
            if (group_owner<E>(l))
#pragma unroll
                for (int k = 0; k < (E + 15) / 16; ++k) store(e + k, s[k], i0, l);
            kc = 0;
            ++gc;
        } else {
            ++kc;
        }
    };

    /* of a ring, the next step's activations, an item or two per wave, fetched ahead of the weights that
       are loaded beside them */
    constexpr int PW = (4 * TQ + WAVES - 1) / WAVES;
    static_assert(PW <= 2, "two phases");
    u32x4 xr[XQ];
    int kx = 1, to = 1;                                          /* a ring's next step to fill, and where */
    auto fill = [&](int k) {                                     /* phase k's item is in xr: into its place */
        const int o = wave + k * WAVES;
        if (o < 4 * TQ) put_x(xr, to * (4 * TQ) + o, here_only(lane));
    };
#pragma unroll 1
    for (int64_t u = 0; u < n; ++u) {
        unit(whole ? kc : to ^ 1, [&](int p) {
            if (whole || !(p == 0 || (p == 2 && PW > 1))) return;
            if (p == 2) fill(0);
            const int o = wave + p / 2 * WAVES;
            if (o < 4 * TQ) fetch_x(xr, kx, o, here_only(lane));
        });
        if (!whole) {
            fill(PW - 1);
            if (++kx == steps) kx = 0;
            to ^= 1;
            lds_barrier();
        }
    }
}

/* ---- rows split over a workgroup's waves --------------------------------------------------------

   Rows [r0, r1) of matrix d for tokens token0 .. token0 + ntok - 1 (ntok <= 4 TQ): in each round the
   four waves take the same 4 RG rows, wave p the chunks of quarter p of every step (its 16 of the 64
   partial sums per row), and join their sums through LDS at the round's end.  A wave needs only its
   quarter's activations, which it loads a step ahead like its weights and turns through an LDS area
   of its own: no barrier before the first product and four waves per round of rows, which suits
   short streams, where the start and the balance of the launch set the time. */
template <int FMT, int TQ> constexpr int split_x_bytes() { return TQ * ColsFmt<FMT>::XQ * 1024; }     /* per wave */
template <int FMT, int TQ, int RG>
constexpr int split_lds_bytes() { return 4 * split_x_bytes<FMT, TQ>() + 4 * (RG * TQ * 4) * 256; }   /* and the joins */

template <int FMT, int TQ, int RG>
__device__ __forceinline__ void rows_split(const DevMat& d, int64_t r0, int64_t r1, int32_t token0, int ntok, int lane_,
                                           int wave, char* lds) {
    using F = ColsFmt<FMT>;
    constexpr int XQ = F::XQ, NP = F::NP, E = RG * 4 * TQ, EW = E / 4;   /* entries; of each wave */
    constexpr bool W16 = FMT != FMT_Q4 && FMT != FMT_I8;
    const int lane = here_only(lane_), b = lane >> 2, j = lane & 3;
    const int nc = (int)d.nc;
    const int64_t rb = (int64_t)nc * 16;
    const int steps = (nc + WAVE - 1) / WAVE;
    const int rounds = (int)((r1 - r0 + 4 * RG - 1) / (4 * RG));
    const int64_t n = (int64_t)rounds * steps;
    const char* x0 = static_cast<const char*>(d.x) + (int64_t)token0 * d.x_stride;
    char* y0 = reinterpret_cast<char*>(d.y) + (int64_t)token0 * d.y_stride;

    auto store = [&](int e, float v, int64_t i, int l) {         /* entry e: row 4 (e / 4 TQ) + l % 4, token e % 4 TQ */
        const int64_t row = i + 4 * (e / (4 * TQ)) + (l & 3);
        const int t = e % (4 * TQ);
        if (row < r1 && t < ntok) {
            if constexpr (FMT == FMT_Q4) v = v * 16777216.0f;    /* undo 2^-24 (exact) */
            if constexpr (FMT == FMT_I8) v = v * 16777216.0f * f16_bits_to_f32(as_global<g_u16*>(d.s)[row]);
            as_global<g_f32*>(y0 + (int64_t)t * d.y_stride)[row] = v;
        }
    };
    if (nc == 0) {                                               /* empty sums */
        for (int64_t i = r0 + wave * 4 * RG; i < r1; i += 16 * RG)
            for (int e = b; e < E; e += 16) store(e, 0.f, i, lane);
        return;
    }

    struct Set {
        u32x4 w[RG];
        uint32_t s[RG];
        u32x4 x[TQ][XQ];
    } next;
    int gl = 0, kl = 0;                                          /* the unit (round, step) being loaded */
    rsrc_t rw = buffer_of(d.w), rs = rw;
    uint32_t vr[RG];
    int last = 0;
    auto aim = [&]() {                                           /* as in rows_cols; all waves the same rows */
        const bool in = gl < rounds;
        const int64_t i = r0 + (int64_t)gl * 4 * RG, i0 = in ? i : r1 - 1;
        last = in ? nc - 1 : 0;
        rw = buffer_of(uniform_ptr(static_cast<const char*>(d.w) + i0 * rb));
        if constexpr (FMT == FMT_Q4) rs = buffer_of(uniform_ptr(static_cast<const char*>(d.s) + i0 * (2 * (int64_t)nc)));
#pragma unroll
        for (int g = 0; g < RG; ++g)
            vr[g] = (uint32_t)(in ? std::min<int64_t>(4 * g + j, r1 - 1 - i0) : 0) * (uint32_t)rb;
    };
    /* 16-byte piece s of the quad's quarter: column s / PIECES (past ntok: the last one again), piece
       s % PIECES of the column's 16 chunks (past the row's end: its last ones again, zeroed below) */
    constexpr int PIECES = 16 * XQ;
    const char* xp[TQ][XQ];
#pragma unroll
    for (int q = 0; q < TQ; ++q)
#pragma unroll
        for (int k = 0; k < XQ; ++k)
            xp[q][k] = x0 + (int64_t)std::min(4 * q + (lane + 64 * k) / PIECES, ntok - 1) * d.x_stride;
    auto load = [&](Set& u) {
        const int c0 = kl * WAVE + 16 * wave;
#pragma unroll
        for (int q = 0; q < TQ; ++q)
#pragma unroll
            for (int k = 0; k < XQ; ++k) {
                const int s = (lane + 64 * k) % PIECES;
                const uint32_t at = (uint32_t)(std::min(c0 + s / XQ, last) * XQ + s % XQ);
                u.x[q][k] = load_reused(as_global<g_u32x4*>(xp[q][k] + (uint64_t)(at * 16)));
            }
        const uint32_t c = (uint32_t)std::min(c0 + b, last);
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            u.w[g] = buf_once(rw, vr[g] + 16 * c, 0);
            if constexpr (FMT == FMT_Q4) u.s[g] = buf_u16(rs, vr[g] / 8 + 2 * c, 0);
        }
        if (++kl == steps) {
            kl = 0;
            ++gl;
            aim();
        }
    };
    aim();
    load(next);

    typename std::conditional<W16, cf4_t, ColsSums>::type acc[RG][TQ];
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int q = 0; q < TQ; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[g][q][i] = 0.f;
    constexpr int NB = NP < 8 ? NP : 8;
    u32x2 B[NB];                                                 /* as in rows_cols */
#pragma unroll
    for (int k = 0; k < NB; ++k) B[k] = u32x2{0u, 0u};
    u32x4* mine = reinterpret_cast<u32x4*>(lds + wave * split_x_bytes<FMT, TQ>());
    float* joins = reinterpret_cast<float*>(lds + 4 * split_x_bytes<FMT, TQ>());

    int gc = 0, kc = 0;                                          /* the unit being multiplied */
#pragma unroll 1
    for (int64_t u = 0; u < n; ++u) {
        const bool past = kc * WAVE + 16 * wave + b >= nc;
        u32x4 w[RG];
        uint32_t ws[RG];
#pragma unroll
        for (int q = 0; q < TQ; ++q)
#pragma unroll
            for (int k = 0; k < XQ; ++k) {
                const int s = lane + 64 * k;
                mine[(q * XQ + s % XQ) * 64 + s % PIECES / XQ * 4 + s / PIECES] = col_order<FMT>(next.x[q][k]);
            }
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            w[g] = next.w[g];
            if constexpr (FMT == FMT_Q4) ws[g] = next.s[g];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        load(next);                                              /* past the last unit: one line */
        __builtin_amdgcn_sched_barrier(0);
        u32x4 x[TQ][XQ];
        float off[TQ][4];
#pragma unroll
        for (int q = 0; q < TQ; ++q) {
#pragma unroll
            for (int k = 0; k < XQ; ++k) {
                x[q][k] = mine[(q * XQ + k) * 64 + lane];
                if (past) x[q][k] = zero4();
            }
            if constexpr (F::OFF) {
                /* lane (b, i) forms column i's offset of chunk b; lane (b, j) needs all four */
                const int o = __float_as_int(col_offset<FMT, XQ>(x[q]));
                off[q][0] = __int_as_float(__builtin_amdgcn_update_dpp(0, o, 0x00, 0xF, 0xF, false));
                off[q][1] = __int_as_float(__builtin_amdgcn_update_dpp(0, o, 0x55, 0xF, 0xF, false));
                off[q][2] = __int_as_float(__builtin_amdgcn_update_dpp(0, o, 0xAA, 0xF, 0xF, false));
                off[q][3] = __int_as_float(__builtin_amdgcn_update_dpp(0, o, 0xFF, 0xF, 0xF, false));
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");   /* read before the next unit writes */
        auto xa = [&](int q, int m) {
            return m % 2 ? u32x2{x[q][m / 2].z, x[q][m / 2].w} : u32x2{x[q][m / 2].x, x[q][m / 2].y};
        };
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            if constexpr (W16)
                if (past) w[g] = zero4();
            auto pair = [&](int k) -> u32x2 {
                B[k % NB][k % 2] = col_pair<FMT>(w[g], k);
                __asm__("" : "+v"(B[k % NB]));
                return B[k % NB];
            };
            if constexpr (FMT == FMT_Q4) {
                const float sc = past ? 0.f : f16_bits_to_f32((uint16_t)ws[g]);
                cf4_t se[TQ], so[TQ];
#pragma unroll
                for (int q = 0; q < TQ; ++q) se[q] = so[q] = cf4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    const u32x2 we = pair(2 * m), wo = pair(2 * m + 1);
#pragma unroll
                    for (int q = 0; q < TQ; ++q) {
                        se[q] = mfma4<FMT_F16>(xa(q, m), we, se[q]);
                        so[q] = mfma4<FMT_F16>(xa(q, m), wo, so[q]);
                    }
                }
#pragma unroll
                for (int q = 0; q < TQ; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        acc[g][q][i] = __builtin_fmaf(sc, __builtin_fmaf(so[q][i], 0.0625f, se[q][i]) - off[q][i], acc[g][q][i]);
                        here_now(acc[g][q][i]);
                    }
            } else if constexpr (FMT == FMT_I8) {
                cf4_t t[TQ];
#pragma unroll
                for (int q = 0; q < TQ; ++q) t[q] = cf4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const u32x2 wk = pair(k);
#pragma unroll
                    for (int q = 0; q < TQ; ++q) t[q] = mfma4<FMT_F16>(xa(q, k / 2), wk, t[q]);
                }
#pragma unroll
                for (int q = 0; q < TQ; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        acc[g][q][i] += t[q][i] - off[q][i];
                        here_now(acc[g][q][i]);
                    }
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const u32x2 wk = pair(k);
#pragma unroll
                    for (int q = 0; q < TQ; ++q) {
                        const u32x2 a = k % 2 ? u32x2{0u, x[q][0][k]} : u32x2{x[q][0][k], 0u};
                        acc[g][q] = mfma4<FMT>(a, wk, acc[g][q]);
                    }
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (kc + 1 == steps) {                                   /* a round's end: join, store, reset */
            const int l = here_only(lane);
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int q = 0; q < TQ; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        joins[(wave * E + (g * TQ + q) * 4 + i) * 64 + l] = acc[g][q][i];   /* [wave][entry][lane] */
                        acc[g][q][i] = 0.f;
                    }
            lds_barrier();
            float s[EW];
#pragma unroll
            for (int k = 0; k < EW; ++k) {
                const float* a = joins + (wave * EW + k) * 64 + l;
                s[k] = (a[0] + a[2 * E * 64]) + (a[E * 64] + a[3 * E * 64]);
            }
            lds_barrier();                                       /* read, before the next round's are written */
            group_sum<EW>(s, l);
            const int e = wave * EW + group_entry<EW>(l);
            const int64_t i0 = r0 + (int64_t)gc * 4 * RG;
            if (group_owner<EW>(l))
#pragma unroll
                for (int k = 0; k < (EW + 15) / 16; ++k) store(e + k, s[k], i0, l);
            kc = 0;
            ++gc;
        } else {
            ++kc;
        }
    }
}

/* Groups of four rows per round of rows_split: four where an activation chunk is larger than its
   weight chunk, two for 16-bit weights (8192 x 8192 bf16 at 4 columns: 25.0 us with two, 33.0 with
   four). */
template <int FMT> constexpr int split_rg() { return FMT == FMT_Q4 || FMT == FMT_I8 ? 4 : 2; }
constexpr int SPLIT_RG_FEW = 2;         /* where those rounds leave half the chip without a workgroup */

/* The workgroup's byte range [lo, hi) of a stream of one format; both ends round up to the next whole
   round of rows of their matrix, the same way for the ranges on both sides. */
template <int FMT, int TQ, int RG>
__device__ __forceinline__ void stream_range_split(const DevMat* __restrict__ tab, const int64_t* __restrict__ cost,
                                                   int nmat, int64_t lo, int64_t hi, int32_t token, int ntok, int lane,
                                                   int wave, char* lds) {
    for (int m = first_matrix(cost, nmat, lo, 0); m < nmat; ++m) {
        const DevMat d = tab[m];
        if (d.cost0 >= hi) break;
        constexpr int64_t g = 4 * RG;
        const int64_t r0 = lo > d.cost0 ? ceil_div(lo - d.cost0, d.row_bytes * g) * g : 0;
        const int64_t e1 = ceil_div(hi - d.cost0, d.row_bytes * g) * g;
        const int64_t r1 = d.M < e1 ? d.M : e1;
        if (r0 >= r1) continue;
        rows_split<FMT, TQ, RG>(d, r0, r1, token, ntok, lane, wave, lds);
    }
}

/* The same for rows_cols, over a stream of one or several formats. */
template <int FMT, int TQ, int WAVES>
__device__ __forceinline__ void stream_range_cols(const DevMat* __restrict__ tab, const int64_t* __restrict__ cost,
                                                  int nmat, int64_t lo, int64_t hi, int32_t token, int ntok, int lane,
                                                  int wave, char* lds) {
    ColsHeld held;
    for (int m = first_matrix(cost, nmat, lo, 0); m < nmat; ++m) {
        const DevMat d = tab[m];
        if (d.cost0 >= hi) break;
        const int fmt = FMT ? FMT : d.fmt;
        constexpr int64_t g = COLS_ROUND;
        const int64_t r0 = lo > d.cost0 ? ceil_div(lo - d.cost0, d.row_bytes * g) * g : 0;
        const int64_t e1 = ceil_div(hi - d.cost0, d.row_bytes * g) * g;
        const int64_t r1 = d.M < e1 ? d.M : e1;
        if (r0 >= r1) continue;
        if ((FMT == 0 || FMT == FMT_F16) && fmt == FMT_F16)
            rows_cols<FMT_F16, TQ, WAVES>(d, r0, r1, token, ntok, lane, wave, lds, held);
        else if ((FMT == 0 || FMT == FMT_BF16) && fmt == FMT_BF16)
            rows_cols<FMT_BF16, TQ, WAVES>(d, r0, r1, token, ntok, lane, wave, lds, held);
        else if constexpr (TQ <= 2) {
            if ((FMT == 0 || FMT == FMT_Q4) && fmt == FMT_Q4)
                rows_cols<FMT_Q4, TQ, WAVES>(d, r0, r1, token, ntok, lane, wave, lds, held);
            else if ((FMT == 0 || FMT == FMT_I8) && fmt == FMT_I8)
                rows_cols<FMT_I8, TQ, WAVES>(d, r0, r1, token, ntok, lane, wave, lds, held);
        }
    }
}

}  // namespace wsr

#endif
