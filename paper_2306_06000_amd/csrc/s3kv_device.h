// Device-side helpers shared by the attention kernels of libs3kv (gfx950): kernel arguments, bounds
// checks of the device arrays, lane reductions, 16-bit dot / accumulate steps, output stores, the
// LDS batch view (work list) and the chunk-partial merge.  Included by the .hip files only.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "s3kv_internal.h"

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

#define S3_MAX_BATCH 4095

struct AttnArgs {
    char *kplane;
    char *vplane;
    const char *q;
    const int64_t *slot_off;
    const int32_t *cur_len;  // rows to attend minus len_add
    void *out;
    // Partials: [slot][H][D] weighted sums and [slot][H] (running max in log2 units, sum).  Slot of a chunk: its
    // position in the work list (one per chunk); vector-ALU kernel for shared heads: b * max_chunks + chunk.
    float *part_acc;
    float2 *part_ml;
    int64_t n_tokens;  // arena capacity N
    int32_t n, H, chunk, max_chunks, out_dtype, max_len;  // H: heads of a K/V row
    int32_t Hq;            // query heads (= H unless grouped-query / multi-query attention)
    int32_t ncls;          // length classes of the work order (1..8)
    int32_t class_rows;    // > 0: one class if the contexts average fewer rows than this
    int32_t few_chunks;    // > 0: few contexts; cut them into about this many chunks (chunk: the longest allowed)
    int32_t len_add;    // 0: cur_len is the context length; 1 (fused step): cur_len is the append position
    float scale_log2e;  // scale * log2(e): scores are kept in log2 units so that exp is v_exp_f32
    // fused step only
    const char *k_new;
    const char *v_new;
    int32_t *len_out;        // may be null
    unsigned int *arrivals;  // [n][n_hgb] chunk-arrival counters, zero between launches
    int32_t merge_sync;      // how chunks that meet inside one launch are ordered: see chunk_arrived()
    unsigned int *queue;     // [2] kernels with a dynamic work list: positions claimed, workgroups gone; zero between launches
    int32_t stream_k;        // matrix-core kernel for shared heads: K rows with the streaming hint (1), plain (0), by launch size (< 0)
    // matrix-core kernel for shared heads: how the rows are divided among the waves
    int32_t group, nqb, columns;          // query heads per cached head, blocks of 16 of them, columns = H * nqb
    int32_t column_shift;                 // log2 of the columns, -1: no power of two
    int32_t wave_shares, team_shares;     // shares per column if every wave takes one, if teams of four waves do
    int32_t max_shares;  // partial slots allow this many publishing units per column (0: none, shares begin and end with contexts)
    float merge_cost;    // time of merging one more piece of a context, in tiles streamed by one wave
    int32_t share_rows;  // > 0: at most this many rows a share (set by the caller)
    int32_t team_lds;    // the launch carries LDS for the pieces of teams of four waves
    // multi-head kernels: > 0: the chunks of a context's heads that run at once (low 16 bits); the contexts may be cut into as
    // many, whatever their rows, or (16 bits and up: 1) as unit_rule() says.  attn_few_kernel: chunks of a context's heads,
    // few_chunks one a compute unit, unit_chunks two; columns head groups.
    int32_t unit_chunks;
};

__device__ __forceinline__ int checked_len(const AttnArgs &a, int64_t off, int32_t raw) {
    const int64_t len = (int64_t)raw + a.len_add;
    const bool ok = off >= 0 && raw >= 0 && len <= a.max_len && off + len <= a.n_tokens;
    return ok ? (int)len : 0;
}
__device__ __forceinline__ int checked_len(const AttnArgs &a, int b) { return checked_len(a, a.slot_off[b], a.cur_len[b]); }

// Entries first .. first+E-1 of the device arrays (length 0 past the end of the batch).  No branch around a load:
// all of them leave together and cost one memory round trip.
template <int E>
__device__ __forceinline__ void load_entries(const AttnArgs &a, int first, int64_t (&off)[E], int (&len)[E]) {
    int32_t raw[E];
#pragma unroll
    for (int e = 0; e < E; e++) {
        const int b = min(first + e, a.n - 1);
        off[e] = a.slot_off[b];
        raw[e] = a.cur_len[b];
    }
#pragma unroll
    for (int e = 0; e < E; e++) len[e] = first + e < a.n ? checked_len(a, off[e], raw[e]) : 0;
}

template <int CTRL>
__device__ __forceinline__ float dpp_sum_step(float v) {
    const int bits = __builtin_bit_cast(int, v);
    const int moved = __builtin_amdgcn_update_dpp(0, bits, CTRL, 0xF, 0xF, true);
    return v + __builtin_bit_cast(float, moved);
}

// Sum, maximum over a lane and those that differ from it in the sixteen (rows of 16 lanes; WIDE: the half) they are in, without the
// LDS unit: the swap brings the even rows (the lower half) of a value into one register, the odd ones (the upper) into another.
// Shared heads, through the LDS unit and by swaps, us a layer: 8q/1kv x 64, 250 contexts of 32..1000 rows 13.1, 12.6, 12q/2kv x 128,
// 100 of 32..1000 17.4, 17.0, 32q/8kv x 128, 1000 of 2..40 29.6, 28.7; 239 launches 0 to 5 % faster, 1.5 % in the mean.  Multi-head rows level.
template <bool WIDE, typename F>
__device__ __forceinline__ float swap_rows(float v, F f) {
    const unsigned u = __builtin_bit_cast(unsigned, v);
    const auto both = WIDE ? __builtin_amdgcn_permlane32_swap(u, u, false, false) : __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned a = both[0], b = both[1];
    return f(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}
__device__ __forceinline__ float max_over_rows(float v) {
    const auto f = [](float a, float b) { return fmaxf(a, b); };
    return swap_rows<true>(swap_rows<false>(v, f), f);
}
__device__ __forceinline__ float sum_over_rows(float v) {
    const auto f = [](float a, float b) { return a + b; };
    return swap_rows<true>(swap_rows<false>(v, f), f);
}

// Sum over groups of LANES adjacent lanes (4, 8, 16 or 32); every lane of a group gets the sum.
template <int LANES>
__device__ __forceinline__ float group_sum(float v) {
    v = dpp_sum_step<0xB1>(v);   // quad_perm [1,0,3,2]: lane ^ 1
    v = dpp_sum_step<0x4E>(v);   // quad_perm [2,3,0,1]: lane ^ 2
    if (LANES >= 8) v = dpp_sum_step<0x141>(v);  // row_half_mirror: the other quad of each 8
    if (LANES >= 16) v = dpp_sum_step<0x140>(v);  // row_mirror: the other 8 of each 16
    if (LANES >= 32) v = swap_rows<false>(v, [](float a, float b) { return a + b; });  // lane ^ 16
    return v;
}

// The value that lane `from` (uniform) holds.
__device__ __forceinline__ float lane_value(float v, int from) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), from));
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Exponent reference of a set of scores whose maximum is m: m, or 0 if every score is -inf, so that exp2(score - reference)
// is 0 for them and not NaN (such rows, a chunk of them or a piece weigh nothing beside rows with finite scores).
__device__ __forceinline__ float exp_reference(float m) { return m == -INFINITY ? 0.f : m; }

// Note: __builtin_bit_cast applied directly to a vector-element expression (v[i]) reads element 0
// with this compiler, so elements are always copied into a scalar first.
template <int DT>
__device__ __forceinline__ float dot8(const u32x4 a, const u32x4 b) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const unsigned ai = a[i], bi = b[i];
        if (DT == S3_F16)
            s = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, ai), __builtin_bit_cast(f16x2, bi), s, false);
        else
            s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, ai), __builtin_bit_cast(bf16x2, bi), s, false);
    }
    return s;
}

template <int DT>
__device__ __forceinline__ void axpy8(float (&acc)[8], const float p, const u32x4 v) {
#pragma unroll
    for (int i = 0; i < 4; i++) {
        float lo, hi;
        const unsigned vi = v[i];
        if (DT == S3_F16) {
            const f16x2 h = __builtin_bit_cast(f16x2, vi);
            lo = (float)h[0];
            hi = (float)h[1];
        } else {
            const unsigned lo_bits = vi << 16, hi_bits = vi & 0xFFFF0000u;
            lo = __builtin_bit_cast(float, lo_bits);
            hi = __builtin_bit_cast(float, hi_bits);
        }
        acc[2 * i] = fmaf(p, lo, acc[2 * i]);
        acc[2 * i + 1] = fmaf(p, hi, acc[2 * i + 1]);
    }
}

__device__ __forceinline__ unsigned f32_to_bf16_rne(float f) {
    unsigned u = __builtin_bit_cast(unsigned, f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;  // NaN stays NaN
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// Store 8 consecutive output elements starting at element index e of `out`.
__device__ __forceinline__ void store_out8(void *out, int out_dtype, int64_t e, const float (&v)[8]) {
    if (out_dtype == S3_F32) {
        f32x4 *p = (f32x4 *)((float *)out + e);
        p[0] = (f32x4){v[0], v[1], v[2], v[3]};
        p[1] = (f32x4){v[4], v[5], v[6], v[7]};
    } else {
        u32x4 w;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            if (out_dtype == S3_F16) {
                const f16x2 h = {(_Float16)v[2 * i], (_Float16)v[2 * i + 1]};
                const unsigned packed = __builtin_bit_cast(unsigned, h);
                w[i] = packed;
            } else {
                w[i] = f32_to_bf16_rne(v[2 * i]) | (f32_to_bf16_rne(v[2 * i + 1]) << 16);
            }
        }
        *(u32x4 *)((uint16_t *)out + e) = w;
    }
}

// One output element.
__device__ __forceinline__ void store_out1(void *out, int out_dtype, int64_t e, const float v) {
    if (out_dtype == S3_F32) ((float *)out)[e] = v;
    else if (out_dtype == S3_F16) ((_Float16 *)out)[e] = (_Float16)v;
    else ((uint16_t *)out)[e] = (uint16_t)f32_to_bf16_rne(v);
}

// Two fp32 values -> their e4m3 codes in one half of a 32-bit word (v_cvt_pk_fp8_f32 rounds to the nearest
// code, ties to even, subnormal codes included).  Magnitudes are clamped to 448 first, so nothing depends on
// the instruction's overflow mode, and NaN is forced to 0x7f afterwards (the clamp turns it into a number).
template <bool HI>
__device__ __forceinline__ unsigned quantize2_e4m3(const float x0, const float x1, const unsigned old) {
    const float c0 = fminf(fmaxf(x0, -448.f), 448.f), c1 = fminf(fmaxf(x1, -448.f), 448.f);
    unsigned w = (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(c0, c1, (int)old, HI);
    constexpr unsigned S = HI ? 16u : 0u;
    if (x0 != x0) w = (w & ~(0xFFu << S)) | (0x7Fu << S);
    if (x1 != x1) w = (w & ~(0xFF00u << S)) | (0x7F00u << S);
    return w;
}

template <int ACT>
__device__ __forceinline__ float widen16(const unsigned short h) {
    if (ACT == S3_F16) return (float)__builtin_bit_cast(_Float16, h);
    const unsigned w = (unsigned)h << 16;
    return __builtin_bit_cast(float, w);
}

// 16 consecutive 16-bit elements (two 128-bit words) -> their 16 codes in element order.
template <int ACT>
__device__ __forceinline__ u32x4 quantize16(const u32x4 lo, const u32x4 hi) {
    u32x4 out;
#pragma unroll
    for (int w = 0; w < 4; w++) {
        const unsigned a = w < 2 ? lo[2 * w] : hi[2 * w - 4], c = w < 2 ? lo[2 * w + 1] : hi[2 * w - 3];
        const unsigned lo2 = quantize2_e4m3<false>(widen16<ACT>((unsigned short)(a & 0xFFFFu)),
                                                   widen16<ACT>((unsigned short)(a >> 16)), 0u);
        out[w] = quantize2_e4m3<true>(widen16<ACT>((unsigned short)(c & 0xFFFFu)), widen16<ACT>((unsigned short)(c >> 16)), lo2);
    }
    return out;
}

typedef float f32x2v __attribute__((ext_vector_type(2)));

// e4m3 codes -> fp32, exact, four codes of one 32-bit word (v_cvt_pk_f32_fp8 reads this format on gfx950).
__device__ __forceinline__ void widen4_e4m3(const unsigned w, float (&f)[4]) {
    const f32x2v lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, false);
    const f32x2v hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, true);
    f[0] = lo[0];
    f[1] = lo[1];
    f[2] = hi[0];
    f[3] = hi[1];
}

template <bool NT>
__device__ __forceinline__ u32x4 load16(const char *p) {
    return NT ? __builtin_nontemporal_load((const u32x4 *)p) : *(const u32x4 *)p;
}

// Quotients of whole numbers from the hardware's reciprocal (an exact integer division is forty instructions, here on
// the way to a launch's first load).  x / y rounded down, exact for x below 2^24: the product is off by less than one, which the
// remainder puts right.  And a whole number not below x / y, by less than 2 above it where x / y is below 2^19.
// Multi-head batch views with divisions and with quotients, us a layer: 16 x 256, 26 contexts of 20..60 rows 8.10, 7.87; 3 x 128, 600 of 5..60
// 16.9, 16.5; 16 x 64, 128 of 20..100 10.9, 10.7; level in longer launches.
__device__ __forceinline__ int quotient(int x, int y) {
    const int q = (int)((float)x * __builtin_amdgcn_rcpf((float)y)), r = x - q * y;
    return q + (r >= y ? 1 : 0) - (r < 0 ? 1 : 0);
}
__device__ __forceinline__ int not_below(int x, int y) { return (int)((float)x * __builtin_amdgcn_rcpf((float)y) * 1.000001f) + 1; }

// Work order of a launch: longest contexts first.  Contexts are put into `ncls` length classes
// relative to the longest context of the batch; the work list holds the chunks of class 0 (the longest)
// in batch order, then class 1, and so on.  Long items therefore start first and the short ones fill
// the end of the kernel (a ragged batch in random order ran 10 % slower), and the cross-workgroup
// merges of multi-chunk contexts overlap with the streaming of the rest.  The whole workgroup builds
// one exclusive prefix sum of chunk counts per class in LDS: pre[c][0..n] at cum[c * (n + 1)].
#define S3_MAX_CLASSES 8
#define S3_MAX_WAVES 16

__device__ __forceinline__ int chunks_of(const AttnArgs &a, int b, int chunk) {
    return (checked_len(a, b) + chunk - 1) / chunk;
}

__device__ __forceinline__ int class_of(int len, int max_len_seen, int ncls) {
    // (the order of the work only: a quotient off by one at a border costs nothing)
    return ncls - 1 - min(ncls - 1, (int)((float)(len * ncls) * __builtin_amdgcn_rcpf((float)(max_len_seen + 1))));
}

// Inclusive prefix sum over the 64 lanes of a wave with DPP row operations (no LDS round trips):
// shifts by 1, 2, 4, 8 inside each row of 16 lanes, then the row totals are carried into the
// following rows (row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_scan_step(int v) {
    return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xF, false);
}
__device__ __forceinline__ int wave_inclusive_scan(int v) {
    v = dpp_scan_step<0x111, 0xF>(v);  // row_shr:1
    v = dpp_scan_step<0x112, 0xF>(v);  // row_shr:2
    v = dpp_scan_step<0x114, 0xF>(v);  // row_shr:4
    v = dpp_scan_step<0x118, 0xF>(v);  // row_shr:8
    v = dpp_scan_step<0x142, 0xA>(v);  // row_bcast:15 -> rows 1, 3
    v = dpp_scan_step<0x143, 0xC>(v);  // row_bcast:31 -> rows 2, 3
    return v;
}

// Maximum of a non-negative value over the 64 lanes, same DPP ladder (lanes shifted in from outside a
// row read as 0, the identity here); every lane gets the result.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_max_step(int v) {
    return max(v, __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xF, false));
}
__device__ __forceinline__ int wave_max_nonneg(int v) {
    v = dpp_max_step<0x111, 0xF>(v);
    v = dpp_max_step<0x112, 0xF>(v);
    v = dpp_max_step<0x114, 0xF>(v);
    v = dpp_max_step<0x118, 0xF>(v);
    v = dpp_max_step<0x142, 0xA>(v);
    v = dpp_max_step<0x143, 0xC>(v);
    return __builtin_amdgcn_readlane(v, 63);
}

// Rows per chunk of a batch of few contexts (total and longest: their rows).  Two bounds.  (1) `few_chunks` chunks in
// all, so that every compute unit has an item and none has two (the host says how many: chunk_slots).
// (2) A context's chunks are merged by one wave, a few per memory round trip, while a chunk's rows stream side by
// side: a chunk of c rows costs about c / 10 of what merging one more chunk costs, so no finer than sqrt(10 * longest).
// One context, 16 heads x 256 fp16, four layers, best chunk of a sweep: 410 rows 64 (36.6 us; whole 72.1), 1417 rows
// 96 to 128 (51; 128), 8050 rows 256 to 384 (114; 181).
__device__ __forceinline__ int few_chunk_rows(const AttnArgs &a, int total, int longest) {
    if (longest <= 128) return a.chunk;  // a cut would save less than a merge costs (14 contexts of 30..68 rows: 7.8 us
                                         // a layer whole, 8.4 in pieces of 32)
    const int even = total / a.few_chunks + 1;
    const int least = (int)__builtin_amdgcn_sqrtf(10.f * (float)longest);
    return min(a.chunk, (max(max(even, least), 64) + 15) & ~15);
}

// Rows per chunk of a batch whose contexts are fewer than the workgroups that run at once (host: chunk_slots): the shortest
// whose chunks all run at once.  `units` less the `n * quarters / 4` chunks by which contexts do not divide evenly; whether
// that was enough is counted (one_wave_view).  Bounds as in few_chunk_rows.
__device__ __forceinline__ int unit_chunk_rows(const AttnArgs &a, int units, int total, int longest, int quarters, int most) {
    if (longest <= 128) return most;
    const int even = total / max(units - ((a.n * quarters + 3) >> 2), 1) + 1;
    const int least = (int)__builtin_amdgcn_sqrtf(10.f * (float)longest);
    return min(most, (max(max(even, least), 64) + 15) & ~15);
}

// 16-bit rows: whether the chunk length above takes the place of few_chunk_rows, or of chunks of 1024 rows (a.chunk), which a
// batch beyond the few contexts gets.  chunks: how many those would be; rows, longest: all rows, and those of the longest
// context.  Two kinds of batch gain:
// (1) few contexts whose chunks turn out more than the compute units (contexts do not divide evenly), so that some units get
// two and the launch lasts as long as those: by more than an eighth at 400 rows a context, by any number at 1000.  (Up to 64
// such contexts are attn_few_kernel's since; what comes here are 65 and more of one or two head groups.)
// (2) beyond the few, a longest chunk that outlasts the rest: u items a compute unit (2 * n / units) of r rows on average take
// the time of u * r rows, a single one streams about twice as fast once the others are done, and the finer division costs as
// much again where it shares out little: the line, measured, is longest / r = 2 * u^2, and 1.6.
// us a layer without and with: (1) 16 x 256, 18 contexts of 1000..2047 rows 94.1, 79.4, 64 x 96, 10 of 400..1400 63.8, 50.5, 12 x
// 128, 52 of 300..600 34.5, 29.7; below the line 64 x 96, 9 of 512..2048 52.1, 56.8.  (2) 16 x 256, 25 of 32..1000 46.4, 41.3, 12 x 128, 67 of 40..2000 with a long tail 48.5, 36.7; below the line 67 of 300..600 35.4, 39.1, 16 x 64, 98 of
// 10..200 13.7, 17.0.  Over 4160 batches (five shapes, thirteen kinds of lengths, 9/16 to 7/4 items a compute unit) those cut
// by (1) took 0.90 of their time, by (2) 0.85, at most 1.074.
__device__ __forceinline__ bool unit_rule(const AttnArgs &a, int units, int chunks, int rows, int longest) {
    if (a.few_chunks > 0)
        return 8 * chunks <= 7 * units && rows >= 400 * a.n && (16 * chunks > 9 * units || (2 * chunks > units && rows >= 1000 * a.n));
    const float most = (float)min(longest, a.chunk), all = (float)rows;
    return 2 * a.n <= units && longest >= 512 && 5.f * most * (float)a.n >= 8.f * all && most * (float)units * (float)units >= 8.f * (float)a.n * all;
}

// ... and whether the contexts stay whole where they would otherwise be cut at 1024 rows.  From 4/3 items a compute unit, no
// context so long that it outlasts the rest: if chunks of 1024 rows were more than run at once by a tenth, so that a second,
// mostly empty round followed, or nearly as many (7/8 and up) of contexts that differ about twofold.  us a layer cut at 1024 and
// whole: 64 x 96, 23 contexts of 400..1400 rows 106.1, 93.9, 23 of 64..1500 81.9, 77.2, 16 x 256, 46 of 200..1800 142.3, 137.7;
// outside the rule 64 x 96, 20 of 900..1100 83.8, 100.2, 16 x 256, 44 of 1000..2047 180.5, 193.  Over the batches above 0.96, at
// most 1.048.
__device__ __forceinline__ bool whole_rule(const AttnArgs &a, int units, int chunks, int rows, int longest) {
    if (a.few_chunks > 0 || 3 * a.n < 2 * units || longest <= a.chunk || 4 * longest > 7 * a.chunk) return false;
    if (chunks > units) return 10 * chunks >= 11 * units;
    return 8 * chunks >= 7 * units && 4 * longest * a.n >= 7 * rows && longest * a.n <= 2 * rows;
}

// LDS picture of the batch built by every workgroup at kernel start (dynamic shared memory):
//   off[n] (int64), len[n] (int32, 0 for refused entries), pre[ncls][n + 1] (int32)
struct BatchView {
    const int64_t *off;
    const int *len;
    const int *pre;
    int n, ncls, total;
    int chunk;  // rows per chunk
    int mean;   // mean rows of a context (0 unless the launch asks for it with class_rows)
};

__device__ __forceinline__ size_t batch_view_bytes(int n, int ncls) {
    return (size_t)n * 8 + (size_t)((n + 1) & ~1) * 4 + (size_t)ncls * (n + 1) * 4;
}

// The one-wave build of the view: lane l owns entries l*E .. l*E+E-1 (n <= 64*E).  `how`, for the other waves, where
// the rows decide: rows per chunk, classes, mean rows of a context.
template <int E, bool UNITS>
__device__ __forceinline__ void one_wave_view(const AttnArgs &a, int64_t *off_s, int *len_s, int *pre, int *how) {
    const int lane = threadIdx.x & 63, n = a.n;
    int chunk = a.chunk, ncls = a.ncls, mean = 0;
    int64_t off[E];
    int len[E], cls[E], cnt[E];
    int mx = 0;
    load_entries<E>(a, lane * E, off, len);
#pragma unroll
    for (int e = 0; e < E; e++) {
        const int b = lane * E + e;
        if (b < n) {
            len_s[b] = len[e];
            off_s[b] = off[e];
        }
        mx = max(mx, len[e]);
    }
    mx = wave_max_nonneg(mx);
    if (a.few_chunks > 0 || a.class_rows > 0 || (UNITS && a.unit_chunks > 0)) {
        int rows = 0;
#pragma unroll
        for (int e = 0; e < E; e++) rows += len[e];
        rows = __builtin_amdgcn_readlane(wave_inclusive_scan(rows), 63);
        if (a.few_chunks > 0) chunk = few_chunk_rows(a, rows, mx);
        auto chunks_of = [&](int rows_each) {
            int count = 0;
#pragma unroll
            for (int e = 0; e < E; e++) count += quotient(len[e] + rows_each - 1, rows_each);
            return __builtin_amdgcn_readlane(wave_inclusive_scan(count), 63);
        };
        const int sixteen = a.unit_chunks >> 16;
        if (UNITS && a.unit_chunks > 0 && (!sixteen || mx >= 400)) {
            // (16-bit rows: chunks of up to 2048 rows, where whole contexts are as many as run at once)
            const int units = a.unit_chunks & 0xFFFF, most = sixteen ? 2 * a.chunk : a.chunk;
            const int before = sixteen && (a.few_chunks > 0 || 2 * n > units) ? chunks_of(chunk) : 0;  // (where a rule asks)
            if (!sixteen || __builtin_expect(unit_rule(a, units, before, rows, mx), 0)) {
#pragma unroll 1
                for (int quarters = 2; quarters <= 4; quarters++) {
                    chunk = unit_chunk_rows(a, units, rows, mx, quarters, most);
                    if (chunk == most || chunks_of(chunk) <= units) break;
                }
            } else if (whole_rule(a, units, before, rows, mx)) {
                chunk = most;
            }
        }
        if (a.class_rows > 0) {
            mean = rows / n;
            if (mean < a.class_rows) ncls = 1;
        }
        if (lane == 0) {
            how[0] = chunk;
            how[1] = ncls;
            how[2] = mean;
        }
    }
#pragma unroll
    for (int e = 0; e < E; e++) {
        cls[e] = class_of(len[e], mx, ncls);
        cnt[e] = quotient(len[e] + chunk - 1, chunk);
    }
    for (int c = 0; c < ncls; c++) {
        int loc[E], lsum = 0;
#pragma unroll
        for (int e = 0; e < E; e++) {
            loc[e] = lsum;
            if (cls[e] == c) lsum += cnt[e];
        }
        const int incl = wave_inclusive_scan(lsum);
#pragma unroll
        for (int e = 0; e < E; e++) {
            const int b = lane * E + e;
            if (b < n) pre[c * (n + 1) + b] = incl - lsum + loc[e];
        }
        if (lane == 63) pre[c * (n + 1) + n] = incl;
    }
}

// The view with one length class, built by the whole workgroup: of every E * threads entries, thread t owns E
// neighbours; two barriers.  Returns the number of chunks.  WITH_ROWS: `rows` receives the rows of all contexts, and if
// they average `most` or more (most > 0) the scan ends there, lengths and offsets in place: -1, with the rows of the
// longest in `longest`.  agg: 2 * S3_MAX_WAVES words that nobody writes before the next barrier after this.
template <int E, bool WITH_ROWS>
__device__ __forceinline__ int block_view(const AttnArgs &a, int chunk, int64_t *off_s, int *len_s, int *pre, int *wave_sums,
                                          int most, int *agg, int64_t *rows, int *longest) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nwaves = blockDim.x >> 6;
    int total = 0;
#pragma unroll 1
    for (int base = 0; base < a.n; base += E * (int)blockDim.x) {
        int64_t off[E];
        int len[E], cnt[E], sum = 0;
        load_entries<E>(a, base + tid * E, off, len);
#pragma unroll
        for (int e = 0; e < E; e++) {
            const int b = base + tid * E + e;
            cnt[e] = quotient(len[e] + chunk - 1, chunk);
            sum += cnt[e];
            if (b < a.n) {
                len_s[b] = len[e];
                off_s[b] = off[e];
            }
        }
        const int incl = wave_inclusive_scan(sum);
        if (lane == 63) wave_sums[wave] = incl;
        if (WITH_ROWS) {
            int mine = 0, mx = 0;
#pragma unroll
            for (int e = 0; e < E; e++) {  // (a wave's rows: at most 256 contexts of 2^20)
                mine += len[e];
                mx = max(mx, len[e]);
            }
            mine = wave_inclusive_scan(mine);
            mx = wave_max_nonneg(mx);
            if (lane == 63) {
                agg[wave] = mine;
                agg[S3_MAX_WAVES + wave] = mx;
            }
        }
        __syncthreads();
        if (WITH_ROWS) {
            for (int w = 0; w < nwaves; w++) {
                *rows += agg[w];
                *longest = max(*longest, agg[S3_MAX_WAVES + w]);
            }
            if (most > 0 && base + E * (int)blockDim.x >= a.n && *rows >= (int64_t)most * a.n) return -1;
        }
        const int upto = wave_inclusive_scan(lane < nwaves ? wave_sums[lane] : 0);
        int run = total + incl - sum + (wave > 0 ? __builtin_amdgcn_readlane(upto, wave - 1) : 0);
        total += __builtin_amdgcn_readlane(upto, nwaves - 1);
#pragma unroll
        for (int e = 0; e < E; e++) {
            const int b = base + tid * E + e;
            if (b < a.n) pre[b] = run;
            run += cnt[e];
        }
        if (tid == 0) pre[a.n] = total;
        __syncthreads();
    }
    return total;
}

// Exclusive prefix sums of the entries' chunks of `rows` rows (len: as the view holds it) into pre[0..n]; returns the
// total.  Whoever reads pre[] before has met a barrier since.
__device__ __forceinline__ int chunk_prefix(int n, const int *len, int rows, int *pre, int *wave_sums) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nwaves = blockDim.x >> 6;
    int total = 0;
#pragma unroll 1
    for (int base = 0; base < n; base += blockDim.x) {
        const int b = base + tid, mine = b < n ? (len[b] + rows - 1) / rows : 0;
        const int incl = wave_inclusive_scan(mine);
        if (lane == 63) wave_sums[wave] = incl;
        __syncthreads();
        const int upto = wave_inclusive_scan(lane < nwaves ? wave_sums[lane] : 0);
        if (b < n) pre[b] = total + incl - mine + (wave > 0 ? __builtin_amdgcn_readlane(upto, wave - 1) : 0);
        total += __builtin_amdgcn_readlane(upto, nwaves - 1);
        if (tid == 0) pre[n] = total;
        __syncthreads();
    }
    return total;
}

// A view with one length class in chunks (tiles) of CHUNK rows; `longest` receives the rows of the longest context.  Kept
// small: every wave runs it before its first load.
template <int CHUNK>
__device__ __forceinline__ BatchView build_tile_view(const AttnArgs &a, char *dyn, int *wave_sums, int &longest) {
    int64_t *off_s = (int64_t *)dyn;
    int *len_s = (int *)(dyn + (size_t)a.n * 8);
    int *pre = len_s + ((a.n + 1) & ~1);
    BatchView v;
    v.off = off_s;
    v.len = len_s;
    v.pre = pre;
    v.n = a.n;
    v.ncls = 1;
    v.chunk = CHUNK;
    v.mean = 0;
    int64_t rows = 0;
    longest = 0;
    v.total = block_view<4, true>(a, CHUNK, off_s, len_s, pre, wave_sums, 0, wave_sums + S3_MAX_WAVES, &rows, &longest);
    return v;
}

// One pass over the device arrays (each entry is read from global memory once and checked once),
// then class-wise exclusive prefix sums of the chunk counts.
template <bool UNITS = false>
__device__ __forceinline__ BatchView build_batch_view(const AttnArgs &a, char *dyn, int *wave_sums) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nthreads = blockDim.x, nwaves = nthreads >> 6;
    const int ncls = a.ncls, chunk = a.chunk, n = a.n;
    int64_t *off_s = (int64_t *)dyn;
    int *len_s = (int *)(dyn + (size_t)n * 8);
    int *pre = len_s + ((n + 1) & ~1);
    if (n <= 64 * 8) {
        // Batches of up to 512 sequences: wave 0 builds the whole view by itself (lane l takes entries
        // l*E .. l*E+E-1; a serial prefix inside the lane, one DPP scan across lanes per class) and the
        // workgroup meets at ONE barrier.  The general path below needs four barriers and LDS round trips
        // between them, which cost every workgroup of a small launch about 1.5 us before its first load.
        // E is a compile-time constant per batch size class: the per-entry work (quotients for its chunks and its
        // class) is not spent on entries a small batch does not have.
        if (wave == 0) {
            if (n <= 64) one_wave_view<1, UNITS>(a, off_s, len_s, pre, wave_sums);
            else if (n <= 128) one_wave_view<2, UNITS>(a, off_s, len_s, pre, wave_sums);
            else if (n <= 256) one_wave_view<4, UNITS>(a, off_s, len_s, pre, wave_sums);
            else one_wave_view<8, UNITS>(a, off_s, len_s, pre, wave_sums);
        }
        __syncthreads();
        BatchView v;
        v.off = off_s;
        v.len = len_s;
        v.pre = pre;
        v.n = n;
        v.chunk = chunk;
        v.ncls = ncls;
        v.mean = 0;
        if (a.few_chunks > 0 || a.class_rows > 0 || (UNITS && a.unit_chunks > 0)) {
            v.chunk = __builtin_amdgcn_readfirstlane(wave_sums[0]);
            v.ncls = __builtin_amdgcn_readfirstlane(wave_sums[1]);
            v.mean = __builtin_amdgcn_readfirstlane(wave_sums[2]);
        }
        v.total = 0;
        for (int c = 0; c < v.ncls; c++) v.total += pre[c * (n + 1) + n];
        return v;
    }
    int mean = 0, mx = 0;
    if (ncls == 1 || a.class_rows > 0) {
        // One class: a scan over the workgroup (the general path below walks the entries three times and costs a
        // batch of 1024 about 5 us before its first load).
        BatchView v;
        v.off = off_s;
        v.len = len_s;
        v.pre = pre;
        v.n = n;
        v.ncls = 1;
        v.chunk = chunk;
        int64_t rows = 0;
        v.total = a.class_rows > 0 ? block_view<4, true>(a, chunk, off_s, len_s, pre, wave_sums, ncls > 1 ? a.class_rows : 0,
                                                         ncls > 1 ? pre + n + 1 : wave_sums + S3_MAX_WAVES, &rows, &mx)
                                   : block_view<4, false>(a, chunk, off_s, len_s, pre, wave_sums, 0, nullptr, nullptr, nullptr);
        v.mean = mean = __builtin_amdgcn_readfirstlane((int)(rows / n));
        if (v.total >= 0) return v;
    }
    const int per = (n + nthreads - 1) / nthreads;
    const int b0 = min(n, tid * per), b1 = min(n, b0 + per);
    if (a.class_rows == 0) {  // (else the scan above has done this)
        for (int b = b0; b < b1; b++) {
            const int len = checked_len(a, b);
            len_s[b] = len;
            off_s[b] = a.slot_off[b];
            mx = max(mx, len);
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) mx = max(mx, __shfl_xor(mx, d));
        if (lane == 0) wave_sums[wave] = mx;
        __syncthreads();
        for (int i = 0; i < nwaves; i++) mx = max(mx, wave_sums[i]);
        __syncthreads();  // wave_sums is reused below
    }
    int cnt[S3_MAX_CLASSES], incl[S3_MAX_CLASSES];
#pragma unroll
    for (int c = 0; c < S3_MAX_CLASSES; c++) cnt[c] = 0;
    for (int b = b0; b < b1; b++) {
        const int len = len_s[b];
        const int k = (len + chunk - 1) / chunk;
        const int cl = class_of(len, mx, ncls);
#pragma unroll
        for (int c = 0; c < S3_MAX_CLASSES; c++) cnt[c] += (c == cl) ? k : 0;
    }
#pragma unroll
    for (int c = 0; c < S3_MAX_CLASSES; c++) {
        if (c < ncls) {  // uniform
            const int v = wave_inclusive_scan(cnt[c]);
            incl[c] = v;
            if (lane == 63) wave_sums[c * S3_MAX_WAVES + wave] = v;
        }
    }
    __syncthreads();
    int run[S3_MAX_CLASSES];
#pragma unroll
    for (int c = 0; c < S3_MAX_CLASSES; c++) {
        run[c] = 0;
        if (c < ncls) {
            int base = 0;
            for (int i = 0; i < wave; i++) base += wave_sums[c * S3_MAX_WAVES + i];
            run[c] = base + incl[c] - cnt[c];
        }
    }
    for (int b = b0; b < b1; b++) {
        const int len = len_s[b];
        const int k = (len + chunk - 1) / chunk;
        const int cl = class_of(len, mx, ncls);
#pragma unroll
        for (int c = 0; c < S3_MAX_CLASSES; c++) {
            if (c < ncls) pre[c * (n + 1) + b] = run[c];
            run[c] += (c == cl) ? k : 0;
        }
    }
    if (tid == nthreads - 1) {
#pragma unroll
        for (int c = 0; c < S3_MAX_CLASSES; c++)
            if (c < ncls) pre[c * (n + 1) + n] = run[c];
    }
    __syncthreads();
    BatchView v;
    v.off = off_s;
    v.len = len_s;
    v.pre = pre;
    v.n = n;
    v.ncls = ncls;
    v.chunk = chunk;
    v.mean = mean;
    v.total = 0;
    for (int c = 0; c < ncls; c++) v.total += pre[c * (n + 1) + n];
    return v;
}

// Partials that cross workgroups inside ONE launch (fused step) must not sit in a cache that another XCD
// cannot see: they are stored and loaded with the sc0 sc1 cache bits (write-through to, and read from,
// memory-side coherence).  No cache write-back or invalidate is needed then (those cost far more than the
// partials themselves).  The accesses are written as machine instructions because the two ways the compiler
// offers are both slower than the exchange itself: `volatile` accesses carry the bits but each one is waited
// for on its own (three memory round trips per partial stored and three per partial merged: a context of 1417
// rows cut into 23 chunks took 27 us against 20 us in 12 chunks), and atomics are at most 64 bits wide.
// A store is left in flight (chunk_arrived() drains the wave's memory counter before the count; the s_nop keeps
// the data registers unwritten for the cycle that a store of more than 64 bits needs); loads wait inside
// their own asm block, so that no register is ever the target of a load the compiler does not know of.
typedef float f32x2 __attribute__((ext_vector_type(2)));
template <bool COHERENT>
__device__ __forceinline__ void put_partial4(float *p, const f32x4 v) {
    if (COHERENT) asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
    else *(f32x4 *)p = v;
}
template <bool COHERENT>
__device__ __forceinline__ void put_partial2(float *p, const f32x2 v) {
    if (COHERENT) asm volatile("global_store_dwordx2 %0, %1, off sc0 sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
    else *(f32x2 *)p = v;
}
__device__ __forceinline__ void put_partial1(float *p, const float v) {
    asm volatile("global_store_dword %0, %1, off sc0 sc1" ::"v"(p), "v"(v) : "memory");
}
// Four partials at once, one memory round trip for all: (max, sum) at ml[u], eight accumulator values at acc[u].
template <bool COHERENT>
__device__ __forceinline__ void get_partials(const float *const (&ml)[4], const float *const (&acc)[4], f32x2 (&m)[4], f32x4 (&lo)[4],
                                             f32x4 (&hi)[4]) {
    if (!COHERENT) {
#pragma unroll
        for (int u = 0; u < 4; u++) {
            m[u] = *(const f32x2 *)ml[u];
            lo[u] = *(const f32x4 *)acc[u];
            hi[u] = *(const f32x4 *)(acc[u] + 4);
        }
        return;
    }
    asm volatile(
        "global_load_dwordx2 %0, %12, off sc0 sc1\n\t"
        "global_load_dwordx2 %1, %13, off sc0 sc1\n\t"
        "global_load_dwordx2 %2, %14, off sc0 sc1\n\t"
        "global_load_dwordx2 %3, %15, off sc0 sc1\n\t"
        "global_load_dwordx4 %4, %16, off sc0 sc1\n\t"
        "global_load_dwordx4 %5, %16, off offset:16 sc0 sc1\n\t"
        "global_load_dwordx4 %6, %17, off sc0 sc1\n\t"
        "global_load_dwordx4 %7, %17, off offset:16 sc0 sc1\n\t"
        "global_load_dwordx4 %8, %18, off sc0 sc1\n\t"
        "global_load_dwordx4 %9, %18, off offset:16 sc0 sc1\n\t"
        "global_load_dwordx4 %10, %19, off sc0 sc1\n\t"
        "global_load_dwordx4 %11, %19, off offset:16 sc0 sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(m[0]), "=&v"(m[1]), "=&v"(m[2]), "=&v"(m[3]), "=&v"(lo[0]), "=&v"(hi[0]), "=&v"(lo[1]), "=&v"(hi[1]),
          "=&v"(lo[2]), "=&v"(hi[2]), "=&v"(lo[3]), "=&v"(hi[3])
        : "v"(ml[0]), "v"(ml[1]), "v"(ml[2]), "v"(ml[3]), "v"(acc[0]), "v"(acc[1]), "v"(acc[2]), "v"(acc[3])
        : "memory");
}

// The matrix-core kernel's loads of partials, as other workgroups of the launch wrote them: 16 or 8 bytes past every cache that another XCD does not see (sc0
// sc1).  Through a buffer descriptor, so that what lies past its end (pieces that are not there, lanes without an element)
// reads as zeros and costs no traffic and no branch: unlike plain loads these never hit a cache (pairs of 64-bit atomic
// loads before, the last piece's repeated for those that are not there: 16q/1kv x 256, 3 contexts of 700..924 rows 17.7 us
// a layer, now 16.7; 512 of 32..1000 81.4 and 78.9).  The compiler tracks them, so any number stays in flight.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t piece_buffer(const float *p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ f32x4 piece_load4(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 17));
}
__device__ __forceinline__ f32x2 piece_load2(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 17));
}

// The arrival counter of context b, head group (column) g of n_groups.  The counter region holds 4096 of each group; smaller
// batches keep theirs apart, up to a cache line each (128 contexts), since atomics on one line wait for each other: eight
// neighbouring counters, on which 200 workgroups counted, cost the last of them 2.5 us.
__device__ __forceinline__ unsigned int *arrival_counter(const AttnArgs &a, int b, int n_groups, int g) {
    const int apart = min(5, __builtin_clz((unsigned)(a.n - 1) | 1u) - 20);  // n << apart <= 4096
    return a.arrivals + (((int64_t)b * n_groups + g) << apart);
}

// A wave has written its chunk's partial: count the chunk on the context's arrival counter.  Returns true
// (to every lane) in the wave that delivered the LAST chunk of the context; that wave then merges the chunks,
// and the counter is back at zero for the next launch.  Called by whole waves in uniform control flow.
// Two orderings of "my partial is visible before my count, the others' partials are visible after theirs":
//   merge_sync 0  the partials are written and read with the write-through / cache-bypassing accesses above,
//                 so they are at the memory side once this wave's vector-memory counter has drained
//                 (s_waitcnt 0); the counter is a relaxed device-scope atomic.  (A host-side test compiles
//                 these helpers and checks the cache bits and the order in the emitted code.)
//   merge_sync 1  the same accesses, ordered by the memory model instead: a device-scope release fence
//                 before the count and an acquire fence in the wave that merges (L2 write-back and
//                 invalidate on this device, which cost far more than the partials themselves).
__device__ __forceinline__ bool chunk_arrived(const AttnArgs &a, unsigned int *cnt, int nchunks) {
    const int lane = threadIdx.x & 63;
    if (a.merge_sync) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // this wave's partial stores have completed
    unsigned int old = 0;
    if (lane == 0) old = atomicAdd(cnt, 1u);
    old = __builtin_amdgcn_readfirstlane(old);
    if (old != (unsigned int)(nchunks - 1)) return false;
    if (lane == 0) atomicExch(cnt, 0u);  // leave the counter clean for the next launch
    if (a.merge_sync) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return true;
}

// Matrix-core kernel.  A context of which this wave or team has left a piece in memory: its pieces are `count` (0:
// nothing left), by the publishing units first, first + 1, ...; unit u keeps its piece of context b in partial slot u + b
// (along the shares either u or b grows from one piece to the next, so no two pieces meet; chunks, which belong to one
// context each, are counted so that u + b is the chunk's number).
struct Pending {
    int b, first, count;
};

// This wave (its team) has written the pieces p0 and p1 (count 0: none): count them on their contexts' arrival
// counters, both in one round trip; bit k of the result: the last piece of p_k's context has arrived, and this wave
// merges it.  See chunk_arrived() for the two orderings.
__device__ __forceinline__ unsigned pieces_arrived(const AttnArgs &a, const Pending &p0, const Pending &p1, int columns, int col) {
    const int lane = threadIdx.x & 63;
    if (a.merge_sync) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // the partial stores have completed
    const int count = lane == 0 ? p0.count : p1.count;
    unsigned int *cnt = arrival_counter(a, lane == 0 ? p0.b : p1.b, columns, col);
    bool mine = false;
    if (lane < 2 && count != 0) {
        mine = atomicAdd(cnt, 1u) == (unsigned int)(count - 1);
        if (mine) atomicExch(cnt, 0u);  // leave the counter clean for the next launch
    }
    const unsigned who = (unsigned)__builtin_amdgcn_ballot_w64(mine);
    if (a.merge_sync && who != 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    asm volatile("" ::: "memory");  // no piece is loaded before this
    return who;
}
// Merge the chunk partials of (sequence b, head h), in slots slot0, slot0 + 1, ..., for this lane's 8-element slice and
// store the final output row slice; H is the head count of the partial and output arrays.  nchunks >= 2.  Four chunks are loaded
// per round, in one memory round trip.
template <int D, bool COHERENT>
__device__ __forceinline__ void merge_chunks(const AttnArgs &a, int64_t slot0, int H, int b, int h, int dl, int nchunks) {
    const int64_t p0 = slot0 * H + h;
    const float *ml = (const float *)a.part_ml;
    float mm = -INFINITY, l = 0.f;
    float o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < nchunks; c0 += 4) {
        float mv[4], lv[4], av[4][8];
        const float *mp[4], *ap[4];
        f32x2 mlv[4];
        f32x4 lo[4], hi[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int64_t pi = p0 + (int64_t)min(c0 + u, nchunks - 1) * H;
            mp[u] = ml + 2 * pi;
            ap[u] = a.part_acc + pi * D + dl * 8;
        }
        get_partials<COHERENT>(mp, ap, mlv, lo, hi);
#pragma unroll
        for (int u = 0; u < 4; u++) {
            mv[u] = mlv[u][0];
            lv[u] = mlv[u][1];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                av[u][i] = lo[u][i];
                av[u][4 + i] = hi[u][i];
            }
        }
        float mn = mm;
#pragma unroll
        for (int u = 0; u < 4; u++) mn = fmaxf(mn, mv[u]);  // repeats of the last chunk do not change the max
        const float ref = exp_reference(mn), alpha = fast_exp2(mm - ref);
        l *= alpha;
#pragma unroll
        for (int i = 0; i < 8; i++) o[i] *= alpha;
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const float wgt = (c0 + u < nchunks) ? fast_exp2(mv[u] - ref) : 0.f;
            l += wgt * lv[u];
#pragma unroll
            for (int i = 0; i < 8; i++) o[i] += wgt * av[u][i];
        }
        mm = mn;
    }
    const float inv = 1.f / l;
#pragma unroll
    for (int i = 0; i < 8; i++) o[i] *= inv;
    store_out8(a.out, a.out_dtype, ((int64_t)b * H + h) * D + dl * 8, o);
}

// What a workgroup item is: chunk c of sequence b for head block hgb.
struct Item {
    int b, c, nchunks, len, hgb;
    int slot0;  // work-list position (partial slot) of the context's first chunk
    int clen;  // rows per chunk of this context: the context is cut into nchunks near-equal pieces
    int64_t off;
};

// Rows per chunk when a context of len rows is cut into nchunks pieces: near-equal pieces; falls
// back to `chunk` if rounding would leave the last piece empty.
__device__ __forceinline__ int balanced_chunk_len(int len, int nchunks, int chunk) {
    if (nchunks <= 1) return chunk;
    const int clen = quotient(len + nchunks - 1, nchunks);
    return (nchunks - 1) * clen < len ? clen : chunk;
}

// Rows [j0, j1) of item `it` that token split ts of TS takes: the item's rows are divided evenly
// (split 0 is never empty; trailing splits may be).
__device__ __forceinline__ void split_rows(const Item &it, int ts, int TS, int &j0, int &j1) {
    const int start = it.c * it.clen;
    const int end = min(it.len, start + it.clen);
    const int per = (end - start + TS - 1) / TS;
    j0 = min(end, start + ts * per);
    j1 = min(end, j0 + per);
}

// The first sequence whose range of a prefix-sum array holds position w: the number of entries b with pre[b + 1] <= w
// (the sums are non-decreasing).  Whole waves, every lane with the same w.  The lanes test every ceil(n/64)-th
// border at once and then the borders between two of those: two LDS round trips whatever the batch.
__device__ __forceinline__ int find_sequence(const int *pre, int n, int w) {
    const int lane = threadIdx.x & 63;
    const int step = (n + 63) >> 6;
    int e = (lane + 1) * step;
    const int at = step * __builtin_popcountll(__builtin_amdgcn_ballot_w64(e <= n && pre[min(e, n)] <= w));
    if (step == 1) return at;
    e = at + lane + 1;
    return at + __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < step - 1 && e <= n && pre[min(e, n)] <= w));
}

// Work-list position -> item.  Called by whole waves (every lane with the same `item`): the class
// totals are read by the first lanes at once and the sequence is found by counting, lanes in parallel,
// the entries whose inclusive prefix does not exceed the position (the prefix sums are non-decreasing,
// so that count is the first sequence whose range holds it): three dependent LDS round trips
// instead of a serial class walk plus a binary search.
__device__ __forceinline__ Item decode_item(const AttnArgs &a, const BatchView &v, int64_t item, int n_hgb) {
    Item it;
    const int lane = threadIdx.x & 63;
    // (items beyond 2^24: whole numbers of 32 bits and more, in forty and a hundred instructions)
    int w = item < (1 << 24) ? quotient((int)item, n_hgb) : (int)(item / n_hgb);
    it.hgb = (int)(item - (int64_t)w * n_hgb);
    it.slot0 = w;
    const int tot = lane < v.ncls ? v.pre[lane * (v.n + 1) + v.n] : 0;
    int cls = v.ncls - 1;
    for (int c = 0; c < v.ncls - 1; c++) {  // which class the item falls into
        const int t = __builtin_amdgcn_readlane(tot, c);
        if (w < t) {
            cls = c;
            break;
        }
        w -= t;
    }
    const int *pre = v.pre + cls * (v.n + 1);
    int lo = find_sequence(pre, v.n, w);
    lo = min(lo, v.n - 1);  // a consistent view never needs this
    it.b = lo;
    it.c = w - pre[lo];
    it.slot0 -= it.c;
    it.nchunks = pre[lo + 1] - pre[lo];
    it.len = v.len[lo];
    it.off = v.off[lo];
    if (it.c < 0 || it.c >= it.nchunks) {  // cannot happen with a consistent view; never index rows from it
        it.c = 0;
        it.nchunks = 1;
        it.len = 0;
        it.slot0 = 0;
    }
    it.clen = balanced_chunk_len(it.len, it.nchunks, v.chunk);
    return it;
}

// A wave-uniform value as the compiler should see it: in scalar registers, so that addresses and branches
// derived from it are scalar too.
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ Item uniform_item(const Item &i) {
    Item o;
    o.b = __builtin_amdgcn_readfirstlane(i.b);
    o.c = __builtin_amdgcn_readfirstlane(i.c);
    o.nchunks = __builtin_amdgcn_readfirstlane(i.nchunks);
    o.slot0 = __builtin_amdgcn_readfirstlane(i.slot0);
    o.len = __builtin_amdgcn_readfirstlane(i.len);
    o.hgb = __builtin_amdgcn_readfirstlane(i.hgb);
    o.clen = __builtin_amdgcn_readfirstlane(i.clen);
    o.off = uniform64(i.off);
    return o;
}

typedef void (*attn_fn)(const AttnArgs);
#define S3_UNIT_VARIANT 1000  // see pick_variant()

// Kernel for shared key/value heads (defined in s3kv_gqa.hip): gq query heads per K/V head and
// lane (1, 2, 4 or 8), shape = index into its (waves, rows per load batch) table, < 0 for the
// default of that gq.  Returns the kernel and its workgroup size, or null.
attn_fn s3i_pick_gqa(int dt, int d, int gq, int shape, int *threads);
// Kernels for 8-bit (e4m3) cache rows (defined in s3kv_fp8.hip): the attention kernel for activation
// type act (S3_F16 / S3_BF16) and its workgroup size, and the append that quantises a new row.
attn_fn s3i_pick_fp8(int act, int d, int shape, int *threads);
typedef void (*append_fp8_fn)(char *, char *, const int64_t *, const int32_t *, const char *, const char *, int32_t,
                              int64_t, int32_t);
append_fp8_fn s3i_pick_append_fp8(int act);
// Matrix-core kernel for shared key/value heads (defined in s3kv_gqa_mfma.hip): q of type act, rows of the same or (kv8) e4m3
// codes; 256 threads per workgroup, one work item per wave, or (wide) 512, one per workgroup; loop: more items than waves.
attn_fn s3i_pick_gqa_mfma(int act, int d, bool kv8, bool wide, bool loop);
attn_fn s3i_pick_gqa_few_heads(int dt, int d, int group, bool wide, bool loop);  // 16-bit rows, two or three query heads per cached head
#define S3_FEW_CONTEXTS 256  // contexts whose view every wave of that kernel builds by itself
