// Matrix-core attention kernel for shared key/value heads (multi-query / grouped-query attention,
// which the paper's related-work section names as a complementary way to shrink the cache), gfx950.
// Launched by the host code in s3kv_kernels.hip through the pointer s3i_pick_gqa_mfma returns.
//
// With one cached head serving `group` query heads, a decode step is no longer one dot product per
// cached row but a small dense contraction: scores S^T[rows x heads] = K[rows x D] . Q^T[D x heads]
// and output O^T[D x heads] = V^T[D x rows] . P^T[rows x heads].  The vector-ALU kernel repeats the
// dot / exp / accumulate work per query head and becomes instruction bound from about eight heads
// per cached head; here both products run on MFMA and every (row, head) score is handled by
// exactly one lane.
//
// With two or three query heads per cached head only the scores are a matrix product (GQ, pick_few_heads).
// Two instances: workgroups of eight waves for launches of no more (context, column) pairs than compute units, which know
// only chunks (eight_wave_plan), and workgroups of four for all others (chunk_plan, share_plan).
// Work division.  A column is one (K/V head, block of 16 query heads); every column has the same rows, in tiles of 16
// or 32.  Many rows: the contexts lie end to end, that length is cut into equal shares and a wave takes one share of one
// column, across the borders of contexts, so the waves end together whatever the lengths of the batch and a context is
// cut only where a share ends (share_plan).  Few rows: every context by itself is cut into chunks, each taken by one
// wave or by all waves of a workgroup (chunk_plan, eight_wave_plan).  A context inside one share or chunk leaves as its final row; a
// piece of a longer one leaves as a partial (max, sum, unnormalised row) and whoever delivers the last piece merges
// them inside this launch.  Dealing chunks of 128 or 256 rows by stride instead let nearly every context leave partials
// (7 to 14 % extra traffic), needed a second launch to merge them (5 to 6 us of device time a step) and left units idle
// in the last round of the stride (16 query heads on one cached head of 256, 256 contexts of 32..1000 rows: 1216
// chunks on 1024 waves).
// Per tile:
//   * K and V rows are loaded whole, 16 bytes a lane, one or two tiles ahead, and pass through a per-wave LDS buffer (row-major;
//     the row strides are at the kernel's start).
//   * K: lane (r = lane % 16, g = lane / 16) reads 16 bytes (8 elements) of row r at element offset 32*ks + 8*g,
//     ks = 0 .. D/32-1: the A operand of v_mfma_f32_16x16x32 (row r, contraction slots of lane group g); Q^T is the B
//     operand, loaded once per context with the same slot assignment (head = lane % 16), so whichever way the
//     instruction numbers its contraction slots, both operands agree.  The accumulator holds S^T[row 4*g + i][head
//     lane % 16], i < 4.
//   * softmax: scale into log2 units, mask rows past the end, tile maximum per head (over the four
//     registers, then across the four lane groups); the exponent reference m follows the maximum
//     lazily (see the loop), p = exp2(s - m), running sum.
//   * V: the accumulator layout of S^T is already the B-operand layout of the second product (rows 4*g .. 4*g+3 of a
//     block of 16, column = head), so P^T needs no shuffle.  The A operand V^T (row of the product = output element d,
//     contraction = cached rows) needs four cached rows at one d per lane, while memory holds eight d of one row per
//     16-byte load: 16-bit rows come out of LDS through the transposing read (ds_read_b64_tr_b16).  With 8-bit rows a
//     lane reads one 32-bit word (four consecutive d) from each of its four rows and transposes the 4 x 4 codes in
//     registers (eight v_perm_b32), which feeds four products at once; the products' operand rows are numbered
//     accordingly (d = 64q + 4n + j) and the results leave in that order.
//   * p enters the second product as two 16-bit operands of the storage type, a high part (p rounded)
//     and a low part (the remainder, rounded), and the product is issued for both, which keeps the
//     weights' error near 2^-16 (bfloat16) / 2^-22 (fp16) instead of 2^-9 / 2^-12: with one part only,
//     values of magnitude 1e2 put the fp16 kernel outside the attention tolerance.
// Accumulators: O^T block db holds O^T[d = 16*db + 4*g + i][head], fp32.  In a decode step the new row is read
// from k_new / v_new and appended by the wave that owns it (8-bit rows: with eight waves, else by a launch before).
#include <type_traits>

#include "s3kv_device.h"

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <int DT>
__device__ __forceinline__ f32x4 mfma_scores(const u32x4 a, const u32x4 b, const f32x4 c) {
    if (DT == S3_F16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// V^T . P^T for RB blocks of 16 rows (two operand words each), P^T as its high and its low part.  Sixteen rows, two dependent products of
// sixteen slots and one of 32, us a layer: 16q/1kv x 256 e4m3, 515 contexts of 100..200 rows 28.0, 27.5, 140 of 32..1000 17.6, 17.3; fp16, 256 of
// 100..200 15.05, 15.22 (the most it loses: 1.2 %); 239 launches level in the mean.
template <int DT, int RB>
__device__ __forceinline__ f32x4 mfma_weights(const unsigned (&v)[2 * RB], const unsigned (&hi)[2 * RB], const unsigned (&lo)[2 * RB], f32x4 c) {
    if constexpr (RB == 2) {
        const u32x4 a = (u32x4){v[0], v[1], v[2], v[3]};
        c = mfma_scores<DT>(a, (u32x4){hi[0], hi[1], hi[2], hi[3]}, c);
        return mfma_scores<DT>(a, (u32x4){lo[0], lo[1], lo[2], lo[3]}, c);
    } else {  // sixteen rows: both parts in the 32 contraction slots of one product, the rows' operand twice
        return mfma_scores<DT>((u32x4){v[0], v[1], v[0], v[1]}, (u32x4){hi[0], hi[1], lo[0], lo[1]}, c);
    }
}

// Lane h (0, 1 or 2) of each sixteen lanes to the lanes of BANKS (four lanes a bit) of that sixteen; the others keep `old`.
template <int BANKS>
__device__ __forceinline__ float head_weight(const float old, const float from, const int h) {
    const int a = __builtin_bit_cast(int, old), b = __builtin_bit_cast(int, from);
    const int r = h == 0   ? __builtin_amdgcn_update_dpp(a, b, 0x150, 0xF, BANKS, false)  // row_newbcast:0
                  : h == 1 ? __builtin_amdgcn_update_dpp(a, b, 0x151, 0xF, BANKS, false)
                           : __builtin_amdgcn_update_dpp(a, b, 0x152, 0xF, BANKS, false);
    return __builtin_bit_cast(float, r);
}

// Between writes to LDS and reads of the same words by other lanes of the wave: the LDS unit serves the wave in issue order,
// so it is only the compiler that must not move the one across the other, nor hand a lane the value it wrote itself.
__device__ __forceinline__ void lds_exchange() {
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ unsigned pack_f16(float lo, float hi) {
    const f16x2 h = {(_Float16)lo, (_Float16)hi};
    return __builtin_bit_cast(unsigned, h);
}
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {  // round to nearest even (v_cvt_pk_bf16_f32)
    const bf16x2 h = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(unsigned, h);
}

// Four consecutive output elements starting at element index e.
__device__ __forceinline__ void store_out4(void *out, int out_dtype, int64_t e, const f32x4 v) {
    if (out_dtype == S3_F32) {
        *(f32x4 *)((float *)out + e) = v;
    } else {
        u32x2 w;
        if (out_dtype == S3_F16) {
            w[0] = pack_f16(v[0], v[1]);
            w[1] = pack_f16(v[2], v[3]);
        } else {
            w[0] = f32_to_bf16_rne(v[0]) | (f32_to_bf16_rne(v[1]) << 16);
            w[1] = f32_to_bf16_rne(v[2]) | (f32_to_bf16_rne(v[3]) << 16);
        }
        *(u32x2 *)((uint16_t *)out + e) = w;
    }
}

// Sixteen lanes read four rows of sixteen 16-bit elements, lane i the four elements of row i / 4 at its own address;
// lane i receives element i of each row.
__device__ __forceinline__ u32x2 lds_transpose4(const char *p) {
    typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(__attribute__((address_space(3))) void *)(void *)p));
}

// Two e4m3 codes (bytes 2*half, 2*half+1 of w) -> one 32-bit word of two DT elements, exact: every e4m3 value
// is an fp16 and a bfloat16 number, and gfx950 converts a pair of codes to either type in one instruction
// (v_cvt_scalef32_pk_{f16,bf16}_fp8 with scale 1).
template <int DT>
__device__ __forceinline__ unsigned widen2_e4m3(const unsigned w, const bool upper) {
    if (DT == S3_F16) {
        const f16x2 h = upper ? __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w, 1.0f, true) : __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w, 1.0f, false);
        return __builtin_bit_cast(unsigned, h);
    }
    const bf16x2 h = upper ? __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true) : __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false);
    return __builtin_bit_cast(unsigned, h);
}

// Bytes j of four words -> one word, j = 0..3 (a 4 x 4 byte transpose in eight v_perm_b32; selector bytes 0-3
// pick from the second operand, 4-7 from the first).
__device__ __forceinline__ void transpose4x4_bytes(const unsigned w0, const unsigned w1, const unsigned w2, const unsigned w3,
                                                   unsigned (&t)[4]) {
    const unsigned a_lo = __builtin_amdgcn_perm(w1, w0, 0x05010400u);  // w0.0 w1.0 w0.1 w1.1
    const unsigned a_hi = __builtin_amdgcn_perm(w1, w0, 0x07030602u);  // w0.2 w1.2 w0.3 w1.3
    const unsigned b_lo = __builtin_amdgcn_perm(w3, w2, 0x05010400u);  // w2.0 w3.0 w2.1 w3.1
    const unsigned b_hi = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
    t[0] = __builtin_amdgcn_perm(b_lo, a_lo, 0x05040100u);  // w0.0 w1.0 w2.0 w3.0
    t[1] = __builtin_amdgcn_perm(b_lo, a_lo, 0x07060302u);
    t[2] = __builtin_amdgcn_perm(b_hi, a_hi, 0x05040100u);
    t[3] = __builtin_amdgcn_perm(b_hi, a_hi, 0x07060302u);
}

// How a launch of few rows divides them (four waves a workgroup): every context by itself, into near-equal
// chunks of at most `per` tiles, one wave or a team of four waves a chunk, all at once.  Nothing is combined that the
// lengths do not force: a context of one chunk is finished by its wave or team.  (The figures of few contexts were taken before
// workgroups of eight took the launches of no more pairs than compute units.)  What bounds such a launch is a chain of
// latencies (view and plan 2.5 us, rows a tile a microsecond and wave, the team's meeting in LDS 1, write-through and count
// 1, merge 2 to 3) and, throughout, instructions that run once.  A layer in microseconds, shares
// across contexts or chunks by one wave -> this rule: 32q/8kv x 128, 3 contexts of 512..8192 rows 18.9 -> 16.2, 8 of
// 32..2000 18.9 -> 15.3, 19 of 70..84 9.7 -> 8.1; 12q/2kv x 128, 17 of 1200..1455 19.8 -> 15.8; 16q/1kv x 256, 3 of
// 700..924 25.0 -> 16.9, 30 of 32..1000 29.0 -> 18.1, 100 30.8 -> 22.8; 64q/8kv x 128 e4m3, 22 of 2000..4793 44.6 -> 41.7,
// 25 of 60..1106 21.4 -> 18.9; beyond 256 contexts 16q/1kv x 256, 300 of 2..40 37.0 -> 15.3, 12q/2kv x 128, 260 of 2..20
// 21.4 -> 9.7.
// Up to S3_FEW_CONTEXTS every wave builds the view for itself (four entries a lane), beyond the workgroup does.
struct ChunkPlan {
    int units, least;  // per column: chunks that run at once, and tiles below which a chunk is not cut (0 units: no chunks)
    int team;
};
// Tiles per chunk, if n / 4 * quarters chunks beyond tiles / per are allowed for (contexts do not divide evenly; 4: always enough).
__device__ __forceinline__ int chunk_tiles(const AttnArgs &a, const ChunkPlan &p, int tiles, int quarters) {
    const int room = min(p.units - ((a.n * quarters + 3) >> 2), a.max_shares);
    return max(not_below(tiles, max(room, 1)), p.least);
}
// One wave a chunk: the wave that merges a context reads its pieces a few per memory round trip while their tiles stream
// side by side, so with `merge_cost` tiles' worth of time per piece (see launch_gqa_mfma) no finer than sqrt(merge_cost *
// tiles of a context); not for chunks beyond 64 KiB of K rows (shares then; 128 KiB beyond 256 contexts of
// sixteen heads of 256, whose pieces of 16 KiB cost shares most: 16q/1kv x 256, 600 of 10..300 rows, chunks of 15 tiles 35.0
// us, shares 42.3; 12q/2kv x 128 e4m3, 702 of 145..518, outside the rule: 41.8, shares 37.5) or contexts of more than 12 pieces on average.
// A team a chunk: no finer than sqrt(1.3 * tiles) or 8 tiles, and contexts of up to 14 tiles whole (one context of 1100
// rows, 32q/8kv x 128, chunks of 4, 8, 12, 16 tiles: 12.6, 11.4, 12.4, 13.1 us; 3 of 512..8192: 18.7, 18.7, 16.8, 15.7, 24:
// 16.6; 16q/1kv x 256, 3 of 700..924: 18.9, 17.8, 18.6, 19.4; 11 of 20..211 rows cut at 8 tiles 10.4, whole 9.5).
// Between the two: the longest wave's tiles, and that a team's four waves merge groups of more than four heads faster
// than one wave does, which small groups' teams lose again at their meeting (16q/8kv x 128 e4m3, 40 contexts of
// 100..1500: waves with 5 tiles 22.1 us, with 5.75 in teams 23.6; 40q/5kv x 128, 30 of 100..2000: 8 tiles 28.8, 5.5 in teams
// 24.0).  That no more than half a chunk a context is allowed for to begin with (the count on the device tells):
// 40q/5kv 25.1 -> 24.2, 64q/8kv e4m3, 22 of 2000..4793, 43.3 -> 41.7.
template <int TR, int ROW_BYTES>
__device__ __forceinline__ ChunkPlan chunk_plan(const AttnArgs &a, int tiles, int longest) {
    ChunkPlan one = {0, 0, 1}, four = {0, 0, 4};
    if (a.max_shares <= 1) return one;
    const float average = (float)tiles * __builtin_amdgcn_rcpf((float)a.n);
    int per = 0;
    if (a.wave_shares > a.n) {
        one.units = a.wave_shares;
        one.least = (int)__builtin_amdgcn_sqrtf(a.merge_cost * 1.5f * average) + 1;
        per = chunk_tiles(a, one, tiles, a.n > S3_FEW_CONTEXTS ? 4 : 2);
        if (per > (a.n > S3_FEW_CONTEXTS && a.merge_cost > 2.f ? 131072 : 65536) / ROW_BYTES / TR || average > 12.f * (float)per) one.units = 0;
    }
    if (a.team_shares > a.n) {
        four.units = a.team_shares;
        const bool whole = longest <= 14;
        four.least = whole ? longest : max(8, (int)__builtin_amdgcn_sqrtf(1.3f * average));
        const int bonus = whole ? 8 : a.merge_cost < 0.5f ? -6 : 8;
        if (min(chunk_tiles(a, four, tiles, 2), longest) <= (one.units > 0 ? 4 * per + bonus : 4 * not_below(tiles, a.wave_shares) + 16)) return four;
    }
    return one;
}

// Teams of eight waves, where the (context, column) pairs are no more than the compute units (launch_gqa_mfma): one workgroup
// a unit, all chunks at once.  With four waves a unit a wave's tile is a chain (rows into LDS, score products, maximum,
// exponents, value products: 1 us at 16 rows x 256) that nothing else on its SIMD fills, and a chunk is as long as four such
// chains; eight waves halve the chain and overlap two of them, and twice the pieces meet in LDS instead of memory.
// Contexts of up to 22 tiles are whole: counting and merging their pieces costs more than the shorter chains give (16q/1kv x
// 256, 16 contexts of 240..300 rows whole 14.0 us a layer, cut 14.6; of 360..450: 16.5, 14.9).  Longer ones in chunks of at
// least a tile a wave, and no finer than sqrt(2 * tiles): 16 of 1000..2000 rows, factor 1, 2, 3: 20.0, 18.5, 18.8; 32q/8kv x
// 128, 3 of 512..8192: 14.9, 14.1, 13.5; one of 8000 rows of 16q/1kv: 22.7, 23.1, 23.8; at least 8, 12, 16 tiles, 16q/1kv, 16 of 360..450:
// 14.9, 15.4, 16.6.  Four waves by the rules above -> eight: 16q/1kv x 256, 256 contexts of 32..1000 rows 44.1 -> 37.2, 200 of
// 1000..2000 86 -> 64, 3 of 32..1000 16.5 -> 14.8; the same of e4m3 rows, 200 of 32..1000, 31.5 -> 25.1 (21.7 with
// the append inside); 32q/8kv x 128, 3 of
// 512..8192 16.4 -> 14.1, 32 of 32..1000 20.9 -> 19.5; 8q/1kv x 64, 256 of 32..1000 16.5 -> 13.3.
__device__ __forceinline__ ChunkPlan eight_wave_plan(const AttnArgs &a, int tiles, int longest) {
    const float average = (float)tiles * __builtin_amdgcn_rcpf((float)a.n);
    return ChunkPlan{a.team_shares, longest <= 22 ? longest : max(8, (int)__builtin_amdgcn_sqrtf(2.f * average)), 8};
}

// The context that holds position w of the work list: its index, the position of its first chunk, its chunks, rows and
// offset.  All fields are wave-uniform.
struct Located {
    int seq, first, count, len;
    int64_t off;
};
// ... from the view in LDS
__device__ __forceinline__ Located locate(const BatchView &v, int w) {
    Located x;
    x.seq = min(find_sequence(v.pre, v.n, w), v.n - 1);
    x.first = __builtin_amdgcn_readfirstlane(v.pre[x.seq]);
    x.count = __builtin_amdgcn_readfirstlane(v.pre[x.seq + 1]) - x.first;
    x.len = __builtin_amdgcn_readfirstlane(v.len[x.seq]);
    x.off = uniform64(v.off[x.seq]);
    return x;
}
// ... from the registers that the view is made in (lane l: entries E*l .. E*l+E-1, `run` chunks before them): a ballot and
// a few lane reads, where the same through LDS is six dependent round trips.
template <int E>
__device__ __forceinline__ Located locate(const int64_t (&off)[E], const int (&len)[E], const int (&cnt)[E], int run, int incl, int w) {
    const int at = min(__builtin_popcountll(__builtin_amdgcn_ballot_w64(incl <= w)), 63);
    Located x;
    x.first = __builtin_amdgcn_readlane(run, at);
    int e = 0;
    x.count = __builtin_amdgcn_readlane(cnt[0], at);
#pragma unroll
    for (int k = 1; k < E; k++) {  // (an entry without chunks holds no position)
        const int c = __builtin_amdgcn_readlane(cnt[k], at);
        const bool on = e == k - 1 && w >= x.first + x.count;
        x.first += on ? x.count : 0;
        x.count = on ? c : x.count;
        e = on ? k : e;
    }
    x.seq = at * E + e;
    x.len = __builtin_amdgcn_readlane(len[0], at);
    int lo = __builtin_amdgcn_readlane((int)off[0], at), hi = __builtin_amdgcn_readlane((int)(off[0] >> 32), at);
#pragma unroll
    for (int k = 1; k < E; k++) {
        const int l = __builtin_amdgcn_readlane(len[k], at), a = __builtin_amdgcn_readlane((int)off[k], at),
                  b = __builtin_amdgcn_readlane((int)(off[k] >> 32), at);
        x.len = e == k ? l : x.len;
        lo = e == k ? a : lo;
        hi = e == k ? b : hi;
    }
    x.off = (int64_t)(((uint64_t)(unsigned)hi << 32) | (unsigned)lo);
    return x;
}

// The view of few contexts, and how they are divided: every wave of the workgroup builds all of it by itself and writes the
// same values to the same words, so that nothing waits at a barrier before its first load (a wave reads behind its own writes).
// Lane l owns entries E*l .. E*l+E-1.  here: the context of position `w`, if there is one (eight waves: the first unit).
template <int E, int TR, int ROW_BYTES, int NW>
__device__ __forceinline__ BatchView few_view(const AttnArgs &a, char *dyn, int &tiles, int &longest, int &per, int &team, int w, Located &here) {
    const int lane = threadIdx.x & 63;
    BatchView v;
    int64_t *off_s = (int64_t *)dyn;
    int *len_s = (int *)(dyn + (size_t)a.n * 8), *pre = len_s + ((a.n + 1) & ~1);
    v.off = off_s;
    v.len = len_s;
    v.pre = pre;
    v.n = a.n;
    v.ncls = 1;
    v.mean = v.chunk = 0;
    int64_t off[E];
    int len[E], cnt[E], sum = 0, most = 0;
    load_entries<E>(a, lane * E, off, len);
#pragma unroll
    for (int e = 0; e < E; e++) {
        cnt[e] = (len[e] + TR - 1) / TR;
        sum += cnt[e];
        most = max(most, cnt[e]);
    }
    int incl = wave_inclusive_scan(sum);
    tiles = __builtin_amdgcn_readlane(incl, 63);
    ChunkPlan plan = {0, 0, 1};
    longest = wave_max_nonneg(most);
    per = a.share_rows / TR;  // the caller's choice (a multiple of 32)
    if (NW == 8) plan = eight_wave_plan(a, tiles, longest);
    else if (per == 0) plan = chunk_plan<TR, ROW_BYTES>(a, tiles, longest);
    team = plan.team;
#pragma unroll 1
    for (int quarters = 2; per > 0 || plan.units > 0; quarters++) {
        if (plan.units > 0) per = min(chunk_tiles(a, plan, tiles, quarters), max(longest, 1));  // (small numbers for quotient())
        sum = 0;
#pragma unroll
        for (int e = 0; e < E; e++) {
            cnt[e] = quotient((len[e] + TR - 1) / TR + per - 1, per);
            sum += cnt[e];
        }
        incl = wave_inclusive_scan(sum);
        if (plan.units == 0 || quarters == 4 || __builtin_amdgcn_readlane(incl, 63) <= min(plan.units, a.max_shares + a.n)) break;
    }
    v.total = __builtin_amdgcn_readlane(incl, 63);
    int run = incl - sum;
    if (NW == 8) here = locate<E>(off, len, cnt, run, incl, w);
#pragma unroll
    for (int e = 0; e < E; e++) {
        const int b = lane * E + e;
        if (b < a.n) {
            off_s[b] = off[e];
            len_s[b] = len[e];
            pre[b] = run;
        }
        run += cnt[e];
    }
    if (lane == 63) pre[a.n] = v.total;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    return v;
}

// How a launch divides its rows: `shares` equal runs of tiles per column, share k = tiles
// [k * base + min(k, rem), ...) with one tile more for the first `rem`.  team 1: every wave works for itself and
// a piece of a context cut by a share's border goes to memory.  team 4: the four waves of a workgroup take four
// consecutive shares of one column and first merge their pieces through LDS.
// whole: both borders of a share move on to where the next context begins, so that no piece leaves a wave.
struct SharePlan {
    int tiles, shares, base, rem, team;
    bool whole;
};

// Whole contexts: where the fixed buffer has no room for pieces (max_shares 0, see s3i_gqa_max_shares); and for short
// contexts, each of which a share's border would cut for about 4 us of counting and merging a launch (10 and more in teams):
// a share of c contexts comes out longer or shorter by one of them, which pays while they average no more than 2c tiles and
// none has more than 16, and instead of teams while none has more than 12.  32q/8kv x 128, 600 contexts of 1..30 rows: 20.6
// us a layer, 25.9 cut; 1400 of 20..200: 138.0, 138.1; 700 of 1..255 (outside the rule): 91.7, 85.8; 400 of 10..60: 22.8, in
// teams 26.6; 64q/8kv, 1010 of 20..200: 114.4, 118.9.

// Why the line between team 1 and team 4 lies at 256 rows a share: a piece costs a write-through store
// and a read of its fp32 rows, 16 query heads x D x 4 bytes twice against D x 4 bytes (16-bit K and V) per
// cached row, so with shares of r rows pieces add up to 2 * 2 * 16 / r of the traffic (two pieces a share; grouped
// heads less, in the ratio of the group to 16): 6 % at a share of 1000 rows, 25 % at 256.  Four waves together
// leave a quarter of that, but meet at barriers at the end of their share, and waves that stream rows of
// adjacent cached heads (team 1: neighbouring waves are neighbouring columns) read whole cached rows between them.
#define S3_TEAM_ROWS 256
// A team's waves take at least this many rows each: below it, what a share costs whatever its length (the meeting in
// LDS, the write-through, the count, the merge of the pieces) outweighs the rows.  Shares of at least 32, 64, 128 rows,
// 8q/1kv x 64, 300 contexts of 20..123 rows: 12.8, 15.2, 18.5 us a layer; 16q/1kv x 256, 300 of 20..200: 28.8, 31.8, 41.6.
#define S3_TEAM_MIN_ROWS 32

// tiles: tiles of TR rows per column.
template <int TR>
__device__ __forceinline__ SharePlan share_plan(const AttnArgs &a, int tiles, int longest) {
    SharePlan sp;
    sp.tiles = tiles;
    sp.team = 1;
    const bool few_rows = tiles < a.wave_shares * (S3_TEAM_ROWS / TR);
    sp.whole = a.max_shares == 0 || (longest <= (few_rows ? 12 : 16) && (few_rows || (int64_t)tiles * a.wave_shares <= 2 * (int64_t)a.n * a.n));
    int shares = sp.whole ? a.wave_shares : min(a.wave_shares, a.max_shares);
    if (a.team_lds && !sp.whole && tiles < shares * (S3_TEAM_ROWS / TR)) {
        sp.team = 4;
        constexpr int LEAST = 4 * (S3_TEAM_MIN_ROWS / TR);
        shares = 4 * min(min(a.team_shares, a.max_shares), (tiles + LEAST - 1) / LEAST);
    }
    sp.shares = max(1, min(shares, tiles));
    sp.base = tiles / sp.shares;
    sp.rem = tiles - sp.base * sp.shares;
    return sp;
}
__device__ __forceinline__ int share_start(const SharePlan &sp, int k) { return k * sp.base + min(k, sp.rem); }
__device__ __forceinline__ int share_of(const SharePlan &sp, int tile) {
    const int cut = sp.rem * (sp.base + 1);
    return tile < cut ? tile / (sp.base + 1) : sp.rem + (tile - cut) / sp.base;
}
// Publishing units (shares, or teams of four) that context b's tiles [t0, t1) touch: the first one and how many.
__device__ __forceinline__ void pieces_of(const SharePlan &sp, int t0, int t1, int &first, int &count) {
    const int sh = sp.team == 4 ? 2 : 0;
    first = share_of(sp, t0) >> sh;
    count = (share_of(sp, t1 - 1) >> sh) - first + 1;
}

// Merge the pieces of query heads hq0 .. hq0+nh-1 of a context and store the final rows; by a wave (nthr 64) or by
// the four or eight (EIGHT) waves of a workgroup in step (nthr 256, 512).  Four waves with at least a thread per quad of elements
// take one quad a thread and deals the pieces over what threads are spare, which meet in LDS (6 floats per thread).
// Kept small: unrolled for every shape, with the code around it, the kernel was 136 KB and a merge of four pieces took 3 us.
template <int D, bool EIGHT>
__device__ __forceinline__ void merge_pieces(const AttnArgs &a, const Pending &p, int hq0, int nh, int tid, int nthr, float *lds) {
    const int64_t row0 = ((int64_t)p.first + p.b) * a.Hq + hq0;
    const int64_t sml = 2 * (int64_t)a.Hq, sacc = (int64_t)a.Hq * D;
    const float *pml = (const float *)a.part_ml + 2 * row0, *pacc = a.part_acc + row0 * D;
    char *out = (char *)a.out;
    const int64_t out0 = ((int64_t)p.b * a.Hq + hq0) * D;
    const int quads = nh * (D / 4);
    if (!EIGHT && nthr == 256 && quads <= 256 && p.count > 4 && (int64_t)p.count * sacc < (1 << 28)) {  // (below 1 GiB)
        const int splits = min(8, 256 / quads);
        const int split = tid / quads, e = tid - split * quads;
        const unsigned sml4 = (unsigned)sml * 4, sacc4 = (unsigned)sacc * 4, last = p.count - 1;
        const __amdgpu_buffer_rsrc_t mls = piece_buffer(pml, last * sml4 + nh * 8), accs = piece_buffer(pacc, last * sacc4 + quads * 16);
        const unsigned eml = 8 * (e / (D / 4)), eacc = 16 * e;
        __syncthreads();  // an earlier merge has read the LDS
        if (split < splits) {
            constexpr int NP = 8;  // pieces per memory round trip
            float m = -INFINITY, l = 0.f;
            f32x4 o = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int c = split; c < p.count; c += NP * splits) {
                f32x2 mv[NP];
                f32x4 av[NP];
#pragma unroll
                for (int u = 0; u < NP; u++) {
                    mv[u] = piece_load2(mls, (c + u * splits) * sml4 + eml);
                    av[u] = piece_load4(accs, (c + u * splits) * sacc4 + eacc);
                }
#pragma unroll
                for (int u = 0; u < NP; u++) mv[u][0] = c + u * splits < p.count ? mv[u][0] : -INFINITY;
                float mn = m;
#pragma unroll
                for (int u = 0; u < NP; u++) mn = fmaxf(mn, mv[u][0]);
                const float ref = exp_reference(mn), alpha = fast_exp2(m - ref);
                l *= alpha;
                o *= alpha;
#pragma unroll
                for (int u = 0; u < NP; u++) {
                    const float w = fast_exp2(mv[u][0] - ref);
                    l += w * mv[u][1];
                    o += w * av[u];
                }
                m = mn;
            }
            *(f32x4 *)(lds + tid * 4) = o;
            *(f32x2 *)(lds + 1024 + tid * 2) = (f32x2){m, l};
        }
        __syncthreads();
        if (tid < quads) {
            float m = -INFINITY, l = 0.f;
            f32x4 o = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int k = 0; k < splits; k++) {  // (a split without a piece: max -inf, sum 0)
                const f32x2 x = *(const f32x2 *)(lds + 1024 + (k * quads + tid) * 2);
                const float mn = fmaxf(m, x[0]), ref = exp_reference(mn), alpha = fast_exp2(m - ref), w = fast_exp2(x[0] - ref);
                l = l * alpha + w * x[1];
                o = o * alpha + w * *(const f32x4 *)(lds + (k * quads + tid) * 4);
                m = mn;
            }
            store_out4(out, a.out_dtype, out0 + tid * 4, o * (1.f / l));
        }
        return;
    }
    // Whole waves in step, every lane EB quads: the piece is uniform, so its address is scalar and a lane adds one 32-bit
    // offset per quad (at most 64 heads' rows of a piece: 64 KiB).
    constexpr int EB = D == 256 && !EIGHT ? 4 : 2, NP = D == 256 && !EIGHT ? 3 : 6;
#pragma unroll 1
    for (int e0 = tid; e0 < quads; e0 += EB * nthr) {
        unsigned eml[EB], eacc[EB];
        float m[EB], l[EB];
        f32x4 o[EB];
#pragma unroll
        for (int i = 0; i < EB; i++) {
            const int e = e0 + i * nthr;  // (past the last quad: past the end of a piece)
            eml[i] = 8 * (e / (D / 4));
            eacc[i] = 16 * e;
            m[i] = -INFINITY;
            l[i] = 0.f;
            o[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll 1
        for (int c = 0; c < p.count; c += NP) {
            f32x2 mv[EB][NP];
            f32x4 av[EB][NP];
#pragma unroll
            for (int u = 0; u < NP; u++) {
                const bool there = c + u < p.count;
                const __amdgpu_buffer_rsrc_t mls = piece_buffer(pml + (c + u) * sml, there ? nh * 8 : 0);
                const __amdgpu_buffer_rsrc_t accs = piece_buffer(pacc + (c + u) * sacc, there ? quads * 16 : 0);
#pragma unroll
                for (int i = 0; i < EB; i++) {
                    mv[i][u] = piece_load2(mls, eml[i]);
                    av[i][u] = piece_load4(accs, eacc[i]);
                }
            }
#pragma unroll
            for (int u = 0; u < NP; u++)
#pragma unroll
                for (int i = 0; i < EB; i++) mv[i][u][0] = c + u < p.count ? mv[i][u][0] : -INFINITY;
#pragma unroll
            for (int i = 0; i < EB; i++) {
                float mn = m[i];
#pragma unroll
                for (int u = 0; u < NP; u++) mn = fmaxf(mn, mv[i][u][0]);
                const float ref = exp_reference(mn), alpha = fast_exp2(m[i] - ref);
                l[i] *= alpha;
                o[i] *= alpha;
#pragma unroll
                for (int u = 0; u < NP; u++) {
                    const float w = fast_exp2(mv[i][u][0] - ref);
                    l[i] += w * mv[i][u][1];
                    o[i] += w * av[i][u];
                }
                m[i] = mn;
            }
        }
#pragma unroll
        for (int i = 0; i < EB; i++)
            if (e0 + i * nthr < quads) store_out4(out, a.out_dtype, out0 + (e0 + i * nthr) * 4, o[i] * (1.f / l[i]));
    }
}

// 16 bytes at byte `off` of the buffer, zeros past its end.
template <bool NT>
__device__ __forceinline__ u32x4 buffer_load16(__amdgpu_buffer_rsrc_t rsrc, unsigned off) {
    return __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, NT ? 2 : 0);
}

// A context as a wave's share sees it.  All fields are wave-uniform.
struct Segment {
    int seq, t0, t_end;  // its index in the batch, its first tile, the tile after its last one in this share
    int t1;              // the tile after its last one
    int len;
    int64_t off;
};

// Rows of a tile.  Cached rows of up to 128 bytes a head: 32, so that a wave's two register sets hold 8 KiB and the work
// per tile (maximum, exponent reference, loop) is spread over twice the rows, and the second product runs at the
// instruction's full 32 contraction slots; longer rows: 16 (the sets and the accumulators fill the registers).
__host__ __device__ constexpr int gqa_tile_rows(int row_bytes) { return row_bytes <= 128 ? 32 : 16; }

// KV8: the cache rows are e4m3 codes (one byte per element) and DT is the type of q; a 16-byte load then
// holds 16 elements, which are widened (exactly) to DT in registers and feed two contraction steps.
// NW: waves of a workgroup, 4 or 8.
// GQ: 2 or 3, the query heads per cached head where these are so few: the scores on the matrix cores, the weighted rows on the
// vector ALU with the weights in fp32 (pick_few_heads); 0: both products on the matrix cores.
// LOOP: there may be more units than waves (teams), see s3i_gqa_units; else every wave (team) takes one, and nothing is computed, and spilled, in
// front of a loop for units that do not come (137 to 169 scalar registers spilled with it, 58 to 105 without).
template <int DT, int D, bool KV8, int NW, int GQ = 0, bool LOOP = false>
__global__ void __launch_bounds__(NW * 64, NW == 8 || D <= 128 ? 2 : 1) attn_gqa_mfma_kernel(const AttnArgs a) {
    constexpr int EB = KV8 ? 1 : 2;       // bytes per cached element
    constexpr int KS = D / 32;            // contraction steps of the score product
    constexpr int CH = KS < 4 ? KS : 4;   // ... in as many chains
    constexpr int DB = D / 16;            // 16-element blocks of an output row
    constexpr int PPR = D * EB / 16;      // 16-byte pieces per cached row of one head
    constexpr int TR = gqa_tile_rows(D * EB), RB = TR / 16;  // rows of a tile, in blocks of 16
    constexpr int NL = TR * PPR / 64;     // 16-byte loads per lane for a tile of K or of V
    constexpr int NK = D * EB / 64;       // 16-byte K operands per lane and row block
    constexpr int RPL = 64 / PPR;         // rows per load instruction
    // LDS row strides, bytes.  K: with 16 bytes of padding the 128-bit reads of sixteen rows cover every bank once.
    // V, 16-bit rows: the transposing reads touch 32 consecutive bytes of sixteen rows, which 32 bytes of padding
    // spread over all banks.  V, 8-bit rows: 16 bytes of padding, so that the four lane groups' 32-bit reads (rows
    // 4g .. 4g+3, sixteen consecutive words each) cover the banks evenly.
    constexpr int KSTRIDE = D * EB + 16;
    constexpr int VSTRIDE = KV8 ? D + 16 : D * 2 + 32;
    constexpr bool CHUNKS = NW == 8;      // eight waves: chunks of contexts by teams, nothing else
    // Register sets of rows on their way: two, or one where two (with the new row of 8-bit rows) do not fit two waves a
    // SIMD: 239 and 229 of 256 registers.
    constexpr bool TWO_SETS = !(NW == 8 && D == 256);
    static_assert(GQ == 0 || (!KV8 && GQ <= 3 && NL * RPL == TR), "16-bit rows, two or three heads");
    constexpr bool APPENDS = !KV8 || CHUNKS;  // takes the new row of a decode step itself (else the host appends it first)
    constexpr float RESCALE_LOG2 = GQ > 0 ? 0.f : 8.f;  // see the softmax step
    extern __shared__ __align__(16) char dyn_lds[];  // the batch view, then the teams' first pieces
    __shared__ int wave_sums[S3_MAX_CLASSES * S3_MAX_WAVES];
    // A wave's LDS: the V and the K tile, or, once its share is done, one piece (16 heads x D floats, padded).
    constexpr int PSTRIDE = D + 4;
    // (GQ: the piece, behind it what each of the RPL groups of lanes has summed)
    constexpr int TILE_BYTES = TR * (VSTRIDE + KSTRIDE), PIECE_BYTES = GQ > 0 ? (GQ * PSTRIDE + RPL * GQ * D) * 4 : 16 * PSTRIDE * 4;
    __shared__ __align__(16) char wave_lds[NW][TILE_BYTES > PIECE_BYTES ? TILE_BYTES : PIECE_BYTES];
    __shared__ float2 piece_ml[2 * NW][16];  // teams: (max, sum) of each wave's first (2w) and last (2w + 1) piece
    __shared__ f32x4 piece_run[CHUNKS ? 1 : 8][16];  // ... a piece's weight in its run of pieces, and the run's (max, sum, 1 / sum)
    __shared__ int piece_b[2 * NW];          // ... and the context it belongs to, -1: none
    __shared__ int merge_mine;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int group = a.group, nqb = a.nqb, columns = a.columns;
    // pre[] counts tiles, or (per > 0) chunks of `per` tiles
    int tiles, longest, per, team = 1;  // (longest: tiles of the longest context)
    BatchView bv;
    Located here = {0, 0, 0, 0, 0};  // (eight waves: the context of the unit at hand)
    if (CHUNKS || a.n <= S3_FEW_CONTEXTS) {
        const int w = __builtin_amdgcn_readfirstlane(a.column_shift >= 0 ? blockIdx.x >> a.column_shift : blockIdx.x / columns);
        bv = a.n <= 64 ? few_view<1, TR, D * EB, NW>(a, dyn_lds, tiles, longest, per, team, w, here)
                       : few_view<S3_FEW_CONTEXTS / 64, TR, D * EB, NW>(a, dyn_lds, tiles, longest, per, team, w, here);
    } else {
        bv = build_tile_view<TR>(a, dyn_lds, wave_sums, longest);
        tiles = __builtin_amdgcn_readfirstlane(bv.total);
        longest = (__builtin_amdgcn_readfirstlane(longest) + TR - 1) / TR;
        per = a.share_rows / TR;  // the caller's chunks (0: none)
        if (per == 0) {
            const ChunkPlan plan = chunk_plan<TR, D * EB>(a, tiles, longest);
            if (plan.units > 0) per = min(chunk_tiles(a, plan, tiles, 4), max(longest, 1));
            team = plan.team;
        }
    }
    SharePlan sp = {tiles, 1, tiles, 0, 1, false};
    int chunks = __builtin_amdgcn_readfirstlane(bv.total);
    if (CHUNKS) {
        per = max(per, 1);
    } else if (per == 0) {
        sp = share_plan<TR>(a, tiles, longest);
        team = sp.team;
    } else if (a.n > S3_FEW_CONTEXTS) {
        chunks = __builtin_amdgcn_readfirstlane(chunk_prefix(a.n, bv.len, TR * per, (int *)bv.pre, wave_sums));
    }

    char *vt = wave_lds[wave];
    char *kt = vt + TR * VSTRIDE;
    // team 4: the first piece of each wave's share waits here (as many heads as the group has) while the share goes on
    const int piece_heads = min(16, group);
    float *first_piece = (float *)(dyn_lds + ((batch_view_bytes(a.n, 1) + 15) & ~(size_t)15)) + (size_t)wave * piece_heads * PSTRIDE;
    float *last_piece = (float *)vt;
    const int64_t rstride = (int64_t)a.H * D * EB;
    const unsigned rs32 = (unsigned)rstride;  // a cached row of all K/V heads: at most 64 KiB
    // The K rows are read with the streaming hint, like the V rows, when this launch has more of them than the
    // memory-side cache holds, so that none survives until the next step; else with plain loads (a batch whose K rows
    // fit finds most of them still cached one step later: 256 sequences of 32q/8kv x 128 in chunks of 128 rows read
    // at 0.76 of peak against 0.63 with the hint; a batch of 1024 the other way round, 0.66 against 0.63).
    const bool stream_k = a.stream_k < 0 ? (int64_t)tiles * TR * rstride > ((int64_t)256 << 20) : a.stream_k != 0;

    // (shares * columns tiles of at least 2 KiB lie in the arena: below 2^31 on any device)
    const unsigned units = tiles == 0 ? 0u : (unsigned)(CHUNKS || per > 0 ? chunks : team == 4 ? (sp.shares + 3) / 4 : sp.shares) * columns;
    const unsigned step = CHUNKS || team == 4 ? gridDim.x : gridDim.x * 4;
    // (chunks: one wave on every compute unit before any unit gets a second one)
#pragma unroll 1
    for (unsigned unit = CHUNKS || team == 4 ? blockIdx.x : per > 0 ? wave * gridDim.x + blockIdx.x : blockIdx.x * 4 + wave; unit < units; unit += step) {
        // publishing unit: this wave's share or chunk, or its team's
        const int pub = __builtin_amdgcn_readfirstlane(a.column_shift >= 0 ? unit >> a.column_shift : unit / columns);
        const int col = __builtin_amdgcn_readfirstlane(unit - (unsigned)pub * columns);
        const int hk = nqb == 1 ? col : col / nqb, qb = col - hk * nqb;
        const int head = qb * 16 + n;  // query head of this lane's column, within the group
        const bool head_ok = head < group;
        const int hq = hk * group + (head_ok ? head : group - 1);
        const int hq0 = hk * group + qb * 16, nheads = min(16, group - qb * 16);
        // This wave's tiles, [t_begin, t_stop): of all contexts laid end to end, or (chunks) of context `seq`.
        int t_begin = 0, t_stop = 0, seq = 0, chunk = 0, nchunks = 0;
        if (CHUNKS || per > 0) {
            if (!CHUNKS) here = locate(bv, pub);
            seq = here.seq;
            nchunks = here.count;
            chunk = pub - here.first;
            const int all = (here.len + TR - 1) / TR;
            // near-equal pieces, none of them empty: the first all % nchunks have a tile more
            const int base = quotient(all, max(nchunks, 1)), rem = all - base * nchunks;
            t_begin = chunk * base + min(chunk, rem);
            t_stop = t_begin + base + (chunk < rem ? 1 : 0);
            if (CHUNKS || team == 4) {  // an equal part each
                const int quarter = (t_stop - t_begin) / NW, more = (t_stop - t_begin) % NW;
                t_begin += wave * quarter + min(wave, more);
                t_stop = t_begin + quarter + (wave < more ? 1 : 0);
            }
        } else {
            const int share = team == 4 ? pub * 4 + wave : pub;
            if (share < sp.shares) {
                t_begin = share_start(sp, share);
                t_stop = share_start(sp, share + 1);
                if (sp.whole) {
                    if (t_begin > 0) t_begin = __builtin_amdgcn_readfirstlane(bv.pre[min(find_sequence(bv.pre, a.n, t_begin - 1) + 1, a.n)]);
                    t_stop = __builtin_amdgcn_readfirstlane(bv.pre[min(find_sequence(bv.pre, a.n, t_stop - 1) + 1, a.n)]);
                }
                seq = min(find_sequence(bv.pre, a.n, t_begin), a.n - 1);
            }
        }
        // contexts this wave or team has left a piece of in memory: at most the first and the last one of its share
        Pending pend0 = {0, 0, 0}, pend1 = {0, 0, 0};
        if ((CHUNKS || team == 4) && lane == 0) piece_b[2 * wave] = piece_b[2 * wave + 1] = -1;

        if (t_begin < t_stop) {
            // Two cursors run over the share's tiles: `ahead` issues the loads of a tile (of the next context, if there
            // is one) into the register set that `now` has just moved to LDS, one tile a set on, so a wave has loads in flight from
            // its first tile to its last.  A tile is read through a buffer descriptor that ends with the context's last
            // row: rows past it, and the tiles after the last one of the share, cost no traffic and read as zeros.
            // Row and column of a lane's 16 bytes never change: the addresses take no vector arithmetic.
            unsigned voff[NL];
#pragma unroll
            for (int i = 0; i < NL; i++) voff[i] = (unsigned)(i * RPL + lane / PPR) * rs32 + (lane % PPR) * 16;
            auto open = [&](int seq, int t) {  // the context of tile t, at or after `seq`
                Segment s;
                s.t0 = 0;
                if (!CHUNKS && per == 0) {
                    while (seq < a.n - 1 && __builtin_amdgcn_readfirstlane(bv.pre[seq + 1]) <= t) seq++;
                    s.t0 = __builtin_amdgcn_readfirstlane(bv.pre[seq]);
                }
                s.seq = seq;
                s.len = CHUNKS ? here.len : __builtin_amdgcn_readfirstlane(bv.len[seq]);
                s.t1 = s.t0 + (s.len + TR - 1) / TR;
                s.t_end = min(t_stop, s.t1);
                s.off = CHUNKS ? here.off : uniform64(bv.off[seq]);
                return s;
            };
            const int64_t head_byte = (int64_t)hk * D * EB;
            Segment now = open(seq, t_begin), ahead = now;
            int t = t_begin, t_ahead = t_begin;
            int rows_ahead = now.len - (t_begin - now.t0) * TR;  // rows of `ahead` from tile t_ahead on
            int64_t at = (now.off + (t_begin - now.t0) * TR) * rstride + head_byte;
            auto load_tile = [&](u32x4 (&kk)[NL], u32x4 (&vv)[NL]) {
                if (t_ahead == ahead.t_end && t_ahead < t_stop) {
                    ahead = open(ahead.seq + 1, t_ahead);
                    at = ahead.off * rstride + head_byte;  // (a context is entered at its first row, but for a share's first)
                    rows_ahead = ahead.len;
                }
                const int bytes = t_ahead < t_stop ? (int)((unsigned)(min(TR, rows_ahead) - 1) * rs32 + D * EB) : 0;
                const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(a.kplane + at, 0, bytes, 0x00020000);
                const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc(a.vplane + at, 0, bytes, 0x00020000);
                if (stream_k) {
#pragma unroll
                    for (int i = 0; i < NL; i++) kk[i] = buffer_load16<true>(krs, voff[i]);
                } else {
#pragma unroll
                    for (int i = 0; i < NL; i++) kk[i] = buffer_load16<false>(krs, voff[i]);
                }
#pragma unroll
                for (int i = 0; i < NL; i++) vv[i] = buffer_load16<true>(vrs, voff[i]);
                t_ahead++;
                at += TR * rstride;
                rows_ahead -= TR;
            };

            u32x4 qop[KS];
            u32x4 knew = (u32x4){0u, 0u, 0u, 0u}, vnew = knew, knew2 = knew, vnew2 = knew;  // (knew2, vnew2: 8-bit rows only)
            f32x4 o[DB];
            float acc[GQ > 0 ? GQ : 1][8];  // GQ: this lane's eight elements of the weighted sums, over its rows of every load
            float m = -INFINITY, lsum = 0.f;
            int jnew = -1;  // decode step: the row of `now` that is still only in k_new / v_new
            auto enter = [&]() {  // start on context `now`
#pragma unroll
                for (int ks = 0; ks < KS; ks++) {
                    // elements of contraction step ks held by lane group g: the same as the K operand's (a 16-byte K
                    // load of 8-bit rows covers 16 elements = steps 2j and 2j+1 of lane group g)
                    const int e0 = KV8 ? (ks >> 1) * 64 + g * 16 + (ks & 1) * 8 : ks * 32 + g * 8;
                    qop[ks] = *(const u32x4 *)(a.q + (((int64_t)now.seq * a.Hq + hq) * D + e0) * 2);
                    if (!head_ok) qop[ks] = (u32x4){0u, 0u, 0u, 0u};  // padding columns: zero scores, never stored
                }
                // Decode step (len_add = 1): row len-1 is still only in k_new / v_new.  Every reader takes it from
                // there; the wave of query block 0 whose tile holds it also writes it into the arena (the append).
                // (8-bit rows: the 16-bit row waits until its tile's turn, so that nothing in flight is waited for here.)
                if (APPENDS && a.len_add) {
                    jnew = now.len - 1;
                    if (jnew < (now.t_end - now.t0) * TR && lane < PPR) {  // in this share
                        const int64_t at = ((int64_t)now.seq * a.H + hk) * D * 2 + lane * (KV8 ? 32 : 16);
                        knew = *(const u32x4 *)(a.k_new + at);
                        vnew = *(const u32x4 *)(a.v_new + at);
                        if (KV8) {
                            knew2 = *(const u32x4 *)(a.k_new + at + 16);
                            vnew2 = *(const u32x4 *)(a.v_new + at + 16);
                        }
                    }
                }
                if constexpr (GQ > 0) {
#pragma unroll
                    for (int h = 0; h < GQ; h++)
#pragma unroll
                        for (int e = 0; e < 8; e++) acc[h][e] = 0.f;
                } else {
#pragma unroll
                    for (int db = 0; db < DB; db++) o[db] = (f32x4){0.f, 0.f, 0.f, 0.f};
                }
                m = -INFINITY;
                lsum = 0.f;
            };
            auto stage_tile = [&](int r0, const u32x4 (&kld)[NL], const u32x4 (&vv)[NL]) {
                // K and V tile through this wave's LDS buffer: K into operand layout, one 128-bit read per contraction
                // load (loading the operand layout directly is 64 separate 16-byte cache accesses per instruction and
                // fetches every 128-byte line twice), V transposed.  The LDS unit serves one wave's operations in
                // issue order; the wave barriers only keep the compiler from moving them across.
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int i = 0; i < NL; i++) *(u32x4 *)(kt + (i * RPL + lane / PPR) * KSTRIDE + (lane % PPR) * 16) = kld[i];
#pragma unroll
                for (int i = 0; i < NL; i++) *(u32x4 *)(vt + (i * RPL + lane / PPR) * VSTRIDE + (lane % PPR) * 16) = vv[i];
                if (APPENDS && jnew >= r0 && jnew < r0 + TR && lane < PPR) {  // this tile holds the new row
                    if (KV8) {  // rounded to codes as the append kernel rounds it
                        knew = quantize16<DT>(knew, knew2);
                        vnew = quantize16<DT>(vnew, vnew2);
                    }
                    __builtin_amdgcn_wave_barrier();
                    *(u32x4 *)(kt + (jnew - r0) * KSTRIDE + lane * 16) = knew;
                    *(u32x4 *)(vt + (jnew - r0) * VSTRIDE + lane * 16) = vnew;
                    if (qb == 0) {  // append it
                        const int64_t at = (now.off + jnew) * rstride + head_byte + lane * 16;
                        *(u32x4 *)(a.kplane + at) = knew;
                        *(u32x4 *)(a.vplane + at) = vnew;
                    }
                }
                __builtin_amdgcn_wave_barrier();
                if constexpr (GQ > 0) lds_exchange();
            };
            auto reduce_tile = [&](int r0) {
                const int end = now.len;
                float sv[RB][4], mt = -INFINITY;
#pragma unroll
                for (int rb = 0; rb < RB; rb++) {
                    // (several short chains of products, added pairwise: a dot product's rounding, and its latency)
                    f32x4 sc[CH];
#pragma unroll
                    for (int c = 0; c < CH; c++) sc[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int j = 0; j < NK; j++) {
                        const u32x4 raw = *(const u32x4 *)(kt + (rb * 16 + n) * KSTRIDE + j * 64 + g * 16);
                        if (KV8) {
#pragma unroll
                            for (int half = 0; half < 2; half++) {
                                u32x4 kk;
#pragma unroll
                                for (int w = 0; w < 2; w++) {
                                    const unsigned word = raw[half * 2 + w];
                                    kk[2 * w] = widen2_e4m3<DT>(word, false);
                                    kk[2 * w + 1] = widen2_e4m3<DT>(word, true);
                                }
                                const int ks = 2 * j + half;
                                sc[ks % CH] = mfma_scores<DT>(kk, qop[ks < KS ? ks : 0], sc[ks % CH]);
                            }
                        } else {
                            sc[j % CH] = mfma_scores<DT>(raw, qop[j], sc[j % CH]);
                        }
                    }
#pragma unroll
                    for (int c = CH / 2; c > 0; c /= 2)
#pragma unroll
                        for (int k = 0; k < c; k++) sc[k] += sc[k + c];
                    const f32x4 s = sc[0];
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        sv[rb][i] = (r0 + rb * 16 + 4 * g + i < end) ? s[i] * a.scale_log2e : -INFINITY;
                        mt = fmaxf(mt, sv[rb][i]);
                    }
                }
                mt = max_over_rows(mt);
                // Lazy reference: m is the exponent reference of the running sums, not necessarily the
                // running maximum.  It moves (and the accumulators are rescaled) only when a tile's
                // maximum exceeds it by more than RESCALE_LOG2, so p stays below 2^RESCALE_LOG2 and the
                // rescale, which would otherwise run for almost every tile, runs for the first tile and
                // then hardly ever.  (max, sum, row) leave the kernel consistent with whatever m is, which
                // is all the merge of pieces needs.  (GQ: the running maximum itself, so that no weight exceeds 1 and sums
                // overflow no earlier than the vector-ALU kernel's; there is little to rescale.)
                const bool move = mt > m + RESCALE_LOG2;  // first tile: m = -inf
                if (__builtin_amdgcn_ballot_w64(move) != 0) {
                    const float mn = move ? mt : m;
                    const float alpha = move ? fast_exp2(m - mn) : 1.f;  // 0 on the first tile
                    lsum *= alpha;
                    if constexpr (GQ > 0) {
#pragma unroll
                        for (int h = 0; h < GQ; h++) {
                            const float f = lane_value(alpha, h);
#pragma unroll
                            for (int e = 0; e < 8; e++) acc[h][e] *= f;
                        }
                    } else {
#pragma unroll
                        for (int db = 0; db < DB; db++) o[db] *= alpha;
                    }
                    m = mn;
                }
                const float ref = exp_reference(m);
                if constexpr (GQ > 0) {
                    // All of it is fp32: a weight keeps its 24 bits however small it is, and an infinite value gives an
                    // infinite element (a 16-bit part of a weight that is 0 or negative would make it NaN).
                    // A lane sums the rows whose weights its sixteen lanes hold (lane h of them those of head h, rows 4g .. 4g+3
                    // of each block), so that the weights come by a broadcast within the sixteen: at D 64 eight lanes
                    // take either block's four rows, at D 256 two sixteens exchange their weights and share eight rows.
                    float p[RB][4];
#pragma unroll
                    for (int rb = 0; rb < RB; rb++) {
#pragma unroll
                        for (int i = 0; i < 4; i++) p[rb][i] = fast_exp2(sv[rb][i] - ref);
                        lsum += (p[rb][0] + p[rb][1]) + (p[rb][2] + p[rb][3]);
                    }
                    float w[GQ][NL];
#pragma unroll
                    for (int h = 0; h < GQ; h++) {
#pragma unroll
                        for (int i = 0; i < 4; i++) {
                            const float own = head_weight<0xF>(p[0][i], p[0][i], h);
                            if constexpr (D == 256) {
                                const auto both = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, own), __builtin_bit_cast(unsigned, own), false, false);
                                const unsigned even = both[0], odd = both[1];
                                w[h][i] = __builtin_bit_cast(float, even);
                                w[h][NL - 4 + i] = __builtin_bit_cast(float, odd);
                            } else {
                                w[h][i] = D == 64 ? head_weight<0xC>(own, p[RB - 1][i], h) : own;
                            }
                        }
                    }
                    const int row = D == 64 ? ((lane >> 3) & 1) * 16 + 4 * g : NL * (lane / PPR);
                    float sum[GQ][8];  // of this tile: the long sums are rounded once a tile
#pragma unroll
                    for (int h = 0; h < GQ; h++)
#pragma unroll
                        for (int e = 0; e < 8; e++) sum[h][e] = 0.f;
#pragma unroll
                    for (int i = 0; i < NL; i++) {
                        const u32x4 v = *(const u32x4 *)(vt + (row + i) * VSTRIDE + (lane % PPR) * 16);
#pragma unroll
                        for (int h = 0; h < GQ; h++) axpy8<DT>(sum[h], w[h][i], v);
                    }
#pragma unroll
                    for (int h = 0; h < GQ; h++)
#pragma unroll
                        for (int e = 0; e < 8; e++) acc[h][e] += sum[h][e];
                    lds_exchange();
                    return;
                }
                // The weights enter the second product as 16-bit operands: a high part (p rounded to the type) and
                // a low part (what the high part misses, rounded again), two products per value block.  Together
                // they carry about twice the type's mantissa, so the weighted sum is as exact as the fp32 weights
                // allow, also for values of large magnitude (one rounded part alone is off by 2^-12 of |p v|).
                // Contraction slots of lane group g: rows 4g .. 4g+3 of each row block.
                unsigned hi[2 * RB], lo[2 * RB];
#pragma unroll
                for (int rb = 0; rb < RB; rb++) {
                    float p[4], r[4];
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        p[i] = fast_exp2(sv[rb][i] - ref);
                        lsum += p[i];
                        r[i] = DT == S3_F16 ? p[i] - (float)(_Float16)p[i] : p[i] - (float)(__bf16)p[i];
                    }
#pragma unroll
                    for (int i = 0; i < 2; i++) {
                        hi[2 * rb + i] = DT == S3_F16 ? pack_f16(p[2 * i], p[2 * i + 1]) : pack_bf16(p[2 * i], p[2 * i + 1]);
                        lo[2 * rb + i] = DT == S3_F16 ? pack_f16(r[2 * i], r[2 * i + 1]) : pack_bf16(r[2 * i], r[2 * i + 1]);
                    }
                }

                if (KV8) {
                    // Four products at a time: this lane's operand row m = n of products 4q .. 4q+3 is output element
                    // d = 64q + 4n + j (j = 0..3), four consecutive codes = ONE 32-bit word per cached row; the words of
                    // rows 4g .. 4g+3 are transposed in registers into the four operands (codes of four rows at one d).
#pragma unroll
                    for (int q4 = 0; q4 < DB / 4; q4++) {
                        unsigned w[RB][4];
#pragma unroll
                        for (int rb = 0; rb < RB; rb++) {
                            const unsigned *src = (const unsigned *)(vt + (rb * 16 + 4 * g) * VSTRIDE + q4 * 64) + n;
                            transpose4x4_bytes(src[0], src[VSTRIDE / 4], src[2 * (VSTRIDE / 4)], src[3 * (VSTRIDE / 4)], w[rb]);
                        }
#pragma unroll
                        for (int j = 0; j < 4; j++) {
                            unsigned vop[2 * RB];
#pragma unroll
                            for (int rb = 0; rb < RB; rb++) {
                                vop[2 * rb] = widen2_e4m3<DT>(w[rb][j], false);
                                vop[2 * rb + 1] = widen2_e4m3<DT>(w[rb][j], true);
                            }
                            o[4 * q4 + j] = mfma_weights<DT, RB>(vop, hi, lo, o[4 * q4 + j]);
                        }
                    }
                } else {
                    const char *src = vt + (4 * g + (n >> 2)) * VSTRIDE + (n & 3) * 8;
#pragma unroll
                    for (int db = 0; db < DB; db++) {
                        unsigned vop[2 * RB];
#pragma unroll
                        for (int rb = 0; rb < RB; rb++) {
                            const u32x2 v4 = lds_transpose4(src + rb * 16 * VSTRIDE + db * 32);
                            vop[2 * rb] = v4[0];
                            vop[2 * rb + 1] = v4[1];
                        }
                        o[db] = mfma_weights<DT, RB>(vop, hi, lo, o[db]);
                    }
                }
                __builtin_amdgcn_wave_barrier();
            };
            // The share's part of context `now` is done: its rows go through the tile buffers (free between tiles) into
            // whole rows, and from there out as final rows (the whole context was here), to memory as a piece (counted
            // and, by whoever is last, merged at the end of a share), or, in a team, to the wave's buffer of first pieces
            // or nowhere: the last piece of a share stays where it is.
            auto leave = [&]() {
                lsum = sum_over_rows(lsum);
                const bool whole = t_begin <= now.t0 && now.t_end == now.t1;
                const bool to_lds = !whole && (CHUNKS || team == 4);
                const float f = whole ? 1.f / lsum : 1.f;
                __builtin_amdgcn_wave_barrier();
                float *sums = last_piece + GQ * PSTRIDE;  // (GQ)
                if constexpr (GQ > 0) {
#pragma unroll
                    for (int h = 0; h < GQ; h++) {
                        float *dst = sums + ((lane / PPR) * GQ + h) * D + (lane % PPR) * 8;
                        *(f32x4 *)dst = (f32x4){acc[h][0], acc[h][1], acc[h][2], acc[h][3]};
                        *(f32x4 *)(dst + 4) = (f32x4){acc[h][4], acc[h][5], acc[h][6], acc[h][7]};
                    }
                    lds_exchange();
                } else if (head_ok) {
#pragma unroll
                    for (int i = 0; i < DB; i++) {
                        // 16-bit rows: accumulator block t holds elements 16t + 4g + i (i = 0..3).  8-bit rows (see the V
                        // product): register i of blocks 4q .. 4q+3 holds elements 64q + 16g + 4i + j.
                        const int q4 = i / 4, j = i % 4;
                        const f32x4 v = KV8 ? (f32x4){o[4 * q4][j], o[4 * q4 + 1][j], o[4 * q4 + 2][j], o[4 * q4 + 3][j]} : o[i];
                        *(f32x4 *)(last_piece + n * PSTRIDE + (KV8 ? q4 * 64 + 16 * g + 4 * j : i * 16 + 4 * g)) = v * f;
                    }
                }
                __builtin_amdgcn_wave_barrier();
                const int slot = 2 * wave + (now.t_end == t_stop ? 1 : 0);
                const int64_t row0 = (int64_t)(whole ? now.seq : per > 0 ? pub : pub + now.seq) * a.Hq + hq0;
                if (to_lds) {
                    if (head_ok && g == 0) piece_ml[slot][n] = make_float2(m, lsum);
                    if (lane == 0) piece_b[slot] = now.seq;
                } else if (!whole) {
                    if (head_ok && g == 0) put_partial2<true>((float *)a.part_ml + 2 * (row0 + n), (f32x2){m, lsum});
                    int first = pub - chunk - seq, count = nchunks;  // (slot of the first piece: first + seq)
                    if (per == 0) pieces_of(sp, now.t0, now.t1, first, count);
                    if (pend0.count == 0) pend0 = Pending{now.seq, first, count};
                    else pend1 = Pending{now.seq, first, count};
                }
                if (GQ > 0 || !(to_lds && (slot & 1))) {
#pragma unroll 1
                    for (int e = lane; e < nheads * (D / 4); e += 64) {
                        const int h = e / (D / 4), d = (e % (D / 4)) * 4;
                        f32x4 v;
                        if constexpr (GQ > 0) {
                            f32x4 part[RPL];
#pragma unroll
                            for (int r = 0; r < RPL; r++) part[r] = *(const f32x4 *)(sums + (r * GQ + h) * D + d);
#pragma unroll
                            for (int r = RPL / 2; r > 0; r /= 2)
#pragma unroll
                                for (int k = 0; k < r; k++) part[k] += part[k + r];
                            v = part[0];
                            float by = lane_value(f, 0);
#pragma unroll
                            for (int k = 1; k < GQ; k++) by = h == k ? lane_value(f, k) : by;
                            v *= by;
                        } else {
                            v = *(const f32x4 *)(last_piece + h * PSTRIDE + d);
                        }
                        if (GQ > 0 && to_lds && (slot & 1)) *(f32x4 *)(last_piece + h * PSTRIDE + d) = v;
                        else if (to_lds) *(f32x4 *)(first_piece + h * PSTRIDE + d) = v;
                        else if (whole) store_out4(a.out, a.out_dtype, row0 * D + 4 * e, v);
                        else put_partial4<true>(a.part_acc + row0 * D + 4 * e, v);
                    }
                }
                __builtin_amdgcn_wave_barrier();
            };

            // One register set: into LDS, refill it, reduce the tile, close the context if that was its last one.  The loop has ONE
            // exit, at its bottom, and every trip issues the same loads in the same order (past the end of the share a
            // half only waits for its set): the compiler derives how many loads may stay in flight at each wait from all
            // paths that reach it.
            auto half = [&](u32x4 (&kk)[NL], u32x4 (&vv)[NL]) {
                const bool rows = t < t_stop;
                if (rows) {
                    stage_tile((t - now.t0) * TR, kk, vv);
                } else {
#pragma unroll
                    for (int i = 0; i < NL; i++) asm volatile("" ::"v"(kk[i]), "v"(vv[i]));
                }
                load_tile(kk, vv);  // the set is in LDS: its next rows leave before this tile's products
                if (rows) {
                    reduce_tile((t - now.t0) * TR);
                    t++;
                    if (t == now.t_end) {
                        leave();
                        if (t < t_stop) {
                            now = open(now.seq + 1, t);
                            enter();
                        }
                    }
                }
            };
            u32x4 k0[NL], v0[NL], k1[NL], v1[NL];
            load_tile(k0, v0);
            enter();
            if (TWO_SETS) load_tile(k1, v1);
            do {
                half(k0, v0);
                if (TWO_SETS) half(k1, v1);
            } while (t < t_stop);
        }
        if (CHUNKS || team == 4) {
            __syncthreads();  // the pieces are in LDS
            if (CHUNKS || per > 0) {
                // The parts of one chunk, left where each wave wrote its last piece; waves 0 .. k-1 had rows.
                const int k = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < NW && piece_b[2 * (lane & (NW - 1)) + 1] >= 0));
                if (k > 1 || nchunks > 1) {
                    if constexpr (D == 256 && NW == 8 && GQ == 0) {
                        // More than a quad of elements a thread: two of one head, whose weights serve both (sixteen heads of 256: one
                        // context of 900 .. 1000 rows 12.24 -> 12.05 us, with 8-bit rows 11.70 -> 11.44).  With heads of several
                        // groups in one tile the division by a variable cost more than it gave (6 / 3 heads: +0.7 %).
                        const bool pairs = nheads > 8;
                        const int log_step = pairs ? 5 : 6;
#pragma unroll 1
                        for (int e = threadIdx.x; e < nheads << log_step; e += NW * 64) {
                            const int h = e >> log_step, d = (e & ((1 << log_step) - 1)) * 4;
                            float m = -INFINITY, l = 0.f;
                            float2 x[NW];
#pragma unroll
                            for (int w = 0; w < NW; w++) {
                                x[w] = w < k ? piece_ml[2 * w + 1][h] : make_float2(-INFINITY, 0.f);
                                m = fmaxf(m, x[w].x);
                            }
                            const float ref = exp_reference(m);
                            f32x4 o[2] = {(f32x4){0.f, 0.f, 0.f, 0.f}, (f32x4){0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                            for (int w = 0; w < NW; w++) {
                                if (w >= k) break;
                                const float wt = fast_exp2(x[w].x - ref);
                                l += wt * x[w].y;
                                const float *src = (const float *)wave_lds[w] + h * PSTRIDE + d;
                                o[0] += wt * *(const f32x4 *)src;
                                if (pairs) o[1] += wt * *(const f32x4 *)(src + D / 2);
                            }
#pragma unroll
                            for (int i = 0; i < 2; i++) {
                                if (i > 0 && !pairs) break;
                                const int at = d + i * (D / 2);
                                if (nchunks == 1) {
                                    store_out4(a.out, a.out_dtype, ((int64_t)seq * a.Hq + hq0 + h) * D + at, o[i] * (1.f / l));
                                } else {
                                    const int64_t pi = (int64_t)pub * a.Hq + hq0 + h;
                                    if (at == 0) put_partial2<true>((float *)a.part_ml + 2 * pi, (f32x2){m, l});
                                    put_partial4<true>(a.part_acc + pi * D + at, o[i]);
                                }
                            }
                        }
                    } else {
#pragma unroll 1
                        for (int e = threadIdx.x; e < nheads * (D / 4); e += NW * 64) {
                            const int h = e / (D / 4), d = (e % (D / 4)) * 4;
                            float m = -INFINITY, l = 0.f;
                            float2 x[NW];
#pragma unroll
                            for (int w = 0; w < NW; w++) {
                                x[w] = w < k ? piece_ml[2 * w + 1][h] : make_float2(-INFINITY, 0.f);
                                m = fmaxf(m, x[w].x);
                            }
                            const float ref = exp_reference(m);
                            f32x4 o = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                            for (int w = 0; w < NW; w++) {
                                if (w >= k) break;
                                const float wt = fast_exp2(x[w].x - ref);
                                l += wt * x[w].y;
                                o += wt * *(const f32x4 *)((const float *)wave_lds[w] + h * PSTRIDE + d);
                            }
                            if (nchunks == 1) {
                                store_out4(a.out, a.out_dtype, ((int64_t)seq * a.Hq + hq0) * D + 4 * e, o * (1.f / l));
                            } else {
                                const int64_t pi = (int64_t)pub * a.Hq + hq0 + h;
                                if (d == 0) put_partial2<true>((float *)a.part_ml + 2 * pi, (f32x2){m, l});
                                put_partial4<true>(a.part_acc + pi * D + d, o);
                            }
                        }
                    }
                    if (nchunks > 1) pend0 = Pending{seq, pub - chunk - seq, nchunks};
                }
            } else if constexpr (!CHUNKS) {
                // Pieces of one context are neighbours: a run.  First the weight of every piece and the sum of every run ...
                const int pb = piece_b[lane & 7];
                int first8 = 0, count8 = 0;  // lane k: the publishing units of piece k's context
                if (pb >= 0) pieces_of(sp, bv.pre[pb], bv.pre[pb + 1], first8, count8);
                if (threadIdx.x < 128) {
                    const int k = threadIdx.x >> 4, h = threadIdx.x & 15;
                    const int mine = piece_b[k];
                    const float2 me = piece_ml[k][h];
                    float2 x[8];
#pragma unroll
                    for (int j = 0; j < 8; j++) x[j] = piece_ml[j][h];
                    float m = me.x, l = 0.f;
#pragma unroll
                    for (int j = 0; j < 8; j++)
                        if (__builtin_amdgcn_readlane(pb, j) == mine) m = fmaxf(m, x[j].x);
                    const float ref = exp_reference(m);
#pragma unroll
                    for (int j = 0; j < 8; j++)
                        if (__builtin_amdgcn_readlane(pb, j) == mine) l += fast_exp2(x[j].x - ref) * x[j].y;
                    if (mine >= 0) piece_run[k][h] = (f32x4){fast_exp2(me.x - ref), m, l, 1.f / l};
                }
                __syncthreads();
                // ... then the rows, all threads together, every thread EB quads of elements at once
                constexpr int EB = D / 64;
                int h[EB], d[EB];
#pragma unroll
                for (int i = 0; i < EB; i++) {
                    const int e = min((int)threadIdx.x + i * 256, nheads * (D / 4) - 1);
                    h[i] = e / (D / 4);
                    d[i] = (e % (D / 4)) * 4;
                }
#pragma unroll 1
                for (int k = 0; k < 8;) {
                    const int b = __builtin_amdgcn_readlane(pb, k);
                    if (b < 0) {
                        k++;
                        continue;
                    }
                    const int first = __builtin_amdgcn_readlane(first8, k), count = __builtin_amdgcn_readlane(count8, k);
                    f32x4 o[EB], r[EB];
#pragma unroll
                    for (int i = 0; i < EB; i++) o[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                    for (; k < 8; k++) {
                        const int kb = __builtin_amdgcn_readlane(pb, k);
                        if (kb < 0) continue;
                        if (kb != b) break;
                        const float *src = (k & 1) ? (const float *)wave_lds[k >> 1] : first_piece + ((k >> 1) - wave) * piece_heads * PSTRIDE;
#pragma unroll
                        for (int i = 0; i < EB; i++) {
                            r[i] = piece_run[k][h[i]];
                            o[i] += r[i][0] * *(const f32x4 *)(src + h[i] * PSTRIDE + d[i]);
                        }
                    }
#pragma unroll
                    for (int i = 0; i < EB; i++) {
                        if ((int)threadIdx.x + i * 256 >= nheads * (D / 4)) continue;
                        if (count == 1) {
                            store_out4(a.out, a.out_dtype, ((int64_t)b * a.Hq + hq0 + h[i]) * D + d[i], o[i] * r[i][3]);
                        } else {
                            const int64_t pi = (int64_t)(pub + b) * a.Hq + hq0 + h[i];
                            if (d[i] == 0) put_partial2<true>((float *)a.part_ml + 2 * pi, (f32x2){r[i][1], r[i][2]});
                            put_partial4<true>(a.part_acc + pi * D + d[i], o[i]);
                        }
                    }
                    if (count > 1) {
                        if (pend0.count == 0) pend0 = Pending{b, first, count};
                        else pend1 = Pending{b, first, count};
                    }
                }
            }
            if (pend0.count != 0) {  // uniform over the workgroup
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // every wave's stores are at the memory side ...
                __syncthreads();                                            // ... before one of them counts the pieces
                if (wave == 0) {
                    const unsigned mine = pieces_arrived(a, pend0, pend1, columns, col);
                    if (lane == 0) merge_mine = (int)mine;
                }
                __syncthreads();
                const int mine = __builtin_amdgcn_readfirstlane(merge_mine);
#pragma unroll 1
                for (int k = 0; k < 2; k++)
                    if ((mine >> k) & 1) merge_pieces<D, CHUNKS>(a, k ? pend1 : pend0, hq0, nheads, threadIdx.x, NW * 64, (float *)wave_lds);
            }
            if (!LOOP) break;
            __syncthreads();  // LDS is free for the next unit
        } else if constexpr (!CHUNKS) {
            if (pend0.count != 0 || pend1.count != 0) {
                const unsigned mine = pieces_arrived(a, pend0, pend1, columns, col);
#pragma unroll 1
                for (int k = 0; k < 2; k++)
                    if ((mine >> k) & 1) merge_pieces<D, false>(a, k ? pend1 : pend0, hq0, nheads, lane, 64, nullptr);
            }
            if (!LOOP) break;
        }
    }
    // What belongs to no row, behind the work: the new lengths (the last workgroup has none in a launch of few rows) ...
    if (a.len_out && blockIdx.x == gridDim.x - 1) {
        for (int b = threadIdx.x; b < a.n; b += NW * 64) a.len_out[b] = a.cur_len[b] + 1;
    }
    // ... and the zero rows of empty or refused contexts, by the workgroups in turn
#pragma unroll 1
    for (int b = blockIdx.x; b < a.n; b += gridDim.x) {
        if (bv.len[b] == 0) {
            const float z[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            for (int e = threadIdx.x; e < a.Hq * D / 8; e += NW * 64) store_out8(a.out, a.out_dtype, ((int64_t)b * a.Hq * D / 8 + e) * 8, z);
        }
    }
}

// Two or three query heads per cached head, 16-bit rows.  The vector-ALU kernel, which serves these where it is faster
// (gqa_on_matrix_cores), keeps the weights in fp32, and so does this one: only the scores are a matrix product (2 or 3 of its
// 16 columns in use), the weighted rows are 2 or 3 multiply-adds an element on the vector ALU, far below what it could issue
// while the rows arrive.  Weights in 16-bit parts on the matrix cores lose what the smallest of them carry (three fp16 parts
// end at 2^-31 of the largest weight: a value of 6e4 under a weight of e^-14 off by 1e-5) and make infinite values NaN; they
// were up to 5 % faster with three heads at 64 and 128 elements a head, level or slower elsewhere.
// Error against 64 bits, relative 2-norm, fp32 outputs, 16q/8kv x 128, 64q/32kv x 128, 16q/8kv x 64, 6q/3kv x 256, 24q/8kv x
// 64, 12q/4kv x 128, 9q/3kv x 256, 8 to 85 contexts: bf16 1.33e-7 to 1.54e-7 where the vector ALU has 1.58e-7 to 1.82e-7, fp16
// 1.38e-7 to 1.61e-7 and 1.66e-7 to 1.85e-7; one context of 37 rows level (bf16 1.11e-7 to 1.37e-7, 1.13e-7 to 1.37e-7).
template <int DT, int NW, bool LOOP>
static attn_fn pick_few_heads(int d, int group) {
    if (d == 64) return group == 2 ? attn_gqa_mfma_kernel<DT, 64, false, NW, 2, LOOP> : attn_gqa_mfma_kernel<DT, 64, false, NW, 3, LOOP>;
    if (d == 128) return group == 2 ? attn_gqa_mfma_kernel<DT, 128, false, NW, 2, LOOP> : attn_gqa_mfma_kernel<DT, 128, false, NW, 3, LOOP>;
    if (d == 256) return group == 2 ? attn_gqa_mfma_kernel<DT, 256, false, NW, 2, LOOP> : attn_gqa_mfma_kernel<DT, 256, false, NW, 3, LOOP>;
    return nullptr;
}
template <int DT>
static attn_fn pick_few_heads(int d, int group, bool wide, bool loop) {
    return wide ? pick_few_heads<DT, 8, false>(d, group) : loop ? pick_few_heads<DT, 4, true>(d, group) : pick_few_heads<DT, 4, false>(d, group);
}
attn_fn s3i_pick_gqa_few_heads(int dt, int d, int group, bool wide, bool loop) {
    return dt == S3_F16 ? pick_few_heads<S3_F16>(d, group, wide, loop) : pick_few_heads<S3_BF16>(d, group, wide, loop);
}

// act: the type of q (and of the rows, unless they are e4m3: kv8).
template <int ACT, int NW, bool LOOP>
static attn_fn pick_waves(int d, bool kv8) {
    if (d == 64) return kv8 ? attn_gqa_mfma_kernel<ACT, 64, true, NW, 0, LOOP> : attn_gqa_mfma_kernel<ACT, 64, false, NW, 0, LOOP>;
    if (d == 128) return kv8 ? attn_gqa_mfma_kernel<ACT, 128, true, NW, 0, LOOP> : attn_gqa_mfma_kernel<ACT, 128, false, NW, 0, LOOP>;
    if (d == 256) return kv8 ? attn_gqa_mfma_kernel<ACT, 256, true, NW, 0, LOOP> : attn_gqa_mfma_kernel<ACT, 256, false, NW, 0, LOOP>;
    return nullptr;
}
template <int ACT>
static attn_fn pick_waves(int d, bool kv8, bool wide, bool loop) {
    return wide ? pick_waves<ACT, 8, false>(d, kv8) : loop ? pick_waves<ACT, 4, true>(d, kv8) : pick_waves<ACT, 4, false>(d, kv8);
}
attn_fn s3i_pick_gqa_mfma(int act, int d, bool kv8, bool wide, bool loop) {
    return act == S3_F16    ? pick_waves<S3_F16>(d, kv8, wide, loop)
           : act == S3_BF16 ? pick_waves<S3_BF16>(d, kv8, wide, loop) : nullptr;
}
