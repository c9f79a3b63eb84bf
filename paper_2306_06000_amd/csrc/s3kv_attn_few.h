// Attention over few contexts of a multi-head cache, 16-bit rows or (KV8) e4m3 codes, gfx950.  Included by s3kv_attn_inst.hip (one translation unit
// per head dimension).
//
// A launch of few rows is a chain of latencies, and most of it instructions that run once.  attn_step_kernel spent, on one
// context of 1450 rows (16 x 256 fp16, MI355X, us from the launch's start): 1.8 until the batch view stood in LDS, 2.7 until a
// workgroup knew its item, 7.9 with its rows (a wave's fifteen in four dependent rounds), 9.9 when the chunk was counted and 12.7
// when one wave had merged twelve pieces.  This one: 1.7 until a workgroup knows its chunk, 5.1 with its rows, 6.7 counted, 8.7 merged.  Here:
//   * one item a workgroup, no loop around it, hence no invariants computed (and spilled) in front of it; the view stays in
//     every wave's registers (lane b: context b) and the item is found by a ballot and lane reads, without LDS or a barrier;
//   * all arguments in one round trip (read where they were used, they cost one each): 0.3 us;
//   * up to twelve rows a wave, all loads leave at once; no load past the share's end but to fill a four (a wave's 16-byte
//     load takes 16 clocks of the unit's L1 whether or not it brings anything);
//   * all eight waves take part in both meetings, of the shares in LDS and of the pieces: two waves take every fourth piece;
//   * the arrival counters are a cache line apart (neighbours in one line, the atomics of 200 workgroups took up to 2.5 us).
// us a layer, attn_step_kernel and this: 16 x 256 fp16, 1 context of 30..40 rows 5.7, 3.9; of 300..400 9.2, 6.6; of 1400..1500
// 12.9, 9.5; of 8000 28.1, 26.1; 4 of 17..128 9.5, 6.6; 4 of 500..1500 17.4, 16.2; 16 of 32..1000 28.1, 26.8; 12 x 128 bf16, 1
// of 1400..1500 12.4, 8.5, 24 of 32..1000 18.1, 17.2; 64 x 96 bf16, 1 of 300..400 9.8, 7.1, 12 of 32..1000 30.2, 31.7 (the
// most it loses, see on_few_kernel); 3 x 128, 8 of 500..1500 12.0, 7.8.  e4m3 rows (attn_fp8_kernel, whose one wave of eight combines a chunk while
// the others wait): 16 x 256, 1 of 300..400 13.9, 7.9, of 8000 32.9, 19.4, 8 of 32..1000 17.8, 11.9, 40 of 32..1000 39.0, 34.9; 12 x 128,
// 4 of 17..128 12.6, 7.0.
#pragma once
#include <type_traits>

#include "s3kv_attn.h"

// Lanes of a wave load: a lane holds 16 bytes of a row, EL elements, LPH lanes a head (USED of them in use), GH heads a load.
template <int D, bool KV8>
struct FewLanes {
    static constexpr int EL = KV8 ? 16 : 8, USED = D / EL, LPH = KV8 ? D / 16 : HeadLanes<D>::LPH, GH = 64 / LPH;
};

// A wave's share of a chunk's rows, for one head group.  DT: the type of q (and of the rows, but for KV8).
template <int DT, int D, bool KV8>
struct FewRows {
    typedef FewLanes<D, KV8> HL;
    static constexpr int EL = HL::EL;
    const char *kb, *vb;      // the share's first row, this head group (wave-uniform)
    const char *knew, *vnew;  // the new row, and whether it is the share's last one (KV8: it is not in `rows`)
    bool fresh;
    int64_t rstride;
    unsigned rs32, tail;      // (tail: bytes of a row in front of this head group)
    unsigned lane_byte;       // this lane's bytes of a row
    int rows;                 // rows of the share
    float scale_log2e;
    u32x4 qv;                 // (16-bit rows)
    float qf[KV8 ? 16 : 1];   // (KV8: q, scaled)

    __device__ __forceinline__ float dot(const u32x4 k) const {
        if constexpr (!KV8) return dot8<DT>(qv, k);
        float d = 0.f;
#pragma unroll
        for (int w = 0; w < 4; w++) {
            float f[4];
            const unsigned word = k[w];
            widen4_e4m3(word, f);
#pragma unroll
            for (int e = 0; e < 4; e++) d = fmaf(qf[KV8 ? 4 * w + e : 0], f[e], d);
        }
        return d;
    }
    __device__ __forceinline__ void axpy(float (&acc)[EL], const float p, const u32x4 v) const {
        if constexpr (!KV8) {
            axpy8<DT>(acc, p, v);
        } else {
#pragma unroll
            for (int w = 0; w < 4; w++) {
                float f[4];
                const unsigned word = v[w];
                widen4_e4m3(word, f);
#pragma unroll
                for (int e = 0; e < 4; e++) acc[4 * w + e] = fmaf(p, f[e], acc[4 * w + e]);
            }
        }
    }

    // Rows j .. j+U-1: zeros (and no traffic) past the share's end.
    template <int U>
    __device__ __forceinline__ void load(int j, u32x4 *kk, u32x4 *vv) const {
        const int left = min(rows - j, U);
        const char *kp = kb + j * rstride, *vp = vb + j * rstride;
        if (!KV8 && __builtin_expect(fresh && left > 0 && j + left == rows, 0)) {  // the last row is the new one
#pragma unroll
            for (int u = 0; u < U; u++) {
                const bool it = u == left - 1;
                const int bytes = u < left ? (int)((unsigned)(u + 1) * rs32 - tail) : 0;
                kk[u] = __builtin_amdgcn_raw_buffer_load_b128(rows_of(it ? knew - u * (int64_t)rs32 : kp, bytes), lane_byte + u * rs32, 0, 2);
                vv[u] = __builtin_amdgcn_raw_buffer_load_b128(rows_of(it ? vnew - u * (int64_t)rs32 : vp, bytes), lane_byte + u * rs32, 0, 2);
            }
            return;
        }
        const int bytes = left > 0 ? (int)((unsigned)left * rs32 - tail) : 0;
        const __amdgpu_buffer_rsrc_t krs = rows_of(kp, bytes), vrs = rows_of(vp, bytes);
#pragma unroll
        for (int u = 0; u < U; u++) kk[u] = __builtin_amdgcn_raw_buffer_load_b128(krs, lane_byte + u * rs32, 0, 2);
#pragma unroll
        for (int u = 0; u < U; u++) vv[u] = __builtin_amdgcn_raw_buffer_load_b128(vrs, lane_byte + u * rs32, 0, 2);
    }
    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_of(const char *p, int bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p), 0, bytes, 0x00020000);
    }

    // `count` of N rows (or more than N: all).
    template <int N>
    __device__ __forceinline__ void reduce(int count, const u32x4 *kk, const u32x4 *vv, float &m, float &l, float (&acc)[EL]) const {
        float s[N], mb = -INFINITY;
#pragma unroll
        for (int u = 0; u < N; u++) s[u] = dot(kk[u]);
#pragma unroll
        for (int u = 0; u < N; u++) s[u] = group_sum<HL::LPH>(s[u]);
#pragma unroll
        for (int u = 0; u < N; u++) {
            s[u] = u < count ? KV8 ? s[u] : s[u] * scale_log2e : -INFINITY;
            mb = fmaxf(mb, s[u]);
        }
        const float mn = fmaxf(m, mb), ref = exp_reference(mn), alpha = fast_exp2(m - ref);
        l *= alpha;
#pragma unroll
        for (int i = 0; i < EL; i++) acc[i] *= alpha;
#pragma unroll
        for (int u = 0; u < N; u++) {
            const float p = fast_exp2(s[u] - ref);
            l += p;
            axpy(acc, p, vv[u]);
        }
        m = mn;
    }
};

// Two workgroups a compute unit (128 registers).  A share beyond sixteen (twelve) rows is walked with two sets of two rows, alternately
// (three at 96 elements a head, whose loads bring 12 of 16 bytes): four or eight a set, which leave room for one workgroup
// only, read level where latencies bound the launch and 5 to 20 % slower where the memory rate does (16 x 256, 8 contexts of
// 500..1500 rows: 24.7 us with two, 26.4 with four, 30.9 with eight).
template <int DT, int D, bool KV8 = false>
__global__ void __launch_bounds__(512, 4) attn_few_kernel(const AttnArgs a) {
    typedef FewLanes<D, KV8> HL;
    constexpr int LPH = HL::LPH, USED = HL::USED, GH = HL::GH, EL = HL::EL, NW = 8, U = D == 96 ? 3 : 2;
    constexpr int ELEMS = GH * D;        // elements of a head group's output
    constexpr int EPT = (ELEMS + 511) / 512;  // ... per thread: one, KV8 two
    __shared__ __align__(16) float comb[NW][ELEMS];
    __shared__ float2 comb_ml[NW][GH];
    __shared__ int last_here;

    // All arguments in one round trip: read where they are used, they cost one each, out of a cold scalar cache.
    asm volatile("" ::"s"(a.kplane), "s"(a.vplane), "s"(a.q), "s"(a.slot_off), "s"(a.cur_len), "s"(a.out), "s"(a.part_acc), "s"(a.part_ml),
                 "s"(a.k_new), "s"(a.v_new), "s"(a.len_out), "s"(a.arrivals), "s"(a.n_tokens), "s"(a.n), "s"(a.H), "s"(a.out_dtype),
                 "s"(a.max_len), "s"(a.len_add), "s"(a.scale_log2e), "s"(a.few_chunks), "s"(a.unit_chunks), "s"(a.columns), "s"(a.column_shift), "s"(a.merge_sync));
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = a.n, n_hg = a.columns;
    // ---- the view, in every wave's registers: lane b holds context b
    const int b = min(lane, n - 1);
    const int64_t off = a.slot_off[b];
    const int raw = a.cur_len[b];
    const int len = lane < n ? checked_len(a, off, raw) : 0;
    const int longest = wave_max_nonneg(len);
    const int total = __builtin_amdgcn_readlane(wave_inclusive_scan(len), 63);
    // As many chunks as workgroups run at once, one a compute unit, or two where a chunk would be long: contexts do not divide
    // evenly, and the launch lasts as long as its longest chunk (16 x 256, 24 contexts of 32..1000 rows: 37.5 us, 46.9 in 32
    // chunks; a single context divides evenly: of 8000 rows 25.4, in twice the chunks 26.4).
    const int units = n > 1 && total > 192 * a.few_chunks ? a.unit_chunks : a.few_chunks;
    int cnt = len > 0 ? 1 : 0, incl = 0;
    // Short contexts stay whole: a cut costs 1.6 us (write-through, count, pieces).  Up to 64 rows, or 128 where the contexts
    // take half of the units as they are (whole and cut: 16 x 256, 4 of 17..128 rows 7.8, 6.8; 64 x 96, 8 of 50..128: 8.1, 8.8).
    if (longest <= (2 * n >= units ? 128 : 64)) {
        incl = wave_inclusive_scan(cnt);
    } else {
        // No finer than sqrt(2 * longest): a chunk's rows stream side by side over eight waves, its piece adds to the merge.
        // Factor 0.1, 1, 2, 4: 12 x 128, one of 1450 rows 11.3, 9.4, 8.8, 9.6 us, of 8050 16.3, 16.3, 15.2, 18.1; 16 x 256, one
        // of 350 8.3, 8.2, 7.1, 7.0.  Half a chunk a context is allowed for to begin with; the count tells.
        const int least = max(16, (int)__builtin_amdgcn_sqrtf(2.f * (float)longest));
#pragma unroll 1
        for (int quarters = 2; quarters <= 4; quarters++) {
            const int room = max(units - ((n * quarters + 3) >> 2), 1);
            const int even = (int)((float)total * __builtin_amdgcn_rcpf((float)room) * 1.000001f) + 1;  // (not below the quotient)
            const int per = min(max(even, least), longest);
            cnt = quotient(len + per - 1, per);
            incl = wave_inclusive_scan(cnt);
            if (__builtin_amdgcn_readlane(incl, 63) <= units) break;
        }
    }
    const int chunks = __builtin_amdgcn_readlane(incl, 63);
    const int w = __builtin_amdgcn_readfirstlane(a.column_shift >= 0 ? (int)(blockIdx.x >> a.column_shift) : quotient(blockIdx.x, n_hg));
    const int hg = blockIdx.x - w * n_hg;
    if (w < chunks) {
        // ---- the chunk of this workgroup: of context `seq`, near-equal pieces, none of them empty
        const int seq = __builtin_popcountll(__builtin_amdgcn_ballot_w64(incl <= w));
        const int nchunks = __builtin_amdgcn_readlane(cnt, seq), first = __builtin_amdgcn_readlane(incl, seq) - nchunks;
        const int all = __builtin_amdgcn_readlane(len, seq), chunk = w - first;
        const int64_t row0 = (int64_t)(((uint64_t)(unsigned)__builtin_amdgcn_readlane((int)(off >> 32), seq) << 32) |
                                       (unsigned)__builtin_amdgcn_readlane((int)off, seq));
        const int base = nchunks == 1 ? all : quotient(all, nchunks), rem = all - base * nchunks;
        const int start = chunk * base + min(chunk, rem), rows = base + (chunk < rem ? 1 : 0);
        const int eighth = rows >> 3, more = rows & 7;
        const int j0 = start + wave * eighth + min(wave, more), share = eighth + (wave < more ? 1 : 0);
        const int g = lane / LPH, dl = lane % LPH;
        const int h = hg * GH + g;
        const int hc = h < a.H ? g : a.H - 1 - hg * GH, dc = dl < USED ? dl : USED - 1;  // (lanes without bytes of their own: a neighbour's)
        const int64_t rstride = (int64_t)a.H * D * (KV8 ? 1 : 2);
        const bool fresh = a.k_new && j0 + share == all && share > 0;  // the new row is this share's last one
        FewRows<DT, D, KV8> st;
        st.rstride = rstride;
        st.rs32 = (unsigned)rstride;
        st.tail = (unsigned)(hg * GH * D * (KV8 ? 1 : 2));
        const unsigned lane_byte = (unsigned)((hc * D + dc * EL) * (KV8 ? 1 : 2));
        st.lane_byte = lane_byte;
        st.kb = a.kplane + (row0 + j0) * rstride + st.tail;
        st.vb = a.vplane + (row0 + j0) * rstride + st.tail;
        st.rows = share - (KV8 && fresh ? 1 : 0);
        st.fresh = fresh;
        st.scale_log2e = a.scale_log2e;
        // q and the new row are 16-bit: this lane's elements of them
        const int64_t in_row = ((int64_t)seq * a.H + hg * GH) * D * 2;
        const unsigned in_lane = KV8 ? 2 * lane_byte : lane_byte;
        st.knew = a.k_new + in_row;
        st.vnew = a.v_new + in_row;
        u32x4 q1;
        st.qv = *(const u32x4 *)(a.q + in_row + in_lane);
        if constexpr (KV8) q1 = *(const u32x4 *)(a.q + in_row + in_lane + 16);
        // (without a branch: what two paths bring into one register is waited for where they meet)
        const int fresh_bytes = fresh ? (int)((a.H - hg * GH) * D * 2) : 0;
        const __amdgpu_buffer_rsrc_t knr = st.rows_of(st.knew, fresh_bytes), vnr = st.rows_of(st.vnew, fresh_bytes);
        u32x4 kn, vn;
        if constexpr (!KV8) {  // (KV8: below, for want of registers)
            kn = __builtin_amdgcn_raw_buffer_load_b128(knr, in_lane, 0, 0);
            vn = __builtin_amdgcn_raw_buffer_load_b128(vnr, in_lane, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < 8; i++) {
                const unsigned w = i < 4 ? st.qv[i] : q1[i - 4];
                st.qf[KV8 ? 2 * i : 0] = widen16<DT>((unsigned short)(w & 0xFFFFu)) * a.scale_log2e;
                st.qf[KV8 ? 2 * i + 1 : 0] = widen16<DT>((unsigned short)(w >> 16)) * a.scale_log2e;
            }
        }
        if (!KV8 && USED < LPH && dl >= USED) st.qv = (u32x4){0u, 0u, 0u, 0u};
        float m = -INFINITY, l = 0.f, acc[EL];
#pragma unroll
        for (int i = 0; i < EL; i++) acc[i] = 0.f;
        // Up to twelve rows (KV8: six): all of them leave at once, in fours (threes; a load past the share's end costs its issue).
        // Up to sixteen, 16-bit heads of less than 256: a second turn of four (the loop below takes four turns of memory for them;
        // us a layer, with it and this way: 12 x 128, 40 contexts of 100..200 rows 12.26, 11.34, 24 of 60..600 12.54, 11.68, 64 x 96, 8
        // of 50..128 8.85, 8.50, 16 x 64, one of 8000 13.50, 13.02, one of 4000 10.62, 10.78).  With 256 the loop is the better
        // one: 16 x 256, 9 of 300..400 13.35, 13.71.  So it is beside a second turn of up to eight: 12 x 128, 24 of 300..400 13.92,
        // 14.40.
        constexpr int FB = KV8 ? 3 : 4;
        auto few = [&](auto times, int j) {
            constexpr int F = decltype(times)::value;
            u32x4 kf[FB * F], vf[FB * F];
#pragma unroll
            for (int f = 0; f < F; f++) st.template load<FB>(j + FB * f, kf + FB * f, vf + FB * f);
#pragma unroll
            for (int f = 0; f < F; f++) st.template reduce<FB>(st.rows - j - FB * f, kf + FB * f, vf + FB * f, m, l, acc);
        };
        if (st.rows <= 2 * FB) {
            if (st.rows > FB) few(std::integral_constant<int, 2>(), 0);
            else if (st.rows > 0) few(std::integral_constant<int, 1>(), 0);
        } else if (!KV8 && st.rows <= (D == 256 ? 3 : 4) * FB) {
            few(std::integral_constant<int, KV8 ? 2 : 3>(), 0);
            if (D != 256 && st.rows > 3 * FB) few(std::integral_constant<int, 1>(), 3 * FB);
        } else {
            float m1 = -INFINITY, l1 = 0.f, acc1[EL];  // the runs before
#pragma unroll
            for (int i = 0; i < EL; i++) acc1[i] = 0.f;
            u32x4 ka[U], va[U], kb[U], vb[U];
            st.template load<U>(0, ka, va);
            st.template load<U>(U, kb, vb);
            int j = 0, turn = 128;
            while (st.rows - j > 2 * U) {
                st.template reduce<U>(U, ka, va, m, l, acc);
                st.template load<U>(j + 2 * U, ka, va);
                st.template reduce<U>(U, kb, vb, m, l, acc);
                st.template load<U>(j + 3 * U, kb, vb);
                j += 2 * U;
                if (j >= turn) {  // (runs of about 128 rows, as attn_step_kernel's longest, so that no fp32 sum is longer)
                    turn = j + 128;
                    const float mm = fmaxf(m1, m), ref = exp_reference(mm), f1 = fast_exp2(m1 - ref), f = fast_exp2(m - ref);
                    m1 = mm;
                    l1 = f1 * l1 + f * l;
#pragma unroll
                    for (int i = 0; i < EL; i++) acc1[i] = f1 * acc1[i] + f * acc[i];
                    m = -INFINITY;
                    l = 0.f;
#pragma unroll
                    for (int i = 0; i < EL; i++) acc[i] = 0.f;
                }
            }
            st.template reduce<U>(st.rows - j, ka, va, m, l, acc);
            if (j + U < st.rows) st.template reduce<U>(st.rows - j - U, kb, vb, m, l, acc);
            const float mm = fmaxf(m1, m), ref = exp_reference(mm), f1 = fast_exp2(m1 - ref), f = fast_exp2(m - ref);
            m = mm;
            l = f1 * l1 + f * l;
#pragma unroll
            for (int i = 0; i < EL; i++) acc[i] = f1 * acc1[i] + f * acc[i];
        }
        if constexpr (KV8) {  // the new row, rounded to codes as the append kernel rounds it, and attended to as they widen
            if (fresh) {
                const u32x4 k0 = __builtin_amdgcn_raw_buffer_load_b128(knr, in_lane, 0, 0), k1 = __builtin_amdgcn_raw_buffer_load_b128(knr, in_lane + 16, 0, 0);
                const u32x4 v0 = __builtin_amdgcn_raw_buffer_load_b128(vnr, in_lane, 0, 0), v1 = __builtin_amdgcn_raw_buffer_load_b128(vnr, in_lane + 16, 0, 0);
                kn = quantize16<DT>(k0, k1);
                vn = quantize16<DT>(v0, v1);
                st.template reduce<1>(1, &kn, &vn, m, l, acc);
            }
        }
        if (fresh && h < a.H && dl < USED) {  // the append
            *(u32x4 *)(const_cast<char *>(st.kb) + (share - 1) * rstride + lane_byte) = kn;
            *(u32x4 *)(const_cast<char *>(st.vb) + (share - 1) * rstride + lane_byte) = vn;
        }
        // ---- the shares meet: every thread one element of the head group's output
        if (dl < USED) {
#pragma unroll
            for (int i = 0; i < EL; i += 4) *(f32x4 *)&comb[wave][g * D + dl * EL + i] = (f32x4){acc[i], acc[i + 1], acc[i + 2], acc[i + 3]};
            if (dl == 0) comb_ml[wave][g] = make_float2(m, l);
        }
        __syncthreads();
        // (element k of this thread: tid + 512 * k of the head group's)
        const int heads = min(GH, a.H - hg * GH);
        const int64_t out0 = (int64_t)seq * a.H * D + hg * ELEMS;
        const auto combine = [&](auto parts, int e, float &top, float &sum, float &val) {
            constexpr int N = decltype(parts)::value;
            float2 x[N];
            float o[N];
            top = -INFINITY;
#pragma unroll
            for (int s = 0; s < N; s++) {
                x[s] = comb_ml[s][e / D];
                o[s] = comb[s][e];
            }
#pragma unroll
            for (int s = 0; s < N; s++) top = fmaxf(top, x[s].x);
            const float ref = exp_reference(top);
            sum = val = 0.f;
#pragma unroll
            for (int s = 0; s < N; s++) {
                const float f = fast_exp2(x[s].x - ref);
                sum += f * x[s].y;
                val += f * o[s];
            }
        };
        const int64_t p0 = (int64_t)first * a.H + hg * GH;  // the context's first piece, this group's first head
#pragma unroll
        for (int k = 0; k < EPT; k++) {
            const int e = ELEMS % 512 == 0 ? tid + 512 * k : min(tid, ELEMS - 1);
            float top, sum, val;
            combine(std::integral_constant<int, NW>(), e, top, sum, val);
            if (e / D < heads && (ELEMS % 512 == 0 || tid < ELEMS)) {
                if (nchunks == 1) {
                    store_out1(a.out, a.out_dtype, out0 + e, val / sum);
                } else {
                    const int64_t pi = p0 + (int64_t)chunk * a.H + e / D;
                    put_partial1(a.part_acc + pi * D + e % D, val);
                    if (e % D == 0) put_partial2<true>((float *)a.part_ml + 2 * pi, (f32x2){top, sum});
                }
            }
        }
        if (nchunks > 1) {
            if (a.merge_sync) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // this wave's stores are at the memory side ...
            __syncthreads();                                             // ... and all the others', before one of them counts
            if (wave == 0) {
                unsigned int *cntp = arrival_counter(a, seq, n_hg, hg);
                unsigned int old = 0;
                if (lane == 0) {
                    old = atomicAdd(cntp, 1u);
                    if (old == (unsigned)(nchunks - 1)) atomicExch(cntp, 0u);
                    last_here = old == (unsigned)(nchunks - 1);
                }
            }
            __syncthreads();
            if (last_here) {
                if (a.merge_sync) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                asm volatile("" ::: "memory");
                // A thread takes four elements of every PARTS-th piece (two waves a piece, KV8 four); the sums meet in LDS.
                constexpr int QUADS = ELEMS / 4, WIDTH = QUADS <= 128 ? 128 : 256, PARTS = 512 / WIDTH;
                const int q = min(tid & (WIDTH - 1), QUADS - 1), qh = 4 * q / D, part = __builtin_amdgcn_readfirstlane(tid / WIDTH);
                const unsigned sml = (unsigned)a.H * 8, sacc = (unsigned)a.H * D * 4;
                const float *pml = (const float *)a.part_ml + 2 * p0, *pacc = a.part_acc + p0 * D;
                float mm = -INFINITY, ll = 0.f;
                f32x4 oo = (f32x4){0.f, 0.f, 0.f, 0.f};
                auto pieces = [&](int c, auto np) {  // pieces c + part, c + part + PARTS, ..., one memory round trip
                    constexpr int NP = decltype(np)::value;
                    const int left = min(nchunks - c, PARTS * NP);
                    const __amdgpu_buffer_rsrc_t mls = piece_buffer(pml + (int64_t)c * a.H * 2, (left - 1) * sml + heads * 8);
                    const __amdgpu_buffer_rsrc_t accs = piece_buffer(pacc + (int64_t)c * a.H * D, (left - 1) * sacc + heads * D * 4);
                    f32x2 mv[NP];
                    f32x4 av[NP];
#pragma unroll
                    for (int u = 0; u < NP; u++) mv[u] = piece_load2(mls, (part + PARTS * u) * sml + 8 * qh);
#pragma unroll
                    for (int u = 0; u < NP; u++) av[u] = piece_load4(accs, (part + PARTS * u) * sacc + 16 * q);
                    float mn = mm;
#pragma unroll
                    for (int u = 0; u < NP; u++) {
                        mv[u][0] = part + PARTS * u < left ? mv[u][0] : -INFINITY;
                        mn = fmaxf(mn, mv[u][0]);
                    }
                    const float r = exp_reference(mn), al = fast_exp2(mm - r);
                    ll *= al;
                    oo *= al;
#pragma unroll
                    for (int u = 0; u < NP; u++) {
                        const float f = fast_exp2(mv[u][0] - r);
                        ll += f * mv[u][1];
                        oo += f * av[u];
                    }
                    mm = mn;
                };
                if (nchunks <= 16) pieces(0, std::integral_constant<int, 16 / PARTS>());
                else
#pragma unroll 1
                    for (int c = 0; c < nchunks; c += 8 * PARTS) pieces(c, std::integral_constant<int, 8>());
                // (the shares in comb have been read: two barriers ago)
                if ((tid & (WIDTH - 1)) < QUADS) {
                    *(f32x4 *)&comb[part][4 * q] = oo;
                    if ((4 * q) % D == 0) comb_ml[part][qh] = make_float2(mm, ll);
                }
                __syncthreads();
#pragma unroll
                for (int k = 0; k < EPT; k++) {
                    const int e = ELEMS % 512 == 0 ? tid + 512 * k : min(tid, ELEMS - 1);
                    float top, sum, val;
                    combine(std::integral_constant<int, PARTS>(), e, top, sum, val);
                    if (e / D < heads && (ELEMS % 512 == 0 || tid < ELEMS)) store_out1(a.out, a.out_dtype, out0 + e, val / sum);
                }
            }
        }
    }
    // ---- what belongs to no row: the new lengths, and the zero rows of empty or refused contexts
    if (a.len_out && blockIdx.x == gridDim.x - 1 && wave == 0 && lane < n) a.len_out[lane] = raw + 1;
    for (int z = blockIdx.x; z < n; z += gridDim.x) {
        if (__builtin_amdgcn_readlane(len, z) != 0) continue;
        const float zero[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int e = tid; e < a.H * D / 8; e += NW * 64) store_out8(a.out, a.out_dtype, ((int64_t)z * a.H * D / 8 + e) * 8, zero);
    }
}
