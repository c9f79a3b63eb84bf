// Launch code of libs3kv for gfx950 (MI355X) and its small kernels: append, plane copies (grow / fill /
// read-back), batch patches, the bandwidth probe, and the host side of every attention call.  The attention
// kernels live in s3kv_attn.h (multi-head 16-bit caches; instantiated per head dimension by
// s3kv_attn_inst.hip), s3kv_gqa.hip, s3kv_gqa_mfma.hip (shared key/value heads) and s3kv_fp8.hip (8-bit
// rows) and are launched from here; the device helpers all of them share are in s3kv_device.h.
//
// Arena layout.  Plane p = 2*layer + (0: K, 1: V) holds N token rows of H*D elements (H = cached
// heads), token-major: element (token t, head h, d) of a plane sits at ((t*H + h)*D + d).  A slot
// is the row range [off, off+cap) in EVERY plane, so one sequence's rows of one plane are one
// contiguous run and the attention kernels stream them with 128-bit loads.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <map>
#include <mutex>

#include "s3kv_internal.h"

#include "s3kv_device.h"

static int hip_fail(const char *what, hipError_t e) {
    s3i_set_hip_error(what, (int)e, hipGetErrorString(e));
    return S3_ERR_HIP;
}
#define HIP_TRY(call)                                     \
    do {                                                  \
        hipError_t e_ = (call);                           \
        if (e_ != hipSuccess) return hip_fail(#call, e_); \
    } while (0)

int s3i_device_cus(int32_t *cus) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    int n = 0;
    HIP_TRY(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
    *cus = n;
    return S3_OK;
}

// ------------------------------------------------------------------------------------------
// plane copies
// ------------------------------------------------------------------------------------------
// Every copied byte is read once and, far more rows than any cache holds being moved, written once: loads carry the
// streaming hint; stores do where it pays (below).  A workgroup moves spans of U * 256 consecutive 16-byte pieces, a
// thread's U loads all leave before its first store.  Admission of 4 contexts of 64..512 rows in 28 layers of 16 x 256
// bf16, one doubling, one eviction and its return (2.7 GB read and written): grid-stride loops, plain accesses 567 us;
// fills with both hints and U = 1: 524 (U = 2, 4: 531, 554; loads only: 569 at U = 4); copies of many planes with the
// load hint and U = 4: 534 (both hints 557; U = 1: 542); together 493.
template <bool NT_STORE, int U>
__device__ __forceinline__ void copy_pieces(const u32x4 *s, u32x4 *d, size_t n16) {
    for (size_t i0 = (size_t)blockIdx.x * (U * 256); i0 < n16; i0 += (size_t)gridDim.x * (U * 256)) {
        if (i0 + U * 256 <= n16) {
            u32x4 v[U];
#pragma unroll
            for (int u = 0; u < U; u++) v[u] = __builtin_nontemporal_load(s + i0 + u * 256 + threadIdx.x);
#pragma unroll
            for (int u = 0; u < U; u++) {
                if (NT_STORE) __builtin_nontemporal_store(v[u], d + i0 + u * 256 + threadIdx.x);
                else d[i0 + u * 256 + threadIdx.x] = v[u];
            }
        } else {
            for (size_t i = i0 + threadIdx.x; i < n16; i += 256) d[i] = __builtin_nontemporal_load(s + i);
        }
    }
}
#define S3_PLANE_U 4
#define S3_FILL_U 1

// blockIdx.y = plane; nbytes is a multiple of 16.
__global__ void __launch_bounds__(256) copy_planes_kernel(const char *src, char *dst, size_t n16,
                                                          size_t src_plane_stride, size_t dst_plane_stride) {
    copy_pieces<false, S3_PLANE_U>((const u32x4 *)(src + (size_t)blockIdx.y * src_plane_stride),
                                   (u32x4 *)(dst + (size_t)blockIdx.y * dst_plane_stride), n16);
}

// Two independent copies in one launch (blockIdx.y picks the pair): the K and V rows of a fill.
__global__ void __launch_bounds__(256) copy_pair_kernel(const char *src0, char *dst0, const char *src1, char *dst1,
                                                        size_t n16) {
    copy_pieces<true, S3_FILL_U>((const u32x4 *)(blockIdx.y ? src1 : src0), (u32x4 *)(blockIdx.y ? dst1 : dst0), n16);
}

// Rewrite a few entries of the per-batch device arrays; the new values travel as kernel arguments.
#define S3_PATCH_MAX 32
struct PatchArgs {
    int64_t off[S3_PATCH_MAX];
    int32_t idx[S3_PATCH_MAX];
    int32_t len[S3_PATCH_MAX];
    int32_t count;
};
__global__ void __launch_bounds__(64) batch_patch_kernel(int64_t *slot_off, int32_t *len, const PatchArgs p) {
    const int i = threadIdx.x;
    if (i < p.count) {
        if (slot_off) slot_off[p.idx[i]] = p.off[i];
        if (len) len[p.idx[i]] = p.len[i];
    }
}

extern "C" int s3_kv_batch_patch(int32_t n, int64_t *slot_off, int32_t *len, int32_t n_updates, const int32_t *idx,
                                 const int64_t *new_off, const int32_t *new_len, void *stream) {
    if (n < 0 || n_updates < 0 || (!slot_off && !len)) return S3_ERR_INVALID;
    if (n_updates == 0) return S3_OK;
    if (!idx || (slot_off && !new_off) || (len && !new_len)) return S3_ERR_INVALID;
    for (int32_t i = 0; i < n_updates; i++)
        if (idx[i] < 0 || idx[i] >= n) return S3_ERR_INVALID;
    for (int32_t first = 0; first < n_updates; first += S3_PATCH_MAX) {
        PatchArgs p;
        p.count = n_updates - first < S3_PATCH_MAX ? n_updates - first : S3_PATCH_MAX;
        for (int32_t i = 0; i < p.count; i++) {
            p.idx[i] = idx[first + i];
            p.off[i] = new_off ? new_off[first + i] : 0;
            p.len[i] = new_len ? new_len[first + i] : 0;
        }
        hipLaunchKernelGGL(batch_patch_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, slot_off, len, p);
        HIP_TRY(hipGetLastError());
    }
    return S3_OK;
}

// Admission of several newcomers in one launch: their prompt rows (K and V of one layer) and, optionally,
// their entries of the running batch's device arrays.  Everything travels as kernel arguments.
#define S3_FILL_MAX 16
struct FillArgs {
    const char *ksrc[S3_FILL_MAX];
    const char *vsrc[S3_FILL_MAX];
    char *kdst[S3_FILL_MAX];
    char *vdst[S3_FILL_MAX];
    int64_t off[S3_FILL_MAX];
    uint64_t n16[S3_FILL_MAX];  // 16-byte pieces of one plane's rows (max_len rows of up to 64 KiB reach 2^32)
    int32_t idx[S3_FILL_MAX];
    int32_t rows[S3_FILL_MAX];
};
// grid (x, 2, entries): blockIdx.z picks the newcomer, blockIdx.y K or V, the x blocks stride over its rows.
__global__ void __launch_bounds__(256) fill_batch_kernel(const FillArgs f, int64_t *slot_off, int32_t *len) {
    const int z = blockIdx.z;
    copy_pieces<true, S3_FILL_U>((const u32x4 *)(blockIdx.y ? f.vsrc[z] : f.ksrc[z]), (u32x4 *)(blockIdx.y ? f.vdst[z] : f.kdst[z]), f.n16[z]);
    if (slot_off && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        slot_off[f.idx[z]] = f.off[z];
        len[f.idx[z]] = f.rows[z];
    }
}

extern "C" int s3_kv_fill_batch(s3_arena *a, int32_t layer, int32_t n_new, const int32_t *slot_id, const int32_t *n_rows,
                                const void *const *k_rows, const void *const *v_rows, int32_t batch_n,
                                int64_t *slot_off, int32_t *len, const int32_t *batch_idx, void *stream) {
    if (!a || !a->base || layer < 0 || layer >= a->cfg.n_layers || n_new < 0) return S3_ERR_INVALID;
    if (n_new == 0) return S3_OK;
    if (!slot_id || !n_rows || !k_rows || !v_rows) return S3_ERR_INVALID;
    const bool patch = slot_off || len;
    if (patch && (!slot_off || !len || !batch_idx || batch_n <= 0)) return S3_ERR_INVALID;
    for (int32_t i = 0; i < n_new; i++) {  // everything is checked before anything is enqueued
        const s3_slot *s = s3i_live_slot(a, slot_id[i]);
        if (!s || n_rows[i] < 0) return S3_ERR_INVALID;
        if (n_rows[i] > s->cap) return S3_ERR_SLOT_FULL;
        if (n_rows[i] > 0 && (!k_rows[i] || !v_rows[i] || ((uintptr_t)k_rows[i] & 15) || ((uintptr_t)v_rows[i] & 15)))
            return S3_ERR_INVALID;
        if (patch && (batch_idx[i] < 0 || batch_idx[i] >= batch_n)) return S3_ERR_INVALID;
    }
    for (int32_t first = 0; first < n_new; first += S3_FILL_MAX) {
        FillArgs f;
        memset(&f, 0, sizeof(f));
        const int count = n_new - first < S3_FILL_MAX ? n_new - first : S3_FILL_MAX;
        size_t most = 1;
        for (int i = 0; i < count; i++) {
            const s3_slot *s = s3i_live_slot(a, slot_id[first + i]);
            const size_t n16 = (size_t)n_rows[first + i] * a->row_bytes / 16;
            f.ksrc[i] = (const char *)k_rows[first + i];
            f.vsrc[i] = (const char *)v_rows[first + i];
            f.kdst[i] = a->plane(layer, 0) + s->off * a->row_bytes;
            f.vdst[i] = a->plane(layer, 1) + s->off * a->row_bytes;
            f.n16[i] = n16;
            f.off[i] = s->off;
            f.idx[i] = patch ? batch_idx[first + i] : 0;
            f.rows[i] = n_rows[first + i];
            if (n16 > most) most = n16;
        }
        size_t blocks = (most + S3_FILL_U * 256 - 1) / (S3_FILL_U * 256);
        // The longest newcomer sets the grid of all: bounded in sum, since a short one's workgroups without work cost about
        // 0.2 ns each (one prompt of 2048 rows and fifteen of 16, 16 x 256 fp16: 131072 workgroups 37.5 us, 16384 14.4,
        // 8192 16.2; sixteen of 300 rows: 27.5, 26.9, 27.1).
        const size_t limit = 16384 / (2 * (size_t)count);
        if (blocks > limit) blocks = limit;
        hipLaunchKernelGGL(fill_batch_kernel, dim3((unsigned)blocks, 2, (unsigned)count), dim3(256), 0, (hipStream_t)stream,
                           f, patch ? slot_off : nullptr, patch ? len : nullptr);
        HIP_TRY(hipGetLastError());
    }
    return S3_OK;
}

int s3i_launch_copy_planes(const char *src, char *dst, size_t nbytes, size_t src_plane_stride,
                           size_t dst_plane_stride, int planes, void *stream) {
    if (nbytes == 0 || planes <= 0) return S3_OK;
    if ((nbytes & 15) || ((uintptr_t)src & 15) || ((uintptr_t)dst & 15)) return S3_ERR_INVALID;
    const size_t n16 = nbytes / 16;
    size_t blocks = (n16 + S3_PLANE_U * 256 - 1) / (S3_PLANE_U * 256);
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(copy_planes_kernel, dim3((unsigned)blocks, (unsigned)planes), dim3(256), 0,
                       (hipStream_t)stream, src, dst, n16, src_plane_stride, dst_plane_stride);
    HIP_TRY(hipGetLastError());
    return S3_OK;
}

// ------------------------------------------------------------------------------------------
// bandwidth probe: what a plain streaming kernel reaches on this device, to put the attention
// kernel's number next to (the attainable HBM rate is below the nominal peak)
// ------------------------------------------------------------------------------------------
static int ensure_scratch(s3_arena *a, size_t need);

// The buffer is read as the attention kernels read a cache: rows of 8 KiB, a wave streams one 1 KiB piece of 128
// consecutive rows, eight non-temporal 128-bit loads per lane in flight; neighbouring waves take neighbouring pieces
// of the same rows.  (A grid-stride loop over the whole buffer, four loads in flight, read 20 % slower here.)
#define S3_PROBE_ROW 8192
#define S3_PROBE_ROWS 128
__global__ void __launch_bounds__(256) read_probe_kernel(const char *src, size_t n_items, unsigned int *sink) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (size_t item = (size_t)blockIdx.x * 4 + wave; item < n_items; item += (size_t)gridDim.x * 4) {
        const char *base = src + (item / 8) * ((size_t)S3_PROBE_ROWS * S3_PROBE_ROW) + (item % 8) * 1024 + lane * 16;
        for (int r = 0; r < S3_PROBE_ROWS; r += 8) {
            u32x4 v[8];
#pragma unroll
            for (int i = 0; i < 8; i++) v[i] = __builtin_nontemporal_load((const u32x4 *)(base + (size_t)(r + i) * S3_PROBE_ROW));
#pragma unroll
            for (int i = 0; i < 8; i++) acc ^= v[i];
        }
    }
    const unsigned int x = acc[0] ^ acc[1] ^ acc[2] ^ acc[3];
    if (x == 0x9E3779B9u) *sink = x;  // practically never: keeps the loads alive
}

extern "C" int s3_kv_probe_bandwidth(s3_arena *a, size_t bytes, int32_t mode, int32_t reps, double *gbps) {
    if (!a || !a->base || !gbps || reps <= 0 || (mode != 0 && mode != 1)) return S3_ERR_INVALID;
    // mode 0 reads whole blocks of 128 rows of 8 KiB (1 MiB); a smaller request reads nothing and is refused
    bytes = mode == 0 ? bytes / ((size_t)S3_PROBE_ROWS * S3_PROBE_ROW) * ((size_t)S3_PROBE_ROWS * S3_PROBE_ROW) : bytes & ~(size_t)15;
    if (bytes == 0 || (mode == 0 ? bytes : 2 * bytes) > a->dev_bytes) return S3_ERR_INVALID;
    const int rc = ensure_scratch(a, 256);
    if (rc != S3_OK) return rc;
    hipEvent_t e0, e1;
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    const size_t n16 = bytes / 16;
    const int cus = a->num_cus > 0 ? a->num_cus : 256;
    for (int r = -2; r < reps; r++) {  // two untimed warm-up passes
        if (r == 0) HIP_TRY(hipEventRecord(e0, nullptr));
        if (mode == 0) {
            hipLaunchKernelGGL(read_probe_kernel, dim3((unsigned)(cus * 2)), dim3(256), 0, nullptr, a->base,
                               bytes / ((size_t)S3_PROBE_ROWS * 1024), (unsigned int *)((char *)a->scratch + 128));
        } else {
            hipLaunchKernelGGL(copy_planes_kernel, dim3((unsigned)(cus * 8), 1), dim3(256), 0, nullptr, a->base,
                               a->base + bytes, n16, (size_t)0, (size_t)0);
        }
        HIP_TRY(hipGetLastError());
    }
    HIP_TRY(hipEventRecord(e1, nullptr));
    HIP_TRY(hipEventSynchronize(e1));
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    *gbps = (double)(mode == 0 ? bytes : 2 * bytes) * reps / (ms * 1e-3) / 1e9;
    return S3_OK;
}

// ------------------------------------------------------------------------------------------
// append
// ------------------------------------------------------------------------------------------
// grid (n, 2): block (b, which) copies one row of H*D elements into row off+pos of the plane.
__global__ void __launch_bounds__(256) append_kernel(char *kplane, char *vplane, const int64_t *slot_off,
                                                     const int32_t *pos, const char *k_new, const char *v_new,
                                                     int64_t row_bytes, int64_t n_tokens, int32_t max_len) {
    const int b = blockIdx.x;
    const int64_t off = slot_off[b];
    const int64_t p = pos[b];
    if (off < 0 || p < 0 || p >= max_len || off + p >= n_tokens) return;  // never leave the arena
    const u32x4 *s = (const u32x4 *)((blockIdx.y ? v_new : k_new) + (int64_t)b * row_bytes);
    u32x4 *d = (u32x4 *)((blockIdx.y ? vplane : kplane) + (off + p) * row_bytes);
    const int n16 = (int)(row_bytes >> 4);
    for (int i = threadIdx.x; i < n16; i += 256) d[i] = s[i];
}

// ------------------------------------------------------------------------------------------
// attention: kernel choice and launchers
// ------------------------------------------------------------------------------------------
// Multi-head kernels, one translation unit per head dimension (s3kv_attn_inst.hip).
attn_fn s3i_pick_mha_d64(int dt, int variant);
attn_fn s3i_pick_mha_d96(int dt, int variant);
attn_fn s3i_pick_mha_d128(int dt, int variant);
attn_fn s3i_pick_mha_d256(int dt, int variant);
attn_fn s3i_pick_few_d64(int act, bool kv8);
attn_fn s3i_pick_few_d96(int act, bool kv8);
attn_fn s3i_pick_few_d128(int act, bool kv8);
attn_fn s3i_pick_few_d256(int act, bool kv8);
attn_fn s3i_pick_merge_d64();
attn_fn s3i_pick_merge_d96();
attn_fn s3i_pick_merge_d128();
attn_fn s3i_pick_merge_d256();
int s3i_default_variant();
int s3i_default_variant_large();
int s3i_variant_threads(int variant);
int s3i_variant_ring_bytes(int variant);
int s3i_variant_dynamic(int variant);
int s3i_variant_stream(int variant);

static attn_fn pick_kernel(int dt, int d, int variant) {
    switch (d) {
        case 64: return s3i_pick_mha_d64(dt, variant);
        case 96: return s3i_pick_mha_d96(dt, variant);
        case 128: return s3i_pick_mha_d128(dt, variant);
        case 256: return s3i_pick_mha_d256(dt, variant);
        default: return nullptr;
    }
}

static attn_fn pick_merge(int d) {
    return d == 64 ? s3i_pick_merge_d64() : d == 96 ? s3i_pick_merge_d96() : d == 128 ? s3i_pick_merge_d128()
                                                                                       : s3i_pick_merge_d256();
}

static attn_fn pick_few(int act, int d, bool kv8) {
    return d == 64 ? s3i_pick_few_d64(act, kv8) : d == 96 ? s3i_pick_few_d96(act, kv8) : d == 128 ? s3i_pick_few_d128(act, kv8)
                                                                                       : d == 256 ? s3i_pick_few_d256(act, kv8) : nullptr;
}

// Heads that one 128-bit wave load of 16-bit elements covers: 512/D, except that a 96-wide head takes a
// group of sixteen lanes of which twelve are used (four heads per load).
static int heads_per_load(int d) { return d == 96 ? 4 : 512 / d; }

static int ensure_scratch(s3_arena *a, size_t need) {
    if (need <= a->scratch_bytes) return S3_OK;
    if (a->scratch) {
        HIP_TRY(hipDeviceSynchronize());
        HIP_TRY(hipFree(a->scratch));
        a->scratch = nullptr;
        a->scratch_bytes = 0;
    }
    HIP_TRY(hipMalloc(&a->scratch, need));
    // The arrival counters at its head must start at zero, for the call's own stream too: a memset of device memory need
    // not be over when hipMemset returns, and a stream that does not wait for the default stream would overtake it.
    HIP_TRY(hipMemset(a->scratch, 0, need));
    HIP_TRY(hipStreamSynchronize(nullptr));
    a->scratch_bytes = need;
    return S3_OK;
}

// ---- the fixed scratch of s3_decode_step_static ------------------------------------------
// Part of the library's device image: every GPU that loads the library holds its own copy at its own
// address until the process ends.  In host code the arrays' names are only handles for the runtime; the
// device addresses are asked for once per device (with that device current) and only those are ever
// handed to kernels.
// The counters have memory of their own, which no call's partials reach whatever its arena or kernel: they are zero
// in the device image and every launch leaves its own at zero, so launches of any layouts may follow one another,
// recorded into graphs or not, and nothing has to be cleared.  (A call's counters and partials together are at most
// S3_STATIC_SCRATCH_BYTES, see place_scratch, so either array holds its part.)
static __device__ __align__(256) unsigned char s3_static_scratch[S3_STATIC_SCRATCH_BYTES];
static __device__ __align__(256) unsigned char s3_static_counters[S3_STATIC_SCRATCH_BYTES];

#define S3_MAX_DEVICES 64
struct StaticScratch {  // device addresses on one device
    char *partials = nullptr, *counters = nullptr;
};
static StaticScratch g_static[S3_MAX_DEVICES];
static std::mutex g_static_guard;

// The current device's addresses, resolved once per device.
static int static_scratch(StaticScratch *out) {
    std::lock_guard<std::mutex> lock(g_static_guard);
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= S3_MAX_DEVICES) return S3_ERR_INVALID;
    StaticScratch &st = g_static[dev];
    if (!st.counters) {
        void *p = nullptr, *c = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(s3_static_scratch)));
        HIP_TRY(hipGetSymbolAddress(&c, HIP_SYMBOL(s3_static_counters)));
        if (!p || !c || ((uintptr_t)p & 255) || ((uintptr_t)c & 255)) return S3_ERR_INVALID;
        st.partials = (char *)p;
        st.counters = (char *)c;
    }
    *out = st;
    return S3_OK;
}

// Called when an arena is created over device memory: the addresses are then known before the first decode step
// (which may run where no runtime query is wanted, e.g. under graph capture).
int s3i_static_scratch_setup() {
    StaticScratch st;
    return static_scratch(&st);
}

// ---- optional event timing of the attention kernels -------------------------------------
static int prof_next_event(s3_arena *a, hipEvent_t *ev) {
    if (a->prof_used == a->prof_events.size()) {
        hipEvent_t e;
        HIP_TRY(hipEventCreate(&e));
        a->prof_events.push_back((void *)e);
    }
    *ev = (hipEvent_t)a->prof_events[a->prof_used++];
    return S3_OK;
}

int s3i_profile_collect(s3_arena *a) {
    for (size_t i = 0; i + 2 < a->prof_used; i += 3) {
        hipEvent_t e0 = (hipEvent_t)a->prof_events[i], e1 = (hipEvent_t)a->prof_events[i + 1],
                   e2 = (hipEvent_t)a->prof_events[i + 2];
        HIP_TRY(hipEventSynchronize(e2));
        float p = 0.f, m = 0.f;
        HIP_TRY(hipEventElapsedTime(&p, e0, e1));
        HIP_TRY(hipEventElapsedTime(&m, e1, e2));
        a->prof_partial_ms += p;
        a->prof_merge_ms += m;
        a->prof_launches++;
        a->prof_durations_ms.push_back(p);
    }
    a->prof_used = 0;
    return S3_OK;
}

void s3i_profile_reset(s3_arena *a) {
    (void)s3i_profile_collect(a);
    a->prof_partial_ms = a->prof_merge_ms = 0.0;
    a->prof_launches = 0;
    a->prof_durations_ms.clear();
    // events are created here, not at the first timed launch: creating one costs tens of microseconds
    while (a->prof_events.size() < 3 * 64) {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) break;
        a->prof_events.push_back((void *)e);
    }
}

extern "C" void s3_kv_arena_destroy(s3_arena *a) {
    if (!a) return;
    if (!a->prof_events.empty()) {
        (void)hipDeviceSynchronize();
        for (void *e : a->prof_events) (void)hipEventDestroy((hipEvent_t)e);
    }
    if (a->scratch) {
        (void)hipDeviceSynchronize();
        (void)hipFree(a->scratch);
    }
    delete a;
}

static bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

// The append of one layer: a bit copy of the new rows, or, for 8-bit caches, their quantisation.
static int launch_append(s3_arena *a, int32_t layer, int32_t n, const int64_t *slot_off, const int32_t *pos,
                         const void *k_new, const void *v_new, void *stream) {
    if (a->cfg.kv_dtype == S3_E4M3) {
        append_fp8_fn fn = s3i_pick_append_fp8(a->cfg.act_dtype);
        if (!fn) return S3_ERR_INVALID;
        hipLaunchKernelGGL(fn, dim3((unsigned)n, 2), dim3(256), 0, (hipStream_t)stream, a->plane(layer, 0),
                           a->plane(layer, 1), slot_off, pos, (const char *)k_new, (const char *)v_new,
                           (int32_t)a->row_bytes, a->n_tokens, a->cfg.max_len);
    } else {
        hipLaunchKernelGGL(append_kernel, dim3((unsigned)n, 2), dim3(256), 0, (hipStream_t)stream, a->plane(layer, 0),
                           a->plane(layer, 1), slot_off, pos, (const char *)k_new, (const char *)v_new, a->row_bytes,
                           a->n_tokens, a->cfg.max_len);
    }
    HIP_TRY(hipGetLastError());
    return S3_OK;
}
static int check_slots_host(const s3_arena *a, int32_t n, const int32_t *slot_id, const int32_t *pos_host);

extern "C" int s3_kv_append(s3_arena *a, int32_t layer, int32_t n, const int32_t *slot_id, const int32_t *pos_host,
                            const int64_t *slot_off, const int32_t *pos, const void *k_new, const void *v_new,
                            void *stream) {
    if (!a || !a->base || layer < 0 || layer >= a->cfg.n_layers || n < 0) return S3_ERR_INVALID;
    if (n == 0) return S3_OK;
    if (!slot_off || !pos || !k_new || !v_new || !aligned16(k_new) || !aligned16(v_new)) return S3_ERR_INVALID;
    const int rc = check_slots_host(a, n, slot_id, pos_host);
    if (rc != S3_OK) return rc;
    return launch_append(a, layer, n, slot_off, pos, k_new, v_new, stream);
}

static int check_slots_host(const s3_arena *a, int32_t n, const int32_t *slot_id, const int32_t *pos_host) {
    if (!slot_id || !pos_host) return S3_OK;  // the caller vouches for the positions
    bool full = false;
    for (int32_t b = 0; b < n; b++) {
        const s3_slot *s = s3i_live_slot(a, slot_id[b]);
        if (!s || pos_host[b] < 0 || pos_host[b] > s->cap) return S3_ERR_INVALID;
        if (pos_host[b] == s->cap) full = true;
    }
    return full ? S3_ERR_SLOT_FULL : S3_OK;
}

// Workgroups of `fn` (threads per workgroup, dynamic LDS bytes) that one CU holds at once.  Asked
// from the runtime once per kernel and LDS size class (4 KiB steps).
static int resident_per_cu(const void *fn, int threads, size_t dyn_lds, int *per_cu) {
    static std::map<std::pair<const void *, size_t>, int> resident;  // (kernel, LDS in 4 KiB) -> workgroups per CU
    static std::mutex guard;  // shared by all arenas, which may live on different threads
    std::lock_guard<std::mutex> lock(guard);
    const std::pair<const void *, size_t> key(fn, (dyn_lds + 4095) / 4096);
    auto it = resident.find(key);
    if (it == resident.end()) {
        if (dyn_lds > 16384)
            HIP_TRY(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(key.second * 4096)));
        int got = 0;
        HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&got, fn, threads, key.second * 4096));
        if (got < 1) return S3_ERR_INVALID;  // does not fit the device at all
        it = resident.emplace(key, got).first;
    }
    *per_cu = it->second;
    return S3_OK;
}

// One attention call as the entry points hand it over.  with_append: s3_decode_step (len_or_pos is the
// append position, the kernels attend over pos + 1 rows and publish len_out).
struct AttnCall {
    int32_t layer, n;
    const void *q;
    const int64_t *slot_off;
    const int32_t *len_or_pos;
    void *out;
    int32_t out_dtype;
    float scale;
    void *stream;
    bool with_append;
    const void *k_new, *v_new;
    int32_t *len_out;
    bool static_scratch;  // s3_decode_step_static: partials and counters in the library's fixed device buffer
};

static size_t batch_view_lds(int n, int ncls);

// Kernel arguments every attention kernel shares.  row_heads: heads of a cached row; q_heads: heads of q / out.
static AttnArgs common_args(const s3_arena *a, const AttnCall &c, int row_heads, int q_heads, int chunk) {
    AttnArgs args;
    memset(&args, 0, sizeof(args));
    args.kplane = a->plane(c.layer, 0);
    args.vplane = a->plane(c.layer, 1);
    args.q = (const char *)c.q;
    args.k_new = (const char *)c.k_new;
    args.v_new = (const char *)c.v_new;
    args.slot_off = c.slot_off;
    args.cur_len = c.len_or_pos;
    args.out = c.out;
    args.n_tokens = a->n_tokens;
    args.n = c.n;
    args.H = row_heads;
    args.Hq = q_heads;
    args.chunk = chunk;
    args.max_chunks = (a->cfg.max_len + chunk - 1) / chunk;
    // length classes of the longest-first work order: small batches gain from it (their kernels are
    // short, the tail matters); for large batches the extra prologue work per class costs more than
    // the order gains.  Measured on MI355X.
    args.ncls = a->ncls > 0 ? a->ncls : c.n <= 128 ? 4 : c.n <= 256 ? 2 : 1;
    // the view must fit LDS beside the kernels' own buffers (up to 67 KiB) whatever the caller asked for:
    // a batch of thousands keeps fewer classes
    while (args.ncls > 1 && batch_view_lds(c.n, args.ncls) > (size_t)96 * 1024) args.ncls--;
    args.out_dtype = c.out_dtype;
    args.max_len = a->cfg.max_len;
    args.len_add = c.with_append ? 1 : 0;
    const float scale = c.scale > 0.f ? c.scale : 1.0f / sqrtf((float)a->cfg.head_dim);
    args.scale_log2e = scale * 1.4426950408889634f;
    args.len_out = c.with_append ? c.len_out : nullptr;
    args.merge_sync = a->merge_sync;
    return args;
}

static size_t scratch_need(const s3_arena *a, int n);

// Library scratch: [arrival counters: cnt_bytes, fixed per arena kind, zero between launches]
// [partial sums][partial (max, sum)], `slots` partials per head of q (one per sequence and chunk, or as
// gqa_partial_slots() counts them).  (s3_decode_step_static: the counters in an array of their own.)
static int place_scratch(s3_arena *a, AttnArgs &args, size_t cnt_bytes, size_t slots, const AttnCall &c) {
    const size_t n_part = slots * args.Hq;
    const size_t acc_bytes = n_part * a->cfg.head_dim * sizeof(float);
    const size_t need = cnt_bytes + acc_bytes + n_part * sizeof(float2);
    char *counters = nullptr, *partials = nullptr;
    if (c.static_scratch) {  // no allocation on this path: the fixed buffers hold the call, or the call is refused
        if (need > (size_t)S3_STATIC_SCRATCH_BYTES) return S3_ERR_SCRATCH;
        StaticScratch st;
        const int rc = static_scratch(&st);
        if (rc != S3_OK) return rc;
        counters = st.counters;
        partials = st.partials;
    } else {
        // The scratch moves only for a batch larger than any before (or after a change of "chunk" or "variant"): a
        // smaller batch may need more than a larger one, since few contexts are cut finer, so a growth takes what
        // every batch up to this one needs.  Recorded graphs keep its address.
        if (args.n > a->scratch_batch || need > a->scratch_bytes) {
            const size_t all = scratch_need(a, args.n);
            const int rc = ensure_scratch(a, all > need ? all : need);
            if (rc != S3_OK) return rc;
            if (args.n > a->scratch_batch) a->scratch_batch = args.n;
        }
        counters = (char *)a->scratch;
        partials = counters + cnt_bytes;
    }
    args.arrivals = (unsigned int *)counters;
    args.queue = cnt_bytes >= 256 ? (unsigned int *)(counters + cnt_bytes - 256) : nullptr;  // the last 256 bytes of the counter region
    args.part_acc = (float *)partials;
    args.part_ml = (float2 *)(partials + acc_bytes);
    return S3_OK;
}

// Bytes of the arrival counters at the head of the scratch: one per (sequence, head group), for the largest
// batch a call takes, so that the partials behind them never move with the batch size.
static size_t counters_bytes(int n_hg) {
    return ((((size_t)(S3_MAX_BATCH + 1) * n_hg * sizeof(unsigned int)) + 255) & ~(size_t)255) + 256;  // + the work-list counters
}

// The matrix-core kernel's share of the scratch.  Cut by the caller's `chunk`, contexts leave one piece per chunk.  With
// the default division a piece of a context sits in slot (publishing unit + sequence), so max_shares units need
// max_shares + n slots; at most one unit per wave and column (waves <= 8 per compute unit, see launch_gqa_mfma).
// What fits the fixed buffer of s3_decode_step_static by its documented rule (chunks of `chunk` rows, or 128 / 256)
// is held to that buffer's size, there and here alike, so that both calls divide their rows the same: by fewer
// shares, or, where that would leave fewer of them than there are contexts, by shares of whole contexts (0; only
// possible where no context is longer than a chunk).  32q/8kv x 128, contexts of 20..200 rows of at most 256, per layer:
// 1900 contexts 232 us in the 108 shares that fit, 181 in whole contexts; 1990: 1201 us in 18 shares, 190; 2008: 21 ms
// in one, 191.
static int64_t gqa_columns(const s3_arena *a) {
    const int group = a->cfg.n_heads / a->cfg.n_kv_heads;
    return (int64_t)a->cfg.n_kv_heads * ((group + 15) / 16);
}
static size_t gqa_slot_bytes(const s3_arena *a) {
    return (size_t)a->cfg.n_heads * ((size_t)a->cfg.head_dim * sizeof(float) + sizeof(float2));
}
// Vector-ALU kernel for shared heads: query heads per lane, and rows per chunk (few (sequence, head group) pairs: contexts
// are cut finer so that the chip still has work everywhere).
static int gqa_heads_per_lane(const s3_arena *a) {
    const int group = a->cfg.n_heads / a->cfg.n_kv_heads;
    return group % 8 == 0 ? 8 : group % 4 == 0 ? 4 : group % 2 == 0 ? 2 : 1;
}
static int gqa_items_per_chunk(const s3_arena *a) {  // K/V head groups x query sub-blocks
    const int GH = 512 / a->cfg.head_dim, group = a->cfg.n_heads / a->cfg.n_kv_heads;
    return ((a->cfg.n_kv_heads + GH - 1) / GH) * (group / gqa_heads_per_lane(a));
}
static int gqa_chunk_rows(const s3_arena *a, int n) {
    const int64_t items = (int64_t)n * gqa_items_per_chunk(a);
    return a->chunk > 0 ? a->chunk : items >= 2048 ? 1024 : items >= 512 ? 512 : 256;
}

// Fewer than four query heads per cached head, 16-bit rows, nothing set by the caller: which kernel serves a batch of n.  The
// matrix cores win where the launch is a chain of latencies (one launch instead of three) and wherever the vector-ALU kernel
// reads the rows once per query head (odd groups).  With two heads it reads them once, and a batch that fills the chip is
// bound by memory either way: more (sequence, cached head) pairs than two a compute unit stay with it (of 256: than one).
// us a layer, bf16, vector ALU and matrix cores: 16q/8kv x 128, 1 context of 30..40 rows 10.8, 6.0, 20 of 32..1000 27.9, 15.5,
// 64 of 100..200 23.6, 15.4, 85 of 32..1000 41.4, 41.8; 64q/32kv x 128, 8 of 32..1000 27.9, 18.5, 64 of 100..200 35.7, 43.0;
// 6q/3kv x 256, 20 of 32..1000 29.0, 14.6, 85 36.8, 32.8 (beyond its line now faster too: 200 75.5, 69.5, 300 of 2..40 17.8,
// 16.4); 24q/8kv x 64, 20 of 32..1000 25.1, 12.4, 700 of 32..1000 392, 132, 300 of 2..40 19.5, 13.3; 9q/3kv x 256, 700 of
// 32..1000 633, 203.
// (Both keep the weights in fp32 and treat infinite values alike, see pick_few_heads.)
static bool gqa_on_matrix_cores(const s3_arena *a, int n) {
    const int kind = s3i_kernel_kind(a);
    if (kind != 1 || a->variant >= 0 || a->chunk > 0) return kind == 2 || kind == 4;
    const int64_t cus = a->num_cus > 0 ? a->num_cus : 256;
    return a->cfg.n_heads / a->cfg.n_kv_heads == 3 || n * gqa_columns(a) <= (a->cfg.head_dim == 256 ? cus : 2 * cus);
}

// Chunks of the documented rule over n contexts, and how many the fixed buffer holds.
static int64_t gqa_chunks(const s3_arena *a, int n) {
    const int chunk = a->chunk > 0 ? a->chunk : n * gqa_columns(a) >= 4096 ? 256 : 128;
    return (int64_t)n * ((a->cfg.max_len + chunk - 1) / chunk);
}
static int64_t gqa_static_slots(const s3_arena *a) {
    return (int64_t)((S3_STATIC_SCRATCH_BYTES - counters_bytes((int)gqa_columns(a))) / gqa_slot_bytes(a));
}
// (kind 1: by the vector-ALU kernel's chunks, without counters, whichever kernel serves the batch)
static bool gqa_fits_static(const s3_arena *a, int n) {
    if (s3i_kernel_kind(a) != 1) return gqa_chunks(a, n) <= gqa_static_slots(a);
    const int chunk = gqa_chunk_rows(a, n);
    return (int64_t)n * ((a->cfg.max_len + chunk - 1) / chunk) <= (int64_t)(S3_STATIC_SCRATCH_BYTES / gqa_slot_bytes(a));
}
// (not for callers of the library: a host test reads it)
extern "C" int64_t s3i_gqa_max_shares(const s3_arena *a, int32_t n) {
    const int64_t columns = gqa_columns(a), waves = (int64_t)(a->num_cus > 0 ? a->num_cus : 256) * 8;
    const int64_t most = (waves + columns - 1) / columns;
    if (!gqa_fits_static(a, n)) return most;
    const int64_t fit = gqa_static_slots(a) - n;
    return fit >= most ? most : fit >= n ? fit : 0;
}
static size_t gqa_partial_slots(const s3_arena *a, int n) {
    if (a->chunk > 0) return (size_t)gqa_chunks(a, n);
    const int64_t shares = s3i_gqa_max_shares(a, n);
    return shares > 1 ? (size_t)(shares + n) : 0;  // one share: no piece ever leaves its wave or team
}

// Kernels whose chunks meet inside the launch (multi-head, 8-bit rows): chunks are of at most `chunk` rows (1024 unless
// the caller says otherwise), and *few, if not 0, is how many chunks in all the kernel cuts a batch of few contexts into
// (the lengths are on the device, so the rows per chunk are chosen there: few_chunk_rows).  Returns the partial slots.
// n_hg: head groups, i.e. work items per chunk.  3/4 of an item per compute unit while the contexts themselves are
// fewer than that (pieces do not divide evenly: with a full item per unit some unit would get two); beyond, whole
// contexts are items enough.  (Up to 64 such contexts are attn_few_kernel's since, if the caller sets neither chunk nor
// variant; these figures are the streaming kernels'.)  Chunk fixed at 1024 -> this rule, 16 heads x 256 fp16, four layers: one context of 410
// rows 74 -> 36 us, of 8050 rows 181 -> 112; 4 contexts of 500..1500 rows 129 -> 68, 8: 143 -> 102, 16: 207 -> 189;
// 32 contexts of 32..1000 rows: 212, and 217 if the line were drawn above them.
// As with s3i_gqa_max_shares, what the fixed buffer takes by its documented rule is held to its size.
// 8-bit rows, *units: beyond those batches, while the contexts' items are fewer than 0.7 of the two workgroups a compute unit
// holds, contexts are cut until the chunks fill these (unit_chunk_rows): a workgroup streams 1000 rows in about 55 us whatever
// the others do, and an item more than run at once starts only when another ends.  Contexts of 32..1000 rows, whole and cut, us
// a layer: 16 heads x 256, 49 contexts 66.0 and 43.6, 64 68.3 and 54.8, 80 75.7 and 69.0, 96 (beyond the line) 90.2 and
// 90.5, 112 97.4 and 98.4; 12 x 128, 97 64.3 and 39.6, 160 76.6 and 63.5.
// 16-bit rows: the same with chunks of up to 2048 rows, where the rows say so on the device: from 9/16 to one item a compute unit
// (unit_rule), and from 4/3 to 7/4 whole contexts (whole_rule), if contexts can be long enough at all.  Batches that the rules
// leave alone pay 0.2 to 1.0 us for the look (half of them less than 0.6), which is why they are not asked in between, where only few gain.
//
// Multi-head rows, nothing set by the caller: attn_few_kernel serves batches of up to 3/4 of an item a compute unit, 8-bit rows
// 4/5 (and 64 contexts, a lane each), in up to 2 * cus / n_hg chunks.  Beyond, whole contexts fill most of the chip and the
// streaming kernels' balance is as good or better.  us a layer, streaming kernel and this one: 16-bit, 16 x 256, 24 contexts
// (the last) of 20..200 rows 14.8, 12.2, of 500..1500 73.7, 68.5, of 32..1000 37.6, 37.5; 26 (beyond) of 500..1500 87.6, 75.7,
// but 40 of 32..1000 60.8, 63.8, 48 70.4, 83.5; 64 x 96, 18 of 20..200 12.8, 14.9.  The lengths are not known here, so a batch below the
// line can be slower where they happen to divide badly (64 x 96, 12 of 32..1000 rows 30.2, 31.7), and one above it could gain; over 60 kinds
// of batches below it, four draws of the lengths each, a kind takes 0.95 of the time, the worst (32 x 128, 24 of 1000..2000) 1.014.  e4m3, 16 x 256, 50 of 20..100 13.2, 10.2, of
// 300..600 38.6, 37.3, of 1000..2000 105.7, 107.1; 64 (beyond) of 20..100 13.8, 10.6, but of 32..1000 53.3, 56.8.  Rows of fewer 8-bit
// heads than a wave load takes, and that divide it, several to a load, stay with attn_fp8_kernel.
static bool on_few_kernel(const s3_arena *a, int n, int n_hg) {
    const int64_t cus = a->num_cus > 0 ? a->num_cus : 256, items = (int64_t)n * n_hg;
    const int kind = s3i_kernel_kind(a), loads = 1024 / a->cfg.head_dim;  // (8-bit rows: heads a wave load)
    if (a->chunk > 0 || a->variant >= 0 || n > 64) return false;
    return kind == 0 ? items <= cus * 3 / 4 : kind == 3 && (a->cfg.n_heads >= loads || loads % a->cfg.n_heads != 0) && items <= cus * 4 / 5;
}
static size_t chunk_slots(const s3_arena *a, int n, int n_hg, size_t slot_bytes, int32_t *few, int32_t *units) {
    const int chunk = a->chunk > 0 ? a->chunk : 1024;
    const int64_t whole = (int64_t)n * ((a->cfg.max_len + chunk - 1) / chunk);
    const int64_t cus = a->num_cus > 0 ? a->num_cus : 256;
    int64_t want = 0;
    if (a->chunk <= 0 && n <= cus * 3 / 4 / n_hg) want = cus * 3 / 4 / n_hg;
    const int64_t fixed = (int64_t)((S3_STATIC_SCRATCH_BYTES - counters_bytes(n_hg)) / slot_bytes);
    if (whole <= fixed && want > fixed - n) want = fixed - n;
    *few = want > 0 ? (int32_t)want : 0;
    const bool free_choice = a->chunk <= 0 && a->variant < 0;
    int64_t fill = free_choice ? 2 * cus / n_hg : 0;
    const bool eight_bit = s3i_kernel_kind(a) == 3;
    if (eight_bit) {
        if (want > 0 || n * 10 > fill * 7) fill = 0;
    } else {
        const bool cut = want > 0 ? n * 32 >= fill * 9 : n * 2 <= fill, uncut = n * 3 >= fill * 2 && n * 8 <= fill * 7;
        if (n > 128 || !(cut ? a->cfg.max_len >= 400 : uncut && a->cfg.max_len > chunk)) fill = 0;
    }
    if (whole <= fixed && fill + n > fixed) fill = 0;
    *units = fill > 0 ? (int32_t)(fill | (eight_bit ? 0 : 1 << 16)) : 0;
    if (fill > want) want = fill;
    if (on_few_kernel(a, n, n_hg)) want = 2 * cus / n_hg;  // (with the n slots below 3 MiB: in the fixed buffer always)
    return (size_t)(want > 0 && want + n > whole ? want + n : whole);
}

// Scratch the attention calls over 1 to n sequences need at most.
static size_t scratch_need(const s3_arena *a, int n) {
    const int D = a->cfg.head_dim, Hq = a->cfg.n_heads, kind = s3i_kernel_kind(a);
    const size_t slot_bytes = (size_t)Hq * ((size_t)D * sizeof(float) + sizeof(float2));
    const int gh = kind == 3 ? 1024 / D : heads_per_load(D), n_hg = (Hq + gh - 1) / gh;  // (kinds 0 and 3)
    size_t most = 0;
    for (int k = 1; k <= n; k++) {
        int32_t few, units;
        size_t slots;
        if (kind != 0 && kind != 3 && gqa_on_matrix_cores(a, k)) {
            slots = gqa_partial_slots(a, k);
        } else if (kind == 0 || kind == 3) {
            slots = chunk_slots(a, k, n_hg, slot_bytes, &few, &units);
        } else {
            const int chunk = gqa_chunk_rows(a, k);
            slots = (size_t)k * ((a->cfg.max_len + chunk - 1) / chunk);
        }
        if (slots > most) most = slots;
    }
    return counters_bytes(kind == 0 || kind == 3 ? n_hg : (int)gqa_columns(a)) + most * slot_bytes;
}

extern "C" int s3_kv_reserve_scratch(s3_arena *a, int32_t max_batch) {
    if (!a || !a->base || max_batch < 1 || max_batch > S3_MAX_BATCH) return S3_ERR_INVALID;
    const int rc = ensure_scratch(a, scratch_need(a, max_batch));
    if (rc == S3_OK && max_batch > a->scratch_batch) a->scratch_batch = max_batch;
    return rc;
}

static size_t batch_view_lds(int n, int ncls) {
    return (size_t)n * 8 + (size_t)((n + 1) & ~1) * 4 + (size_t)ncls * (n + 1) * 4;
}

// Grid of a kernel that walks the work list with a stride: the workgroups that are resident at once
// (every workgroup pays the batch-view prologue once), times `rounds`; or what the caller set.
static int stride_grid(const s3_arena *a, const void *fn, int threads, size_t dyn_lds, int rounds, int *blocks,
                       int max_per_cu = 0) {
    if (a->grid_blocks > 0) {
        *blocks = a->grid_blocks;
        return S3_OK;
    }
    int per_cu = 0;
    const int rc = resident_per_cu(fn, threads, dyn_lds, &per_cu);
    if (rc != S3_OK) return rc;
    if (max_per_cu > 0 && per_cu > max_per_cu) per_cu = max_per_cu;
    *blocks = (a->num_cus > 0 ? a->num_cus : 256) * per_cu * rounds;
    return S3_OK;
}

// Launch the attention kernel and, if merge_heads > 0, attn_merge_kernel over that many heads of q / out
// (it finishes multi-chunk contexts and writes the zero rows of empty ones).  Every k-th call (the
// "profile" parameter) is bracketed with events: before, after the attention kernel, after the merge.
static int launch_attn_kernels(s3_arena *a, attn_fn fn, int blocks, int threads, size_t dyn_lds, void *stream,
                               const AttnArgs &args, int merge_heads, bool may_time) {
    hipEvent_t ev[3] = {nullptr, nullptr, nullptr};
    const bool timed = may_time && a->profile > 0 && (a->prof_tick++ % a->profile) == 0;
    if (timed) {
        for (int i = 0; i < 3; i++) {
            const int prc = prof_next_event(a, &ev[i]);
            if (prc != S3_OK) return prc;
        }
        // the events take the kernel's own start and end times (not the times at which markers around it
        // pass through the queue), so the duration is the one a profiler reports for the dispatch
        AttnArgs copy = args;
        void *kargs[] = {(void *)&copy};
        HIP_TRY(hipExtLaunchKernel((const void *)fn, dim3((unsigned)blocks), dim3((unsigned)threads), kargs, dyn_lds,
                                   (hipStream_t)stream, ev[0], ev[1], 0));
    } else {
        hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3((unsigned)threads), dyn_lds, (hipStream_t)stream, args);
        HIP_TRY(hipGetLastError());
    }
    if (merge_heads > 0) {
        const int D = a->cfg.head_dim;
        AttnArgs margs = args;
        margs.H = merge_heads;  // the merge kernel indexes partials and output by head of q
        const int GH = heads_per_load(D);
        const unsigned mblocks = (unsigned)(((int64_t)args.n * ((merge_heads + GH - 1) / GH) + 3) / 4);
        attn_fn mfn = pick_merge(D);
        if (timed) {
            void *kargs[] = {(void *)&margs};
            HIP_TRY(hipExtLaunchKernel((const void *)mfn, dim3(mblocks), dim3(256), kargs, 0, (hipStream_t)stream, nullptr,
                                       ev[2], 0));
        } else {
            hipLaunchKernelGGL(mfn, dim3(mblocks), dim3(256), 0, (hipStream_t)stream, margs);
            HIP_TRY(hipGetLastError());
        }
    } else if (timed) {
        HIP_TRY(hipEventRecord(ev[2], (hipStream_t)stream));
    }
    return S3_OK;
}

// What the matrix-core kernel's workgroups of four, per_cu of them a compute unit, make of a column: at most so many shares (or
// chunks) by single waves, or by teams of the four waves of a workgroup.  Returns whether these units can be more than run at
// once, so that the instance with the loop over units is needed: chunks of the caller's size, grids of the caller's, and more
// columns than workgroups, since a column has at least one unit and a team's unit takes a whole workgroup.
// (not for callers of the library: a host test reads it)
extern "C" int32_t s3i_gqa_units(const s3_arena *a, int32_t per_cu, int32_t *wave_shares, int32_t *team_shares) {
    const int64_t columns = gqa_columns(a), workgroups = (int64_t)(a->num_cus > 0 ? a->num_cus : 256) * per_cu;
    *wave_shares = (int32_t)(4 * workgroups > columns ? 4 * workgroups / columns : 1);
    *team_shares = (int32_t)(workgroups > columns ? workgroups / columns : 1);
    return a->chunk > 0 || a->grid_blocks > 0 || columns > workgroups;
}

// Shared key/value heads, matrix-core kernel: one launch (with workgroups of four over 8-bit rows an append before it).
static int launch_gqa_mfma(s3_arena *a, const AttnCall &c) {
    const int D = a->cfg.head_dim, Hq = a->cfg.n_heads, Hkv = a->cfg.n_kv_heads;
    const bool eight_bit = s3i_kernel_kind(a) == 4;
    const int group = Hq / Hkv;
    const bool few_heads = !eight_bit && group < 4;
    const auto pick = [&](bool wide, bool loop) {
        return few_heads ? s3i_pick_gqa_few_heads(a->cfg.kv_dtype, D, group, wide, loop) : s3i_pick_gqa_mfma(a->cfg.act_dtype, D, eight_bit, wide, loop);
    };
    attn_fn fn = pick(false, false);
    if (!fn) return S3_ERR_INVALID;
    if (c.static_scratch && !gqa_fits_static(a, c.n)) return S3_ERR_SCRATCH;
    const int64_t columns = gqa_columns(a);
    AttnArgs args = common_args(a, c, Hkv, Hq, 16);  // (the kernel's batch view counts its own tiles)
    args.ncls = 1;
    args.stream_k = a->gqa_stream;
    args.share_rows = a->chunk;
    args.max_shares = (int32_t)s3i_gqa_max_shares(a, c.n);
    int rc = place_scratch(a, args, counters_bytes((int)columns), gqa_partial_slots(a, c.n), c);
    if (rc != S3_OK) return rc;
    // LDS behind the view: the first pieces of a team's four waves.  A batch whose view leaves no room for them has
    // thousands of contexts, i.e. long shares, and works without teams.
    const size_t view = batch_view_lds(c.n, 1), group16 = Hq / Hkv < 16 ? Hq / Hkv : 16;
    const size_t pieces = 4 * group16 * (size_t)(D + 4) * sizeof(float);
    args.team_lds = c.n <= 1024;
    const size_t dyn_lds = args.team_lds ? ((view + 15) & ~(size_t)15) + pieces : view;
    int per_cu = 0;
    const int cus = a->num_cus > 0 ? a->num_cus : 256;
    args.group = group;
    args.nqb = (args.group + 15) / 16;
    args.columns = (int32_t)columns;
    args.column_shift = (columns & (columns - 1)) == 0 ? __builtin_ctzll((unsigned long long)columns) : -1;
    // No more (context, column) pairs than compute units: workgroups of eight waves, one a unit, which take a context or a
    // chunk of one (eight_wave_plan).  Beyond, pairs would wait for a unit of their own (32q/8kv x 128, 34 contexts of
    // 32..1000 rows 22.0 us a layer against 21.5 with workgroups of four, 64 contexts 34.2 against 30.5).
    if (a->chunk <= 0 && c.n <= S3_FEW_CONTEXTS && c.n * columns <= cus) {
        attn_fn wide = pick(true, false);
        args.team_shares = (int32_t)(cus / columns);
        rc = resident_per_cu((const void *)wide, 512, view, &per_cu);
        if (rc != S3_OK) return rc;
        const int blocks = (int)(args.team_shares * columns);  // one chunk a workgroup
        return launch_attn_kernels(a, wide, blocks, 512, view, c.stream, args, 0, !c.static_scratch);
    }
    // Workgroups of four over 8-bit rows: the append is its own launch.  (Taken into the kernel, as it is with eight waves, the
    // rounding of 16 codes a lane in the middle of the row stream costs a long launch more than the 5 us: 32q/8kv x 128, 1024
    // contexts of 32..1000 rows 208.9 us, folded 212.2; 24q/8kv x 64, 500 of 5..60 18.1, 18.4.)
    if (c.with_append && eight_bit) {
        rc = launch_append(a, c.layer, c.n, c.slot_off, c.len_or_pos, c.k_new, c.v_new, c.stream);
        if (rc != S3_OK) return rc;
    }
    bool loop = false;
    while (true) {
        rc = resident_per_cu((const void *)fn, 256, dyn_lds, &per_cu);
        if (rc != S3_OK) return rc;
        if (per_cu > 2) per_cu = 2;
        if (!s3i_gqa_units(a, per_cu, &args.wave_shares, &args.team_shares) || loop) break;
        loop = true;
        fn = pick(false, true);
    }
    // What one more piece costs the wave that merges a context, in tiles streamed by one wave: a memory round trip of
    // about two tiles brings two quads of elements a lane of six pieces (D 256: four quads of three).
    const int eb = D == 256 ? 4 : 2, quads = (int)group16 * (D / 4), passes = (quads + 64 * eb - 1) / (64 * eb);
    args.merge_cost = 2.f * passes / (eb == 4 ? 3 : 6);
    const int blocks = a->grid_blocks > 0 ? a->grid_blocks : cus * per_cu;
    return launch_attn_kernels(a, fn, blocks, 256, dyn_lds, c.stream, args, 0, !c.static_scratch);
}

// Shared key/value heads, vector-ALU kernel: append as its own launch, attention, merge.
static int launch_gqa(s3_arena *a, const AttnCall &c) {
    const int D = a->cfg.head_dim, Hq = a->cfg.n_heads, Hkv = a->cfg.n_kv_heads;
    // Variant indices of a shared-K/V arena: the shapes of the vector-ALU kernel, then the matrix-core kernel.
    if (gqa_on_matrix_cores(a, c.n)) return launch_gqa_mfma(a, c);
    int threads = 256;
    attn_fn fn = s3i_pick_gqa(a->cfg.kv_dtype, D, gqa_heads_per_lane(a), a->variant, &threads);
    if (!fn) return S3_ERR_INVALID;
    if (c.with_append) {
        const int arc = launch_append(a, c.layer, c.n, c.slot_off, c.len_or_pos, c.k_new, c.v_new, c.stream);
        if (arc != S3_OK) return arc;
    }
    AttnArgs args = common_args(a, c, Hkv, Hq, gqa_chunk_rows(a, c.n));
    // The arena's scratch keeps the matrix-core kernel's counter region (zero between launches) in front of the
    // partials: both kernels of a shared-head arena run in turn (by the batch, or the "variant" parameter).  The fixed
    // scratch of s3_decode_step_static has its counters elsewhere and needs no such room.
    int rc = place_scratch(a, args, c.static_scratch ? 0 : counters_bytes((int)gqa_columns(a)), (size_t)args.n * args.max_chunks, c);
    if (rc != S3_OK) return rc;
    const size_t dyn_lds = batch_view_lds(c.n, args.ncls);
    int blocks = 0;
    rc = stride_grid(a, (const void *)fn, threads, dyn_lds, 1, &blocks);
    if (rc != S3_OK) return rc;
    return launch_attn_kernels(a, fn, blocks, threads, dyn_lds, c.stream, args, Hq, !c.static_scratch);
}

static int launch_few(s3_arena *a, AttnArgs &args, int n_hg, bool kv8, const AttnCall &c) {
    const int cus = a->num_cus > 0 ? a->num_cus : 256;
    attn_fn fn = pick_few(a->cfg.act_dtype, a->cfg.head_dim, kv8);
    if (!fn) return S3_ERR_INVALID;
    args.few_chunks = cus / n_hg;
    args.unit_chunks = 2 * cus / n_hg;
    args.columns = n_hg;
    args.column_shift = (n_hg & (n_hg - 1)) == 0 ? __builtin_ctz((unsigned)n_hg) : -1;
    return launch_attn_kernels(a, fn, args.unit_chunks * n_hg, 512, 0, c.stream, args, 0, !c.static_scratch);
}

// Scratch of a kernel whose chunks meet inside the launch.
static int place_chunk_scratch(s3_arena *a, AttnArgs &args, int n_hg, const AttnCall &c) {
    const size_t slot_bytes = (size_t)args.Hq * ((size_t)a->cfg.head_dim * sizeof(float) + sizeof(float2));
    const size_t slots = chunk_slots(a, c.n, n_hg, slot_bytes, &args.few_chunks, &args.unit_chunks);
    return place_scratch(a, args, counters_bytes(n_hg), slots, c);
}

// 8-bit cache rows: one kernel, which in a decode step also quantises and appends the new row, merges
// chunks and publishes the new lengths.
static int launch_fp8(s3_arena *a, const AttnCall &c) {
    const int D = a->cfg.head_dim, H = a->cfg.n_heads;
    int threads = 0;
    attn_fn fn = s3i_pick_fp8(a->cfg.act_dtype, D, a->variant, &threads);
    if (!fn) return S3_ERR_INVALID;
    AttnArgs args = common_args(a, c, H, H, a->chunk > 0 ? a->chunk : 1024);
    const int n_hg = (H + 1024 / D - 1) / (1024 / D);  // head groups: 1024/D heads per 128-bit wave load of bytes
    int rc = place_chunk_scratch(a, args, n_hg, c);
    if (rc != S3_OK) return rc;
    if (on_few_kernel(a, c.n, n_hg)) return launch_few(a, args, n_hg, true, c);
    const size_t dyn_lds = batch_view_lds(c.n, args.ncls);
    int blocks = 0;
    rc = stride_grid(a, (const void *)fn, threads, dyn_lds, c.n > 128 ? 2 : 1, &blocks);
    if (rc != S3_OK) return rc;
    return launch_attn_kernels(a, fn, blocks, threads, dyn_lds, c.stream, args, 0, !c.static_scratch);  // the kernel merges by itself
}

// Mean rows of a context below which a dynamic list has one length class.  The rows decide, on the device, and not the
// entry point.  One class against four, two layers, append + attention: 12 x 128, 300 contexts of 20..300 rows 64.3 us and
// 59.2, 953 of 100..200 152.6 and 156.4, 953 of 2..25 48.1 and 51.5; 32 x 128, 1000 of 5..60 134.9 and 144.6; 16 x 256,
// 512 of 40..1600 531 and 513.  (A batch beyond 512 that is found to need the classes pays 0.5 us for the look.)
#define S3_CLASS_ROWS 128
// Shared by s3_decode_attention and s3_decode_step (with_append: the kernel also appends and publishes the new
// lengths).
static int launch_attention(s3_arena *a, const AttnCall &c) {
    if (a->cfg.n_kv_heads < a->cfg.n_heads) return launch_gqa(a, c);
    if (a->cfg.kv_dtype == S3_E4M3) return launch_fp8(a, c);
    const int D = a->cfg.head_dim, H = a->cfg.n_heads;
    // Defaults from sweeps on MI355X: large chunks keep most contexts in one piece (no cross-workgroup
    // merge), eight waves share an item's rows evenly, each with two batches of two rows in flight
    // alternately (1 % ahead of one batch of four rows on the ragged batch of 64, level on the others).
    const int variant = a->variant >= 0 ? a->variant : c.n > 128 ? s3i_default_variant_large() : s3i_default_variant();
    attn_fn fn = pick_kernel(a->cfg.kv_dtype, D, variant);
    if (!fn) return S3_ERR_INVALID;
    const int GH = heads_per_load(D);
    const int n_hg = (H + GH - 1) / GH;
    AttnArgs args = common_args(a, c, H, H, a->chunk > 0 ? a->chunk : 1024);
    // A dynamic work list is a longest-processing-time schedule only if the long items come first: four length classes
    // whatever the batch size (with a fixed stride, large batches did better without the classes' prologue), unless the
    // contexts are so short that the prologue outweighs the order; see S3_CLASS_ROWS.
    if (a->ncls <= 0 && s3i_variant_dynamic(variant)) {
        args.ncls = 4;
        while (args.ncls > 1 && batch_view_lds(c.n, args.ncls) > (size_t)96 * 1024) args.ncls--;
        args.class_rows = S3_CLASS_ROWS;
    }
    int rc = place_chunk_scratch(a, args, n_hg, c);
    if (rc != S3_OK) return rc;
    if (on_few_kernel(a, c.n, n_hg)) return launch_few(a, args, n_hg, false, c);
    if (args.unit_chunks > 0) fn = pick_kernel(a->cfg.kv_dtype, D, S3_UNIT_VARIANT);
    const int threads = s3i_variant_threads(variant);
    const size_t view = batch_view_lds(c.n, args.ncls);
    const size_t dyn_lds = s3i_variant_ring_bytes(variant) ? ((view + 15) & ~(size_t)15) + s3i_variant_ring_bytes(variant) : view;
    int blocks = 0;
    // fixed stride: large batches balance better over two rounds of resident workgroups; a dynamic work list
    // needs exactly the resident ones
    const int rounds = s3i_variant_dynamic(variant) ? 1 : c.n > 128 ? 2 : 1;
    // the shapes that carry the row stream across items keep a compute unit's memory pipeline full from one
    // workgroup; a second resident one (their register count admits it) measured 2 % slower
    rc = stride_grid(a, (const void *)fn, threads, dyn_lds, rounds, &blocks, s3i_variant_stream(variant) ? 1 : 0);
    if (rc != S3_OK) return rc;
    return launch_attn_kernels(a, fn, blocks, threads, dyn_lds, c.stream, args, 0, !c.static_scratch);  // the kernel merges by itself
}

extern "C" int s3_decode_attention(s3_arena *a, int32_t layer, int32_t n, const void *q, const int64_t *slot_off,
                                   const int32_t *cur_len, void *out, int32_t out_dtype, float scale, void *stream) {
    if (!a || !a->base || layer < 0 || layer >= a->cfg.n_layers || n < 0 || n > S3_MAX_BATCH) return S3_ERR_INVALID;
    if (n == 0) return S3_OK;
    if (!q || !slot_off || !cur_len || !out || !aligned16(q) || !aligned16(out)) return S3_ERR_INVALID;
    if (out_dtype != S3_F32 && out_dtype != S3_F16 && out_dtype != S3_BF16) return S3_ERR_INVALID;
    const AttnCall c = {layer, n, q, slot_off, cur_len, out, out_dtype, scale, stream, false, nullptr, nullptr, nullptr, false};
    return launch_attention(a, c);
}

static int decode_step(s3_arena *a, int32_t layer, int32_t n, const int32_t *slot_id, const int32_t *pos_host,
                       const int64_t *slot_off, const int32_t *pos, const void *q, const void *k_new, const void *v_new,
                       void *out, int32_t out_dtype, float scale, int32_t *len_out, void *stream, bool static_scratch) {
    if (!a || !a->base || layer < 0 || layer >= a->cfg.n_layers || n < 0 || n > S3_MAX_BATCH) return S3_ERR_INVALID;
    if (n == 0) return S3_OK;
    if (!q || !k_new || !v_new || !slot_off || !pos || !out) return S3_ERR_INVALID;
    if (!aligned16(q) || !aligned16(k_new) || !aligned16(v_new) || !aligned16(out)) return S3_ERR_INVALID;
    if (len_out == pos) return S3_ERR_INVALID;  // other workgroups still read pos while len_out is written
    if (out_dtype != S3_F32 && out_dtype != S3_F16 && out_dtype != S3_BF16) return S3_ERR_INVALID;
    const int rc = check_slots_host(a, n, slot_id, pos_host);
    if (rc != S3_OK) return rc;
    const AttnCall c = {layer, n, q, slot_off, pos, out, out_dtype, scale, stream, true, k_new, v_new, len_out, static_scratch};
    return launch_attention(a, c);
}

extern "C" int s3_decode_step(s3_arena *a, int32_t layer, int32_t n, const int32_t *slot_id, const int32_t *pos_host,
                              const int64_t *slot_off, const int32_t *pos, const void *q, const void *k_new,
                              const void *v_new, void *out, int32_t out_dtype, float scale, int32_t *len_out,
                              void *stream) {
    return decode_step(a, layer, n, slot_id, pos_host, slot_off, pos, q, k_new, v_new, out, out_dtype, scale, len_out,
                       stream, false);
}

extern "C" int s3_decode_step_static(s3_arena *a, int32_t layer, int32_t n, const int32_t *slot_id,
                                     const int32_t *pos_host, const int64_t *slot_off, const int32_t *pos, const void *q,
                                     const void *k_new, const void *v_new, void *out, int32_t out_dtype, float scale,
                                     int32_t *len_out, void *stream) {
    return decode_step(a, layer, n, slot_id, pos_host, slot_off, pos, q, k_new, v_new, out, out_dtype, scale, len_out,
                       stream, true);
}

extern "C" int s3_kv_fill(s3_arena *a, int32_t slot_id, int32_t layer, int32_t first_row, int32_t n_rows,
                          const void *k_rows, const void *v_rows, void *stream) {
    const s3_slot *s = s3i_live_slot(a, slot_id);
    if (!s || !a->base || layer < 0 || layer >= a->cfg.n_layers || first_row < 0 || n_rows < 0) return S3_ERR_INVALID;
    if ((int64_t)first_row + n_rows > s->cap) return S3_ERR_SLOT_FULL;
    if (n_rows == 0) return S3_OK;
    if (!k_rows || !v_rows) return S3_ERR_INVALID;
    const size_t nbytes = (size_t)n_rows * a->row_bytes;
    const int64_t row0 = s->off + first_row;
    if (((uintptr_t)k_rows & 15) || ((uintptr_t)v_rows & 15)) return S3_ERR_INVALID;
    const size_t n16 = nbytes / 16;
    size_t blocks = (n16 + S3_FILL_U * 256 - 1) / (S3_FILL_U * 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(copy_pair_kernel, dim3((unsigned)blocks, 2), dim3(256), 0, (hipStream_t)stream,
                       (const char *)k_rows, a->plane(layer, 0) + row0 * a->row_bytes, (const char *)v_rows,
                       a->plane(layer, 1) + row0 * a->row_bytes, n16);
    HIP_TRY(hipGetLastError());
    return S3_OK;
}

// ---- evict to / restore from host memory (the paper's own misprediction path, section 3 and 4.3) ----
extern "C" int64_t s3_kv_evict_bytes(const s3_arena *a, int32_t len) {
    if (!a || len < 0 || len > a->cfg.max_len) return S3_ERR_INVALID;
    return (int64_t)2 * a->cfg.n_layers * len * a->row_bytes;
}

extern "C" int s3_kv_evict(s3_arena *a, int32_t slot_id, int32_t len, void *host_buf, void *stream) {
    const s3_slot *s = s3i_live_slot(a, slot_id);
    if (!s || !a->base || len < 0 || len > s->cap || (len > 0 && !host_buf)) return S3_ERR_INVALID;
    const size_t piece = (size_t)len * (size_t)a->row_bytes;
    const int planes = 2 * a->cfg.n_layers;
    for (int p = 0; p < planes && piece; p++)
        HIP_TRY(hipMemcpyAsync((char *)host_buf + (size_t)p * piece,
                               a->base + (int64_t)p * a->plane_bytes + s->off * a->row_bytes, piece,
                               hipMemcpyDeviceToHost, (hipStream_t)stream));
    return s3_kv_free(a, slot_id);
}

extern "C" int s3_kv_restore(s3_arena *a, int32_t predicted_len, int32_t len, const void *host_buf, int32_t *slot_id,
                             int64_t *slot_off, int32_t *slot_cap, void *stream) {
    if (!a || !a->base || !slot_id || len < 0 || predicted_len < len || (len > 0 && !host_buf)) return S3_ERR_INVALID;
    if (len > a->cfg.max_len) return S3_ERR_INVALID;
    int32_t id = -1, cap = 0;
    int64_t off = -1;
    const int admitted = s3_kv_alloc(a, 1, &predicted_len, &id, &off, &cap);
    if (admitted < 0) return admitted;
    if (admitted == 0) return S3_ERR_NOMEM;
    const size_t piece = (size_t)len * (size_t)a->row_bytes;
    const int planes = 2 * a->cfg.n_layers;
    for (int p = 0; p < planes && piece; p++) {
        const hipError_t e = hipMemcpyAsync(a->base + (int64_t)p * a->plane_bytes + off * a->row_bytes,
                                            (const char *)host_buf + (size_t)p * piece, piece, hipMemcpyHostToDevice,
                                            (hipStream_t)stream);
        if (e != hipSuccess) {
            (void)s3_kv_free(a, id);
            return hip_fail("hipMemcpyAsync(restore)", e);
        }
    }
    *slot_id = id;
    if (slot_off) *slot_off = off;
    if (slot_cap) *slot_cap = cap;
    return S3_OK;
}

// Rows [0, len) of every plane of a live slot to / from one contiguous device buffer laid out like the host
// buffer of s3_kv_evict: the device-side halves of an eviction and of a re-admission that cross the host link
// off the decode stream.  One launch each.
extern "C" int s3_kv_gather_rows(s3_arena *a, int32_t slot_id, int32_t len, void *dev_buf, void *stream) {
    const s3_slot *s = s3i_live_slot(a, slot_id);
    if (!s || !a->base || len < 0 || len > s->cap || (len > 0 && (!dev_buf || ((uintptr_t)dev_buf & 15)))) return S3_ERR_INVALID;
    const size_t piece = (size_t)len * (size_t)a->row_bytes;
    return s3i_launch_copy_planes(a->base + s->off * a->row_bytes, (char *)dev_buf, piece, (size_t)a->plane_bytes, piece,
                                  2 * a->cfg.n_layers, stream);
}

extern "C" int s3_kv_scatter_rows(s3_arena *a, int32_t slot_id, int32_t len, const void *dev_buf, void *stream) {
    const s3_slot *s = s3i_live_slot(a, slot_id);
    if (!s || !a->base || len < 0 || len > s->cap || (len > 0 && (!dev_buf || ((uintptr_t)dev_buf & 15)))) return S3_ERR_INVALID;
    const size_t piece = (size_t)len * (size_t)a->row_bytes;
    return s3i_launch_copy_planes((const char *)dev_buf, a->base + s->off * a->row_bytes, piece, piece, (size_t)a->plane_bytes,
                                  2 * a->cfg.n_layers, stream);
}

// A copy that deliberately occupies few compute units, and occupies them alone: `workgroups` workgroups of 1024
// threads move `bytes` with four 16-byte pieces in flight per thread, and every workgroup reserves nearly all of a
// compute unit's LDS so that no attention workgroup shares the unit with waves that wait on the host link.  For
// transfers between device memory and mapped pinned host memory beside the decode steps.  How many workgroups
// is the caller's trade: the copy's rate grows with them (measured device -> host: 1: 17 GB/s, 2: 31, 4: 43,
// 8: 55 = the link's rate), but so does the number of writes queued for the link at once, and beyond four the
// queue hurts everything else that runs - with eight, whatever kernel was running when a copy started (an
// attention launch, a doubling's copy) took 3-5 times as long for the copy's first milliseconds (attention
// launches of the 28-layer workload under a kernel trace: average 769-780 us, up to 3.5 ms; the runtime's own
// copy kernels, which spread over every unit: 821 us, up to 5.5 ms), with one, two or four: 746-748 us, none above
// 1.0 ms.  The decode loop uses two.
#define S3_LINK_THREADS 1024
#define S3_LINK_LDS (152 * 1024)
__global__ void __launch_bounds__(S3_LINK_THREADS) link_copy_kernel(const char *src, char *dst, size_t n16) {
    const u32x4 *s = (const u32x4 *)src;
    u32x4 *d = (u32x4 *)dst;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + 3 * stride < n16; i += 4 * stride) {
        const u32x4 a = s[i], b = s[i + stride], c = s[i + 2 * stride], e = s[i + 3 * stride];
        d[i] = a;
        d[i + stride] = b;
        d[i + 2 * stride] = c;
        d[i + 3 * stride] = e;
    }
    for (; i < n16; i += stride) d[i] = s[i];
}

extern "C" int s3_kv_link_copy(void *dst, const void *src, size_t bytes, int32_t workgroups, void *stream) {
    if (bytes == 0) return S3_OK;
    if (!dst || !src || (bytes & 15) || ((uintptr_t)dst & 15) || ((uintptr_t)src & 15)) return S3_ERR_INVALID;
    if (workgroups < 1 || workgroups > 1024) return S3_ERR_INVALID;
    static std::once_flag once;
    static hipError_t attr = hipSuccess;
    std::call_once(once, [] {
        attr = hipFuncSetAttribute((const void *)link_copy_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, S3_LINK_LDS);
    });
    if (attr != hipSuccess) return hip_fail("hipFuncSetAttribute(link_copy_kernel)", attr);
    hipLaunchKernelGGL(link_copy_kernel, dim3((unsigned)workgroups), dim3(S3_LINK_THREADS), S3_LINK_LDS, (hipStream_t)stream,
                       (const char *)src, (char *)dst, bytes / 16);
    HIP_TRY(hipGetLastError());
    return S3_OK;
}

extern "C" int s3_kv_read_rows(s3_arena *a, int32_t slot_id, int32_t layer, int32_t which, int32_t first_row,
                               int32_t n_rows, void *dst, void *stream) {
    const s3_slot *s = s3i_live_slot(a, slot_id);
    if (!s || !a->base || layer < 0 || layer >= a->cfg.n_layers || first_row < 0 || n_rows < 0 ||
        (which != 0 && which != 1))
        return S3_ERR_INVALID;
    if ((int64_t)first_row + n_rows > s->cap) return S3_ERR_INVALID;
    if (n_rows == 0) return S3_OK;
    if (!dst) return S3_ERR_INVALID;
    return s3i_launch_copy_planes(a->plane(layer, which) + (s->off + first_row) * a->row_bytes, (char *)dst,
                                  (size_t)n_rows * a->row_bytes, 0, 0, 1, stream);
}
