// copy.hip -- retrieve scatter and store gather between staged chunks and
// paged KV blocks, for CDNA4 (gfx950).
//
// Vocabulary.  A segment is the B tokens of one layer's K or V plane that
// form one paged block: B*H*D*e contiguous bytes on both sides (32 KiB for
// block 16 x 8 heads x 128 dims x bf16).  A plane is the C/B segments of one
// (job, layer, K or V): contiguous in the staged chunk, one paged block each.
// A row is 1 KiB of contiguous memory, one 16-byte vector per lane of a wave.
//
// A window is V consecutive rows of a staged slot.  The staged side of a window
// is contiguous; on the paged side it covers parts of one or more segments, of
// one or two planes, whatever the segment size.
//
// Both directions run copy_window: one wave per window, T/64 consecutive
// windows of the launch's order (window.h) per workgroup, all loads of a window
// before its stores.  What bounds a copy is how the memory system takes its
// order of reads and writes, so the shapes differ in how much a wave moves and
// which windows are in flight together:
//
//   Store and streaming retrieve (no staged byte read twice): job-major order,
//   each XCD taking one contiguous range of it, non-temporal on both sides.
//   Large launches move 16 KiB per wave in 1024-lane workgroups; small ones
//   mostly 2 KiB per wave, so that every CU has work and the first store is
//   issued early (stream_shape in window.h has the sizes and times, and where
//   a streaming retrieve reads through the caches).
//
//   Retrieve where jobs share staged chunks: 4 KiB per wave (2 KiB in small
//   launches), 256-lane workgroups, in groups of windows (shared_shape in
//   window.h: 32 KiB to 1 MiB); a group of one job is followed by the same group
//   of the next job, and each XCD takes one contiguous range of that order.
//   Jobs that share a chunk (adjacent once the job list is grouped by slot) read
//   the group through one XCD's L2 while it is there, and a paged block is
//   written by workgroups that run together.  Loads are cached, paged writes
//   non-temporal.
//
//   Staged chunks in host memory: shapes of their own (window.h), since what
//   bounds those copies is the link.
//
// A further retrieve, the four-job-window retrieve (one segment of four
// consecutive jobs per 1024-lane workgroup), runs where a caller names it: 3.69
// to 3.83 ms against 3.18 to 3.65 for the windows at the 32-layer batch on three
// pools, 1.55 against 0.79 ms at 4 KiB segments.
//
// Generic path: any segment size that is a multiple of 16 bytes, one
// 256-lane workgroup per segment.

#include "internal.h"
#include "window.h"

namespace tkv {
namespace {

typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef int32_t v4i __attribute__((ext_vector_type(4)));
// Uniform reads through the scalar cache: loads from the constant address
// space with wave-uniform addresses become s_load instructions.
typedef const __attribute__((address_space(4))) v4i *const_job_ptr;
typedef const __attribute__((address_space(4))) int32_t *const_i32_ptr;

template <bool kNT>
__device__ __forceinline__ v4u load16(const v4u *p) {
    if constexpr (kNT) return __builtin_nontemporal_load(p);
    else return *p;
}

__device__ __forceinline__ bool job_ok(const CopyParams &p, const v4i jb) {
    return jb.x >= 0 && jb.x < p.num_slots && jb.y >= 0 && jb.y < p.num_reqs && jb.z >= 0 &&
           ((int64_t)jb.z + 1) * p.nseg <= p.bt_stride;
}

__device__ __forceinline__ bool blk_ok(const CopyParams &p, int32_t blk) {
    return blk >= 0 && blk < p.num_blocks;
}

// --------------------------------------------------------------------------
// Window copy.  Bound by the memory system: ~5.8-6.0 TB/s (read + write) for a
// large store of 32 KiB segments and 5.3-5.6 TB/s for a retrieve, which is what
// dense copies in the same shapes reach.
//
// Lane i of a wave looks up the paged address of the i-th segment that the
// window touches; rows then take their segment's address from that lane
// (kRow): 2, the first lane's for the whole window, where it lies in one
// segment; 1, by v_readlane, where a row never crosses a segment (segments of
// whole KiB); 0, lane by lane through ds_bpermute.  So any segment of at least
// kMinWindowSeg bytes fills its lanes, where one workgroup per segment leaves
// three of four waves of a 1 KiB segment without work: 512 jobs of 1 KiB
// segments store in 0.19 ms (one workgroup per segment: 0.75 ms), retrieve with
// shared chunks (1,422 jobs) in 0.37 ms (2.07 ms).
//
// The division of a row's vector index by the segment size is a multiply by
// magic = ceil(2^32 / segv), exact while index * (magic * segv - 2^32) < 2^32:
// the index is below segv + 1024 and the bracket below segv, so it holds for
// segv <= 32768 (kMaxWindowSeg).
// --------------------------------------------------------------------------
// Modes (plain numbers, so that a profiler's kernel names show them).
constexpr int kWinStore = 0, kWinStream = 1, kWinShared = 2;

template <int T, int V, int kMode, int kRow>
__device__ __forceinline__ void copy_window(const CopyParams &p, const WindowParams &w) {
    static_assert(V * 64 <= 1024, "the bound of magic and the lane table allow 1024 vectors a window");
    constexpr uint32_t W = T / 64;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t jobs = (uint32_t)p.num_jobs;
    const uint32_t per_xcd = window_wgs_per_xcd(w.total, W);
    for (uint32_t b = blockIdx.x; b < per_xcd * kXcds; b += gridDim.x) {
        const uint32_t g = window_of_wave(b, wave, W, per_xcd);
        if (g >= w.total) continue;
        uint32_t q = 0, wi = 0;
        window_at(w, jobs, kMode != kWinShared, g, q, wi);
        const uint32_t v0 = wi * (V * 64);   // first vector of the window in its slot
        if (v0 >= w.slotv) continue;
        const v4i jb = ((const_job_ptr)p.jobs)[q];
        if (!job_ok(p, jb)) continue;

        const uint32_t s0 = v0 / w.segv;
        const uint32_t rel0 = v0 - s0 * w.segv;
        uint32_t base_lo = 0, base_hi = 0;   // lane i: paged address of segment s0 + i, 0 where nothing is copied
        const uint32_t s = s0 + lane;
        if (s < w.nsegs && s * w.segv < v0 + V * 64) {
            const uint32_t pl = s / (uint32_t)p.nseg;   // layer * 2 + plane
            const int32_t blk = p.bt[(int64_t)jb.y * p.bt_stride + (int64_t)jb.z * p.nseg + (s - pl * p.nseg)];
            if (blk_ok(p, blk)) {
                const uint64_t a = (uint64_t)(p.layers[pl >> 1] + (int64_t)(pl & 1) * p.kv_stride +
                                              (int64_t)blk * p.block_stride);
                base_lo = (uint32_t)a;
                base_hi = (uint32_t)(a >> 32);
            }
        }
        // paged address of this lane's vector in row k, or null
        auto paged = [&](int k) -> v4u * {
            uint32_t lo, hi, off;
            if constexpr (kRow == 2) {
                off = rel0 + k * 64 + lane;
                lo = __builtin_amdgcn_readfirstlane(base_lo);
                hi = __builtin_amdgcn_readfirstlane(base_hi);
            } else if constexpr (kRow == 1) {
                const uint32_t rel = rel0 + k * 64;
                const uint32_t j = (uint32_t)(((uint64_t)rel * w.magic) >> 32);
                off = rel - j * w.segv + lane;
                lo = __builtin_amdgcn_readlane(base_lo, j);
                hi = __builtin_amdgcn_readlane(base_hi, j);
            } else {
                const uint32_t rel = rel0 + k * 64 + lane;
                const uint32_t j = __umulhi(rel, w.magic);
                off = rel - j * w.segv;
                lo = __builtin_amdgcn_ds_bpermute(j << 2, base_lo);
                hi = __builtin_amdgcn_ds_bpermute(j << 2, base_hi);
            }
            v4u *base = reinterpret_cast<v4u *>(((uint64_t)hi << 32) | lo);
            return base && v0 + k * 64 + lane < w.slotv ? base + off : nullptr;
        };
        v4u *stg = reinterpret_cast<v4u *>(p.staging + (int64_t)jb.x * p.slot_bytes) + v0 + lane;
        v4u r[V];
        if constexpr (kMode == kWinStore) {
            uint32_t copied = 0;
#pragma unroll
            for (int k = 0; k < V; ++k)
                if (const v4u *src = paged(k)) {
                    copied |= 1u << k;
                    r[k] = __builtin_nontemporal_load(src);
                }
#pragma unroll
            for (int k = 0; k < V; ++k)
                if ((copied >> k) & 1) __builtin_nontemporal_store(r[k], stg + k * 64);
        } else {
            // a segment whose block id is invalid is read but not written
#pragma unroll
            for (int k = 0; k < V; ++k)
                if (v0 + k * 64 + lane < w.slotv) r[k] = load16<kMode == kWinStream>(stg + k * 64);
#pragma unroll
            for (int k = 0; k < V; ++k)
                if (v4u *dst = paged(k)) __builtin_nontemporal_store(r[k], dst);
        }
    }
}

// Large launches: store, streaming retrieve (16 vectors a lane) and the
// retrieve with shared chunks (4 vectors a lane).
template <int T, int kRow, bool kRetrieve>
__global__ __launch_bounds__(T) void group_copy_kernel(CopyParams p, WindowParams w) {
    copy_window<T, 16, kRetrieve ? kWinStream : kWinStore, kRow>(p, w);
}

template <int kRow>
__global__ __launch_bounds__(256) void retrieve_unit_kernel(CopyParams p, WindowParams w) {
    copy_window<256, 4, kWinShared, kRow>(p, w);
}

// The other shapes: launches of up to 1 GiB.
template <int T, int V, int kMode, int kRow>
__global__ __launch_bounds__(T) void small_copy_kernel(CopyParams p, WindowParams w) {
    copy_window<T, V, kMode, kRow>(p, w);
}

// --------------------------------------------------------------------------
// Retrieve, windows of four jobs (R rows of 4 KiB per segment): a unit is
// (layer, plane, window of jobs 4w..4w+3, segment s), copied by one 1024-lane
// workgroup whose quarter j moves job 4w+j's segment s.  Jobs of a window that
// share a staged chunk load the same bytes at the same time, so one load comes
// from memory and the others from L2.  Units are (layer, plane)-major, then
// groups of kQuadGroup windows (32 jobs), then segment, then window, in plain
// dispatch order: the workgroups in flight write one segment of 32 jobs at a
// time.  (Window-major order, and groups of 1, 2 or 4 windows, measured 2-7 %
// slower.)
// --------------------------------------------------------------------------
constexpr int kQuadGroup = 8;

template <int R>
__global__ __launch_bounds__(1024) void retrieve_quad_kernel(CopyParams p) {
    constexpr int T = 256;
    // the quarter is uniform within each 64-lane wave
    const int j = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int tid = threadIdx.x & (T - 1);
    const int64_t ngroup = ((int64_t)p.num_jobs + 4 * kQuadGroup - 1) / (4 * kQuadGroup);
    const int64_t units = ngroup * kQuadGroup * p.nseg * p.L * 2;
    for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
        const int32_t h = (int32_t)(u % kQuadGroup);
        const int64_t t = u / kQuadGroup;
        const int32_t s = (int32_t)(t % p.nseg);
        const int64_t g = t / p.nseg;
        const int64_t q = ((g % ngroup) * kQuadGroup + h) * 4 + j;
        const int64_t pl = g / ngroup;   // layer * 2 + plane
        if (q >= p.num_jobs) continue;
        const v4i jb = ((const_job_ptr)p.jobs)[q];
        if (!job_ok(p, jb)) continue;
        const int32_t blk = ((const_i32_ptr)p.bt)[(int64_t)jb.y * p.bt_stride + (int64_t)jb.z * p.nseg + s];
        if (!blk_ok(p, blk)) continue;
        const int32_t kv = (int32_t)(pl & 1);
        const int32_t l = (int32_t)(pl >> 1);
        const v4u *src = reinterpret_cast<const v4u *>(p.staging + (int64_t)jb.x * p.slot_bytes +
                                                       (pl * p.nseg + s) * p.seg_bytes) + tid;
        v4u *dst = reinterpret_cast<v4u *>(p.layers[l] + kv * p.kv_stride + (int64_t)blk * p.block_stride) + tid;
        v4u a[R];
#pragma unroll
        for (int r = 0; r < R; ++r) a[r] = src[r * T];
#pragma unroll
        for (int r = 0; r < R; ++r) __builtin_nontemporal_store(a[r], dst + r * T);
    }
}

// --------------------------------------------------------------------------
// Generic path: one 256-lane workgroup per segment, any multiple of 16 bytes.
// --------------------------------------------------------------------------
constexpr int kGenThreads = 256;
constexpr int kGenUnroll = 8;

template <bool kSrcNT>
__device__ __forceinline__ void copy_segment(v4u *__restrict__ dst, const v4u *__restrict__ src, int64_t bytes,
                                             int tid) {
    const int64_t n = bytes >> 4;
    for (int64_t base = 0; base < n; base += (int64_t)kGenThreads * kGenUnroll) {
        v4u r[kGenUnroll];
#pragma unroll
        for (int k = 0; k < kGenUnroll; ++k) {
            const int64_t v = base + k * kGenThreads + tid;
            if (v < n) r[k] = load16<kSrcNT>(src + v);
        }
#pragma unroll
        for (int k = 0; k < kGenUnroll; ++k) {
            const int64_t v = base + k * kGenThreads + tid;
            if (v < n) __builtin_nontemporal_store(r[k], dst + v);
        }
    }
}

template <bool kRetrieve>
__global__ __launch_bounds__(kGenThreads) void copy_generic_kernel(CopyParams p) {
    const int tid = threadIdx.x;
    const int64_t total = (int64_t)p.num_jobs * p.L * 2 * p.nseg;
    for (int64_t g = blockIdx.x; g < total; g += gridDim.x) {
        const int64_t q = g % p.num_jobs;
        int64_t t = g / p.num_jobs;
        const int32_t i = (int32_t)(t % p.nseg);
        t /= p.nseg;
        const int32_t kv = (int32_t)(t & 1);
        const int32_t l = (int32_t)(t >> 1);
        const v4i jb = ((const_job_ptr)p.jobs)[q];
        if (!job_ok(p, jb)) continue;
        const int32_t blk = ((const_i32_ptr)p.bt)[(int64_t)jb.y * p.bt_stride + (int64_t)jb.z * p.nseg + i];
        if (!blk_ok(p, blk)) continue;
        char *stg = p.staging + (int64_t)jb.x * p.slot_bytes + (((int64_t)l * 2 + kv) * p.nseg + i) * p.seg_bytes;
        char *pg = p.layers[l] + kv * p.kv_stride + (int64_t)blk * p.block_stride;
        if constexpr (kRetrieve)
            copy_segment<false>(reinterpret_cast<v4u *>(pg), reinterpret_cast<const v4u *>(stg), p.seg_bytes, tid);
        else
            copy_segment<true>(reinterpret_cast<v4u *>(stg), reinterpret_cast<const v4u *>(pg), p.seg_bytes, tid);
    }
}

constexpr int64_t kMaxGrid = int64_t(1) << 30;

unsigned grid_of(int64_t items) { return (unsigned)(items < kMaxGrid ? items : kMaxGrid); }

// Workgroups of a launch: one per T/64 windows, at most 2^31 work-items (the rest by the kernels' grid-stride loops).
template <int T>
unsigned window_grid(uint32_t total) {
    const uint32_t grid = window_wgs_per_xcd(total, T / 64) * kXcds;
    constexpr uint32_t cap = (1u << 31) / T;
    return grid < cap ? grid : cap;
}

#define TKV_LAUNCH_WINDOW(T, kernel)                                                                          \
    hipLaunchKernelGGL((kernel), dim3(window_grid<T>(w.total)), dim3(T), 0, s, p, w)

template <int T, bool kRetrieve>
void launch_group(const CopyParams &p, const WindowParams &w, hipStream_t s) {
    if constexpr (T == 1024) {   // (256-lane workgroups run segments below 16 KiB)
        if (p.seg_bytes % (16 << 10) == 0) {
            TKV_LAUNCH_WINDOW(T, (group_copy_kernel<T, 2, kRetrieve>));
            return;
        }
    }
    if (p.seg_bytes % 1024 == 0)
        TKV_LAUNCH_WINDOW(T, (group_copy_kernel<T, 1, kRetrieve>));
    else
        TKV_LAUNCH_WINDOW(T, (group_copy_kernel<T, 0, kRetrieve>));
}

template <int T, int V, int kMode>
void launch_small(const CopyParams &p, const WindowParams &w, hipStream_t s) {
    if (p.seg_bytes % 1024 == 0)
        TKV_LAUNCH_WINDOW(T, (small_copy_kernel<T, V, kMode, 1>));
    else
        TKV_LAUNCH_WINDOW(T, (small_copy_kernel<T, V, kMode, 0>));
}

// Whether a device-accessible pointer maps host memory (0.24 us on the host).
bool in_host_memory(const void *ptr) {
    hipPointerAttribute_t at;
    if (hipPointerGetAttributes(&at, ptr) != hipSuccess) {
        (void)hipGetLastError();   // memory that HIP did not allocate
        return false;
    }
    return at.type == hipMemoryTypeHost;
}

double payload_of(const CopyParams &p) { return (double)p.slot_bytes * p.num_jobs; }

template <bool kRetrieve>
bool launch_stream_shape(const CopyParams &p, const CopyShape &c, hipStream_t s) {
    constexpr int kMode = kRetrieve ? kWinStream : kWinStore;
    WindowParams w;
    if (!window_params(p.seg_bytes, p.slot_bytes, p.num_jobs, c.vectors, c.group, w)) return false;
    if (kRetrieve && c.cached && c.vectors == 2) launch_small<256, 2, kWinShared>(p, w, s);
    else if (kRetrieve && c.cached) launch_small<256, 8, kWinShared>(p, w, s);
    else if (c.vectors == 2) launch_small<256, 2, kMode>(p, w, s);
    else if (c.vectors == 8) launch_small<256, 8, kMode>(p, w, s);
    else if (c.threads == 512) launch_small<512, 16, kMode>(p, w, s);
    else if (kRetrieve && c.threads == 256) launch_group<256, true>(p, w, s);
    else launch_group<1024, kRetrieve>(p, w, s);
    return true;
}

template <bool kRetrieve>
bool launch_stream(const CopyParams &p, hipStream_t s) {
    const double payload = payload_of(p);
    const bool host = stream_asks_host(kRetrieve, payload) && in_host_memory(p.staging);
    return launch_stream_shape<kRetrieve>(p, stream_shape(kRetrieve, payload, p.seg_bytes, host), s);
}

bool launch_shared(const CopyParams &p, hipStream_t s) {
    const double payload = payload_of(p);
    const bool host = (p.num_jobs == 1 || !shared_small(payload, p.seg_bytes)) && in_host_memory(p.staging);
    if (host && p.num_jobs == 1)
        return launch_stream_shape<true>(p, stream_shape(true, payload, p.seg_bytes, true), s);
    const CopyShape c = shared_shape(payload, p.seg_bytes, p.seg_bytes * p.nseg, host);
    WindowParams w;
    if (!window_params(p.seg_bytes, p.slot_bytes, p.num_jobs, c.vectors, c.group, w)) return false;
    if (c.vectors == 2)
        launch_small<256, 2, kWinShared>(p, w, s);
    else if (p.seg_bytes % 1024 == 0)
        TKV_LAUNCH_WINDOW(256, (retrieve_unit_kernel<1>));
    else
        TKV_LAUNCH_WINDOW(256, (retrieve_unit_kernel<0>));
    return true;
}

#undef TKV_LAUNCH_WINDOW

// Rows of `row_bytes` per segment if the segment is 1, 2, 4, 8 or 16 rows.
int rows_of(int64_t seg_bytes, int64_t row_bytes) {
    if (seg_bytes % row_bytes) return 0;
    const int64_t r = seg_bytes / row_bytes;
    return (r == 1 || r == 2 || r == 4 || r == 8 || r == 16) ? (int)r : 0;
}

template <int R>
void launch_retrieve_quad_r(const CopyParams &p, hipStream_t s) {
    const int64_t units = ((int64_t)p.num_jobs + 4 * kQuadGroup - 1) / (4 * kQuadGroup) * kQuadGroup * p.nseg * p.L * 2;
    hipLaunchKernelGGL(retrieve_quad_kernel<R>, dim3(grid_of(units)), dim3(1024), 0, s, p);
}

bool launch_retrieve_quad(const CopyParams &p, hipStream_t s) {
    switch (rows_of(p.seg_bytes, 256 * 16)) {
    case 1: launch_retrieve_quad_r<1>(p, s); return true;
    case 2: launch_retrieve_quad_r<2>(p, s); return true;
    case 4: launch_retrieve_quad_r<4>(p, s); return true;
    case 8: launch_retrieve_quad_r<8>(p, s); return true;
    case 16: launch_retrieve_quad_r<16>(p, s); return true;
    default: return false;
    }
}

}  // namespace

hipError_t launch_copy(const CopyParams &p, CopyKind kind, hipStream_t stream) {
    if (p.total_segs <= 0) return hipSuccess;
    (void)hipGetLastError();   // clear an error left by an unrelated earlier call
    const bool retrieve = kind != kStore;
    const bool fast = kind == kRetrieve         ? launch_shared(p, stream)
                      : kind == kRetrieveQuad   ? launch_retrieve_quad(p, stream) || launch_shared(p, stream)
                      : kind == kRetrieveStream ? launch_stream<true>(p, stream)
                                                : launch_stream<false>(p, stream);
    if (!fast) {
        const unsigned grid = grid_of(p.total_segs);
        if (retrieve)
            hipLaunchKernelGGL(copy_generic_kernel<true>, dim3(grid), dim3(kGenThreads), 0, stream, p);
        else
            hipLaunchKernelGGL(copy_generic_kernel<false>, dim3(grid), dim3(kGenThreads), 0, stream, p);
    }
    return hipGetLastError();
}

}  // namespace tkv
