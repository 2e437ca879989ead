// window.h -- which windows a window copy consists of and in what order its
// waves take them (the kernels are in copy.hip).  Plain C++ (no HIP header),
// constexpr where the kernels call it, so that the order can be tested on its
// own.
#pragma once

#include <stdint.h>

namespace tkv {

// Accelerator complex dies on MI355X; consecutive workgroups of a launch are
// dispatched to them round-robin.  Only performance depends on this value.
constexpr uint32_t kXcds = 8;

constexpr int64_t kMinWindowSeg = 512;   // 16 rows of 1 KiB touch at most 33 segments: one lane each
constexpr int64_t kMaxWindowSeg = 512 << 10;

struct WindowParams {
    uint32_t segv;     // 16-byte vectors of a segment
    uint32_t slotv;    // ... of a slot
    uint32_t nsegs;    // segments of a slot
    uint32_t magic;    // ceil(2^32 / segv)
    uint32_t group;    // consecutive windows of one job
    uint32_t total;    // windows of the launch: jobs * groups of a slot * group
};

// Parameters of a copy of `jobs` slots in windows of V * 64 vectors and groups
// of about `group` windows (0: a job's windows are one group).  A slot's
// windows are divided evenly over its groups, so that slots smaller than a
// group, or no multiple of one, leave fewer than one window a group without
// work (100,000 jobs on slots of 8 KiB: 0.16 ms; 1.78 ms with every slot
// padded to a 512 KiB group, 0.29 with one workgroup per segment).  False where the window copy does not apply: segment size, or vector
// indexes beyond 32 bits or window numbers beyond 31.
inline bool window_params(int64_t seg_bytes, int64_t slot_bytes, int64_t jobs, int V, int64_t group,
                          WindowParams &w) {
    if (seg_bytes < kMinWindowSeg || seg_bytes > kMaxWindowSeg) return false;
    const int64_t slotv = slot_bytes / 16;
    const int64_t nwin = (slotv + V * 64 - 1) / (V * 64);
    const int64_t ngroups = group ? (nwin + group - 1) / group : 1;
    const int64_t per_group = (nwin + ngroups - 1) / ngroups;
    // the grid rounds the windows up by at most 16 waves on each XCD
    if (slotv > (int64_t(1) << 30) || ngroups * per_group > ((int64_t(1) << 31) - 256) / jobs) return false;
    w.segv = (uint32_t)(seg_bytes / 16);
    w.slotv = (uint32_t)slotv;
    w.nsegs = (uint32_t)(slotv / w.segv);
    w.magic = (uint32_t)(((uint64_t(1) << 32) + w.segv - 1) / w.segv);
    w.group = (uint32_t)per_group;
    w.total = (uint32_t)(ngroups * per_group * jobs);
    return true;
}

// Workgroups of `waves` waves that each XCD takes: workgroup b runs on XCD
// b mod 8, which copies a contiguous range of the order.
constexpr uint32_t window_wgs_per_xcd(uint32_t total, uint32_t waves) {
    return ((total + waves - 1) / waves + kXcds - 1) / kXcds;
}

// Position in the order of wave `wave` of workgroup b (total or more: none).
constexpr uint32_t window_of_wave(uint32_t b, uint32_t wave, uint32_t waves, uint32_t per_xcd) {
    return ((b % kXcds) * per_xcd + b / kXcds) * waves + wave;
}

// Window `g` of the order: job q, window wi of its slot (may start past the
// slot's end).  Groups of one job follow the same groups of the job before.
constexpr void window_at(const WindowParams &w, uint32_t jobs, bool one_group, uint32_t g, uint32_t &q, uint32_t &wi) {
    const uint32_t h = g / w.group;
    q = h;
    wi = g - h * w.group;
    if (!one_group) {
        const uint32_t sw = h / jobs;
        q = h - sw * jobs;
        wi += sw * w.group;
    }
}

// ---------------------------------------------------------------------------
// Launch shapes: lanes a workgroup, vectors a lane (KiB a window) and windows a
// group (0: a job's windows are one group), from the launch's payload in bytes.
// cached: a streaming retrieve that reads through the caches.
// ---------------------------------------------------------------------------
struct CopyShape {
    int threads, vectors, group;
    bool cached = false;
};

constexpr double kMiB = 1 << 20;

// Store and streaming retrieve.  Median us over rotating buffers, 32 KiB
// segments unless noted, store / retrieve:
//   payload      2 KiB a wave    8 KiB          16 KiB, T=512   16 KiB, T=1024
//   8 MiB (4K)     6.0 /   5.8    8.1 /   6.4    12.2 /  11.3     13.6 /  14.0
//   32 MiB        14.7 /  14.3   13.3 /  13.6    16.9 /  14.7     18.4 /  17.5
//   96 MiB        36.7 /  37.0   37.7 /  40.9    33.4 /  35.0     41.9 /  42.6
//   128 MiB       49.4 /  46.7   54.8 /  55.5    53.4 /  57.6     48.6 /  53.1
//   512 MiB        182 /   183    203 /   207     199 /   209      197 /   204
//   8 GiB         2968 /  3147      -            2912 /  3164     2889 /  3131
//   8 GiB (64K)   2780 /  2875      -            2791 /  2754     2743 /  2695
// The edges (24, 48 and 96 MiB) are those of the table.  A CU holds 24 waves of
// the 16 KiB shape, so 96 MiB is one full set of them; above it short waves win
// until the launch is long enough for its start and end not to matter.  (A
// large streaming retrieve of segments below 16 KiB runs 256-lane workgroups:
// 796 against 792 us with 1024 lanes at 2 GiB of 4 KiB segments; the store
// keeps 1024: 738 against 745 us.)
//
// With the staged chunks in host memory the link sets the time.  Up to 96 MiB
// it wants reads that are issued early and together, 16 KiB a wave, and writes
// in short waves (us at 32 KiB segments, retrieve / store):
//   payload      2 KiB a wave    8 KiB          16 KiB, T=512   16 KiB, T=1024
//   16 MiB         324 /   338    333 /   354     314 /   364      306 /   364
//   36 MiB         696 /   728    734 /   738     703 /   764      700 /   782
//   60 MiB        1152 /  1184   1177 /  1189    1168 /  1243     1170 /  1258
// and above the shapes differ by 1 %.
//
// Non-temporal loads suit chunks that come from HBM; chunks that were just
// staged or stored may still lie in the 256 MiB memory-side cache, and cached
// loads read them faster (us, cached / non-temporal; cached 8 KiB a wave up to
// 48 MiB, then 2 KiB):
//   segments, payload        from HBM        from the cache
//   20 KiB,  40 MiB        19.2 / 18.4       16.0 / 17.4
//   20 KiB,  60 MiB        27.1 / 26.0       18.9 / 25.7
//   20 KiB, 130 MiB        56.0 / 54.8       35.2 / 54.3
//   32 KiB,  60 MiB        27.3 / 25.8       18.5 / 23.0
//   32 KiB,  90 MiB        38.1 / 35.7       25.0 / 32.0
// Segments of 4 KiB x 2^n (up to 256 KiB) take the non-temporal side of that
// trade, 5-7 % from HBM, where a reused chunk comes from in ordinary use; for
// other sizes that side is worth at most 8 % from HBM, mostly under 3 %, and
// costs up to 1.7 times from the cache (7,936-byte segments), so they take the
// cached side.
constexpr bool stream_cached(double payload, int64_t seg_bytes) {
    const bool pow2 = seg_bytes >= 4096 && seg_bytes <= (256 << 10) && (seg_bytes & (seg_bytes - 1)) == 0;
    return !pow2 && payload > 24 * kMiB && payload <= 256 * kMiB;
}

constexpr bool stream_asks_host(bool retrieve, double payload) {
    return payload <= 96 * kMiB && (retrieve || payload > 24 * kMiB);
}

constexpr CopyShape stream_shape(bool retrieve, double payload, int64_t seg_bytes, bool host) {
    if (host && payload <= 96 * kMiB)
        return retrieve && payload <= 48 * kMiB ? CopyShape{1024, 16, 0} : CopyShape{256, 2, 0};
    if (retrieve && stream_cached(payload, seg_bytes)) return {256, payload > 48 * kMiB ? 2 : 8, 0, true};
    if (payload > 1024 * kMiB) return {retrieve && seg_bytes < 16384 ? 256 : 1024, 16, 0};
    if (payload > 96 * kMiB || payload <= 24 * kMiB) return {256, 2, 0};
    if (payload > 48 * kMiB) return {512, 16, 0};
    return {256, 8, 0};
}

// Retrieve with shared chunks.  Large launches: groups of 512 KiB, or of 1 MiB
// where a plane's segments are more than 512 KiB: median ms by KiB a group, 4 KiB
// a wave, 8 requests per chunk:
//   segment    16    128    512   1024
//   4 KiB    1.08   0.98   0.93   0.94
//   16 KiB   2.11   1.95   1.58   1.59
//   20 KiB   1.68   1.67   1.60   1.60   (ragged sharing)
//   32 KiB   3.90   3.81   3.12   3.10
//   64 KiB   4.65   3.82   3.77   3.46
// Below, the pieces of a block are written far apart in time; 2 KiB and 8 KiB
// a wave are 5-40 % slower at these sizes.  Segments below 32 KiB with planes of
// 128 KiB to 512 KiB take groups of a plane, 256 KiB at least: within 1 % on
// lists grouped by slot and up to 1.5 times as fast on lists that are not, where
// a group is read again only after the same group of every other chunk (us by
// KiB a group, 8 requests per chunk):
//                     grouped: 64   128   256   512   not grouped: 64   128   256   512
//   8 KiB,  3 GiB             803   695   674   676               682   762   762   768
//   8 KiB,  6 GiB            1586  1382  1349  1339              1508  1540  1572  2395
//   16 KiB, 3 GiB             894   751   672   663               680   673   892  1149
// Smaller planes keep 512 KiB: 4 KiB segments, 6 GiB, 1.31 ms grouped against
// 1.37 in groups of 256 KiB, 2.36 against 2.32 not grouped.
//
// Launches of up to 1 GiB in segments below 32 KiB live in the caches.  Up to
// 512 MiB 2 KiB a wave in groups of 32 KiB is the fastest (500 MiB of 4 KiB
// segments, 8 requests per chunk: 90 us; 98 with 4 KiB a wave in groups of 64
// KiB, 103 in groups of 512 KiB), from there to 1 GiB 4 KiB a wave in groups of
// 64 KiB (us by requests per chunk, and 8 on a list that is not grouped):
//                                  1     2     8   not grouped
//   700 MiB of 4 KiB,  64 KiB    277   205   134   135
//                     512 KiB    281   208   144   162
//   600 MiB of 4 KiB,  64 KiB    238   170   117   117
//                      32 KiB    238   183   111   117
//   600 MiB of 16 KiB, 64 KiB    237   168   119   118
//                      32 KiB    236   193   110   115
//
// Staged chunks in host memory are read through the link: the jobs sharing a
// chunk should read the same bytes at the same time, yet write enough of a
// block together.  Groups of 16 KiB, 4 KiB a wave, do both (ms by KiB a group;
// 2,016 jobs of 32 MiB on 12 chunks, 2,568 on 24, 3,072 on 48; 32 KiB segments;
// with ragged sharing, 3,072 on 48 take 29.3 in groups of 16 KiB, 30.2 of 32):
//                2 KiB a wave: 8    32   128    4 KiB a wave: 16    32    64   512
//   on 12 chunks            13.9  12.3  12.7                12.5  12.4  12.4  13.5
//   on 24                   17.3  14.3  17.4                14.2  14.2  14.6  18.5
//   on 48                   28.3  28.2  32.6                28.2  28.1  33.3  33.1
// Launches of up to 512 MiB run 2 KiB a wave in groups of 32 KiB, as the small
// launches of small segments do (24 MiB, three jobs: 158 against 163 us).  A
// single job shares nothing and takes the streaming shape (8 MiB: 158 us; 191
// in groups).
constexpr bool shared_small(double payload, int64_t seg_bytes) {
    return payload <= 512 * kMiB && seg_bytes < 32768;
}

constexpr CopyShape shared_shape(double payload, int64_t seg_bytes, int64_t plane_bytes, bool host) {
    if (shared_small(payload, seg_bytes)) return {256, 2, 16};
    if (host) return payload <= 512 * kMiB ? CopyShape{256, 2, 16} : CopyShape{256, 4, 4};
    if (seg_bytes < 32768) {
        if (payload <= 1024 * kMiB) return {256, 4, 16};
        if (plane_bytes >= (128 << 10) && plane_bytes <= (512 << 10))
            return {256, 4, plane_bytes < (256 << 10) ? 64 : (int)((plane_bytes + 4095) / 4096)};
    }
    return {256, 4, plane_bytes > (512 << 10) ? 256 : 128};
}

}  // namespace tkv
