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

}  // namespace tkv
