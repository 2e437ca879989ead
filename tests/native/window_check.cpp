// Check of the window copies' order (paper_2609_35065_amd/csrc/window.h) over
// random launches: every window of every job is taken by exactly one wave, and
// no more waves than one a group (and the rounding of the grid) are without
// work, however small the slot.  Built by tests/test_window_order.py.
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <random>
#include <vector>

#include "window.h"

#define CHECK(c)                                                     \
    do {                                                             \
        if (!(c)) {                                                  \
            fprintf(stderr, "check failed line %d: %s (seed %llu)\n", __LINE__, #c, (unsigned long long)seed); \
            return 1;                                                \
        }                                                            \
    } while (0)

static int run(uint64_t seed) {
    std::mt19937_64 rng(seed);
    auto pick = [&](std::vector<int64_t> v) { return v[rng() % v.size()]; };
    const int V = (int)pick({2, 4, 8, 16});
    const uint32_t W = (uint32_t)pick({4, 8, 16});
    const int64_t seg = pick({512, 528, 1024, 1040, 4096, 7936, 20480, 32768, 65536, 524288});
    const int64_t nsegs = 1 + (int64_t)(rng() % (uint64_t)std::max<int64_t>(1, (256 << 10) / seg));
    const int64_t slot = seg * 2 * nsegs;
    const int64_t jobs = 1 + (int64_t)(rng() % 60);
    const int64_t group = pick({0, 1, 4, 5, 16, 32, 128, 256});
    tkv::WindowParams w;
    CHECK(tkv::window_params(seg, slot, jobs, V, group, w));
    const uint32_t nwin = (uint32_t)((slot / 16 + V * 64 - 1) / (V * 64));
    CHECK(w.nsegs == 2 * nsegs && w.total % jobs == 0 && w.total % w.group == 0);
    const int64_t ngroups = w.total / w.group / jobs;
    CHECK(group ? w.group <= group : ngroups == 1);
    CHECK((int64_t)w.total < (nwin + ngroups) * jobs);   // less than a window a group without work
    std::vector<int> seen((size_t)(jobs * nwin), 0);
    const uint32_t per_xcd = tkv::window_wgs_per_xcd(w.total, W);
    CHECK(per_xcd * tkv::kXcds * W < w.total + (tkv::kXcds + 1) * W);
    // a grid of one workgroup per item, or a capped one with the kernels' stride
    const uint32_t grid = (rng() & 1) ? per_xcd * tkv::kXcds : std::min<uint32_t>(per_xcd, 2) * tkv::kXcds;
    for (uint32_t b0 = 0; b0 < grid; ++b0)
        for (uint32_t b = b0; b < per_xcd * tkv::kXcds; b += grid)
            for (uint32_t wave = 0; wave < W; ++wave) {
                const uint32_t g = tkv::window_of_wave(b, wave, W, per_xcd);
                if (g >= w.total) continue;
                uint32_t q = 0, wi = 0;
                tkv::window_at(w, (uint32_t)jobs, group == 0, g, q, wi);
                CHECK(q < jobs);
                if (wi >= nwin) continue;
                CHECK(!seen[(size_t)q * nwin + wi]++);
            }
    for (int s : seen) CHECK(s == 1);
    return 0;
}

int main() {
    uint64_t seed = 0;
    for (; seed < 4000; ++seed)
        if (run(seed)) return 1;
    // limits: segment size, vector indexes of a slot, windows of a launch
    tkv::WindowParams w;
    CHECK(!tkv::window_params(496, 992, 1, 2, 0, w) && !tkv::window_params(528 << 10, 1056 << 10, 1, 2, 0, w));
    CHECK(tkv::window_params(1 << 16, int64_t(1) << 34, 1, 4, 128, w));
    CHECK(!tkv::window_params(1 << 16, (int64_t(1) << 34) + (1 << 17), 1, 4, 128, w));
    CHECK(tkv::window_params(1024, 2048, 0x7fffff00, 2, 16, w) && w.total == 0x7fffff00u);
    CHECK(!tkv::window_params(1024, 2048, 0x7fffff01, 2, 16, w));
    // launch shapes: with the chunks in host memory a retrieve of up to 48 MiB reads 16 KiB a wave, other small
    // copies move 2 KiB a wave, and jobs that share a chunk take groups of 32 KiB up to 512 MiB and of 16 KiB
    // above; the question is asked wherever the answer matters
    for (double mib = 0.5; mib < 4096; mib *= 1.1)
        for (int64_t seg : {1024, 20480, 32768, 65536})
            for (int retrieve = 0; retrieve < 2; ++retrieve) {
                const double bytes = mib * tkv::kMiB;
                const tkv::CopyShape d = tkv::stream_shape(retrieve, bytes, seg, false);
                const tkv::CopyShape h = tkv::stream_shape(retrieve, bytes, seg, true);
                if (mib <= 96) CHECK(h.vectors == (retrieve && mib <= 48 ? 16 : 2));
                if (!tkv::stream_asks_host(retrieve, bytes)) CHECK(d.threads == h.threads && d.vectors == h.vectors);
                const tkv::CopyShape sh = tkv::shared_shape(bytes, seg, 16 * seg, true);
                const tkv::CopyShape sd = tkv::shared_shape(bytes, seg, 16 * seg, false);
                CHECK(sh.vectors == (mib <= 512 ? 2 : 4) && sh.group == (mib <= 512 ? 16 : 4));
                if (tkv::shared_small(bytes, seg)) CHECK(sh.vectors == sd.vectors && sh.group == sd.group);
                // cached loads: from 24 to 256 MiB of segments that are not 4 KiB x 2^n
                CHECK(d.cached == (retrieve && (seg == 1024 || seg == 20480) && mib > 24 && mib <= 256));
                CHECK((!d.cached || d.vectors == (mib > 48 ? 2 : 8)) && !(h.cached && mib <= 96));
                // groups (4 KiB a wave): 64 KiB up to 1 GiB of small segments, then no more than a plane, unless
                // it is smaller than 128 KiB
                if (seg < 32768 && !tkv::shared_small(bytes, seg))
                    CHECK(sd.vectors == 4 && sd.group == (mib <= 1024 ? 16 : seg == 20480 ? 80 : 128));
                if (seg >= 32768) CHECK(sd.vectors == 4 && sd.group == (seg == 32768 ? 128 : 256));
                CHECK(d.group == 0 && h.group == 0 && sd.group > 0 && sh.group > 0);
            }
    CHECK(tkv::shared_shape(3e9, 8192, 128 << 10, false).group == 64);
    CHECK(tkv::shared_shape(3e9, 16384, 256 << 10, false).group == 64);
    puts("window check ok");
    return 0;
}
