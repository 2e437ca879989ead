// hash.hip -- chained prefix hash and prefix lookup kernels for CDNA4 (gfx950).
//
// Hash.  h_{-1} = seed, h_b = M(h_{b-1} ^ d_b ^ G), d_b = sum_j M(word(j, tok))
// over the 16 tokens of block b, M = SplitMix64's finalizer.  The digests are
// independent and computed one block per lane; the chain is sequential, so
// its latency sets the rate: it runs on the scalar ALU of one wave per
// request.  One wave issues at most one instruction every four cycles, so what
// counts is how many it issues per block: 19 scalar ones (two 64-bit multiplies
// of six 32-bit instructions each, three xor-shifts, the xor with the digest),
// two v_readlane for the digest and, in the last tile of a request, two
// v_writelane for the hash.  In the tiles before it the chain keeps only every
// eighth hash and the workgroup's other waves, which also digest the next
// tile, compute the seven between, eight blocks to a lane: 4,096 blocks take
// 163 us (172 us with every hash kept by the chain).
//
// Lookup.  One wave per request probes up to 64 chunk keys at once in the
// device open-addressing table and turns the 64 hit flags into the length of
// the leading run of hits with one ballot and a count of trailing ones.  What
// bounds it is the longest chain of dependent loads of any key, so a lane
// reads kProbes consecutive entries at a time: in a table half full, walks of
// 15 to 30 entries occur among a few thousand keys (1,024 requests of 4 chunks:
// 7.4 us an entry at a time, 4.0 by four, 3.7 by eight).  Where full waves are
// many, the address rate bounds it instead, and most walks end at their first
// entry: those lanes read it alone first (4,096 requests of 64 present chunks
// 8.6 us, 11.3 without, 10.8 an entry at a time; of 256, 33 us, 42 and 40).  The
// rule asks for 2,048 requests, and 64 chunks of this one: 100,000 requests of 4
// chunks take 46 us with it and 41 without, 64 requests of 4,096 89 and 68; at
// 1,024 requests of 64 both take 3.7.  Smaller batches run a kernel without the
// question: it would cost them 0.3 of 2.8 us.

#include "internal.h"

namespace tkv {
namespace {

constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;
constexpr int kWave = 64;
constexpr int kHashThreads = 256;
constexpr int kProbes = 8;
constexpr int32_t kFirstRequests = 2048;
constexpr int64_t kFirstChunks = 64;
static_assert(64 % kProbes == 0, "tables have at least 64 entries, a power of two");

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ uint64_t readlane64(uint64_t v, int lane) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// Lane K of `old` takes the wave-uniform value `val` (v_writelane_b32 with
// an inline-constant lane number); the other lanes keep theirs.
template <int K>
__device__ __forceinline__ uint32_t writelane(uint32_t old, uint32_t val) {
    asm("v_writelane_b32 %0, %1, %2" : "+v"(old) : "s"(val), "n"(K));
    return old;
}

// Steps K..K+7 of the chain over a full group of 64 blocks, unrolled so that
// every lane number is an immediate.  The eight digests are read into scalar
// registers before the eight dependent steps, keeping v_readlane latency off
// the chain.  kAll: lane K+j takes hash K+j; otherwise lane K/8 takes the hash
// before step K.  The last group of a request runs its `left` blocks, a multiple
// of eight (62 blocks, 56 of them here: 5.8 us a launch, 7.3 as a loop of single
// steps).
template <bool kAll, int K>
struct ChainGroup {
    static __device__ __forceinline__ void run(uint64_t &h, uint64_t d, uint32_t &lo, uint32_t &hi, int left) {
        if (kAll && K >= left) return;
        uint64_t dk[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) dk[j] = readlane64(d, K + j);
        if constexpr (!kAll) {
            lo = writelane<K / 8>(lo, (uint32_t)h);
            hi = writelane<K / 8>(hi, (uint32_t)(h >> 32));
        }
        __builtin_amdgcn_sched_barrier(0);   // keep the reads ahead of the steps
        uint64_t hk[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            h = mix64(h ^ dk[j]);
            hk[j] = h;
        }
        if constexpr (kAll) Park<K, 0>::run(hk, lo, hi);
        ChainGroup<kAll, K + 8>::run(h, d, lo, hi, left);
    }
    template <int B, int J>
    struct Park {
        static __device__ __forceinline__ void run(const uint64_t *hk, uint32_t &lo, uint32_t &hi) {
            lo = writelane<B + J>(lo, (uint32_t)hk[J]);
            hi = writelane<B + J>(hi, (uint32_t)(hk[J] >> 32));
            Park<B, J + 1>::run(hk, lo, hi);
        }
    };
    template <int B>
    struct Park<B, 8> {
        static __device__ __forceinline__ void run(const uint64_t *, uint32_t &, uint32_t &) {}
    };
};
template <bool kAll>
struct ChainGroup<kAll, 64> {
    static __device__ __forceinline__ void run(uint64_t &, uint64_t, uint32_t &, uint32_t &, int) {}
};

__device__ __forceinline__ uint64_t block_digest(const int32_t *tp) {
    uint64_t d = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) d += mix64((uint64_t)(uint32_t)tp[j] + ((uint64_t)(j + 1) << 32));
    return d ^ kGamma;   // the chain's constant, folded in here, off the chain
}

// One 256-lane workgroup per request, blocks in tiles of 256.  The digests
// of a tile are independent: all four waves compute the first tile into LDS;
// afterwards wave 0 runs the chain over tile t while waves 1-3 digest tile
// t+1 into another LDS buffer and wave 1 fills in the hashes of tile t-1 from
// every eighth one.  The chain runs with wave-uniform values, so it executes on
// the scalar ALU: for each group of 64 blocks, lane k holds digest k and
// v_readlane moves it to scalar registers.  In the last tile v_writelane parks
// h_k in lane k, which then stores the group's 64 hashes in one write, so that
// nothing is left to do when the chain ends.  The last one to seven blocks run
// as single steps: where requests are many and short, workgroups wait for their
// turn on a CU and every step counts (100,000 requests of one block 91 us, 130
// with eight steps for it; 20,000 of nine 27 against 35).  All waves have the
// same priority: raised for the chain it holds up the digests that the other
// chains on the CU wait for (2,000 requests of 512 blocks 50 us, 61 with it).
__global__ __launch_bounds__(kHashThreads) void hash_kernel(const int32_t *__restrict__ tokens,
                                                           const int64_t *__restrict__ tok_off, uint64_t seed,
                                                           const int64_t *__restrict__ blk_off,
                                                           uint64_t *__restrict__ out) {
    __shared__ uint64_t dig[3][kHashThreads];
    __shared__ uint64_t every8[2][kHashThreads / 8];
    const int r = blockIdx.x;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);   // wave-uniform by construction
    const int lane = tid % kWave;
    const int64_t t0 = tok_off[r];
    const int64_t n = tok_off[r + 1] - t0;
    int64_t nb = n > 0 ? n / 16 : 0;
    const int64_t o0 = blk_off[r];
    const int64_t span = blk_off[r + 1] - o0;
    if (span < nb) nb = span > 0 ? span : 0;
    const int64_t ntiles = (nb + kHashThreads - 1) / kHashThreads;
    const int32_t *tk = tokens + t0;

    if (tid < nb) dig[0][tid] = block_digest(tk + (int64_t)tid * 16);
    __syncthreads();
    uint64_t h = seed;   // live in wave 0 only
    int cur = 0;         // t mod 3
    for (int64_t t = 0; t < ntiles; ++t) {
        const int64_t tb = t * kHashThreads;
        const int next = cur == 2 ? 0 : cur + 1, prev = cur == 0 ? 2 : cur - 1;
        if (wave == 0) {
            const uint64_t *dt = dig[cur];
            if (t + 1 < ntiles) {                      // a full tile
                for (int g = 0; g < kHashThreads; g += kWave) {
                    uint32_t lo = 0, hi = 0;
                    ChainGroup<false, 0>::run(h, dt[g + lane], lo, hi, kWave);
                    if (lane < 8) every8[t & 1][g / 8 + lane] = ((uint64_t)hi << 32) | lo;
                }
            } else {
                const int left = (int)(nb - tb);
                for (int g = 0; g < left; g += kWave) {
                    const uint64_t d = dt[g + lane];
                    const int cnt = left - g < kWave ? left - g : kWave;
                    uint32_t mine_lo = 0, mine_hi = 0;
                    ChainGroup<true, 0>::run(h, d, mine_lo, mine_hi, cnt & ~7);
                    for (int k = cnt & ~7; k < cnt; ++k) {
                        h = mix64(h ^ readlane64(d, k));
                        if (lane == k) {
                            mine_lo = (uint32_t)h;
                            mine_hi = (uint32_t)(h >> 32);
                        }
                    }
                    if (g + lane < left) out[o0 + tb + g + lane] = ((uint64_t)mine_hi << 32) | mine_lo;
                }
            }
        } else {
            if (t + 1 < ntiles) {
                const int64_t nt = tb + kHashThreads;
                for (int i = tid - kWave; i < kHashThreads; i += kHashThreads - kWave)
                    if (nt + i < nb) dig[next][i] = block_digest(tk + (nt + i) * 16);
            }
            if (t > 0 && wave == 1 && lane < kHashThreads / 8) {   // tile t-1, a full one
                uint64_t hb = every8[(t - 1) & 1][lane];
                uint64_t *o = out + o0 + tb - kHashThreads + lane * 8;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    hb = mix64(hb ^ dig[prev][lane * 8 + k]);
                    o[k] = hb;
                }
            }
        }
        if (t + 1 == ntiles) break;   // nothing reads the tiles any more
        __syncthreads();
        cur = next;
    }
}

template <bool kLarge>
__global__ __launch_bounds__(64) void lookup_kernel(const IndexEntry *__restrict__ table, int log2cap,
                                                    const uint64_t *__restrict__ bh,
                                                    const int64_t *__restrict__ blk_off, int32_t bpc,
                                                    const int64_t *__restrict__ chunk_off,
                                                    int32_t *__restrict__ chunk_slot,
                                                    int32_t *__restrict__ hit_chunks) {
    const int r = blockIdx.x;
    const int lane = threadIdx.x;
    const int64_t b0 = blk_off[r];
    int64_t nb = blk_off[r + 1] - b0;
    if (nb < 0) nb = 0;
    int64_t nc = nb / bpc;
    const int64_t c0 = chunk_off[r];
    const int64_t cspan = chunk_off[r + 1] - c0;
    if (cspan < nc) nc = cspan > 0 ? cspan : 0;
    const uint64_t mask = (uint64_t(1) << log2cap) - 1;

    const bool first_alone = kLarge && nc >= kFirstChunks;
    int32_t hits = 0;
    bool alive = true;
    for (int64_t base = 0; base < nc; base += 64) {
        const int64_t j = base + lane;
        int32_t slot = -1;
        if (j < nc) {
            const uint64_t key = bh[b0 + (j + 1) * bpc - 1];
            uint64_t pos = index_home(key, log2cap);
            bool open = true;
            if (first_alone) {
                const IndexEntry e = table[pos];
                if (e.state == kLive && e.key == key) slot = e.slot;
                open = e.state != kEmpty && slot < 0;
                pos = (pos + 1) & mask;
            }
            // bounded: a full table ends the walk (its size is a multiple of kProbes)
            for (uint64_t probe = 0; open && probe <= mask; probe += kProbes) {
                IndexEntry e[kProbes];
#pragma unroll
                for (int k = 0; k < kProbes; ++k) e[k] = table[(pos + k) & mask];
#pragma unroll
                for (int k = 0; k < kProbes; ++k) {
                    if (!open) continue;
                    if (e[k].state == kLive && e[k].key == key) slot = e[k].slot;
                    open = e[k].state != kEmpty && slot < 0;
                }
                pos = (pos + kProbes) & mask;
            }
            chunk_slot[c0 + j] = slot;
        }
        const uint64_t present = __ballot(j < nc && slot >= 0);
        if (alive) {
            const uint64_t missing = ~present;
            const int run = missing ? __builtin_ctzll(missing) : 64;
            hits += run;
            alive = (run == 64);
        }
    }
    if (lane == 0) hit_chunks[r] = hits;
}

}  // namespace

hipError_t launch_hash(const int32_t *tokens, const int64_t *tok_off, int32_t num_reqs, uint64_t seed,
                       const int64_t *blk_off, uint64_t *out, hipStream_t stream) {
    if (num_reqs <= 0) return hipSuccess;
    (void)hipGetLastError();
    hipLaunchKernelGGL(hash_kernel, dim3(num_reqs), dim3(kHashThreads), 0, stream, tokens, tok_off, seed, blk_off,
                       out);
    return hipGetLastError();
}

hipError_t launch_lookup(const IndexEntry *table, int log2cap, const uint64_t *block_hash,
                         const int64_t *blk_off, int32_t num_reqs, int32_t bpc, const int64_t *chunk_off,
                         int32_t *chunk_slot, int32_t *hit_chunks, hipStream_t stream) {
    if (num_reqs <= 0) return hipSuccess;
    (void)hipGetLastError();
    hipLaunchKernelGGL(num_reqs >= kFirstRequests ? lookup_kernel<true> : lookup_kernel<false>, dim3(num_reqs), dim3(64),
                       0, stream, table, log2cap, block_hash, blk_off, bpc, chunk_off, chunk_slot, hit_chunks);
    return hipGetLastError();
}

}  // namespace tkv
