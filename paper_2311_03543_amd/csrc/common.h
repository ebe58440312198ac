// Device helpers shared by the gfx950 kernels of libcompar.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace cmp {

constexpr int kXcds = 8;   // MI355X: 8 accelerator complex dies, 32 CUs each

// Workgroups are dispatched round-robin over the XCDs (id % 8 lands on XCD
// id % 8).  Renumber so that each XCD receives one contiguous range of tile
// ids: neighbouring tiles then share that XCD's L2.  Bijective on [0, nb).
__device__ __forceinline__ int xcd_remap(int b, int nb) {
    const int per = nb / kXcds, rem = nb % kXcds;
    const int x = b % kXcds, idx = b / kXcds;
    return x * per + (x < rem ? x : rem) + idx;
}

// Tile coordinates from a linear id with "grouped" ordering: walk `group`
// tile-rows at a time, column by column, so consecutive ids reuse the same
// B column panel and a small set of A row panels.
__device__ __forceinline__ void grouped_tile(int id, int tiles_m, int tiles_n, int group,
                                             int& tm, int& tn) {
    const int per_group = group * tiles_n;
    const int g = id / per_group;
    const int first_m = g * group;
    const int gm = (tiles_m - first_m) < group ? (tiles_m - first_m) : group;
    const int local = id - g * per_group;
    tm = first_m + local % gm;
    tn = local / gm;
}

// Panel images: the operand layout the MFMA kernels stream.  An operand with
// Mp rows (a multiple of 256) and Kb bytes of K per row (a multiple of 64) is
// cut into blocks of 256 rows x 64 bytes (16 KiB); block (rb, kb) starts at
// byte (rb * nkb + kb) * 16 KiB, nkb = Kb / 64.  The K extent of one 256-row
// panel is therefore contiguous, and one block is exactly one LDS slab of one
// pipeline stage, copied linearly.  Inside a block, row r occupies bytes
// [64 r, 64 r + 64) and its 16-byte chunk c sits at position c ^ ((r / 4) % 4):
// the LDS bank swizzle, applied once by the writer of the image.
constexpr int kPanelRows = 256, kPanelRowBytes = 64, kPanelBlock = 16384;

__host__ __device__ __forceinline__ int64_t panel_offset(int64_t row, int64_t kbyte, int64_t nkb) {
    const int64_t rb = row >> 8, kb = kbyte >> 6;
    const int r = (int)(row & 255), c = (int)((kbyte >> 4) & 3);
    return ((rb * nkb + kb) << 14) + (r << 6) + ((c ^ ((r >> 2) & 3)) << 4) + (kbyte & 15);
}

// MX FP6 panel images (E2M3 codes packed 6 bits each, code j of a 32-value K
// half at bit 6 j, little endian): per operand three arrays, hi codes, lo
// codes and scales, cut like the panel images into blocks of 256 rows by one
// 64-value K block; block (rb, kb) is block number rb * nkb + kb of each array.
// A code block is 256 rows x 48 bytes (12 KiB); row r holds, at 48 r,
//   [half 0 bytes 0-15 | half 1 bytes 0-15 | half 0 bytes 16-23 | half 1 bytes 16-23]
// so that a lane's 24 bytes are one 16-byte and one 8-byte aligned read.  A
// scale block is 256 rows x 4 bytes (1 KiB): row r holds the E8M0 bytes
// (half 0 hi, half 0 lo, half 1 hi, half 1 lo) at 4 r, so one 16-bit read
// gives a lane both levels' scales of its half.
constexpr int kMx6RowBytes = 48, kMx6Block = kPanelRows * kMx6RowBytes, kMx6ScaleBlock = 1024;

__host__ __device__ __forceinline__ int64_t mx6_code_offset(int64_t row, int64_t kb, int h, int byte,
                                                            int64_t nkb) {
    const int64_t rb = row >> 8;
    const int r = (int)(row & 255);
    const int pos = byte < 16 ? 16 * h + byte : 32 + 8 * h + (byte - 16);
    return (rb * nkb + kb) * kMx6Block + r * kMx6RowBytes + pos;
}
__host__ __device__ __forceinline__ int64_t mx6_scale_offset(int64_t row, int64_t kb, int h, int level,
                                                             int64_t nkb) {
    return (((row >> 8) * nkb + kb) << 10) + (row & 255) * 4 + 2 * h + level;
}

// Workgroup `blk` of a launch that runs ta workgroups of one kind and tb of
// another (the operand pre-passes of A and B in one launch), spread evenly:
// the second kind sits at the blocks where floor(blk * tb / (ta + tb)) steps,
// so both kinds stream side by side in proportion for the whole launch.
// *index is the workgroup's number within its kind.
__device__ __forceinline__ bool second_kind(int64_t blk, int64_t ta, int64_t tb, int64_t* index) {
    const int64_t total = ta + tb;
    const int64_t before = blk * tb / total, upto = (blk + 1) * tb / total;
    *index = upto > before ? before : blk - before;
    return upto > before;
}

// The same over groups of eight consecutive workgroups, which the hardware
// hands to the eight XCDs in turn: every XCD gets its share of both kinds
// (a plain A, B, A, B order would put all of A on four XCDs).  A launch of
// paired_blocks(ta, tb) workgroups; returns 0 (first kind), 1 (second kind)
// or -1 for the few workgroups past the end of a kind's last group.
__host__ __device__ __forceinline__ int64_t paired_blocks(int64_t ta, int64_t tb) {
    return 8 * ((ta + 7) / 8 + (tb + 7) / 8);
}
__device__ __forceinline__ int paired_kind(int64_t blk, int64_t ta, int64_t tb, int64_t* index) {
    int64_t g;
    const bool second = second_kind(blk >> 3, (ta + 7) / 8, (tb + 7) / 8, &g);
    *index = 8 * g + (blk & 7);
    if (*index >= (second ? tb : ta)) return -1;
    return second ? 1 : 0;
}

// Largest i in [0, count) with start(i) <= value, for non-decreasing starts and
// start(0) <= value (count >= 1): the problem a workgroup of a grouped launch
// belongs to.  Every lane of a wave takes part and gets the same answer; a
// round narrows 64-fold, so 1024 problems take two dependent loads where a
// binary search takes ten (each 0.5 us or more when another XCD wrote the list).
template <class F>
__device__ __forceinline__ int wave_find_last(int count, int value, F&& start) {
    const int lane = threadIdx.x & 63;
    int lo = 0, n = count;                        // the answer lies in [lo, lo + n)
    while (n > 1) {
        const int step = (n + 63) / 64;
        const int i = lane * step;                // lane 0 always passes
        const bool below = i < n && start(lo + i) <= value;
        const int k = 63 - __builtin_clzll(__ballot(below) | 1ull);
        lo += k * step;
        n = n - k * step < step ? n - k * step : step;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

// Tile queues of a persistent grouped launch: the tile list is cut into one
// list per XCD, tiles [start[x], start[x + 1]), so that the tiles of a problem
// run on one XCD and read its panels through one L2.  Workgroup b belongs to
// list b % 8 (the hardware hands consecutive workgroups to the XCDs in turn)
// and starts with entry b / 8 of it; further entries are claimed from the
// list's counter, and from the other lists' once the own one is empty.
// `counters` holds one 32-bit counter per list and one of the workgroups that
// are done, kQueuePitch words apart, zero before the first launch; the last
// workgroup leaves them zero for the next one (a kernel that zeroed them took
// 4.6 us).
struct TileQueues {
    int start[kXcds + 1];
};
constexpr int kQueuePitch = 16;                   // 64 bytes: one counter per cache line
constexpr int kQueueWords = (kXcds + 1) * kQueuePitch;

// The end of a workgroup of a launch that claimed from `lists` counters (thread
// 0, all claims answered): the launch's last workgroup zeroes them.  The counter
// of the done ones follows them and wraps at the grid size by itself, never
// stored to: were two launches of the same counters to overlap, which is not
// allowed, the last workgroup of all would still be one that wraps it, so the
// next launch finds every counter zero.  (A stored zero could drop the other
// launch's arrivals, and then every later launch zeroed the lists too early.)
__device__ __forceinline__ void end_claims(unsigned* counters, int lists) {
    const unsigned last = gridDim.x - 1;
    if (threadIdx.x == 0 && atomicInc(counters + lists * kQueuePitch, last) == last)
        for (int x = 0; x < lists; ++x)
            __hip_atomic_store(counters + x * kQueuePitch, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct TileClaims {
    const TileQueues& q;
    unsigned* counters;
    int home;
    unsigned ticket;

    __device__ __forceinline__ TileClaims(const TileQueues& queues, unsigned* c)
        : q(queues), counters(c), home(blockIdx.x % kXcds), ticket(0) {}
    __device__ __forceinline__ int size(int x) const { return q.start[x + 1] - q.start[x]; }
    // entries of list x that workgroups start with
    __device__ __forceinline__ int started(int x) const {
        const int wgs = ((int)gridDim.x - x + kXcds - 1) / kXcds;
        return wgs < size(x) ? wgs : size(x);
    }
    // Claim the next entry of the own list (thread 0).  Called as a tile's stores
    // begin, so that the answer arrives under them; claimed at the start of a long
    // tile, an entry would wait for it while other workgroups idle.  The opaque
    // zero keeps the compiler from waiting for it here.
    __device__ __forceinline__ void prefetch() {
        int zero = 0;
        asm volatile("" : "+v"(zero));
        if (threadIdx.x == 0) ticket = atomicAdd(counters + home * kQueuePitch + zero, 1u);
    }
    // An entry of any list with one left (the own list first), or -1 when all
    // are empty.  Wave 0 only; every repetition has seen another list emptied.
    __device__ __forceinline__ int steal() const {
        const int lane = threadIdx.x & 63;
        for (;;) {
            int x = (home + lane) % kXcds;
            bool left = false;
            if (lane < kXcds)
                left = __hip_atomic_load(counters + x * kQueuePitch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
                       (unsigned)(size(x) - started(x));
            const uint64_t any = __ballot(left);
            if (!any) return -1;
            x = (home + (int)__builtin_ctzll(any)) % kXcds;
            unsigned got = 0;
            if (lane == 0) got = atomicAdd(counters + x * kQueuePitch, 1u);
            got = (unsigned)__builtin_amdgcn_readfirstlane((int)got);
            if (got < (unsigned)(size(x) - started(x))) return q.start[x] + started(x) + (int)got;
        }
    }
    // The workgroup's first tile and its next one (every thread; -1: none left).
    // `slot` is an LDS word of this object's own.
    __device__ __forceinline__ int first(int* slot) const {
        const int i = blockIdx.x / kXcds;
        if (i < size(home)) return q.start[home] + i;   // uniform
        return share(slot, threadIdx.x < 64 ? steal() : 0);
    }
    __device__ __forceinline__ int next(int* slot) const {
        int tile = -1;
        if (threadIdx.x < 64) {
            const unsigned t = (unsigned)__builtin_amdgcn_readfirstlane((int)ticket);
            tile = t < (unsigned)(size(home) - started(home)) ? q.start[home] + started(home) + (int)t : steal();
        }
        return share(slot, tile);
    }

    // After the last tile: every claim of this workgroup has been answered.
    __device__ __forceinline__ void finish() const { end_claims(counters, kXcds); }

  private:
    __device__ __forceinline__ static int share(int* slot, int tile) {
        __syncthreads();                          // the last value has been read
        if (threadIdx.x == 0) *slot = tile;
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(*slot);
    }
};

}  // namespace cmp
