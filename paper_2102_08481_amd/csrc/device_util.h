// Device helpers shared by the proposal and ROI kernels: order-preserving score keys,
// a block-wide sort, greedy suppression among 64 rows, box decoding and the NMS overlap test.  All geometry is
// plain fp32 with singly rounded operations (the library is built with
// -ffp-contract=off), so that orderings and keep decisions are reproducible.
#pragma once
#include "thia_internal.h"

namespace thia {

// Monotone map float -> uint32 (larger float = larger key); -0 and +0 map to the same key.
__device__ inline uint32_t score_key(float s) {
    const uint32_t b = __float_as_uint(s + 0.0f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ inline float key_score(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// n2 keys (a power of two, at least 64) in LDS, sorted descending by the whole block: every wavefront sorts runs of 64 in
// registers (a bitonic network over the lanes), then pairs of runs are merged, each key finding its place by a binary search
// in the other run.  Two buffers of n2 keys; returns the one that holds the result.  A merge level is ~10 dependent LDS
// reads and one barrier; the 66-stage network in LDS it replaces paid a round trip through LDS per stage (the
// top-k tail on up to 2048 keys: 26.4 -> 22.6 us, now bound by the random LDS reads of the searches).  The caller's writes to `keys` need no barrier of their own.
__device__ inline uint64_t* block_sort_desc(uint64_t* keys, uint64_t* tmp, int n2) {
    const int lane = threadIdx.x & 63;
    __syncthreads();
    for (int i = threadIdx.x; i < n2; i += blockDim.x) {   // (n2 and the block size are multiples of 64: whole wavefronts)
        uint64_t v = keys[i];
        for (int k = 2; k <= 64; k <<= 1)
            for (int j = k >> 1; j > 0; j >>= 1) {
                const uint64_t o = __shfl_xor((unsigned long long)v, j);
                const bool larger = ((lane & k) == 0) == ((lane & j) == 0);   // this lane keeps the larger of the two
                v = (o > v) == larger ? o : v;
            }
        keys[i] = v;
    }
    __syncthreads();
    for (int len = 64; len < n2; len <<= 1) {
        for (int i = threadIdx.x; i < n2; i += blockDim.x) {
            const uint64_t v = keys[i];
            const int run = i & ~(len - 1);
            const bool second = (run & len) != 0;
            const uint64_t* other = keys + (run ^ len);
            // keys of the other run that come first (equal keys, i.e. padding: the first run's)
            int lo = 0;
            for (int step = len; step > 0; step >>= 1)
                if (lo + step <= len && (second ? other[lo + step - 1] >= v : other[lo + step - 1] > v)) lo += step;
            tmp[(run & ~len) + (i - run) + lo] = v;
        }
        __syncthreads();
        uint64_t* t = keys; keys = tmp; tmp = t;
    }
    return keys;
}

// Greedy suppression among up to 64 rows, one per lane, decided by a whole wavefront: `open` = rows not suppressed from
// outside, `earlier` = this lane's earlier rows that overlap it.  A row is kept once all of its overlapping earlier rows
// are suppressed, and suppressed once one of them is kept; the lowest open row is decided in every round, and usually all
// rows are after a few, where stepping from one kept row to the next costs ~120 cycles for each of them.
__device__ inline uint64_t greedy_keep(uint64_t open, uint64_t earlier) {
    const uint64_t me = 1ull << (threadIdx.x & 63);
    uint64_t kept = 0ull;
    while (open != 0ull) {
        kept |= __ballot((open & me) != 0ull && (earlier & (open | kept)) == 0ull);
        open &= ~kept;
        open &= ~__ballot((open & me) != 0ull && (earlier & kept) != 0ull);
    }
    return kept;
}

// Bitonic network with a block barrier after every stage: keys may live in LDS or in global memory.
__device__ inline void bitonic_sort_desc(uint64_t* keys, int n2) {
    for (int k = 2; k <= n2; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < n2; i += blockDim.x) {
                const int p = i ^ j;
                if (p > i) {
                    const uint64_t a = keys[i], b = keys[p];
                    const bool desc = (i & k) == 0;
                    if (desc ? (a < b) : (a > b)) { keys[i] = b; keys[p] = a; }
                }
            }
            __syncthreads();
        }
}

struct Box { float x1, y1, x2, y2; };

// Decoding of (dx,dy,dw,dh) against a reference box given as centre/size, unit weights,
// dw/dh clamped at ln(1000/16), corners clipped to the frame.  Returns false for boxes
// narrower or lower than 1e-3 px after clipping.
__device__ inline bool decode_box(float cx, float cy, float w, float h, float dx, float dy, float dw, float dh, float imgW,
                                  float imgH, Box& o) {
    const float clampv = 4.135166556742356f;
    dw = dw < clampv ? dw : clampv;
    dh = dh < clampv ? dh : clampv;
    const float ncx = cx + dx * w, ncy = cy + dy * h;
    const float nw = w * expf(dw), nh = h * expf(dh);
    const float hw = 0.5f * nw, hh = 0.5f * nh;
    o.x1 = fminf(fmaxf(ncx - hw, 0.f), imgW);
    o.y1 = fminf(fmaxf(ncy - hh, 0.f), imgH);
    o.x2 = fminf(fmaxf(ncx + hw, 0.f), imgW);
    o.y2 = fminf(fmaxf(ncy + hh, 0.f), imgH);
    return (o.x2 - o.x1 >= 1e-3f) && (o.y2 - o.y1 >= 1e-3f);
}

// Division-free overlap test: IoU(a, b) > thr  <=>  union > 0 and inter > thr * union.
__device__ inline bool iou_over(const Box& a, const Box& b, float thr) {
    float iw = fminf(a.x2, b.x2) - fmaxf(a.x1, b.x1);
    float ih = fminf(a.y2, b.y2) - fmaxf(a.y1, b.y1);
    iw = fmaxf(iw, 0.f);
    ih = fmaxf(ih, 0.f);
    const float inter = iw * ih;
    const float aa = (a.x2 - a.x1) * (a.y2 - a.y1);
    const float ab = (b.x2 - b.x1) * (b.y2 - b.y1);
    const float uni = (aa + ab) - inter;
    const float t = thr * uni;
    return uni > 0.f && inter > t;
}

}  // namespace thia
