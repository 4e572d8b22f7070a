// First layers of the bf16 image classifier, straight from the uint8 frames (gfx950 matrix cores).
//
// The first 3x3 layer contracts 27 values per output.  Padded to a K tile of 64 channels per tap it cost 576, and its padded
// input had to be written first; here a normalised pixel is 4 bf16 (the fourth is 0) in LDS and K runs over 10 taps x 8 (four
// zeros behind each pixel, the tenth tap's weights zero): five 32x32x16 products per tile, one 8-byte LDS read per lane each.
//
// Both layers give the values of the general kernel bit for bit, so an answer does not depend on which of them ran: taps in
// filter order, a tap's channels 16 at a time, each sum on its own, from the bias on.  The matrix instruction adds the 8 products of lanes 0..31
// first and then those of lanes 32..63, each 8 as one sum: two taps in the two halves round like a product per tap, two taps
// within a half (three products per tile instead of five) do not.
//
// first_layer_kernel: that layer alone.  64 pictures of 224 x 224, 64 channels: 173 us, against 94 + 470 as packing and general
// kernel.  Its matrix work is 13 us; it writes 411 MB at 2.4 TB/s, half of a copy's rate: 16 bytes of a pixel per lane, so that
// a store touches 32 lines.
// first_pair_kernel: 3 -> 64 -> 64 layers (and the 2x2 max-pool behind them) in one launch.  The 64-channel tensor between
// them is as large as the network's largest and is never written: a block computes it for its own tile and halo in LDS.
// Bound by the matrix pipe (237 GFLOP at 0.88 PFLOP/s); 64 pictures of 224 x 224: 269 us, against 1 232 us as packing, two
// layers on the general kernel and pool (258 us with sums in another order: four taps per product in the first layer, input
// rows innermost in the second).
#include <algorithm>
#include <type_traits>

#include "thia_internal.h"

namespace thia {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;

namespace {

template <int I, int N, typename F>
__device__ inline void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

__device__ inline void mma(f32x16_t& acc, const u32x4_t& a, const u32x4_t& b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), acc, 0, 0, 0);
}

constexpr int kTaps = 9, kCin = 64;   // weights of both layers: bf16 [Cout][9][64] (the first layer's channels 3..63 are zeros)

constexpr int kSteps1 = 5;   // products per tile of the first layer: taps 2 s (lanes 0..31) and 2 s + 1 (lanes 32..63)

// First layer's weights of this lane's output channel and its half's tap of step s.
__device__ inline u32x2_t first_weights(const bf16_t* __restrict__ w, int ch, int s, int g) {
    const int tap = 2 * s + g;
    if (tap >= kTaps) return u32x2_t{0u, 0u};
    return *reinterpret_cast<const u32x2_t*>(w + ((size_t)ch * kTaps + tap) * kCin);
}

// Byte offsets, from a pixel's (tap 0) position in the raw patch of COLS columns, of the taps that lane half g feeds to the
// steps.  The tenth tap has zero weights and re-reads the ninth.
template <int COLS>
__device__ inline void first_offsets(int g, int off[kSteps1]) {
#pragma unroll
    for (int s = 0; s < kSteps1; ++s) {
        const int a = 2 * s, b = 2 * s + 1 < kTaps ? 2 * s + 1 : kTaps - 1;
        off[s] = g ? ((b / 3) * COLS + b % 3) * 8 : ((a / 3) * COLS + a % 3) * 8;
    }
}

__device__ inline u32x2_t first_pixels(const unsigned char* px, const int off[kSteps1], int s) {
    return *reinterpret_cast<const u32x2_t*>(px + off[s]);
}

__device__ inline u32x4_t tap_operand(const u32x2_t& v) { return u32x4_t{v.x, v.y, 0u, 0u}; }

__device__ inline f32x16_t bias_tile(const float* bias, int g) {   // accumulator element e: channel 8 (e / 4) + 4 g + e % 4
    f32x16_t r;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const f32x4_t q = *reinterpret_cast<const f32x4_t*>(bias + 8 * v + 4 * g);
        r[4 * v] = q.x; r[4 * v + 1] = q.y; r[4 * v + 2] = q.z; r[4 * v + 3] = q.w;
    }
    return r;
}

// ReLU'd channels 8 v + 4 g .. + 3 of this lane's pixel, rounded.
__device__ inline u32x2_t relu_pack(const f32x16_t& a, int v) {
    return u32x2_t{pack_bf16x2(fmaxf(a[4 * v], 0.f), fmaxf(a[4 * v + 1], 0.f)), pack_bf16x2(fmaxf(a[4 * v + 2], 0.f), fmaxf(a[4 * v + 3], 0.f))};
}

// Stores the 32 channels of a tile: the two lane halves of a pixel swap quads, so that each holds 8 consecutive channels and
// every store is 16 bytes (channel group 2 h + g of 8).
__device__ inline void store_tile(const f32x16_t& a, bf16_t* __restrict__ dst, int g, bool ok) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const u32x2_t v0 = relu_pack(a, 2 * h), v1 = relu_pack(a, 2 * h + 1);
        const u32x2_t give = g ? v0 : v1;
        const u32x2_t got = {(uint32_t)__shfl_xor((int)give.x, 32), (uint32_t)__shfl_xor((int)give.y, 32)};
        const u32x4_t o = g ? u32x4_t{got.x, got.y, v1.x, v1.y} : u32x4_t{v0.x, v0.y, got.x, got.y};
        if (ok) *reinterpret_cast<u32x4_t*>(dst + (2 * h + g) * 8) = o;
    }
}

// Normalised pixel (iy, ix) of a frame as 4 bf16; zeros outside (padding follows the normalisation).
__device__ inline u32x2_t raw_pixel(const uint8_t* __restrict__ f, size_t HW, int iy, int ix, int H, int W, const bf16_t* lut) {
    u32x2_t r = {0u, 0u};
    if ((unsigned)iy < (unsigned)H && (unsigned)ix < (unsigned)W) {
        const uint8_t* p = f + (size_t)iy * W + ix;
        r.x = (uint32_t)lut[p[0]] | ((uint32_t)lut[p[HW]] << 16);
        r.y = lut[p[2 * HW]];
    }
    return r;
}

// ------------------------------------------------------------------------------------------------ the first layer alone
constexpr int F1R = 8, F1C = 32;   // output tile: a wavefront takes two rows

__global__ __launch_bounds__(256) void first_layer_kernel(const uint8_t* __restrict__ frames, int H, int W, const bf16_t* __restrict__ w,
                                                          const float* __restrict__ bias, int Cout, float mean, float stdv,
                                                          bf16_t* __restrict__ out, int tiles_x, int tiles_y) {
    __shared__ __align__(16) unsigned char raw[(F1R + 2) * (F1C + 2) * 8];
    __shared__ bf16_t lut[256];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, g = lane >> 5, col = lane & 31;
    const int img = blockIdx.x / (tiles_x * tiles_y), rem = blockIdx.x - img * tiles_x * tiles_y;
    const int oy0 = (rem / tiles_x) * F1R, ox0 = (rem % tiles_x) * F1C;
    const size_t HW = (size_t)H * W;
    lut[t] = f32_to_bf16(((float)t - mean) / stdv);
    __syncthreads();
    for (int i = t; i < (F1R + 2) * (F1C + 2); i += 256) {
        const int py = i / (F1C + 2), px = i - py * (F1C + 2);
        *reinterpret_cast<u32x2_t*>(raw + i * 8) = raw_pixel(frames + (size_t)img * 3 * HW, HW, oy0 - 1 + py, ox0 - 1 + px, H, W, lut);
    }
    __syncthreads();
    int off[kSteps1];
    first_offsets<F1C + 2>(g, off);
    u32x2_t px[2][kSteps1];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int s = 0; s < kSteps1; ++s) px[r][s] = first_pixels(raw + ((2 * wv + r) * (F1C + 2) + col) * 8, off, s);
    for (int c0 = 0; c0 < Cout; c0 += 32) {
        f32x16_t acc[2];
        acc[0] = acc[1] = bias_tile(bias + c0, g);
#pragma unroll
        for (int s = 0; s < kSteps1; ++s) {
            const u32x4_t a = tap_operand(first_weights(w, c0 + col, s, g));
#pragma unroll
            for (int r = 0; r < 2; ++r) mma(acc[r], a, tap_operand(px[r][s]));
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int oy = oy0 + 2 * wv + r, ox = ox0 + col;
            store_tile(acc[r], out + (((size_t)img * H + oy) * W + ox) * Cout + c0, g, oy < H && ox < W);
        }
    }
}

// ------------------------------------------------------------------------------------- the first two layers and their pool
// Output tile 16 x 32 pixels, 8 wavefronts: wavefront wv owns channels 32 (wv & 1) .. + 31 of the four rows 4 (wv >> 1) .. + 3.
// Its 36 weight fragments (144 registers) stay in registers over all tiles of the persistent block.  A fragment of one input
// row at one column shift serves the output rows above, at and below it, so the contraction reads 6 fragments per 12 products:
// half of the 128 bytes/cycle of LDS at the full matrix rate, where reading a fragment per product would need all of it.
// Input rows are walked outermost: an output row then meets its taps in filter order (the order of the general kernel).
constexpr int PR = 16, PC = 32;                       // output tile
constexpr int MR = PR + 2, MC = PC + 2;               // first layer's tile with the second's halo
constexpr int RR = MR + 2, RC = MC + 2;               // raw patch
constexpr int MPITCH = 128 + 16;                      // bytes per pixel (padded: 16 consecutive pixels on 16 different 16-byte slots)
constexpr int MTILES = (MR * MC + 31) / 32;           // 32-pixel tiles of the first layer (the last one is partly outside)
constexpr int RAW_PT = (RR * RC + 511) / 512;         // raw pixels per thread

template <bool POOL>
__global__ __launch_bounds__(512, 2) void first_pair_kernel(const uint8_t* __restrict__ frames, int H, int W, const bf16_t* __restrict__ w1,
                                                            const float* __restrict__ b1, const bf16_t* __restrict__ w2,
                                                            const float* __restrict__ b2, float mean, float stdv,
                                                            bf16_t* __restrict__ out, int tiles_x, int tiles_y, int total) {
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* mid = smem;                                   // [MR * MC][MPITCH]
    unsigned char* raw = mid + MR * MC * MPITCH;                 // [RR * RC][8]
    unsigned char* wf1 = raw + RR * RC * 8;                      // [2][kSteps1][64 lanes][8]
    float* sb = reinterpret_cast<float*>(wf1 + 2 * kSteps1 * 512);   // both layers' biases
    bf16_t* lut = reinterpret_cast<bf16_t*>(sb + 128);
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6), g = lane >> 5, col = lane & 31;
    const int cn = wv & 1, rg = wv >> 1;
    const size_t HW = (size_t)H * W;

    if (t < 256) lut[t] = f32_to_bf16(((float)t - mean) / stdv);
    if (t < 64) sb[t] = b1[t];
    else if (t < 128) sb[t] = b2[t - 64];
    for (int q = wv; q < 2 * kSteps1; q += 8)
        *reinterpret_cast<u32x2_t*>(wf1 + (q * 64 + lane) * 8) = first_weights(w1, (q / kSteps1) * 32 + col, q % kSteps1, g);
    u32x4_t w[36];
#pragma unroll
    for (int k = 0; k < 36; ++k) w[k] = *reinterpret_cast<const u32x4_t*>(w2 + (size_t)(cn * 32 + col) * (kTaps * kCin) + k * 16 + g * 8);
    int off[kSteps1];
    first_offsets<RC>(g, off);

    struct Org { int img, y, x; };
    auto origin = [&](int tile) {
        Org o;
        o.img = tile / (tiles_x * tiles_y);
        const int rem = tile - o.img * tiles_x * tiles_y;
        o.y = (rem / tiles_x) * PR; o.x = (rem % tiles_x) * PC;
        return o;
    };
    // raw pixels of the next tile are requested before the current one is multiplied
    uint32_t bytes[RAW_PT];   // three bytes each, bit 24 set inside the frame
    auto load_raw = [&](const Org& o) {
        const uint8_t* f = frames + (size_t)o.img * 3 * HW;
#pragma unroll
        for (int q = 0; q < RAW_PT; ++q) {
            const int i = q * 512 + t, py = i / RC, px = i - py * RC, iy = o.y - 2 + py, ix = o.x - 2 + px;
            bytes[q] = 0u;
            if (i < RR * RC && (unsigned)iy < (unsigned)H && (unsigned)ix < (unsigned)W) {
                const uint8_t* p = f + (size_t)iy * W + ix;
                bytes[q] = (uint32_t)p[0] | ((uint32_t)p[HW] << 8) | ((uint32_t)p[2 * HW] << 16) | (1u << 24);
            }
        }
    };
    int tile = blockIdx.x;   // (the grid has no more blocks than tiles)
    Org cur = origin(tile);
    load_raw(cur);
    __syncthreads();         // table, biases and weights are in LDS
    for (; tile < total; tile += gridDim.x) {
#pragma unroll
        for (int q = 0; q < RAW_PT; ++q) {
            const int i = q * 512 + t;
            if (i < RR * RC) {
                u32x2_t r = {0u, 0u};
                if (bytes[q] >> 24) {
                    r.x = (uint32_t)lut[bytes[q] & 0xffu] | ((uint32_t)lut[(bytes[q] >> 8) & 0xffu] << 16);
                    r.y = lut[(bytes[q] >> 16) & 0xffu];
                }
                *reinterpret_cast<u32x2_t*>(raw + i * 8) = r;
            }
        }
        __syncthreads();     // raw patch complete; every wavefront has read the previous tile's `mid`
        const Org nxt = origin(min(tile + (int)gridDim.x, total - 1));
        load_raw(nxt);
        // ---- first layer on the tile and its halo; pixels outside the frame are the second layer's zero padding
        {
            u32x4_t a[kSteps1];
#pragma unroll
            for (int s = 0; s < kSteps1; ++s) a[s] = tap_operand(*reinterpret_cast<const u32x2_t*>(wf1 + ((cn * kSteps1 + s) * 64 + lane) * 8));
            const f32x16_t bt = bias_tile(sb + cn * 32, g);
            for (int mt = rg; mt < MTILES; mt += 4) {
                const int p = mt * 32 + col, pc = min(p, MR * MC - 1), py = pc / MC, px = pc - py * MC;
                f32x16_t acc = bt;
#pragma unroll
                for (int s = 0; s < kSteps1; ++s) mma(acc, a[s], tap_operand(first_pixels(raw + (py * RC + px) * 8, off, s)));
                const bool in = (unsigned)(cur.y - 1 + py) < (unsigned)H && (unsigned)(cur.x - 1 + px) < (unsigned)W;
                if (p < MR * MC) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const u32x2_t o = relu_pack(acc, v);
                        *reinterpret_cast<u32x2_t*>(mid + p * MPITCH + (cn * 32 + 8 * v + 4 * g) * 2) = in ? o : u32x2_t{0u, 0u};
                    }
                }
            }
        }
        __syncthreads();     // `mid` complete
        // ---- second layer: steps in the order (input row, column shift, 16 channels); a ring of four fragments runs three ahead
        f32x16_t acc[4];
        acc[0] = acc[1] = acc[2] = acc[3] = bias_tile(sb + 64 + cn * 32, g);
        const unsigned char* base = mid + (rg * 4 * MC + col) * MPITCH + g * 16;
        constexpr int STEPS = 6 * 3 * 4, AHEAD = 3;
        u32x4_t f[AHEAD + 1];
        auto fragment = [&](int i) {
            const int row = i / 12, kx = (i / 4) % 3, ks = i % 4;
            return *reinterpret_cast<const u32x4_t*>(base + (row * MC + kx) * MPITCH + ks * 32);
        };
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) f[i] = fragment(i);
        static_for<0, STEPS>([&](auto ic) {
            constexpr int i = decltype(ic)::value, row = i / 12, kx = (i / 4) % 3, ks = i % 4;
            if constexpr (i + AHEAD < STEPS) f[(i + AHEAD) % (AHEAD + 1)] = fragment(i + AHEAD);
            static_for<0, 3>([&](auto kc) {
                constexpr int ky = decltype(kc)::value, r = row - ky;
                if constexpr (r >= 0 && r < 4) mma(acc[r], w[(ky * 3 + kx) * 4 + ks], f[i % (AHEAD + 1)]);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (POOL) {
            // ReLU and rounding are monotonic: the maximum is taken on the sums.  Neighbouring columns are neighbouring lanes;
            // the even one of a pair keeps the tile's first 16 channels, the odd one the others.
            const int Ho = H / 2, Wo = W / 2, ox = (cur.x + col) >> 1;
#pragma unroll
            for (int pr = 0; pr < 2; ++pr) {
                f32x16_t m;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float v = fmaxf(acc[2 * pr][e], acc[2 * pr + 1][e]);
                    m[e] = fmaxf(v, __shfl_xor(v, 1));
                }
                const int oy = (cur.y >> 1) + 2 * rg + pr;
                const bool ok = oy < Ho && ox < Wo;
                bf16_t* dst = out + (((size_t)cur.img * Ho + oy) * Wo + ox) * 64 + cn * 32;
                const bool odd = col & 1;
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    const u32x2_t lo = relu_pack(m, v), hi = relu_pack(m, v + 2);
                    const u32x2_t o = odd ? hi : lo;
                    if (ok) *reinterpret_cast<u32x2_t*>(dst + (odd ? 16 : 0) + 8 * v + 4 * g) = o;
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int oy = cur.y + rg * 4 + r, ox = cur.x + col;
                store_tile(acc[r], out + (((size_t)cur.img * H + oy) * W + ox) * 64 + cn * 32, g, oy < H && ox < W);
            }
        }
        cur = nxt;
    }
}

constexpr size_t kPairLds = (size_t)MR * MC * MPITCH + RR * RC * 8 + 2 * kSteps1 * 512 + 128 * 4 + 256 * 2;

}  // namespace

hipError_t launch_first_layer(const uint8_t* frames, int n, int H, int W, const bf16_t* w, const float* bias, int Cout, float mean, float stdv,
                              bf16_t* out, hipStream_t s) {
    const long long tx = (W + F1C - 1) / F1C, ty = (H + F1R - 1) / F1R, blocks = tx * ty * n;
    if (n <= 0 || H <= 0 || W <= 0 || Cout <= 0 || Cout % 32 || blocks >= (1ll << 31)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(first_layer_kernel, dim3((unsigned)blocks), dim3(256), 0, s, frames, H, W, w, bias, Cout, mean, stdv, out, (int)tx, (int)ty);
    return hipGetLastError();
}

hipError_t launch_first_pair(const uint8_t* frames, int n, int H, int W, const bf16_t* w1, const float* b1, const bf16_t* w2, const float* b2,
                             bool pool, float mean, float stdv, bf16_t* out, hipStream_t s) {
    const long long tx = (W + PC - 1) / PC, ty = (H + PR - 1) / PR, tiles = tx * ty * n;
    if (n <= 0 || H <= 0 || W <= 0 || tiles >= (1ll << 30)) return hipErrorInvalidValue;
    const auto kern = pool ? first_pair_kernel<true> : first_pair_kernel<false>;
    const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), kPairLds);
    if (e != hipSuccess) return e;
    const unsigned grid = (unsigned)std::min<long long>(tiles, 256);   // one resident block on each of the 256 CUs (registers)
    hipLaunchKernelGGL(kern, dim3(grid), dim3(512), kPairLds, s, frames, H, W, w1, b1, w2, b2, mean, stdv, out, (int)tx, (int)ty, (int)tiles);
    return hipGetLastError();
}

}  // namespace thia
