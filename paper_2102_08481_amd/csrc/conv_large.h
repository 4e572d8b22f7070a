// Large tiles of the bf16 layer kernel (gfx950): 256 or 192 pixels x 256 or 128 channels per block of eight wavefronts, for
// layers with many pixels and a long contraction, with the fused RPN predictors and the expansion tail (256 x 256).  The
// contraction, its operand layout and the order of its sums are those of conv_igemm.hip: same values bit for bit.
//
// What bounds it is the matrix pipe: per K tile (64 values of every row) a 256 x 256 block has 2048 cycles of products, 192 KB of
// fragment reads and 64 requests of 1 KiB at the CU's address unit (17 to 28 cycles each), which have to run side by side.
// A K tile is therefore multiplied in phases, each a memory part (fragment reads and requests) and a product part with a block
// barrier behind either, and wavefronts 4..7 run one part behind wavefronts 0..3.  w and w + 4 share a SIMD: while one of the
// two multiplies, the other reads its fragments and issues its two or three requests.
//
// 256 channels: a K tile lies in LDS as four halves, W0, W1 (the weight rows of each wavefront's first and second 32
// channels) and X0, X1 (the pixel rows of each wavefront's first 64 and of its other pixels), two buffers of each:
//   phase    reads           requests (two tiles ahead)    products
//     1      X0 of t         W0 of t + 2                   W0 X0
//     2      W1 of t         X0 of t + 2                   W1 X0
//     3      X1 of t         W1 of t + 2                   W0 X1
//     4      W0 of t + 1     X1 of t + 2                   W1 X1
// A half that is read in phase i is requested anew in phase i + 1: the reads are waited for (lgkmcnt) in front of the
// barrier that ends the memory part, the later group's one barrier further on, and that barrier lies in front of the
// earlier group's next memory part.  A half that phase j reads has landed for all wavefronts when phase j starts: each
// waits in phase j - 1, in front of its barrier, until no more of its requests are outstanding than it issued behind that
// half (vmcnt counts them in order).  So a request has six phases (1.5 K tiles) to arrive and no wait is for everything.
// 128 channels: a wavefront's 64 x 64 or 96 x 32 tile has too few products for four phases; a phase takes all of them for two
// of the K tile's four k-steps, three buffers hold whole K tiles, and tile t + 2 is requested into the buffer of t - 1.
// Requests are buffer loads: 32-bit offsets (a descriptor per block, a scalar offset per K tile), so that a request costs no
// 64-bit address arithmetic, and lanes without a pixel or with a padded tap point behind the descriptor's end and read zeros.
//
// Measured against the loop before (fragments read in front of the products that use them, every wavefront requesting a whole
// K tile's share at once), 32 frames at 540 x 960: RPN 3x3 + predictors at exit 1 1 249 -> 1 022 us (1 011 -> 1 236 TFLOP/s; a
// library product of the same size: 1 069), at exit 2 328 -> 261, 3x3 256 -> 256 + expansion 149 -> 131 (119 with the tail as below), 1024 -> 256 39 -> 33, first
// FC layer (192 x 256) 291 -> 207.  A K tile takes 1.0 us while a third of the CUs work and 1.38 when all do: the chip's clock
// comes down under matrix work.
//
// Part of conv_igemm.hip, which includes it once, at its end: it has no translation unit of its own.
namespace thia {

// MODE 0: any filter size; 1: 1x1 unpadded (no tap bookkeeping); 2: 1x1 with a second source tensor;
// 4: any filter size, followed by the expansion tail (ConvArgs::tail_*) on the block's output tile.
template <int BM, int BN, int MODE>
__global__ __launch_bounds__(512, 1) void conv_large_kernel(const ConvArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
    using T = bf16_t;
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    typedef __attribute__((address_space(3))) u32x4_t lds_u32x4;
    // Lanes whose offset is not below the descriptor's size read zeros: padded filter taps and rows beyond the last pixel.
    constexpr uint32_t OUTSIDE = 0x80000000u;
    constexpr bool ONE = MODE == 1 || MODE == 2, DUAL = MODE == 2;
    constexpr bool QUAD = BN == 256;                     // four phases of a product of halves; else two of half the k-steps
    constexpr int BK = 64, ROW = 128;                    // K values and bytes of a tile row
    constexpr int WAVES_N = QUAD || BM == 192 ? 4 : 2, WAVES_M = 8 / WAVES_N;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;  // wavefront tile (pixels x channels)
    constexpr int TM = WM / 32, TN = WN / 32;            // 32x32 matrix tiles per wavefront
    constexpr int TM1 = TM - 2;                          // of them in the second pixel half (QUAD)
    constexpr int KK = 4;                                // k-steps of a K tile
    constexpr int PB = BM / 64, PA = BN / 64;            // pixel and weight rows a thread requests per K tile
    // LDS.  QUAD: weights [2][256 rows], pixels [2][256 rows]; else [3][weights, pixels]
    constexpr uint32_t BUF = QUAD ? 256 * ROW : (BN + BM) * ROW, XOFF = QUAD ? 2 * BUF : BN * ROW;
    static_assert(!QUAD || TM == 3 || TM == 4, "the halves are two and one or two matrix tiles");
    constexpr int LPP = WN / 8;                // epilogue: lanes per pixel (8 channels each)
    constexpr int PPI = 64 / LPP;              // epilogue: pixels per wavefront instruction
    constexpr int NIT = 32 / PPI;              // epilogue: instructions per 32-pixel sub-tile
    constexpr int EPITCH = WN * 4 + 16;        // epilogue: padded fp32 row pitch in LDS (bytes)
    static_assert(8 * 32 * EPITCH <= 3 * BUF, "epilogue tile must fit in the pipeline buffers");

    extern __shared__ __align__(128) unsigned char smem[];

    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wv % WAVES_M, wn = wv / WAVES_M;
    const int HoWo = a.Ho * a.Wo;
    const int M = a.N * HoWo;
    const int K = a.kh * a.kw * a.Cin + (DUAL ? a.Cin2 : 0);
    const int KT = K / BK;
    const int tiles_n = a.Cout / BN;
    // Workgroups are dealt round-robin to the 8 XCDs (each with its own L2): give every XCD a contiguous range of tiles so
    // that tiles sharing an activation tile hit the same L2.
    const int total_tiles = ((M + BM - 1) / BM) * tiles_n;
    const int per_xcd = (total_tiles + 7) >> 3;
    const int tile = (int)(blockIdx.x & 7u) * per_xcd + (int)(blockIdx.x >> 3);
    if (tile >= total_tiles) return;
    const int tile_m = a.by_tiles(tile), tile_n = tile - tile_m * tiles_n;
    const int m0 = tile_m * BM, n0 = tile_n * BN;

    // ---- bias: where the sums start
    f32x16_t acc[TN][TM];
    f32x4_t bias_q[TN][4];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v)   // element e of lane l: channel 8 (e / 4) + 4 (l / 32) + e % 4
            bias_q[i][v] = *reinterpret_cast<const f32x4_t*>(a.bias + n0 + wn * WN + i * 32 + 8 * v + 4 * (lane >> 5));

    // ---- requests.  One wavefront instruction fills 8 whole rows of a tile in LDS (lane l's 16 bytes at base + 16 l); a lane
    // fetches the 16-byte chunk (slot ^ swz(row)) of its row, swz(row) = (row & 7) ^ ((row >> 3) & 1), so that the fragment
    // reads of 16 consecutive rows at one chunk fall on 16 different 16-byte slots modulo 256 bytes.
    // q: the thread's row among the 64 of one pass of the block.
    const int q = wv * 8 + (lane >> 3);
    const int chunk = ((lane & 7) ^ (lane >> 3) ^ (wv & 1)) & 7;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte*)smem;
    // weights: pass u of half g is row 128 u + 64 (q / 32) + 32 g + q % 32 (QUAD), or pass p is row 64 p + q
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(static_cast<const T*>(a.w) + (size_t)n0 * K), 0, 0x80000000, 0x00020000);
    const int row_bytes = K * 2;
    const uint32_t w_off = (uint32_t)((QUAD ? (q >> 5) * 64 + (q & 31) : q) * row_bytes + chunk * 16);
    const uint32_t w_dst = lds0 + (uint32_t)((QUAD ? (wv >> 2) * 64 + (wv & 3) * 8 : wv * 8) * ROW);
    auto request_w = [&](int g, int kt, uint32_t buf) {   // half g
#pragma unroll
        for (int u = 0; u < PA / 2; ++u) {
            const int row = QUAD ? 128 * u + 32 * g : 64 * g;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_byte*)(uintptr_t)(w_dst + buf + (uint32_t)(row * ROW)), 16, w_off, row * row_bytes + kt * ROW, 0, 0);
        }
    };
    request_w(0, 0, 0);   // (they need no pixel arithmetic)
    request_w(1, 0, 0);
    // pixels: row of pass p.  QUAD: halves of 256: passes 0, 1 and 2, 3; of 192: 0, 1 and 2 (32 rows of either wavefront row).
    auto x_row = [&](int p, int r) {
        if constexpr (!QUAD) return 64 * p + r;
        else if constexpr (BM == 256) return (p & 1) * 128 + (p >> 1) * 64 + r;
        else return p < 2 ? p * 96 + r : (r < 32 ? 64 + r : 128 + r);
    };
    // offsets count from tap 0 of the first pixel of the block's first row (large_first_row), so that they have 31 bits whatever the
    // size of an image
    const int img0 = a.by_hw(m0), oy0 = a.by_w(m0 - img0 * HoWo), row0 = large_first_row(oy0, a.stride, a.H);
    const T* x_base = static_cast<const T*>(a.in) + (((long long)img0 * a.H + row0) * a.W - (ONE ? 0 : (long long)a.pad * (a.W + 1))) * a.Cin;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(x_base), 0, 0x80000000, 0x00020000);
    const __amdgpu_buffer_rsrc_t rx2 = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(static_cast<const T*>(DUAL ? a.in2 : a.in) + (DUAL ? ((long long)img0 * a.H2 + oy0 * a.stride2) * a.W2 * a.Cin2 : 0)), 0, 0x80000000, 0x00020000);
    uint32_t x_off[PB], x_off2[DUAL ? PB : 1], x_taps[ONE ? 1 : PB];
    uint32_t every_row = 0;
    if constexpr (!ONE)
        for (int ky = 0; ky < a.kh; ++ky) every_row |= 1u << (ky * a.kw);
#pragma unroll
    for (int p = 0; p < PB; ++p) {
        const int m = m0 + x_row(p, q);
        const int img = a.by_hw(m), rem = m - img * HoWo;
        const int oy = a.by_w(rem), ox = rem - oy * a.Wo;
        const bool ok = m < M;
        x_off[p] = (uint32_t)((((img - img0) * a.H + oy * a.stride - row0) * a.W + ox * a.stride) * a.Cin * 2 + chunk * 16);
        if constexpr (ONE) {
            x_off[p] = ok ? x_off[p] : OUTSIDE;
        } else {
            x_taps[p] = ok ? tap_mask(oy * a.stride - a.pad, ox * a.stride - a.pad, a.H, a.W, a.kh, a.kw, every_row) : 0u;
        }
        if constexpr (DUAL)
            x_off2[p] = ok ? (uint32_t)((((img - img0) * a.H2 + (oy - oy0) * a.stride2) * a.W2 + ox * a.stride2) * a.Cin2 * 2 + chunk * 16) : OUTSIDE;
    }
    const uint32_t x_dst = lds0 + XOFF;
    const int cin_tiles = a.Cin / BK;   // K tiles of a tap, or of the first source
    int x_kt = 0, x_c = 0, x_kx = 0, x_tap = 0, x_so = 0;   // K tile that the next pixel requests are for: tile, channel tile, tap, byte offset
    auto request_x = [&](auto hc, uint32_t buf) {
        constexpr int h = decltype(hc)::value;
        static_for<2 * h, (h == 0 ? 2 : PB)>([&](auto pc) {
            constexpr int p = decltype(pc)::value;
            lds_byte* dst = (lds_byte*)(uintptr_t)(x_dst + buf + (uint32_t)(x_row(p, wv * 8) * ROW));
            if constexpr (DUAL) {
                if (x_kt < cin_tiles) __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, dst, 16, x_off[p], x_kt * ROW, 0, 0);
                else __builtin_amdgcn_raw_ptr_buffer_load_lds(rx2, dst, 16, x_off2[DUAL ? p : 0], (x_kt - cin_tiles) * ROW, 0, 0);
            } else if constexpr (ONE) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, dst, 16, x_off[p], x_kt * ROW, 0, 0);
            } else {
                const uint32_t off = (x_taps[ONE ? 0 : p] >> x_tap) & 1u ? x_off[p] : OUTSIDE;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, dst, 16, off, x_so, 0, 0);
            }
        });
    };
    auto next_x = [&]() {
        ++x_kt;
        if constexpr (!ONE) {
            x_so += ROW;
            if (++x_c == cin_tiles) {   // next tap: along the filter row, then to the next input row
                x_c = 0;
                ++x_tap;
                if (++x_kx == a.kw) { x_kx = 0; x_so += (a.W - a.kw) * a.Cin * 2; }
            }
        }
    };
    constexpr std::integral_constant<int, 0> H0{};
    constexpr std::integral_constant<int, 1> H1{};
    request_x(H0, 0);
    request_x(H1, 0);
    next_x();
    request_w(0, 1, BUF);
    request_x(H0, BUF);
    request_w(1, 1, BUF);
    request_x(H1, BUF);
    next_x();

    // ---- fragments: lane l holds row l % 32, k = 8 (l / 32) .. + 7 of a k-step
    const int frag_row = lane & 31, frag_off = (lane >> 5) * 16;
    uint32_t w_at[KK], x_at[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        const uint32_t slot = (uint32_t)(((2 * kk + (lane >> 5)) ^ (frag_row & 7) ^ ((frag_row >> 3) & 1)) * 16);
        w_at[kk] = lds0 + (uint32_t)((wn * WN + frag_row) * ROW) + slot;
        x_at[kk] = lds0 + XOFF + (uint32_t)((wm * WM + frag_row) * ROW) + slot;
    }
    u32x4_t wf[TN][KK], xf[QUAD ? 2 : TM][KK];
    auto read_w = [&](auto gc) {
        constexpr int g = decltype(gc)::value;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) wf[g][kk] = *(const lds_u32x4*)(uintptr_t)(w_at[kk] + (uint32_t)(g * 32 * ROW));
    };
    auto read_x = [&](auto hc) {
        constexpr int h = decltype(hc)::value;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
            for (int j = 0; j < (h == 0 ? 2 : TM1); ++j) xf[j][kk] = *(const lds_u32x4*)(uintptr_t)(x_at[kk] + (uint32_t)((h * 64 + j * 32) * ROW));
    };
    auto multiply = [&](auto gc, auto hc) {
        constexpr int g = decltype(gc)::value, h = decltype(hc)::value;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
            for (int j = 0; j < (h == 0 ? 2 : TM1); ++j) mma_step<T>(acc[g][2 * h + j], wf[g][kk], xf[j][kk]);
    };
    // waits for nothing but the other wavefronts: LDS accesses that others depend on are waited for (lgkmcnt) in front of it
    auto barrier = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // vmcnt(n) lgkmcnt(0), nothing moves across
    auto wait = [&](auto nc) {
        constexpr int n = decltype(nc)::value;
        static_assert(n >= 0 && n < 64, "vmcnt counts to 63");
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0070 | (n & 15) | ((n >> 4) << 14));
    };
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                acc[i][j][4 * v] = bias_q[i][v].x; acc[i][j][4 * v + 1] = bias_q[i][v].y;
                acc[i][j][4 * v + 2] = bias_q[i][v].z; acc[i][j][4 * v + 3] = bias_q[i][v].w;
            }
    if constexpr (QUAD) {
        // requests of one thread in phase 1..4, and those outstanding behind the half that phase j + 1 reads when the last
        // `skip` of the phases j - 5 .. j requested nothing (the end of the loop)
        constexpr auto left = [](int j, int skip) {
            int n = 0;
            for (int i = j - 5; i <= j - skip; ++i) n += ((i + 7) & 3) == 3 ? TM1 : 2;
            return n;
        };

        // ---- loop.  TAIL: K tiles behind this one, if fewer than two (2: two or more)
        auto k_tile = [&](auto tail, int kt, uint32_t buf) {
            constexpr int TAIL = decltype(tail)::value;
            constexpr int S0 = TAIL == 2 ? 1 : TAIL == 1 ? 1 : 5;   // phases without requests, counted at phase 1 (TAIL 2: none)
            static_for<1, 5>([&](auto pc) {
                constexpr int P = decltype(pc)::value;
                if constexpr (P == 1) read_x(H0);
                if constexpr (P == 2) read_w(H1);
                if constexpr (P == 3) read_x(H1);
                if constexpr (P == 4) {
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk) { w_at[kk] ^= BUF; x_at[kk] ^= BUF; }
                    if constexpr (TAIL > 0) read_w(H0);
                }
                if constexpr (TAIL == 2) {
                    if constexpr (P == 1) request_w(0, kt + 2, buf);
                    if constexpr (P == 2) request_x(H0, buf);
                    if constexpr (P == 3) request_w(1, kt + 2, buf);
                    if constexpr (P == 4) { request_x(H1, buf); next_x(); }
                }
                constexpr int skip = TAIL == 2 ? 0 : S0 + P - 1;
                wait(std::integral_constant<int, left(P, skip < 6 ? skip : 6)>{});
                barrier();
                __builtin_amdgcn_s_setprio(1);
                if constexpr (P == 1) multiply(H0, H0);
                if constexpr (P == 2) multiply(H1, H0);
                if constexpr (P == 3) multiply(H0, H1);
                if constexpr (P == 4) multiply(H1, H1);
                __builtin_amdgcn_s_setprio(0);
                barrier();
            });
        };
        // all of tile 1 and nothing of the first three halves requested (W0, W1, X0 of tile 0) may be on its way
        wait(std::integral_constant<int, TM1 + 4 + PB>{});
        barrier();
        read_w(H0);
        wait(std::integral_constant<int, TM1 + 4 + PB>{});
        barrier();
        if (wv >= 4) barrier();
        uint32_t buf = 0;
        int kt = 0;
        for (; kt + 2 < KT; ++kt) {
            k_tile(std::integral_constant<int, 2>{}, kt, buf);
            buf ^= BUF;
        }
        k_tile(std::integral_constant<int, 1>{}, kt, buf);
        k_tile(std::integral_constant<int, 0>{}, kt + 1, buf ^ BUF);
    } else {
        constexpr int PER_TILE = PA + PB;
        auto read_half = [&](auto hc) {
            constexpr int h = decltype(hc)::value;
#pragma unroll
            for (int kk = 2 * h; kk < 2 * h + 2; ++kk) {
#pragma unroll
                for (int i = 0; i < TN; ++i) wf[i][kk] = *(const lds_u32x4*)(uintptr_t)(w_at[kk] + (uint32_t)(i * 32 * ROW));
#pragma unroll
                for (int j = 0; j < TM; ++j) xf[j][kk] = *(const lds_u32x4*)(uintptr_t)(x_at[kk] + (uint32_t)(j * 32 * ROW));
            }
        };
        auto multiply_half = [&](auto hc) {
            constexpr int h = decltype(hc)::value;
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int kk = 2 * h; kk < 2 * h + 2; ++kk)
#pragma unroll
                for (int i = 0; i < TN; ++i)
#pragma unroll
                    for (int j = 0; j < TM; ++j) mma_step<T>(acc[i][j], wf[i][kk], xf[j][kk]);
            __builtin_amdgcn_s_setprio(0);
        };
        uint32_t at = 0, to = 2 * BUF;   // buffers of tile kt and of tile kt + 2
        auto k_tile = [&](auto tail, int kt) {
            constexpr int TAIL = decltype(tail)::value;
            read_half(H0);
            if constexpr (TAIL == 2) { request_x(H0, to); request_w(0, kt + 2, to); }
            wait(std::integral_constant<int, 63>{});
            barrier();
            multiply_half(H0);
            barrier();
            read_half(H1);
            if constexpr (TAIL == 2) { request_x(H1, to); request_w(1, kt + 2, to); next_x(); }
            const uint32_t step = at == 2 * BUF ? (uint32_t)(0 - 2 * BUF) : BUF;   // to the next tile's buffer
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) { w_at[kk] += step; x_at[kk] += step; }
            to = at;
            at += step;
            wait(std::integral_constant<int, TAIL == 2 ? PER_TILE : 0>{});
            barrier();
            multiply_half(H1);
            barrier();
        };
        wait(std::integral_constant<int, PER_TILE>{});   // tile 0 has landed
        barrier();
        if (wv >= 4) barrier();
        int kt = 0;
        for (; kt + 2 < KT; ++kt) k_tile(std::integral_constant<int, 2>{}, kt);
        k_tile(std::integral_constant<int, 1>{}, kt);
        k_tile(std::integral_constant<int, 0>{}, kt + 1);
    }
    if (wv < 4) barrier();
    // (every wavefront has read its last fragments and no request is on its way: LDS is free)

    // ---- fused RPN predictors (large bf16 tile only): the block's ReLU'd 256 x 256 tile, rounded to bf16 as the
    // stored tensor would be, stays in LDS and is contracted with the 1x1 predictor weights right away.
    if constexpr (BM == 256 && BN == 256 && MODE == 0) {
        if (a.head_w != nullptr) {
            constexpr int YP = BN * 2 + 16;            // LDS row pitch of the bf16 tile
            constexpr int HKS = BN / 16;               // k-steps of the predictor contraction (16)
            constexpr int HP = 96 * 4 + 16;            // fp32 row pitch of the per-wavefront output tile
            static_assert(BM * YP <= 160 * 1024 && 32 * HP <= 32 * YP, "tile and output staging fit (launch_large_cfg requests BM * YP bytes)");
            const u32x4_t* __restrict__ hwf = reinterpret_cast<const u32x4_t*>(a.head_w) + lane;
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int i = 0; i < TN; ++i)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int ch = wn * WN + i * 32 + 8 * v + 4 * (lane >> 5);
                        u32x2_t o = {pack_bf16x2(fmaxf(acc[i][j][4 * v], 0.f), fmaxf(acc[i][j][4 * v + 1], 0.f)),
                                     pack_bf16x2(fmaxf(acc[i][j][4 * v + 2], 0.f), fmaxf(acc[i][j][4 * v + 3], 0.f))};
                        *reinterpret_cast<u32x2_t*>(smem + (size_t)(wm * WM + j * 32 + frag_row) * YP + ch * 2) = o;
                    }
            // predictor weight fragments (3 channel tiles per k-step) run HRING k-steps ahead of their use; the first
            // ones and the bias tile are requested once the accumulators are parked, in flight across the barrier
            constexpr int HRING = 4;   // (8 spills and is slower)
            __builtin_amdgcn_sched_barrier(0);   // (hoisted above the parking loop they would spill)
            u32x4_t hw[HRING * 3];
#pragma unroll
            for (int ks = 0; ks < HRING; ++ks)
#pragma unroll
                for (int i = 0; i < 3; ++i) hw[ks * 3 + i] = hwf[(i * HKS + ks) * 64];
            f32x16_t hacc[3];
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const f32x4_t q = *reinterpret_cast<const f32x4_t*>(a.head_b + i * 32 + 8 * v + 4 * (lane >> 5));
                    hacc[i][4 * v] = q.x; hacc[i][4 * v + 1] = q.y; hacc[i][4 * v + 2] = q.z; hacc[i][4 * v + 3] = q.w;
                }
            __syncthreads();
            // wavefront wv: pixels 32 wv .. 32 wv + 31 of the tile against all 96 (padded) predictor rows
            const unsigned char* yrow = smem + (size_t)(wv * 32 + frag_row) * YP + frag_off;
            static_for<0, HKS>([&](auto kc) {
                constexpr int ks = decltype(kc)::value;
                const u32x4_t b = *reinterpret_cast<const u32x4_t*>(yrow + ks * 32);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    mma_step<T>(hacc[i], hw[(ks % HRING) * 3 + i], b);
                    if (ks + HRING < HKS) hw[(ks % HRING) * 3 + i] = hwf[(i * HKS + ks + HRING) * 64];
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            // the wavefront's own 32 rows of the tile are dead now: fp32 results go there, then out in dense rows
            unsigned char* hp = smem + (size_t)(wv * 32) * YP;
            __builtin_amdgcn_s_waitcnt(0xc07f);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    f32x4_t r = {hacc[i][4 * v], hacc[i][4 * v + 1], hacc[i][4 * v + 2], hacc[i][4 * v + 3]};
                    *reinterpret_cast<f32x4_t*>(hp + (size_t)frag_row * HP + (i * 32 + 8 * v + 4 * (lane >> 5)) * 4) = r;
                }
            __builtin_amdgcn_s_waitcnt(0xc07f);
            __builtin_amdgcn_wave_barrier();
            const int A = a.head_a;
            const int mbase = m0 + wv * 32;
            for (int e = lane; e < 32 * A; e += 64) {
                const int px = e / A, an = e - px * A;
                if (mbase + px >= M) continue;
                const f32x4_t d = *reinterpret_cast<const f32x4_t*>(hp + (size_t)px * HP + an * 16);
                *reinterpret_cast<f32x4_t*>(a.head_deltas + ((size_t)(mbase + px) * A + an) * 4) = d;
                a.head_logits[(size_t)(mbase + px) * A + an] = *reinterpret_cast<const float*>(hp + (size_t)px * HP + (4 * A + an) * 4);
            }
            return;
        }
    }

    // ---- expansion tail (256 x 256 tile only): the block's ReLU'd tile, rounded to bf16 as the stored tensor would be, is
    // parked in LDS (unpadded 512-byte rows, 16-byte chunk index XOR-ed with the row) and contracted with the next 1x1 layer's
    // weights (fragment order).  The eight wavefronts take 32 channels each of 256 at a time, for one 128-pixel half of the
    // tile after the other.  It is bound by memory: residual and result are four times the tile (268 MB for 65 280 pixels, 53 us at
    // the rate of a copy) and nothing else of the launch touches memory much.  So the residual of the next half is requested
    // as soon as the registers of this one's are free, with the products of a half to arrive under, and the weights stay in
    // registers for both halves (refilled under the second): loads complete in order, a weight fetched from L2 behind the
    // residual would wait for it.  Residual and result pass through a 4 KB wavefront-private LDS region as bf16, so that global
    // loads and stores are 16 bytes per lane and cover whole lines together with the neighbouring wavefront's; the sum is formed
    // in accumulator layout in fp32 and rounded once.
    if constexpr (MODE == 4) {
        constexpr int TKS = BN / 16;               // k-steps of the tail contraction (16)
        const int lh = lane >> 5;
        auto yoff = [](int row, int byteoff) { return row * 512 + ((((byteoff >> 4) ^ row) & 31) << 4) + (byteoff & 15); };
        auto roff = [](int row, int byteoff) { return row * 64 + ((((byteoff >> 4) ^ (row >> 2)) & 3) << 4) + (byteoff & 15); };
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int ch = wn * WN + i * 32 + 8 * v + 4 * lh;
                    u32x2_t o = {pack_bf16x2(fmaxf(acc[i][j][4 * v], 0.f), fmaxf(acc[i][j][4 * v + 1], 0.f)),
                                 pack_bf16x2(fmaxf(acc[i][j][4 * v + 2], 0.f), fmaxf(acc[i][j][4 * v + 3], 0.f))};
                    *reinterpret_cast<u32x2_t*>(smem + yoff(wm * WM + j * 32 + frag_row, ch * 2)) = o;
                }
        __builtin_amdgcn_sched_barrier(0);
        const int N3 = a.tail_n, groups = N3 / 256;
        // descriptors over the tile's rows that exist: reads of the others give zeros, stores are dropped
        const uint32_t tile_bytes = (uint32_t)((M - m0 < BM ? M - m0 : BM) * N3 * 2);
        const __amdgpu_buffer_rsrc_t rt = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.tail_w), 0, (uint32_t)N3 * 512, 0x00020000);
        const __amdgpu_buffer_rsrc_t rres = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(static_cast<const T*>(a.tail_res) + (size_t)m0 * N3), 0, tile_bytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(static_cast<T*>(a.tail_out) + (size_t)m0 * N3, 0, tile_bytes, 0x00020000);
        const uint32_t piece = (uint32_t)((lane >> 2) * N3 * 2 + (lane & 3) * 16);   // the lane's 16 bytes of a row's 64; rows lane / 4 + 16 it
        auto place = [&](int hp, int j, int it) { return piece + (uint32_t)((hp * 128 + j * 32 + 16 * it) * N3 * 2); };
        u32x4_t wt[TKS], rq[4][2];
        f32x4_t bq[4];
        auto fetch_w = [&](int g, int ks) { return __builtin_amdgcn_raw_buffer_load_b128(rt, (uint32_t)lane * 16, ((8 * g + wv) * TKS + ks) * 1024, 0); };
        auto fetch_b = [&](int g, int v) { return *reinterpret_cast<const f32x4_t*>(a.tail_b + (8 * g + wv) * 32 + 8 * v + 4 * lh); };
        auto fetch_res = [&](int g, int hp, int j, int it) { return __builtin_amdgcn_raw_buffer_load_b128(rres, place(hp, j, it), (8 * g + wv) * 64, 0); };
#pragma unroll
        for (int v = 0; v < 4; ++v) bq[v] = fetch_b(0, v);
#pragma unroll
        for (int ks = 0; ks < TKS; ++ks) wt[ks] = fetch_w(0, ks);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int it = 0; it < 2; ++it) rq[j][it] = fetch_res(0, 0, j, it);
        wait(std::integral_constant<int, 63>{});   // the wavefront's part of the tile is in LDS (the loads stay on their way)
        barrier();
        unsigned char* R = smem + 256 * 512 + wv * 4096;
        // pixel operand of the tail's MFMAs: row hp * 128 + j * 32 + frag_row, logical chunk 2 ks + lane / 32; the rows of one
        // fragment differ in their low five bits only (= frag_row), so the swizzled chunk is (x0 ^ 2 ks) for every j and hp
        const int x0 = (lh ^ frag_row) & 31;
        const unsigned char* ylane = smem + frag_row * 512;
        // one half of the tile against 256 channels; MORE: channels come behind these
        auto half = [&](auto hc, auto more, int g) {
            constexpr int hp = decltype(hc)::value;
            constexpr bool MORE = decltype(more)::value != 0, NEXT = hp == 0 || MORE;
            f32x16_t t4[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) { t4[j][4 * v] = bq[v].x; t4[j][4 * v + 1] = bq[v].y; t4[j][4 * v + 2] = bq[v].z; t4[j][4 * v + 3] = bq[v].w; }
            u32x4_t y[2][4];   // the next k-step's pixels are read while this one's are multiplied
            auto read_y = [&](int ks, u32x4_t* to) {
#pragma unroll
                for (int j = 0; j < 4; ++j) to[j] = *reinterpret_cast<const u32x4_t*>(ylane + (hp * 128 + j * 32) * 512 + ((x0 ^ (2 * ks)) << 4));
            };
            read_y(0, y[0]);
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, TKS>([&](auto kc) {
                constexpr int ks = decltype(kc)::value;
                if constexpr (ks + 1 < TKS) read_y(ks + 1, y[(ks + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 4; ++j) mma_step<T>(t4[j], wt[ks], y[ks & 1][j]);
                if constexpr (hp == 1 && MORE) wt[ks] = fetch_w(g + 1, ks);
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (hp == 1 && MORE) {
#pragma unroll
                for (int v = 0; v < 4; ++v) bq[v] = fetch_b(g + 1, v);
            }
            static_for<0, 2>([&](auto pc) {   // two 32-pixel sub-tiles at a time
                constexpr int j0 = 2 * decltype(pc)::value;
#pragma unroll
                for (int j = j0; j < j0 + 2; ++j)
#pragma unroll
                    for (int it = 0; it < 2; ++it) *reinterpret_cast<u32x4_t*>(R + (j - j0) * 2048 + roff((lane >> 2) + 16 * it, (lane & 3) * 16)) = rq[j][it];
                if constexpr (NEXT) {
#pragma unroll
                    for (int j = j0; j < j0 + 2; ++j)
#pragma unroll
                        for (int it = 0; it < 2; ++it) rq[j][it] = fetch_res(hp == 0 ? g : g + 1, 1 - hp, j, it);
                }
                __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the region is private to this wavefront
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int j = j0; j < j0 + 2; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        unsigned char* pp = R + (j - j0) * 2048 + roff(frag_row, (8 * v + 4 * lh) * 2);
                        const u32x2_t r = *reinterpret_cast<const u32x2_t*>(pp);
                        const float r0 = fmaxf(t4[j][4 * v] + __uint_as_float(r.x << 16), 0.f);
                        const float r1 = fmaxf(t4[j][4 * v + 1] + __uint_as_float(r.x & 0xffff0000u), 0.f);
                        const float r2 = fmaxf(t4[j][4 * v + 2] + __uint_as_float(r.y << 16), 0.f);
                        const float r3 = fmaxf(t4[j][4 * v + 3] + __uint_as_float(r.y & 0xffff0000u), 0.f);
                        const u32x2_t o = {pack_bf16x2(r0, r1), pack_bf16x2(r2, r3)};
                        *reinterpret_cast<u32x2_t*>(pp) = o;   // the lane rewrites exactly the bytes it has read
                    }
                __builtin_amdgcn_s_waitcnt(0xc07f);
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int j = j0; j < j0 + 2; ++j)
#pragma unroll
                    for (int it = 0; it < 2; ++it) {
                        const u32x4_t o = *reinterpret_cast<const u32x4_t*>(R + (j - j0) * 2048 + roff((lane >> 2) + 16 * it, (lane & 3) * 16));
                        __builtin_amdgcn_raw_buffer_store_b128(o, rout, place(hp, j, it), (8 * g + wv) * 64, 0);
                    }
                __builtin_amdgcn_s_waitcnt(0xc07f);
                __builtin_amdgcn_wave_barrier();
            });
        };
        int g = 0;
        for (; g + 1 < groups; ++g) {
            half(H0, H1, g);
            half(H1, H1, g);
        }
        half(H0, H0, g);
        half(H1, H0, g);
        return;
    }

    // ---- epilogue.  Accumulator element e of lane l: channel 8*(e/4) + 4*(l/32) + e%4, pixel l%32.
    T* __restrict__ out0 = static_cast<T*>(a.out0);
    const T* __restrict__ res = static_cast<const T*>(a.res);
    {
        // Coalesced path, one 32-pixel sub-tile at a time: the wavefront parks its 32 pixel x WN channel
        // fp32 tile in its own LDS region (the pipeline buffers are free now) and re-reads it so
        // that each lane owns 8 consecutive channels of one pixel: residual loads and output stores are
        // 16-byte and the lanes of one instruction cover whole lines of the NHWC tensors.
        unsigned char* ep = smem + (size_t)wv * (32 * EPITCH);
        {
            // No residual: ReLU and the rounding to bf16 are applied in accumulator layout, and the tile goes through
            // LDS already rounded - half the LDS traffic, one 16-byte read per store (same values as the fp32 round trip).
            if (res == nullptr) {
                constexpr int EPB = WN * 2 + 16;   // bf16 row pitch
                const bool relu = a.relu != 0;
                static_for<0, TM>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
#pragma unroll
                    for (int i = 0; i < TN; ++i)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            float r0 = acc[i][j][4 * v], r1 = acc[i][j][4 * v + 1], r2 = acc[i][j][4 * v + 2], r3 = acc[i][j][4 * v + 3];
                            if (relu) { r0 = fmaxf(r0, 0.f); r1 = fmaxf(r1, 0.f); r2 = fmaxf(r2, 0.f); r3 = fmaxf(r3, 0.f); }
                            const u32x2_t o = {pack_bf16x2(r0, r1), pack_bf16x2(r2, r3)};
                            *reinterpret_cast<u32x2_t*>(ep + (size_t)frag_row * EPB + (i * 32 + 8 * v + 4 * (lane >> 5)) * 2) = o;
                        }
                    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the region is private to this wavefront
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int it = 0; it < NIT; ++it) {
                        const int pxl = it * PPI + lane / LPP, ck = lane % LPP;
                        const int pix = m0 + wm * WM + j * 32 + pxl, ch = n0 + wn * WN + ck * 8;
                        const u32x4_t q = *reinterpret_cast<const u32x4_t*>(ep + (size_t)pxl * EPB + ck * 16);
                        if (pix < M) *reinterpret_cast<u32x4_t*>(out0 + (size_t)pix * a.ld0 + ch) = q;
                    }
                    __builtin_amdgcn_s_waitcnt(0xc07f);
                    __builtin_amdgcn_wave_barrier();
                });
                return;
            }
        }
        // residual: fetched one sub-tile ahead of its use
        Vec8<T> rq0[NIT], rq1[NIT];
        auto fetch_res = [&](int j, Vec8<T>* dst) {
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
                const int pix = m0 + wm * WM + j * 32 + it * PPI + lane / LPP, ch = n0 + wn * WN + (lane % LPP) * 8;
                if (pix < M) dst[it] = *reinterpret_cast<const Vec8<T>*>(res + (size_t)pix * a.Cout + ch);
            }
        };
        fetch_res(0, rq0);
        static_for<0, TM>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            Vec8<T>* rnow = (j & 1) ? rq1 : rq0;
            if (j + 1 < TM) fetch_res(j + 1, (j & 1) ? rq0 : rq1);
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int chl = i * 32 + 8 * v + 4 * (lane >> 5);
                    f32x4_t r = {acc[i][j][4 * v], acc[i][j][4 * v + 1], acc[i][j][4 * v + 2], acc[i][j][4 * v + 3]};
                    *reinterpret_cast<f32x4_t*>(ep + (size_t)frag_row * EPITCH + chl * 4) = r;
                }
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the region is private to this wavefront
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
                const int pxl = it * PPI + lane / LPP, ck = lane % LPP;
                const int pix = m0 + wm * WM + j * 32 + pxl, ch = n0 + wn * WN + ck * 8;
                if (pix >= M) continue;
                const f32x4_t lo = *reinterpret_cast<const f32x4_t*>(ep + (size_t)pxl * EPITCH + ck * 32);
                const f32x4_t hi = *reinterpret_cast<const f32x4_t*>(ep + (size_t)pxl * EPITCH + ck * 32 + 16);
                float r[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                float rv[8];
                unpack8(rnow[it], rv);
#pragma unroll
                for (int e = 0; e < 8; ++e) r[e] += rv[e];
                if (a.relu) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) r[e] = fmaxf(r[e], 0.f);
                }
                store8(out0 + (size_t)pix * a.ld0 + ch, r);
            }
            __builtin_amdgcn_s_waitcnt(0xc07f);
            __builtin_amdgcn_wave_barrier();
        });
    }
#endif
}

template <int BM, int BN, int MODE>
static hipError_t launch_large_cfg(const ConvArgs& args, hipStream_t s) {
    ConvArgs a = args;
    a.by_hw = FastDiv(a.Ho * a.Wo);
    a.by_w = FastDiv(a.Wo);
    a.by_tiles = FastDiv(a.Cout / BN);
    // two buffers of 256 rows per operand; the fused predictors park a padded 256 x 528-byte tile instead, the expansion tail an
    // unpadded 256 x 512-byte tile and 4 KB per wavefront beside it (the CU's whole LDS)
    const size_t lds = BN != 256 ? (size_t)3 * (BN + BM) * 128 : MODE == 4 ? (size_t)160 * 1024 : BM == 256 && MODE == 0 ? (size_t)256 * 528 : (size_t)128 * 1024;
    auto kern = conv_large_kernel<BM, BN, MODE>;
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    const long long M = (long long)a.N * a.Ho * a.Wo;
    const long long tiles = ((M + BM - 1) / BM) * (a.Cout / BN);
    if (tiles <= 0 || tiles >= (1ll << 30)) return hipErrorInvalidValue;
    const long long grid = ((tiles + 7) / 8) * 8;  // 8 XCDs x equal ranges; surplus workgroups exit at once
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(512), lds, s, a);
    return hipGetLastError();
}

// Bytes of the source [H][W][Cin] from where a block's offsets count (large_first_row) to the end of what its pixels' taps reach.
// bm pixels lie in at most `down` + 1 output rows: from the first on, `stride` input rows for each, at the end of an image also the rows that
// no filter starts in, and the rows by which the first filter may start below its image.
static long long large_span(const ConvArgs& a, int bm, int stride, int H, int W, int Cin) {
    const long long down = (bm - 1 + a.Wo - 1) / a.Wo, images = (down + a.Ho - 1) / a.Ho;
    const long long unused = H - (long long)a.Ho * stride, below = (a.Ho - 1ll) * stride - H;
    const long long rows = down * stride + (unused > 0 ? images * unused : 0) + (below > 0 ? below : 0) + a.kh - 1;
    return (rows * W + W + a.pad) * Cin * 2;
}

bool conv_large_supported(const ConvArgs& a, int precision, int bm, int bn) {
    if (precision != 1 || !conv_supported(a, precision) || a.Cout % bn != 0 || a.out1 != nullptr || (a.ld0 & 7) != 0) return false;
    const long long K = (long long)a.kh * a.kw * a.Cin + (a.in2 ? a.Cin2 : 0);
    if (K < 128) return false;   // the loops have two K tiles under way
    // byte offsets within a block have 31 bits: of its weight rows, and of the input rows that its pixels read
    if (bn * K * 2 >= 1ll << 31 || large_span(a, bm, a.stride, a.H, a.W, a.Cin) >= 1ll << 31) return false;
    return a.in2 == nullptr || large_span(a, bm, a.stride2, a.H2, a.W2, a.Cin2) < 1ll << 31;
}

template <int BM, int BN>
static hipError_t launch_large(const ConvArgs& a, hipStream_t s) {
    if (a.in2) return launch_large_cfg<BM, BN, 2>(a, s);
    return a.kh == 1 && a.kw == 1 && a.pad == 0 ? launch_large_cfg<BM, BN, 1>(a, s) : launch_large_cfg<BM, BN, 0>(a, s);
}

hipError_t launch_conv_large(const ConvArgs& a, int bm, int bn, hipStream_t s) {
    if (!conv_large_supported(a, 1, bm, bn)) return hipErrorInvalidValue;
    if (bm == 256 && bn == 256) return a.tail_w ? launch_large_cfg<256, 256, 4>(a, s) : launch_large<256, 256>(a, s);
    if (a.head_w || a.tail_w) return hipErrorInvalidValue;
    if (bm == 192 && bn == 256) return launch_large<192, 256>(a, s);
    if (bm == 256 && bn == 128) return launch_large<256, 128>(a, s);
    if (bm == 192 && bn == 128) return launch_large<192, 128>(a, s);
    return hipErrorInvalidValue;
}

}  // namespace thia
