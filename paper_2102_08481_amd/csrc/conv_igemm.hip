// Implicit-GEMM convolution on the CDNA4 matrix cores (gfx950).
//
// Every convolution and fully connected layer of the detector (bottleneck 1x1/3x3,
// shortcut, exit lateral, RPN 3x3 and heads, FC layers and predictors) is the
// contraction  out[m, n] = sum_k W[n, k] * X[m, k]  with m = (image, oy, ox),
// n = output channel and k = (ky, kx, ci); activations are NHWC so a K tile of one
// filter tap is a contiguous run of input channels of one input pixel.
//
// Tiling: a block owns BM pixels x BN channels (32 x 32 to 128 x 128 here, 192 x 128 to 256 x 256 in conv_large.h, chosen
// by the layer's size in launch_conv) and walks K in 128-byte steps (64 bf16 / 32 fp32 per row).  Operand tiles go from
// global memory straight into LDS, two buffers requested by the multiplying wavefronts or, in calls with few pixels, a ring
// of 4 to 16 filled by wavefronts of its own; the streaming tile of the short-K layers (64-byte rows) stages them in registers.  Each wavefront owns part of
// the tile as 32x32 MFMA tiles.  The weights are the MFMA "A" operand (rows = channels) and the activations the
// "B" operand (columns = pixels): each lane then holds 4 consecutive channels of one
// pixel per accumulator quad, which is the contiguous direction of the NHWC output.
// Sums start from the bias (fp32), here as in the single-kernel blocks, the fused predictors and the expansion tail, so a
// layer's result does not depend on which of them a call's size picks.  Epilogue: [+ residual] [ReLU], then one rounding
// to the output type.
#include "conv_common.h"

namespace thia {

// 16 bytes per lane from global memory straight into LDS: lane l's bytes land at lds + 16 l (lds is uniform over the
// wavefront).  Counted by vmcnt like any vector memory load.  (The builtin exists in the device pass only.)
__device__ inline void load_to_lds16(const void* g, void* lds) {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_global_load_lds(g, lds, 16, 0, 0);
#endif
}

// 16 zero bytes (and some more) in global memory: what a padded filter tap fetches on the direct-to-LDS path
__device__ __align__(256) unsigned char g_zero_page[256];

// MODE 0: any filter size; 1: 1x1 unpadded (no tap bookkeeping); 2: 1x1 with a second source tensor.
// STAGES 2: double-buffered operand tiles; more: a ring of that many, U of them handed over at a time (see RING below).
template <typename T, int BM, int BN, int BKB, int WAVES_M, int WAVES_N, int MODE, typename OutT, int STAGES = 2, int PROD = 0, int U = 1>
__global__ __launch_bounds__(64 * (WAVES_M * WAVES_N + PROD), BKB == 64 ? 4 : 1) void conv_igemm_kernel(const ConvArgs a) {
    // (64-byte K rows: streaming layers, which want four blocks per CU, that is 128 registers)
    constexpr bool ONE = MODE == 1 || MODE == 2, DUAL = MODE == 2;
    constexpr int NW = WAVES_M * WAVES_N;       // wavefronts that multiply
    constexpr int NT = PROD ? 64 * PROD : 64 * NW;  // threads that load: all, or PROD wavefronts that do nothing else (ring)
    constexpr int BK = BKB / (int)sizeof(T);   // K elements per tile row
    constexpr int EPC = 16 / (int)sizeof(T);   // elements per 16-byte chunk
    constexpr int CPR = BKB / 16;              // 16-byte chunks per tile row
    constexpr int RPP = NT / CPR;              // tile rows covered by one pass of the block's threads
    constexpr int PB = BM / RPP, PA = BN / RPP;  // chunks staged per thread (activations, weights)
    // DIRECT (128-byte K rows): operand tiles go from global memory straight into LDS (global_load_lds_dwordx4: lane l of
    // a wavefront instruction lands at the instruction's LDS base + 16 l, i.e. one instruction fills 8 whole tile rows),
    // without staging registers or LDS-write instructions.  Rows are unpadded; instead a lane fetches the 16-byte chunk
    // (slot ^ swz(row)) of its row, swz(row) = (row & 7) ^ ((row >> 3) & 1), so that the fragment reads of 16 consecutive
    // rows at one logical chunk fall on 16 different 16-byte slots modulo 256 bytes (and any 8 aligned rows on 8 modulo 128).
    constexpr bool DIRECT = BKB == 128;
    constexpr int LDS_ROW = DIRECT ? BKB : BKB + 16;   // staged path: padded row pitch (an odd multiple of 16 bytes)
    constexpr bool RING = STAGES > 2;
    static_assert(RING ? STAGES % U == 0 && STAGES / U > 2 : U == 1, "the ring holds whole groups of tiles");
    static_assert(RING == (PROD > 0), "the ring is filled by loading wavefronts, the other paths have none");
    static_assert(!RING || DIRECT, "the ring holds direct-to-LDS tiles");
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;  // wavefront tile (pixels x channels)
    // F16 (ring): a wavefront owns one 16x16 tile instead, so that four times as many wavefronts share the work of a short call; the
    // contraction takes its k in the order of the 32x32 tiles (bf16: the 16x16x32 instruction adds its four groups of eight
    // products one after the other, as two 32x32x16 do their two: the same bits).
    constexpr bool F16 = WM == 16 && WN == 16, F32 = std::is_same<T, float>::value;
    static_assert(!F16 || STAGES > 2, "16x16 tiles: ring only");
    constexpr int KK = F16 && !F32 ? BKB / 64 : BKB / 32;   // MFMA k-steps per tile row (16 bytes for each of 4 lane groups, or 2 lane halves)
    constexpr int TM = F16 ? 1 : WM / 32, TN = F16 ? 1 : WN / 32;  // 32x32 MFMA tiles per wavefront
    constexpr int LPP = WN / 8;                // epilogue: lanes per pixel (8 channels each)
    constexpr int PPI = 64 / LPP;              // epilogue: pixels per wavefront instruction
    constexpr int NIT = 32 / PPI;              // epilogue: instructions per 32-pixel sub-tile
    constexpr int EPITCH = WN * 4 + 16;        // epilogue: padded fp32 row pitch in LDS (bytes)
    static_assert(TM * NIT <= 8, "the residual tile is held across the K loop");
    static_assert(DIRECT || !DUAL, "the staged path has one source");
    static_assert(WAVES_M * WAVES_N * 32 * EPITCH <= STAGES * (BN + BM) * LDS_ROW, "epilogue tile must fit in the pipeline buffers");
    static_assert(!DIRECT || (CPR == 8 && (NT / 64) % 2 == 0), "direct loads: 8 chunks per row, an even number of wavefronts");
    static_assert(BM % RPP == 0 && BN % RPP == 0, "tile rows must be a multiple of the rows staged per pass");

    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* sA = smem;                          // [STAGES][BN][LDS_ROW]
    unsigned char* sB = smem + STAGES * BN * LDS_ROW;  // [STAGES][BM][LDS_ROW]

    const int lane = threadIdx.x & 63, wave = RING ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6;
    const bool loads = PROD == 0 || wave >= NW;      // this wavefront requests operand tiles
    const bool multiplies = PROD == 0 || !loads;
    const int wv = PROD && loads ? wave - NW : wave, t = wv * 64 + lane;             // position among the wavefronts of its kind
    const int wm = wv % WAVES_M, wn = wv / WAVES_M;
    const int HoWo = a.Ho * a.Wo;
    const int M = a.N * HoWo;
    const int K = a.kh * a.kw * a.Cin + (DUAL ? a.Cin2 : 0);
    const int tiles_n = (a.Cout + BN - 1) / BN;
    // Workgroups are dealt round-robin to the 8 XCDs (each with its own L2): give every XCD a
    // contiguous range of tiles so that tiles sharing an activation tile hit the same L2.
    const int total_tiles = ((M + BM - 1) / BM) * tiles_n;
    const int per_xcd = (total_tiles + 7) >> 3;
    const int tile = (int)(blockIdx.x & 7u) * per_xcd + (int)(blockIdx.x >> 3);
    if (tile >= total_tiles) return;
    // (ring: with fewer pixels than output channels an XCD's range walks the pixel tiles of one channel tile first, so
    // that the larger operand, the weights, is read by one XCD only instead of by all eight)
    const int tiles_m = (M + BM - 1) / BM;
    const bool pixels_first = RING && M < a.Cout;
    const int slow = a.by_tiles(tile), fast = tile - slow * (pixels_first ? tiles_m : tiles_n);
    const int tile_n = pixels_first ? slow : fast, tile_m = pixels_first ? fast : slow;
    const int m0 = tile_m * BM, n0 = tile_n * BN;

    const T* __restrict__ in = static_cast<const T*>(a.in);
    const T* __restrict__ wgt = static_cast<const T*>(a.w);

    // ---- per-thread load coordinates: tile row lrow + RPP*p, 16-byte chunk lchunk of the row
    const int lrow = t / CPR;
    // staged path: the thread's chunk of the row; direct path: the chunk whose LDS slot is t % CPR (see DIRECT above;
    // row & 7 = lane / 8 and (row >> 3) & 1 = wavefront & 1 for every row lrow + RPP * p of this thread)
    const int lchunk = DIRECT ? ((t % CPR) ^ ((lane >> 3) ^ (wv & 1))) & 7 : t % CPR;
    // weight rows first: they need no pixel arithmetic, and on the direct path the first K tile's weight requests go out
    // before the (division-heavy) pixel coordinates are worked out
    size_t a_base[PA];
    bool a_ok[PA];
#pragma unroll
    for (int p = 0; p < PA; ++p) {
        const int n = n0 + lrow + RPP * p;
        a_ok[p] = n < a.Cout;
        a_base[p] = (size_t)(a_ok[p] ? n : 0) * K + (size_t)lchunk * EPC;
    }
    if (DIRECT && loads) {
        unsigned char* dA0 = sA + (size_t)((wv * 64) / CPR) * LDS_ROW;
#pragma unroll
        for (int p = 0; p < PA; ++p) load_to_lds16(wgt + a_base[p], dA0 + (size_t)(RPP * p) * LDS_ROW);
    }
    size_t b_base[PB];
    size_t b_base2[DUAL ? PB : 1];
    const T* __restrict__ in2 = static_cast<const T*>(a.in2);
    // general filters: signed element offset of the (tap 0, channel 0) input of the row's pixel and, per filter tap, one
    // bit "tap lies inside the image" (kh * kw <= 32)
    long long b_off0[ONE ? 1 : PB];
    uint32_t b_taps[ONE ? 1 : PB];
    bool b_ok[PB];
    uint32_t every_row = 0;
    if constexpr (!ONE)
        for (int ky = 0; ky < a.kh; ++ky) every_row |= 1u << (ky * a.kw);
#pragma unroll
    for (int p = 0; p < PB; ++p) {
        const int m = m0 + lrow + RPP * p;
        b_ok[p] = m < M;
        const int mm = b_ok[p] ? m : 0;   // (rows beyond M are clamped to row 0: they only feed outputs that are never stored)
        const int img = a.by_hw(mm), rem = mm - img * HoWo;
        const int oy = a.by_w(rem), ox = rem - oy * a.Wo;
        const int iy0 = oy * a.stride - a.pad, ix0 = ox * a.stride - a.pad;
        b_base[p] = (size_t)img * a.H * a.W * a.Cin + (size_t)lchunk * EPC;
        // 1x1, unpadded: the row's input pixel is fixed for the whole K loop
        if constexpr (ONE) {
            b_base[p] += ((size_t)iy0 * a.W + ix0) * a.Cin;
        } else {
            b_off0[p] = (long long)b_base[p] + ((long long)iy0 * a.W + ix0) * a.Cin;
            b_taps[p] = tap_mask(iy0, ix0, a.H, a.W, a.kh, a.kw, every_row);
        }
        if constexpr (DUAL)
            b_base2[p] = (((size_t)img * a.H2 + (size_t)oy * a.stride2) * a.W2 + (size_t)ox * a.stride2) * a.Cin2 + (size_t)lchunk * EPC;
    }
    const int cin_tiles = a.Cin / BK;
    const int KT = K / BK;

    // zmask: bit p set = activation chunk p is a padded tap and is written to LDS as zeros.  (The select is applied at
    // the LDS write, one step after the load: applied right after the load it would make every step wait for its data.)
    struct Stage { u32x4_t a[PA]; u32x4_t b[PB]; uint32_t zmask; };
    Stage st0;
    auto load_tiles = [&](int kt, Stage& st) {
        // All loads are unconditional: rows beyond M / Cout are clamped to row 0 (they only feed outputs that are
        // never stored), padded filter taps are fetched from a valid in-image address and zeroed at the LDS write.
        st.zmask = 0;
        if constexpr (ONE) {
#pragma unroll
            for (int p = 0; p < PB; ++p) st.b[p] = *reinterpret_cast<const u32x4_t*>(in + b_base[p] + (size_t)kt * BK);
#pragma unroll
            for (int p = 0; p < PA; ++p) st.a[p] = *reinterpret_cast<const u32x4_t*>(wgt + a_base[p] + (size_t)kt * BK);
            return;
        }
        const int tap = kt / cin_tiles;
        const int c0 = (kt - tap * cin_tiles) * BK;
        const int ky = tap / a.kw, kx = tap - ky * a.kw;
        const long long tap_off = ((long long)ky * a.W + kx) * a.Cin + c0;   // uniform over the block
        uint32_t zm = 0;
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const bool ok = (b_taps[ONE ? 0 : p] >> tap) & 1u;
            // a padded tap reads the row's (always valid) image base instead and is replaced by zeros at the LDS write
            const long long off = ok ? b_off0[ONE ? 0 : p] + tap_off : (long long)b_base[p];
            st.b[p] = *reinterpret_cast<const u32x4_t*>(in + off);
            zm |= ok ? 0u : (1u << p);
        }
        st.zmask = zm;
#pragma unroll
        for (int p = 0; p < PA; ++p) st.a[p] = *reinterpret_cast<const u32x4_t*>(wgt + a_base[p] + (size_t)kt * BK);
    };
    auto store_tiles = [&](int buf, const Stage& st) {
#pragma unroll
        for (int p = 0; p < PA; ++p)
            *reinterpret_cast<u32x4_t*>(sA + (size_t)(buf * BN + lrow + RPP * p) * LDS_ROW + lchunk * 16) = st.a[p];
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const u32x4_t z = {0u, 0u, 0u, 0u};
            const u32x4_t v = (!ONE && ((st.zmask >> p) & 1u)) ? z : st.b[p];
            *reinterpret_cast<u32x4_t*>(sB + (size_t)(buf * BM + lrow + RPP * p) * LDS_ROW + lchunk * 16) = v;
        }
    };

    // direct path: request K tile kt into LDS buffer buf (PA + PB wavefront instructions, each filling 8 rows)
    auto issue_tiles = [&](int kt, int buf) {
        unsigned char* dA = sA + (size_t)(buf * BN + (wv * 64) / CPR) * LDS_ROW;
        unsigned char* dB = sB + (size_t)(buf * BM + (wv * 64) / CPR) * LDS_ROW;
        if constexpr (ONE) {
            const int kt1 = a.Cin / BK;  // K tiles of the first source
            if (!DUAL || kt < kt1) {
#pragma unroll
                for (int p = 0; p < PB; ++p)
                    load_to_lds16(in + b_base[p] + (size_t)kt * BK, dB + (size_t)(RPP * p) * LDS_ROW);
            } else {
#pragma unroll
                for (int p = 0; p < PB; ++p)
                    load_to_lds16(in2 + b_base2[DUAL ? p : 0] + (size_t)(kt - kt1) * BK, dB + (size_t)(RPP * p) * LDS_ROW);
            }
        } else {
            const int tap = kt / cin_tiles;
            const int c0 = (kt - tap * cin_tiles) * BK;
            const int ky = tap / a.kw, kx = tap - ky * a.kw;
            const long long tap_off = ((long long)ky * a.W + kx) * a.Cin + c0;   // uniform over the block
#pragma unroll
            for (int p = 0; p < PB; ++p) {
                // a padded tap reads 16 zero bytes instead
                const bool ok = (b_taps[ONE ? 0 : p] >> tap) & 1u;
                const T* src = ok ? in + (b_off0[ONE ? 0 : p] + tap_off) : reinterpret_cast<const T*>(g_zero_page);
                load_to_lds16(src, dB + (size_t)(RPP * p) * LDS_ROW);
            }
        }
        if (kt == 0) return;   // the first tile's weight rows were requested at the top of the kernel
#pragma unroll
        for (int p = 0; p < PA; ++p)
            load_to_lds16(wgt + a_base[p] + (size_t)kt * BK, dA + (size_t)(RPP * p) * LDS_ROW);
    };

    // Sums start from the bias.  Its loads go out with the first tile's requests and are used behind the wait for that tile.
    f32x16_t acc[TN][TM];
    f32x4_t acc4 = {0.f, 0.f, 0.f, 0.f};                // F16: element e of lane l is channel 4 (l / 16) + e, pixel l % 16
    f32x4_t bias_q[TN][F16 ? 1 : 4];
    auto load_bias = [&]() {
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int v = 0; v < (F16 ? 1 : 4); ++v) {   // element e of lane l: channel 8 (e / 4) + 4 (l / 32) + e % 4
                const int ch = n0 + wn * WN + (F16 ? 4 * (lane >> 4) : i * 32 + 8 * v + 4 * (lane >> 5));
                f32x4_t q = {0.f, 0.f, 0.f, 0.f};
                if (ch + 4 <= a.Cout) {
                    q = *reinterpret_cast<const f32x4_t*>(a.bias + ch);
                } else {
                    if (ch < a.Cout) q.x = a.bias[ch];
                    if (ch + 1 < a.Cout) q.y = a.bias[ch + 1];
                    if (ch + 2 < a.Cout) q.z = a.bias[ch + 2];
                }
                bias_q[i][v] = q;
            }
    };
    auto start_sums = [&]() {
        if constexpr (F16) {
            acc4 = bias_q[0][0];
        } else {
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int j = 0; j < TM; ++j) {
                        acc[i][j][4 * v] = bias_q[i][v].x; acc[i][j][4 * v + 1] = bias_q[i][v].y;
                        acc[i][j][4 * v + 2] = bias_q[i][v].z; acc[i][j][4 * v + 3] = bias_q[i][v].w;
                    }
        }
    };

    // 8-channel-per-lane epilogue needs Cout, ld0 multiples of 8 and one dense output
    const bool vec = (a.out1 == nullptr) && ((a.Cout & 7) == 0) && ((a.ld0 & 7) == 0);
    const T* __restrict__ res = static_cast<const T*>(a.res);
    Vec8<T> rres[TM * NIT];
    if (RING && multiplies) load_bias();   // (in front of the residual: the sums wait for the bias only)
    struct alignas(4 * sizeof(T)) Quad { T v[4]; };
    Quad rquad = {};                                     // F16: the residual of the lane's four channels
    const bool quads = F16 && res != nullptr && (a.Cout & 3) == 0;
    if (quads && multiplies) {
        const int pix = m0 + wm * WM + (lane & 15), ch = n0 + wn * WN + 4 * (lane >> 4);
        if (pix < M && ch < a.Cout) rquad = *reinterpret_cast<const Quad*>(res + (size_t)pix * a.Cout + ch);
    }
    if (!F16 && multiplies && vec && res != nullptr) {  // residual tile: issued now, consumed after the K loop
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
                const int pix = m0 + wm * WM + j * 32 + it * PPI + lane / LPP, ch = n0 + wn * WN + (lane % LPP) * 8;
                if (pix < M && ch < a.Cout) rres[j * NIT + it] = *reinterpret_cast<const Vec8<T>*>(res + (size_t)pix * a.Cout + ch);
            }
    }

    const int frag_row = lane & 31, frag_off = (lane >> 5) * 16;
    // direct path: slot of logical chunk c in this lane's fragment row is c ^ frag_swz (tile row offsets are multiples of 16)
    const int frag_swz = (frag_row & 7) ^ ((frag_row >> 3) & 1);
    struct Frags { u32x4_t a[TN], b[TM]; };
    auto read_frags = [&](int buf, int kk, Frags& f) {
        if constexpr (F16) {
            const int row = lane & 15, slot = ((4 * kk + (lane >> 4)) ^ (row & 7) ^ (row >> 3)) * 16;
            f.a[0] = *reinterpret_cast<const u32x4_t*>(sA + (size_t)(buf * BN + wn * WN + row) * LDS_ROW + slot);
            f.b[0] = *reinterpret_cast<const u32x4_t*>(sB + (size_t)(buf * BM + wm * WM + row) * LDS_ROW + slot);
            return;
        }
        const int koff = DIRECT ? ((2 * kk + (lane >> 5)) ^ frag_swz) * 16 : kk * 32 + frag_off;
#pragma unroll
        for (int i = 0; i < TN; ++i)
            f.a[i] = *reinterpret_cast<const u32x4_t*>(sA + (size_t)(buf * BN + wn * WN + i * 32 + frag_row) * LDS_ROW + koff);
#pragma unroll
        for (int j = 0; j < TM; ++j)
            f.b[j] = *reinterpret_cast<const u32x4_t*>(sB + (size_t)(buf * BM + wm * WM + j * 32 + frag_row) * LDS_ROW + koff);
    };
    auto mma_frags = [&](const Frags& f) {
        if constexpr (F16) {
            acc4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, f.a[0]), __builtin_bit_cast(bf16x8_t, f.b[0]), acc4, 0, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j) mma_step<T>(acc[i][j], f.a[i], f.b[j]);
        }
    };
    auto compute = [&](int buf) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            Frags f;
            read_frags(buf, kk, f);
            mma_frags(f);
        }
    };

    // Software pipeline of the staged path: while tile kt is multiplied out of LDS buffer kt & 1, the loads of tile kt + 1 are in
    // flight into registers; they are written to the other buffer at the end of the step.  (A second register stage costs the
    // second resident block per CU and is slower.)
    if constexpr (RING) {
        // Ring of STAGES operand tiles, STAGES - 1 of them requested ahead: a call with few pixels has no more than one or
        // two blocks per CU, so the time of a K step is the latency of its operands (0.65 us from L2 with one tile in
        // flight) unless several tiles are in flight.  The order of the sums is the two-buffer loop's: same values bit for bit.
        // PROD wavefronts do nothing but request tiles: issued by the multiplying wavefronts the requests stand in line with
        // their fragment reads and products (300 x 1024, K 12544, before groups and with the reads in front of the products: 128 us
        // with two buffers, 60 with the ring, 39 / 32 with two / four loading wavefronts; the ring's depth beyond 4 changes nothing).
        // U tiles (a group) are handed over per barrier: a step is one barrier, one round trip of the fragment reads and the products
        // of a group, of which only the products grow with U.  U 1 / U, K 12544 to 1024 channels: 32 x 32, U 4, 100 rows 33.0 / 19.1 us;
        // 32 x 64, U 3, 300 rows 35.4 / 27.7; 64 x 64, U 2, 900 rows 46.2 / 40.1; 64 x 128, U 2, 1500 rows 62.0 / 54.7; fp32 32 x 32, U 2, 200 rows
        // 102.4 / 95.0; fp32 64 x 64, U 2, 600 rows 237 / 217.  Larger groups need larger rings: where two blocks share a CU U is 1.
        // A layer of one or two groups gains nothing: up to K 320 (fp32: 128) it takes 0.1 to 0.2 us longer than with the shorter
        // loop before (256 -> 75, 3 136 pixels 4.6 / 4.4; fp32 64 -> 64, 2 352 pixels 3.6 / 3.4).
        // Step g: the fragments of group g are in registers; group g + 1 is waited for (the newest STAGES / U - 2 groups may
        // still be on their way; loads complete in order), and past the barrier every wavefront has group g in registers,
        // so its buffers take group g + STAGES / U while the fragments of g + 1 are read under the products of g.
        constexpr int GROUPS = STAGES / U;                      // groups the ring holds
        constexpr int PER_TILE = PA + PB;                       // requests of one thread per tile
        constexpr int LEFT = (GROUPS - 2) * U * PER_TILE;       // requests that may be outstanding when the next group is needed
        static_assert(LEFT < 64, "vmcnt counts to 63");
        constexpr int WAIT_LEFT = 0x0070 | (LEFT & 15) | ((LEFT >> 4) << 14);   // vmcnt(LEFT) lgkmcnt(0)
        const int KG = (KT + U - 1) / U;                        // groups of the layer; the last one may lack tiles
        int q_kt = 0, q_c = 0, q_kx = 0, q_tap = 0;
        long long q_off = 0;                                    // element offset of (tap, first channel) from the pixel's tap 0
        const int kt1 = DUAL ? a.Cin / BK : 0;
        auto request = [&](int buf) {                           // next tile in K order into buffer buf
            unsigned char* dA = sA + (size_t)(buf * BN + (wv * 64) / CPR) * LDS_ROW;
            unsigned char* dB = sB + (size_t)(buf * BM + (wv * 64) / CPR) * LDS_ROW;
#pragma unroll
            for (int p = 0; p < PB; ++p) {
                const T* src;
                if constexpr (ONE) {
                    src = (!DUAL || q_kt < kt1) ? in + b_base[p] + (size_t)q_kt * BK : in2 + b_base2[DUAL ? p : 0] + (size_t)(q_kt - kt1) * BK;
                } else {
                    const bool ok = (b_taps[ONE ? 0 : p] >> q_tap) & 1u;
                    src = ok ? in + (b_off0[ONE ? 0 : p] + q_off) : reinterpret_cast<const T*>(g_zero_page);
                }
                load_to_lds16(src, dB + (size_t)(RPP * p) * LDS_ROW);
            }
            if (q_kt > 0) {
#pragma unroll
                for (int p = 0; p < PA; ++p) load_to_lds16(wgt + a_base[p] + (size_t)q_kt * BK, dA + (size_t)(RPP * p) * LDS_ROW);
            }
            ++q_kt;
            if constexpr (!ONE) {
                q_off += BK;
                if (++q_c == cin_tiles) {                       // next tap: along the filter row, then to the next input row
                    q_c = 0;
                    ++q_tap;
                    if (++q_kx == a.kw) { q_kx = 0; q_off += (long long)(a.W - a.kw) * a.Cin; }
                }
            }
        };
        auto barrier = [&]() {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };
        auto landed = [&](bool steady) {                        // what this thread requested of the next tile has arrived
            asm volatile("" ::: "memory");
            if (steady) __builtin_amdgcn_s_waitcnt(WAIT_LEFT);
            else __builtin_amdgcn_s_waitcnt(0x0070);            // the last tiles: vmcnt(0) lgkmcnt(0)
        };
        auto request_group = [&](int buf) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (q_kt < KT) request(buf * U + u);
        };
        if (loads) {
#pragma unroll
            for (int s = 0; s < GROUPS - 1; ++s) request_group(s);
            landed(KT >= (GROUPS - 1) * U);
            barrier();
            request_group(GROUPS - 1);
            int buf = 0;
            for (int g = 0; g + 1 < KG; ++g) {
                landed((g + GROUPS) * U <= KT);
                barrier();
                request_group(buf);
                buf = buf + 1 == GROUPS ? 0 : buf + 1;
            }
            barrier();                                          // the one in front of the epilogue
            return;
        }
        auto in_registers = [&]() {                             // the fragments read last are in registers
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0xc07f);                 // lgkmcnt(0)
        };
        int buf = 0;                                            // buffer of the group read last
        if constexpr (F16 && F32) {
            // The matrix instruction wants one k of four from each lane group: 0, 4, 1, 5 of a group of 8, then 2, 6, 3, 7 (the order of
            // the 32x32 tiles).  Lanes read 16 bytes instead, lanes 0..31 of k group 2 p and lanes 32..63 of 2 p + 1, and swap
            // halves in registers (4-byte reads conflict in the banks: 124 us against 115 at 200 x 1024, K 12544).  A product is 32
            // cycles and waits for the one before; everything else stands between the products of group g, one thing behind
            // each: the swaps of group g + 1 and the reads of group g + 2, in three sets of registers.  200 x 1024, K 12544: swaps in front
            // of the products 115 us, between them 103, the reads as well 96 (the products alone are 44).
            struct Raw { uint32_t a[U][KK / 2][4], b[U][KK / 2][4]; } r0, r1, r2;
            auto read_one = [&](int group, Raw& r, int u, int p, bool weights) {
                const int row = lane & 15, koff = ((2 * (2 * p + (lane >> 5)) + ((lane >> 4) & 1)) ^ (row & 7) ^ (row >> 3)) * 16;
                const unsigned char* at = weights ? sA + (size_t)((group * U + u) * BN + wn * WN + row) * LDS_ROW : sB + (size_t)((group * U + u) * BM + wm * WM + row) * LDS_ROW;
                const u32x4_t v = *reinterpret_cast<const u32x4_t*>(at + koff);
                uint32_t* to = weights ? r.a[u][p] : r.b[u][p];
#pragma unroll
                for (int e = 0; e < 4; ++e) to[e] = v[e];
            };
            auto read_group = [&](int group, Raw& r) {
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int p = 0; p < KK / 2; ++p) { read_one(group, r, u, p, true); read_one(group, r, u, p, false); }
            };
            // x: lanes 0..31 of x and of y, y: lanes 32..63 of x and of y
            auto swap = [&](uint32_t& x, uint32_t& y) {
#if defined(__HIP_DEVICE_COMPILE__)
                const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
                x = r[0];
                y = r[1];
#endif
            };
            auto deal = [&](Raw& r, int u, int p, int part) {   // one of the four swaps of k groups 2 p, 2 p + 1
                if (part == 0) swap(r.a[u][p][0], r.a[u][p][1]);
                if (part == 1) swap(r.b[u][p][0], r.b[u][p][1]);
                if (part == 2) swap(r.a[u][p][2], r.a[u][p][3]);
                if (part == 3) swap(r.b[u][p][2], r.b[u][p][3]);
            };
            in_registers();
            barrier();                                          // group 0 has landed
            start_sums();
            // (the bias is waited for here: left to the first product, the compiler puts that wait into every step of the loop)
            asm volatile("" : "+v"(acc4));
            read_group(0, r0);
            in_registers();
            if (KG > 1) { barrier(); buf = 1; read_group(1, r1); }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int p = 0; p < KK / 2; ++p)
#pragma unroll
                    for (int part = 0; part < 4; ++part) deal(r0, u, p, part);
            auto step = [&](int g, Raw& now, Raw& next, Raw& read) {
                in_registers();
                if (g + 2 < KG) barrier();
                buf = buf + 1 == GROUPS ? 0 : buf + 1;          // (past the last group the ring's old contents are read and not used)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (u > 0 && g * U + u >= KT) break;        // (only the last group lacks tiles: nothing to deal either)
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int p = 0; p < KK / 2; ++p)
#pragma unroll
                        for (int part = 0; part < 4; ++part) {
                            constexpr int at[4] = {0, 2, 1, 3};   // k group 2 p: words 0 and 2; 2 p + 1: 1 and 3
                            acc4 = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(now.a[u][p][at[part]]), __uint_as_float(now.b[u][p][at[part]]), acc4, 0, 0, 0);
                            deal(next, u, p, part);
                            if (part % 2 == 0) read_one(buf, read, u, p, part == 0);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                }
            };
            for (int g = 0; g < KG; g += 3) {
                step(g, r0, r1, r2);
                if (g + 1 < KG) step(g + 1, r1, r2, r0);
                if (g + 2 < KG) step(g + 2, r2, r0, r1);
            }
        } else {
            struct TileFrags { Frags k[U][KK]; };
            TileFrags g0, g1;
            in_registers();
            barrier();                                          // group 0 has landed
            start_sums();
            if constexpr (F16) {                                // (as above)
                asm volatile("" : "+v"(acc4));
            } else {
#pragma unroll
                for (int i = 0; i < TN; ++i)
#pragma unroll
                    for (int j = 0; j < TM; ++j) asm volatile("" : "+v"(acc[i][j]));
            }
#pragma unroll
            for (int i = 0; i < U * KK; ++i) read_frags(i / KK, i % KK, g0.k[i / KK][i % KK]);
            auto step = [&](int g, const TileFrags& now, TileFrags& next) {
                // The next group's fragments are read between the products, two k-steps behind each of the first half: in front of all
                // products they queue at the LDS (300 x 1024, K 12544 31.2 / 27.8 us, 1500 x 1024 59 / 55, 3x3 256 -> 256 at 4 715 pixels 14.9 / 14.0).
                in_registers();
                if (g + 1 < KG) barrier();
                buf = buf + 1 == GROUPS ? 0 : buf + 1;          // (past the last group the ring's old contents are read and not used)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (u > 0 && g * U + u >= KT) break;        // (only the last group lacks tiles)
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk) {
                        __builtin_amdgcn_sched_barrier(0);
                        mma_frags(now.k[u][kk]);
#pragma unroll
                        for (int i = 2 * (u * KK + kk); i < 2 * (u * KK + kk) + 2; ++i)
                            if (i < U * KK) read_frags(buf * U + i / KK, i % KK, next.k[i / KK][i % KK]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            for (int g = 0; g < KG; g += 2) {
                step(g, g0, g1);
                if (g + 1 < KG) step(g + 1, g1, g0);
            }
        }
        // (a wavefront's epilogue region lies in other wavefronts' operand tiles)
        in_registers();
        barrier();
        if constexpr (F16) {
            const int pix = m0 + wm * WM + (lane & 15), ch = n0 + wn * WN + 4 * (lane >> 4);
            if (pix >= M) return;
            OutT* o0 = static_cast<OutT*>(a.out0);
            OutT* o1 = static_cast<OutT*>(a.out1);
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool in_range = ch + e < a.Cout;
                v[e] = acc4[e];
                if (quads) v[e] += load_elem(&rquad.v[e]);
                else if (res != nullptr && in_range) v[e] += load_elem(res + (size_t)pix * a.Cout + ch + e);
                if (a.relu) v[e] = fmaxf(v[e], 0.f);
            }
            if (o1 == nullptr && (a.Cout & 3) == 0 && (a.ld0 & 3) == 0) {
                if (ch < a.Cout) store4(o0 + (size_t)pix * a.ld0 + ch, v);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int c = ch + e;
                    if (c < a.n_split) { if (c < a.Cout) store_elem(o0 + (size_t)pix * a.ld0 + c, v[e]); }
                    else if (c < a.Cout) store_elem(o1 + (size_t)pix * a.ld1 + (c - a.n_split), v[e]);
                }
            }
            return;
        }
    } else if constexpr (DIRECT) {
        // Two LDS buffers: tile kt + 1 is requested as soon as every wavefront has finished reading its buffer (the
        // barrier that ends step kt - 1) and has the whole of step kt to arrive.
        // The fragments of k-step kk + 1 are read while k-step kk is multiplied, and the barrier sits in front of a
        // tile's LAST k-step: by then every wavefront has read the whole tile (so its buffer can be refilled) and still
        // has a k-step of matrix work queued, which covers the first fragment reads of the next tile.
        static_assert(KK % 2 == 0, "the fragment double buffer alternates per k-step");
        issue_tiles(0, 0);
        load_bias();
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
        __syncthreads();
        start_sums();
        if (KT > 1) issue_tiles(1, 1);
        Frags f0, f1;
        read_frags(0, 0, f0);
        for (int kt = 0; kt < KT; ++kt) {
            const int buf = kt & 1;
            static_for<0, KK - 1>([&](auto kc) {
                constexpr int kk = decltype(kc)::value;
                read_frags(buf, kk + 1, (kk & 1) ? f0 : f1);
                mma_frags((kk & 1) ? f1 : f0);
            });
            __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this thread's part of tile kt + 1 is in LDS
            __syncthreads();
            if (kt + 2 < KT) issue_tiles(kt + 2, buf);
            if (kt + 1 < KT) read_frags(buf ^ 1, 0, f0);
            mma_frags(f1);
        }
    } else {
    load_tiles(0, st0);
    load_bias();
    store_tiles(0, st0);
    if (KT > 1) load_tiles(1, st0);
    start_sums();
    __syncthreads();
    // The requests for tile kt + 2 go out right after the LDS write of tile kt + 1 has freed the staging
    // registers, so the data has a whole step to arrive.
    for (int kt = 0; kt < KT; ++kt) {
        const int buf = kt & 1;
        // the wavefront that multiplies wins issue arbitration over the SIMD's other wavefront, which is staging
        // (LDS writes, global loads) at that moment: measured 0.5-1 % on the whole sweep
        __builtin_amdgcn_s_setprio(3);
        compute(buf);
        __builtin_amdgcn_s_setprio(0);
        if (kt + 1 < KT) store_tiles(buf ^ 1, st0);
        if (kt + 2 < KT) load_tiles(kt + 2, st0);
        __syncthreads();
    }
    }

    // ---- epilogue.  Accumulator element e of lane l: channel 8*(e/4) + 4*(l/32) + e%4, pixel l%32.
    OutT* __restrict__ out0 = static_cast<OutT*>(a.out0);
    OutT* __restrict__ out1 = static_cast<OutT*>(a.out1);
    if (vec) {
        // Coalesced path, one 32-pixel sub-tile at a time: the wavefront parks its 32 pixel x WN channel
        // fp32 tile in its own LDS region (the pipeline buffers are free now) and re-reads it so
        // that each lane owns 8 consecutive channels of one pixel: residual loads and output stores are
        // 16-byte and the lanes of one instruction cover whole lines of the NHWC tensors.
        unsigned char* ep = smem + (size_t)wv * (32 * EPITCH);
        if constexpr (std::is_same<OutT, bf16_t>::value && std::is_same<T, bf16_t>::value) {
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
                        const int pxl = it * PPI + lane / LPP, chunk = lane % LPP;
                        const int pix = m0 + wm * WM + j * 32 + pxl, ch = n0 + wn * WN + chunk * 8;
                        const u32x4_t q = *reinterpret_cast<const u32x4_t*>(ep + (size_t)pxl * EPB + chunk * 16);
                        if (pix < M && ch < a.Cout) *reinterpret_cast<u32x4_t*>(out0 + (size_t)pix * a.ld0 + ch) = q;
                    }
                    __builtin_amdgcn_s_waitcnt(0xc07f);
                    __builtin_amdgcn_wave_barrier();
                });
                return;
            }
        }
        static_for<0, TM>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
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
                const int pxl = it * PPI + lane / LPP, chunk = lane % LPP;
                const int pix = m0 + wm * WM + j * 32 + pxl, ch = n0 + wn * WN + chunk * 8;
                if (pix >= M || ch >= a.Cout) continue;
                const f32x4_t lo = *reinterpret_cast<const f32x4_t*>(ep + (size_t)pxl * EPITCH + chunk * 32);
                const f32x4_t hi = *reinterpret_cast<const f32x4_t*>(ep + (size_t)pxl * EPITCH + chunk * 32 + 16);
                float r[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                if (res) {
                    float q[8];
                    unpack8(rres[j * NIT + it], q);
#pragma unroll
                    for (int e = 0; e < 8; ++e) r[e] += q[e];
                }
                if (a.relu) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) r[e] = fmaxf(r[e], 0.f);
                }
                store8(out0 + (size_t)pix * a.ld0 + ch, r);
            }
            __builtin_amdgcn_s_waitcnt(0xc07f);
            __builtin_amdgcn_wave_barrier();
        });
        return;
    }
    // General path (split outputs, channel counts that are not multiples of 8): the same LDS round trip,
    // then one element per lane with consecutive lanes on consecutive channels of a pixel, so that stores
    // stay contiguous within each output row.
    {
        unsigned char* ep = smem + (size_t)wv * (32 * EPITCH);
        static_for<0, TM>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int chl = i * 32 + 8 * v + 4 * (lane >> 5);
                    f32x4_t r = {acc[i][j][4 * v], acc[i][j][4 * v + 1], acc[i][j][4 * v + 2], acc[i][j][4 * v + 3]};
                    *reinterpret_cast<f32x4_t*>(ep + (size_t)frag_row * EPITCH + chl * 4) = r;
                }
            __builtin_amdgcn_s_waitcnt(0xc07f);
            __builtin_amdgcn_wave_barrier();
            for (int e = lane; e < 32 * WN; e += 64) {
                const int pxl = e / WN, cl = e - pxl * WN;
                const int pix = m0 + wm * WM + j * 32 + pxl, c = n0 + wn * WN + cl;
                if (pix >= M || c >= a.Cout) continue;
                float val = *reinterpret_cast<const float*>(ep + (size_t)pxl * EPITCH + cl * 4);
                if (res) val += load_elem(res + (size_t)pix * a.Cout + c);
                if (a.relu) val = fmaxf(val, 0.f);
                if (c < a.n_split) store_elem(out0 + (size_t)pix * a.ld0 + c, val);
                else store_elem(out1 + (size_t)pix * a.ld1 + (c - a.n_split), val);
            }
            __builtin_amdgcn_s_waitcnt(0xc07f);
            __builtin_amdgcn_wave_barrier();
        });
    }
}

// Whether a layer gets the 256 x 256 bf16 tile of conv_large.h for the sake of the predictors that it alone can fuse.  The 200
// tiles are from the loop that this tile had before; with the present one a launch pays from fewer on, and the line has not been
// moved yet (3x3 256 -> 256 with predictors, one launch / two in us: 96 tiles 43.0 / 39.0, 128 tiles 44.8 / 46.3, 160 tiles 50.9 / 61.2).
static bool takes_large_tile(const ConvArgs& a) {
    const long long M = (long long)a.N * a.Ho * a.Wo;
    const long long K = (long long)a.kh * a.kw * a.Cin;
    return K >= 512 && ((M + 255) / 256) * (a.Cout / 256) >= 200 && conv_large_supported(a, 1, 256, 256);
}

bool conv_heads_supported(const ConvArgs& a, int precision) {
    if (precision != 1 || a.head_w == nullptr || a.head_b == nullptr || a.head_logits == nullptr || a.head_deltas == nullptr) return false;
    if (a.Cout != 256 || a.in2 != nullptr || a.res != nullptr || !a.relu || a.head_a < 1 || 5 * a.head_a > 96) return false;
    if (a.kh == 1 && a.kw == 1 && a.pad == 0) return false;   // only the general-filter instantiation carries the predictor path
    return conv_supported(a, precision) && takes_large_tile(a);
}

bool conv_supported(const ConvArgs& a, int precision) {
    const int bk = precision ? 64 : 32;
    if (a.Cin <= 0 || a.Cin % bk) return false;
    if (a.kh < 1 || a.kw < 1 || a.kh * a.kw > 32) return false;   // one validity bit per filter tap
    if (a.N <= 0 || a.Cout <= 0 || a.Ho <= 0 || a.Wo <= 0) return false;
    if (a.in2 != nullptr) {
        if (a.kh != 1 || a.kw != 1 || a.pad != 0 || a.Cin2 <= 0 || a.Cin2 % bk || a.stride2 < 1) return false;
        if ((a.Ho - 1) * a.stride2 >= a.H2 || (a.Wo - 1) * a.stride2 >= a.W2) return false;
    }
    if ((long long)a.N * a.Ho * a.Wo >= (1ll << 31)) return false;
    if ((long long)a.N * a.H * a.W * a.Cin >= (1ll << 40)) return false;
    return true;
}

template <typename T, int BM, int BN, int BKB, int WAVES_M, int WAVES_N, int MODE, typename OutT, int STAGES = 2, int PROD = 0, int U = 1>
static hipError_t launch_cfg(const ConvArgs& args, hipStream_t s) {
    ConvArgs a = args;
    const int tiles_m = (int)(((long long)a.N * a.Ho * a.Wo + BM - 1) / BM), tiles_n = (a.Cout + BN - 1) / BN;
    a.by_hw = FastDiv(a.Ho * a.Wo);
    a.by_w = FastDiv(a.Wo);
    a.by_tiles = FastDiv(PROD > 0 && (long long)a.N * a.Ho * a.Wo < a.Cout ? tiles_m : tiles_n);
    const size_t lds = (size_t)STAGES * (BN + BM) * (BKB == 128 ? BKB : BKB + 16);
    auto kern = conv_igemm_kernel<T, BM, BN, BKB, WAVES_M, WAVES_N, MODE, OutT, STAGES, PROD, U>;
    {
        hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
        if (e != hipSuccess) return e;
    }
    const long long M = (long long)a.N * a.Ho * a.Wo;
    const long long tiles = ((M + BM - 1) / BM) * ((a.Cout + BN - 1) / BN);
    if (tiles <= 0 || tiles >= (1ll << 30)) return hipErrorInvalidValue;
    const long long grid = ((tiles + 7) / 8) * 8;  // 8 XCDs x equal ranges; surplus workgroups exit at once
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * (WAVES_M * WAVES_N + PROD)), lds, s, a);
    return hipGetLastError();
}

// 1x1 unpadded convolutions (and the FC layers) get the variant without filter-tap bookkeeping.
template <typename T, int BM, int BN, int BKB, int WAVES_M, int WAVES_N, typename OutT, bool ALLOW_DUAL = false, int STAGES = 2, int PROD = 0, int U = 1>
static hipError_t launch_one(const ConvArgs& a, hipStream_t s) {
    if (a.in2 != nullptr) {
        if constexpr (ALLOW_DUAL) return launch_cfg<T, BM, BN, BKB, WAVES_M, WAVES_N, 2, OutT, STAGES, PROD, U>(a, s);
        else return hipErrorInvalidValue;
    }
    if (a.kh == 1 && a.kw == 1 && a.pad == 0) return launch_cfg<T, BM, BN, BKB, WAVES_M, WAVES_N, 1, OutT, STAGES, PROD, U>(a, s);
    return launch_cfg<T, BM, BN, BKB, WAVES_M, WAVES_N, 0, OutT, STAGES, PROD, U>(a, s);
}

bool conv_tail_supported(const ConvArgs& a, int precision) {
    if (!conv_large_supported(a, precision, 256, 256)) return false;
    if (!a.tail_w || !a.tail_b || !a.tail_res || !a.tail_out || a.tail_res == a.tail_out) return false;
    if (a.tail_n < 512 || a.tail_n % 512 || a.tail_n > 4096) return false;
    if (a.Cout != 256 || !a.relu || a.res != nullptr || a.out1 != nullptr || a.in2 != nullptr || a.head_w != nullptr) return false;
    const long long M = (long long)a.N * a.Ho * a.Wo;
    return M * a.tail_n < (1ll << 31);
}

// Tiles of bm x bn, in rounds of one block per CU.
static long long tile_rounds(const ConvArgs& a, int bm, int bn) {
    const long long M = (long long)a.N * a.Ho * a.Wo;
    return (((M + bm - 1) / bm) * ((a.Cout + bn - 1) / bn) + 255) / 256;
}

// Calls with few pixels.  A 128 x 128 tile of two operand tiles takes 0.64 us per K step (64 bf16 / 32 fp32 of every row) however few
// blocks there are, because a block waits for the one tile it has in flight; the ring tiles take, per K step and round of 256
// blocks: 32 x 64 0.16 us, 64 x 64 0.24, 64 x 128 0.31, 128 x 128 0.49 (measured at K 12544; 0.13, 0.20, 0.28, 0.49 since reads
// stand between the products, which gives the same order from K 1024 on).  The rule takes the cheapest by the first count.
// Measured in us, two-buffer tile / ring tile: K 12544 to 1024 channels: 300 rows 127 / 28 (32 x 64), 1 020 128 / 42 (64 x 64), 1 500
// 125 / 56 (64 x 128), 3 000 124 / 92 (128 x 128); 3x3 256 -> 256: 2 040 pixels 24 / 9.3, 8 160 25 / 15.6; 3x3 512 -> 512: 510
// pixels 44 / 12.5, 4 080 54 / 26, 8 160 56 / 47.5.  From K 768 on what a layer takes without the ring is one of the large tiles; the
// rule does not ask for their time, which is no less in all but the last sizes of the range (best large tile / ring tile: 300 rows
// 85 / 28, 1 500 86 / 56, 3 000 91 / 92; 3x3 256 -> 256: 8 160 pixels 25 / 15.6, 12 240 25 / 22.4, 16 320 26 / 24.2; 3x3 512 -> 512: 4 080
// pixels 44 / 26, 8 160 49.8 / 47.5; 1024 -> 256: 8 160 pixels 11.2 / 8.1, 16 320 13.3 / 15.1).  Below K 512 more than 256 tiles
// of 128 x 128 run two blocks per CU and overlap each other: no ring tile is faster there.  The count holds for long K; for
// short K a launch is set-up and epilogue, of which one large block per CU hides nothing.  So 64 x 128 runs from K 512 and in
// one round only (256 channels, 8 160 pixels, two-buffer tile / ring tile: K 512 7.5 / 6.1, K 768 9.3 / 7.4), and 128 x 128 from K 768,
// where the two are even (9 000 pixels: K 768 9.4 / 9.7, K 1024 11.0 / 11.3; 12 240 pixels, K 2304 25.6 / 22.4).  64 x 64 pays from K 256 in up to two rounds
// (8 160 pixels, 256 channels, K 256 7.0 / 6.4, K 448 9.3 / 7.7).  Below K 256 the detectors have K 64 and 128 only, the streaming
// tile's; at K 192 the small tiles would pay too (2 040 pixels, 256 channels 5.4 / 4.0).  Up to 256 tiles of 32 x 32 (four
// wavefronts of one 16x16 tile, K tiles of 8 KB) that tile is the one that uses most CUs, 32 x 64 / 32 x 32: 510 pixels, 3x3 512 -> 512 14.9 /
// 12.7, 2048 -> 256 6.6 / 5.7, 100 rows x 1024, K 12544 26.8 / 19.1, 500 x 512, K 384 3.7 / 3.9.  Returns false if no ring tile pays.
static bool launch_ring_bf16(const ConvArgs& a, long long K, hipStream_t s, hipError_t* e) {
    if (K < 256 || a.out1 != nullptr) return false;
    const bool narrow = a.Cout <= 64;
    if (narrow ? tile_rounds(a, 64, 64) > 1 : tile_rounds(a, 128, 128) > 1) return false;
    if (tile_rounds(a, 32, 32) == 1) {
        *e = launch_one<bf16_t, 32, 32, 128, 2, 2, bf16_t, true, 16, 4, 4>(a, s);
        return true;
    }
    const long long c32 = 16 * tile_rounds(a, 32, 64), c64 = 24 * tile_rounds(a, 64, 64);
    const long long c64w = K >= 512 && !narrow && tile_rounds(a, 64, 128) == 1 ? 31 : 1000, c128 = K >= 768 && !narrow ? 49 : 1000;
    const long long best = c32 < c64 ? c32 : c64, wide = c64w < c128 ? c64w : c128;
    if ((best < wide ? best : wide) >= 64) return false;
    if (best <= wide)
        *e = c32 < c64                     ? launch_one<bf16_t, 32, 64, 128, 1, 2, bf16_t, true, 9, 4, 3>(a, s)
             : tile_rounds(a, 64, 64) == 1 ? launch_one<bf16_t, 64, 64, 128, 2, 2, bf16_t, true, 6, 4, 2>(a, s)
                                           : launch_one<bf16_t, 64, 64, 128, 2, 2, bf16_t, true, 5, 4>(a, s);
    else
        *e = c64w <= c128 ? launch_one<bf16_t, 64, 128, 128, 2, 2, bf16_t, true, 6, 4, 2>(a, s) : launch_one<bf16_t, 128, 128, 128, 2, 2, bf16_t, true, 4, 4>(a, s);
    return true;
}

// fp32.  Per K step and round of 256 blocks: 128 x 128 2.1 us and 64 x 64 ring 0.6, both bound by the fp32 matrix instructions
// (1024 cycles per K step of a 64 x 64 tile), so that what counts is how many SIMDs share the work; 32 x 32 ring (16x16 matrix
// tiles, four wavefronts) 0.24 in one round, half of it matrix instructions, and 0.23 to 0.28 in several.  The rule counts 0.28 for it.  Measured
// in us, 128 x 128 / 64 x 64 / 32 x 32: 200 x 1024, K 12544: 820 / 234 / 96; 600 x 1024: 833 / 250 / 304; 3x3 256 -> 256,
// 1 020 pixels 164 / 50 / 22, 2 040 165 / 52 / 34, 4 080 168 / 56 / 77, 16 320 186 / 180 / 266; 1x1 64 -> 64, 8 160 pixels 64 x 64
// 5.9, 32 x 32 5.1, 9 000 pixels 5.9 / 6.8.
// Up to 64 channels the two-buffer tile is 128 x 64: 1.5 us with one block per CU, 1.06 a round where two share it, so that
// the ring pays while its last round is not full (64 x 64 ring / 128 x 64: 3x3 64 -> 64, 32 400 pixels 31.2 / 33.8, 66 000 64.6 / 69.9,
// 64 800 54.8 / 52.6, 259 200 188 / 176), with few K steps in up to two rounds (1x1 64 -> 64: 32 400 pixels 8.7 / 9.4, 33 000
// 11.3 / 10.8, 259 200 43.0 / 36.2).
static hipError_t launch_fp32(const ConvArgs& a, long long K, hipStream_t s) {
    const bool narrow = a.Cout <= 64;
    const long long r64 = tile_rounds(a, 64, 64), rw = tile_rounds(a, 128, 64);
    const long long c32 = 28 * tile_rounds(a, 32, 32), c64 = 57 * r64;
    const long long base = narrow ? (rw == 1 ? 150 : 106 * rw) : 207 * tile_rounds(a, 128, 128);
    if (c32 < c64 && c32 < base) return launch_one<float, 32, 32, 128, 2, 2, float, true, 8, 4, 2>(a, s);
    if (c64 < base && !(narrow && K < 256 && r64 > 2))
        return r64 == 1 ? launch_one<float, 64, 64, 128, 2, 2, float, true, 6, 4, 2>(a, s) : launch_one<float, 64, 64, 128, 2, 2, float, true, 5, 4>(a, s);
    return narrow ? launch_one<float, 128, 64, 128, 2, 2, float>(a, s) : launch_one<float, 128, 128, 128, 2, 2, float, true>(a, s);
}

// fp32 outputs of bf16 tensors (the predictors, at most a few channel tiles wide): the general epilogue's time goes with the
// tile.  Measured, 128-pixel tile / ring: 75 channels, K 256: 300 pixels 17.3 / 5.7 us (32 x 64), 510 pixels 32 x 64 / 32 x 32 4.5 / 3.6, 16 320 17.5 / 8.2 and
// 32 640 18.3 / 14.2 (64 x 64); 55 channels, K 1024, 4 800 rows: 15.5 / 7.5.  Up to 64 channels the 128-pixel tile is no wider
// than the ring's: 60 channels, K 256, 48 000 pixels 14.5 / 14.2, 64 800 15.7 / 17.5.
static hipError_t launch_out_f32(const ConvArgs& a, hipStream_t s) {
    if (tile_rounds(a, 32, 32) <= 1) return launch_one<bf16_t, 32, 32, 128, 2, 2, float, false, 16, 4, 4>(a, s);
    if (tile_rounds(a, 32, 64) <= 1) return launch_one<bf16_t, 32, 64, 128, 1, 2, float, false, 9, 4, 3>(a, s);
    if (tile_rounds(a, 64, 64) <= (a.Cout <= 64 ? 3 : 4)) return launch_one<bf16_t, 64, 64, 128, 2, 2, float, false, 5, 4>(a, s);
    return a.Cout <= 64 ? launch_one<bf16_t, 128, 64, 128, 2, 2, float>(a, s) : launch_one<bf16_t, 128, 128, 128, 2, 2, float>(a, s);
}

// Layers with more pixels.  A round of 256 blocks of a large tile takes, in 1/100 us, step for every K tile and fixed for what does
// not grow with K (set-up, first operands, epilogue, stores); a last round that is not full costs less, its blocks having the
// caches and the power budget of the others.  The tile with the least sum is taken, the larger one if they are equal.  Measured
// in us, 256 x 256 / 192 x 256 / 256 x 128 / 192 x 128 / 128 x 128 (two buffers, two blocks per CU): K 12544 to 1024
// channels: 9 600 rows 228 / 199 / 254 / 268 / 274, 4 800 198 / 168 / 124 / 118 / 175; K 1024, 9 600 rows 27 / 23 / 29 / 25 / 30; 3x3
// 512 -> 512: 16 320 pixels 90 / 81 / 72 / 105 / 94, 12 544 80 / 69 / 62 / 98 / 85, 50 176 192 / 234 / 243 / 261 / 247; 3x3 256 -> 256:
// 32 640 49 / 44 / 38 / 58 / 49, 130 560 123 / 141 / 146 / 185 / 147; 3x3 128 -> 128, 802 816: - / - / 273 / 306 / 307.  Below K 512 a launch is
// mostly epilogue (256 -> 1024 channels with a residual, 32 640 pixels: 40 / 41 / 44 / 46 / 38), which the two resident blocks of
// 128 x 128 overlap with each other's K loop, except with a second source, where 200 tiles pay from K 384 on.  Up to K 704 the
// 128 x 128 tile's smaller set-up and epilogue also win where one round of it holds the layer (512 -> 256, 11 468 pixels 7.5 against 7.8
// on 192 x 128; 512 -> 2048 with a residual, 2 007 pixels 8.5 / 9.5; 3x3 64 -> 128, 27 840 pixels 9.6 / 10.2; K 704 to 512 channels, 5 734
// pixels 8.8 / 9.0), from K 768 on no longer (10.2 / 9.7); in two rounds it does not (3x3 64 -> 128, 36 000 pixels 13.6 / 10.5).
static bool launch_large_bf16(const ConvArgs& a, long long K, hipStream_t s, hipError_t* e) {
    const struct { int bm, bn, step, fixed; } tiles[4] = {{256, 256, 138, 900}, {192, 256, 106, 800}, {256, 128, 84, 700}, {192, 128, 64, 600}};
    const long long M = (long long)a.N * a.Ho * a.Wo, KT = K / 64;
    if (K < 512) {
        if (a.in2 == nullptr || K < 384 || ((M + 255) / 256) * (a.Cout / 256) < 200 || !conv_large_supported(a, 1, 256, 256)) return false;
        *e = launch_conv_large(a, 256, 256, s);
        return true;
    }
    if (K < 768 && tile_rounds(a, 128, 128) <= 1) return false;
    long long best = 0;
    int pick = -1;
    for (int i = 0; i < 4; ++i) {
        if (!conv_large_supported(a, 1, tiles[i].bm, tiles[i].bn)) continue;
        const long long n = ((M + tiles[i].bm - 1) / tiles[i].bm) * (a.Cout / tiles[i].bn), last = n % 256;
        const long long rounds = 100 * (n / 256) + (last ? 60 + 40 * last / 256 : 0);   // in 1/100
        const long long cost = rounds * (KT * tiles[i].step + tiles[i].fixed);
        if (pick < 0 || cost < best) { best = cost; pick = i; }
    }
    if (pick < 0) return false;
    *e = launch_conv_large(a, tiles[pick].bm, tiles[pick].bn, s);
    return true;
}

hipError_t launch_conv(const ConvArgs& a, int precision, bool out_f32, hipStream_t s) {
    if (!conv_supported(a, precision)) return hipErrorInvalidValue;
    if (a.tail_w != nullptr) {   // expansion tail: one kernel variant only
        if (out_f32 || !conv_tail_supported(a, precision)) return hipErrorInvalidValue;
        return launch_conv_large(a, 256, 256, s);
    }
    if (a.head_w != nullptr) {   // fused predictors exist in one kernel variant only
        if (out_f32 || !conv_heads_supported(a, precision)) return hipErrorInvalidValue;
        return launch_conv_large(a, 256, 256, s);
    }
    const bool narrow = a.Cout <= 64;
    if (precision == 0) return launch_fp32(a, (long long)a.kh * a.kw * a.Cin + (a.in2 ? a.Cin2 : 0), s);
    if (out_f32) return launch_out_f32(a, s);
    const long long M = (long long)a.N * a.Ho * a.Wo;
    const long long K = (long long)a.kh * a.kw * a.Cin + (a.in2 ? a.Cin2 : 0);
    // Short-K layers are pure streaming: what matters is how many independent tiles a CU has in
    // flight, so they take the small-footprint 128 x 64 tile (4 blocks of 4 wavefronts per CU).
    if (K <= 128 && a.out1 == nullptr && a.in2 == nullptr) return launch_one<bf16_t, 128, 64, 64, 2, 2, bf16_t>(a, s);
    hipError_t e;
    if (((M + 255) / 256) * ((a.Cout + 255) / 256) < 200 && launch_ring_bf16(a, K, s, &e)) return e;
    if (launch_large_bf16(a, K, s, &e)) return e;
    return narrow ? launch_one<bf16_t, 128, 64, 64, 2, 2, bf16_t>(a, s) : launch_one<bf16_t, 128, 128, 128, 2, 4, bf16_t, true>(a, s);
}

}  // namespace thia

// The kernel of the large tiles: part of this translation unit, so that whoever links the layer kernels needs one object.
#include "conv_large.h"
