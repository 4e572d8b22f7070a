// ROI head kernels: ROIAlign gather on the NHWC head feature map, class scores and
// per-class box decoding, and the final detection selection (threshold, ordering,
// same-class greedy NMS, top-D).
#include "device_util.h"

#include <type_traits>

namespace thia {

// ------------------------------------------------------------------ ROIAlign
// One block per ROI, in calls with few ROIs two or four that share its bins and channels; threads run over channels, so
// every tap is one contiguous run of Ch elements of the NHWC map.  Convention: texel j has centre j + 0.5; a sample more than one
// texel outside the map contributes zero; otherwise its coordinates are clamped to the
// texel-centre range.  Output layout [(ph*P + pw)][c].
//
// A bin averages 2 x 2 samples of 2 x 2 texels each, and both the sample grid and the bilinear
// weights are products of a row factor and a column factor.  So a bin is sum_y sum_x Wy[y] Wx[x] F[y][x]
// over the DISTINCT rows and columns its samples touch (2 to 4 of each), with the weights of coinciding
// texels added up: a bin narrower than two texels gathers 4, 6 or 9 texels instead of 16.  The per-axis
// lists are built once per ROI (2 P threads), expanded to one tap table per bin in LDS (texel offset and
// weight, the 1/4 of the average folded in, entries past the bin's count zero), and every work item runs
// the smallest unrolled gather that covers its bin's count.
constexpr int ROI_TAPS = 16;   // most taps per bin (4 rows x 4 columns)

__host__ __device__ inline size_t roialign_lds_bytes(int P) {
    return (size_t)P * P * (ROI_TAPS * 8 + 4) + (size_t)2 * P * (4 * 8 + 4);
}

template <typename T>
__global__ __launch_bounds__(256) void roialign_kernel(const T* __restrict__ feat, const float* __restrict__ rois, int post,
                                                       int Hk, int Wk, int Ch, float scale, int P, int parts, T* __restrict__ out) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int nb = P * P;
    int* s_off = reinterpret_cast<int*>(smem_raw);             // [nb][16] texel offsets (in pixels of the map)
    float* s_w = reinterpret_cast<float*>(s_off + ROI_TAPS * nb);   // [nb][16]
    int* s_nt = reinterpret_cast<int*>(s_w + ROI_TAPS * nb);   // [nb] taps of the bin
    int* ax_i = s_nt + nb;                                     // [2 P][4] distinct texel rows (first P lists) / columns
    float* ax_w = reinterpret_cast<float*>(ax_i + 8 * P);      // [2 P][4] their summed weights
    int* ax_n = reinterpret_cast<int*>(ax_w + 8 * P);          // [2 P] entries per list
    const int roi = blockIdx.x / parts, part = blockIdx.x - roi * parts, f = roi / post;
    const float4 r = *reinterpret_cast<const float4*>(rois + 4 * (size_t)roi);
    const float x1 = r.x * scale, y1 = r.y * scale;
    const float bw = (r.z * scale - x1) / (float)P, bh = (r.w * scale - y1) / (float)P;
    if ((int)threadIdx.x < 2 * P) {
        const int lst = threadIdx.x, isx = lst >= P, p = isx ? lst - P : lst;
        const float start = isx ? x1 : y1, b = isx ? bw : bh;
        const int L = isx ? Wk : Hk;
        int n = 0;
        auto add = [&](int j, float w) {
            for (int k = 0; k < n; ++k)
                if (ax_i[4 * lst + k] == j) { ax_w[4 * lst + k] += w; return; }
            ax_i[4 * lst + n] = j; ax_w[4 * lst + n] = w; ++n;
        };
        for (int i = 0; i < 2; ++i) {
            float tc = start + (float)p * b + ((float)i + 0.5f) * b * 0.5f - 0.5f;
            if (tc < -1.f || tc > (float)L) continue;
            tc = fminf(fmaxf(tc, 0.f), (float)(L - 1));
            const int i0 = (int)floorf(tc), i1 = i0 + 1 < L ? i0 + 1 : L - 1;
            const float l = tc - (float)i0;
            add(i0, 1.f - l);
            add(i1, l);
        }
        ax_n[lst] = n;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < ROI_TAPS * nb; e += blockDim.x) {
        const int bin = e / ROI_TAPS, k = e - bin * ROI_TAPS, ph = bin / P, pw = bin - ph * P;
        const int ny = ax_n[ph], nx = ax_n[P + pw], nt = ny * nx;
        int off = 0;
        float w = 0.f;
        if (k < nt) {
            const int ia = k / nx, ib = k - ia * nx;
            off = ax_i[4 * ph + ia] * Wk + ax_i[4 * (P + pw) + ib];
            w = ax_w[4 * ph + ia] * ax_w[4 * (P + pw) + ib] * 0.25f;
        }
        s_off[e] = off;
        s_w[e] = w;
        if (k == 0) s_nt[bin] = nt;
    }
    __syncthreads();
    const T* fm = feat + (size_t)f * Hk * Wk * Ch;
    T* o = out + (size_t)roi * nb * Ch;
    // one work item = one bin x one 16-byte run of channels; consecutive threads take consecutive runs
    constexpr int VEC = 16 / (int)sizeof(T);
    const int runs = Ch / VEC;
    for (int i = part * blockDim.x + threadIdx.x; i < nb * runs; i += parts * blockDim.x) {
        const int bin = i / runs, c = (i - bin * runs) * VEC;
        const int nt = s_nt[bin];
        const int* toff = s_off + ROI_TAPS * bin;
        const float* tw = s_w + ROI_TAPS * bin;
        float sum[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) sum[e] = 0.f;
        auto gather = [&](auto nc) {
            constexpr int N = decltype(nc)::value;
            uint4 raw[N];
#pragma unroll
            for (int k = 0; k < N; ++k) raw[k] = *reinterpret_cast<const uint4*>(fm + (size_t)toff[k] * Ch + c);
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const float w = tw[k];
                if constexpr (sizeof(T) == 2) {
                    const uint32_t wd[4] = {raw[k].x, raw[k].y, raw[k].z, raw[k].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        sum[2 * e] += w * __uint_as_float(wd[e] << 16);
                        sum[2 * e + 1] += w * __uint_as_float(wd[e] & 0xffff0000u);
                    }
                } else {
                    sum[0] += w * __uint_as_float(raw[k].x); sum[1] += w * __uint_as_float(raw[k].y);
                    sum[2] += w * __uint_as_float(raw[k].z); sum[3] += w * __uint_as_float(raw[k].w);
                }
            }
        };
        if (nt <= 4) gather(std::integral_constant<int, 4>{});
        else if (nt <= 6) gather(std::integral_constant<int, 6>{});
        else if (nt <= 9) gather(std::integral_constant<int, 9>{});
        else if (nt <= 12) gather(std::integral_constant<int, 12>{});
        else gather(std::integral_constant<int, 16>{});
        uint4 pk;
        if constexpr (sizeof(T) == 2) {
            pk = make_uint4(pack_bf16x2(sum[0], sum[1]), pack_bf16x2(sum[2], sum[3]), pack_bf16x2(sum[4], sum[5]),
                            pack_bf16x2(sum[6], sum[7]));
        } else {
            pk = make_uint4(__float_as_uint(sum[0]), __float_as_uint(sum[1]), __float_as_uint(sum[2]), __float_as_uint(sum[3]));
        }
        *reinterpret_cast<uint4*>(o + (size_t)bin * Ch + c) = pk;
    }
}

hipError_t launch_roialign(const void* feat, const float* rois, int n, int post, int Hk, int Wk, int Ch, int stride, int P,
                           int precision, void* out, hipStream_t s) {
    if (n <= 0 || post <= 0 || P <= 0 || P > 16 || Ch % 8) return hipErrorInvalidValue;
    const size_t lds = roialign_lds_bytes(P);
    const float scale = 1.0f / (float)stride;
    // One block per ROI leaves a call with few of them waiting for its ~6 rounds of gathers (fp32: ~12): few ROIs are split over
    // two or four blocks, which repeat the (short) tap lists.  Measured in us with 1 / 2 / 4 blocks per ROI, proposals of
    // 540 x 960 frames at exits 1, 2 and 4: bf16, 300 ROIs 16.0 / 11.9 / 13.4, 15.1 / 11.4 / 11.6 and 12.0 / 10.0 / 12.6; 600
    // 17.1 / 15.6 / 19.4, 16.3 / 13.6 / 17.0 and 14.2 / 15.3 / 17.9; fp32, 300 ROIs 17.4 / 13.8 / 13.4, 16.7 / 12.4 / 10.6 and
    // 14.2 / 11.3 / 10.7; 600 26.3 / 22.2 / 25.7, 19.1 / 15.4 / 16.1 and 16.5 / 14.5 / 17.2; four 128 x 128 frames (200, fp32)
    // 15.7 / 12.0 / 10.4.  Random ROIs, one block / four: 50 bf16 12.3 / 7.7, 200 bf16 14.0 / 10.8; 700 19.3 / 24.9 and fp32 31.4 / 32.9.
    const long long rois_all = (long long)n * post;
    const int parts = rois_all <= (precision ? 200 : 300) ? 4 : rois_all <= 600 ? 2 : 1;
    const unsigned blocks = (unsigned)n * (unsigned)post * (unsigned)parts;
    if (precision)
        hipLaunchKernelGGL(roialign_kernel<bf16_t>, dim3(blocks), dim3(256), lds, s, static_cast<const bf16_t*>(feat), rois, post,
                           Hk, Wk, Ch, scale, P, parts, static_cast<bf16_t*>(out));
    else
        hipLaunchKernelGGL(roialign_kernel<float>, dim3(blocks), dim3(256), lds, s, static_cast<const float*>(feat), rois, post, Hk,
                           Wk, Ch, scale, P, parts, static_cast<float*>(out));
    return hipGetLastError();
}

// ------------------------------------------------------------------ scores + per-class boxes
// One thread per ROI and class: softmax over Kc logits (max subtracted; every thread of a ROI forms the same sum in the same
// order) and, for a foreground class, the ROI decoded with that class's deltas and clipped.  (One thread per ROI walked the
// classes one by one in a handful of wavefronts: 300 ROIs, 8 classes 6.4 us, now 4.5; 8 000 of 20 14.9, 7.4.)
__global__ __launch_bounds__(128) void scores_boxes_kernel(const float* __restrict__ cls, const float* __restrict__ deltas,
                                                           const float* __restrict__ rois, long long total, int Kc, float imgW, float imgH,
                                                           float* __restrict__ scores, float* __restrict__ boxes) {
    const long long e = (long long)blockIdx.x * 128 + threadIdx.x;
    if (e >= total) return;
    const long long r = e / Kc;
    const int c = (int)(e - r * Kc);
    const float4 q = *reinterpret_cast<const float4*>(rois + 4 * r);
    const float4 d = *reinterpret_cast<const float4*>(deltas + 4 * e);
    const float* x = cls + r * Kc;
    const float mine = x[c];
    float mx = x[0];
    for (int k = 1; k < Kc; ++k) mx = fmaxf(mx, x[k]);
    float sum = 0.f;
    for (int k = 0; k < Kc; ++k) sum += expf(x[k] - mx);
    scores[e] = expf(mine - mx) / sum;
    const float rw = q.z - q.x, rh = q.w - q.y;
    const float cx = q.x + 0.5f * rw, cy = q.y + 0.5f * rh;
    Box b = {0.f, 0.f, 0.f, 0.f};
    if (c > 0) decode_box(cx, cy, rw, rh, d.x, d.y, d.z, d.w, imgW, imgH, b);
    *reinterpret_cast<float4*>(boxes + 4 * e) = make_float4(b.x1, b.y1, b.x2, b.y2);
}

hipError_t launch_scores_boxes(const float* cls, const float* deltas, const float* rois, int n, int post, int Kc, float imgW,
                               float imgH, float* scores, float* boxes, hipStream_t s) {
    const long long total = (long long)n * post * Kc, blocks = (total + 127) / 128;
    if (n <= 0 || post <= 0 || Kc <= 0 || blocks >= (1ll << 31)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(scores_boxes_kernel, dim3((unsigned)blocks), dim3(128), 0, s, cls, deltas, rois, total, Kc, imgW, imgH,
                       scores, boxes);
    return hipGetLastError();
}

// ------------------------------------------------------------------ detection selection
// One block per frame.  Candidates (roi < roi_n, class >= 1, score > thr, non-empty box)
// get the key (order-preserving score) << 32 | (2^32 - 1 - (roi*Kc + class)); the keys are
// sorted descending (LDS when they fit, else in the global scratch), then wavefront 0
// runs greedy same-class NMS 64 candidates at a time against the list of kept boxes.
constexpr int SEL_LDS_KEYS = 4096;
constexpr int SEL_MAX_D = 512;

__global__ __launch_bounds__(1024) void select_kernel(const float* __restrict__ scores, const float* __restrict__ boxes,
                                                      const int32_t* __restrict__ roi_n, int post, int Kc, float score_thr,
                                                      float nms_thr, int D, uint64_t* __restrict__ gkeys, int key_cap,
                                                      float* __restrict__ out_boxes, float* __restrict__ out_scores,
                                                      int32_t* __restrict__ out_labels, int32_t* __restrict__ out_n) {
    __shared__ uint64_t lkeys[SEL_LDS_KEYS];
    __shared__ Box kbox[SEL_MAX_D];
    __shared__ int klab[SEL_MAX_D];
    __shared__ float kscore[SEL_MAX_D];
    __shared__ int s_count, s_nk;
    const int f = blockIdx.x, t = threadIdx.x;
    int nr = roi_n[f];
    nr = nr < post ? nr : post;
    const float* sc = scores + (size_t)f * post * Kc;
    const float* bx = boxes + (size_t)f * post * Kc * 4;
    uint64_t* gk = gkeys + (size_t)f * key_cap;
    if (t == 0) { s_count = 0; s_nk = 0; }
    __syncthreads();
    const int total = nr * Kc;
    for (int j = t; j < total; j += 1024) {
        const int c = j % Kc;
        if (c == 0) continue;
        const float s = sc[j];
        if (!(s > score_thr)) continue;
        const float4 b = *reinterpret_cast<const float4*>(bx + 4 * (size_t)j);
        if (!((b.z - b.x >= 1e-3f) && (b.w - b.y >= 1e-3f))) continue;
        const int slot = atomicAdd(&s_count, 1);
        gk[slot] = ((uint64_t)score_key(s) << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)j);
    }
    __syncthreads();
    const int nc = s_count;
    int n2 = 1;
    while (n2 < nc) n2 <<= 1;
    uint64_t* keys;
    if (n2 <= SEL_LDS_KEYS) {
        for (int i = t; i < n2; i += 1024) lkeys[i] = i < nc ? gk[i] : 0ull;
        keys = lkeys;
    } else {
        for (int i = nc + t; i < n2; i += 1024) gk[i] = 0ull;
        keys = gk;
    }
    __syncthreads();
    bitonic_sort_desc(keys, n2);

    if (t < 64) {
        const int lane = t;
        int nk = 0;
        for (int s0 = 0; s0 < nc && nk < D; s0 += 64) {
            const int i = s0 + lane;
            bool alive = i < nc;
            Box me = {0.f, 0.f, 0.f, 0.f};
            int lab = -1;
            float myscore = 0.f;
            if (alive) {
                const uint64_t key = keys[i];
                const uint32_t j = 0xFFFFFFFFu - (uint32_t)(key & 0xFFFFFFFFull);
                const float4 b = *reinterpret_cast<const float4*>(bx + 4 * (size_t)j);
                me = {b.x, b.y, b.z, b.w};
                lab = (int)(j % (uint32_t)Kc);
                myscore = key_score((uint32_t)(key >> 32));
                for (int q = 0; q < nk; ++q)
                    if (klab[q] == lab && iou_over(kbox[q], me, nms_thr)) { alive = false; break; }
            }
            for (int b = 0; b < 64 && nk < D; ++b) {
                const int ab = __shfl((int)alive, b);
                if (!ab) continue;
                const Box kb = {__shfl(me.x1, b), __shfl(me.y1, b), __shfl(me.x2, b), __shfl(me.y2, b)};
                const int kl = __shfl(lab, b);
                const float ks = __shfl(myscore, b);
                if (lane == 0) { kbox[nk] = kb; klab[nk] = kl; kscore[nk] = ks; }
                ++nk;
                if (lane > b && alive && lab == kl && iou_over(kb, me, nms_thr)) alive = false;
            }
            __builtin_amdgcn_wave_barrier();
            __threadfence_block();
        }
        if (lane == 0) s_nk = nk;
    }
    __syncthreads();
    const int nk = s_nk;
    for (int d = t; d < D; d += 1024) {
        float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
        float s = 0.f;
        int l = -1;
        if (d < nk) { b = make_float4(kbox[d].x1, kbox[d].y1, kbox[d].x2, kbox[d].y2); s = kscore[d]; l = klab[d]; }
        *reinterpret_cast<float4*>(out_boxes + ((size_t)f * D + d) * 4) = b;
        out_scores[(size_t)f * D + d] = s;
        out_labels[(size_t)f * D + d] = l;
    }
    if (t == 0 && out_n) out_n[f] = nk;
}

// Same selection with blocks that take the foreground classes of a frame one by one, then one block per frame that merges
// (post <= 1024, (Kc - 1) * min(D, post) <= 8192).  Same-class NMS never looks across classes and the global walk stops after
// D kept boxes, so the result equals: per class, greedy NMS over that class's candidates in key order, cut after its first D
// kept; then the D largest keys among all kept.  A class's candidates are sorted in LDS and resolved 64 at a time: the
// wavefronts share the tests against the kept boxes and the group's overlap words, one wavefront decides.  What bounds it is
// the chain of groups (one block for all classes of a frame: 72 us for 32 frames of 300 ROIs x 7 classes, 15 + 7 now; the
// single chain over all classes in select_kernel: 346 us for 8 frames of 1000 ROIs x 19 classes, 10 to 18 + 6 to 8 now).
constexpr int SELC_MAX_POST = 1024, SELC_MAX_KEPT = 8192, SELC_THREADS = 512;
constexpr int SELC_FEW = 8;             // most classes merged by binary search
constexpr int SELC_RESIDENT = 768, SELC_MAX_GROUP = 4;   // blocks the chip holds (LDS: three per CU); most classes per block

// gkeys [n][key_cap]: class c's kept keys at c * Dc (sorted descending), the classes' counts behind all of them.  GROUPED: a
// block takes up to four classes where a call has more than 32 of them and more than the chip holds blocks; it first looks
// which of its classes have a score above the threshold (their scores lie side by side).  Of many classes most are usually
// empty, and a block for each of them costs 2 to 3 us a round: 32 frames, 90 classes without a candidate 12 -> 3 us, with
// 300 candidates each 23 -> 24.  (With few candidates select_kernel's one block per frame is as fast, 3 to 14 us; with many it
// takes 25 to 360.)
template <bool GROUPED>
__global__ __launch_bounds__(SELC_THREADS) void select_class_kernel(const float* __restrict__ scores, const float* __restrict__ boxes,
                                                                    const int32_t* __restrict__ roi_n, int post, int Kc, int group,
                                                                    float score_thr, float nms_thr, int Dc, uint64_t* __restrict__ gkeys,
                                                                    int key_cap) {
    __shared__ uint64_t lkeys[2 * SELC_MAX_POST];
    __shared__ float4 sbox[SELC_MAX_POST];                               // boxes in key order
    __shared__ float4 kbox[SELC_MAX_POST];                               // kept boxes
    __shared__ uint64_t early[64];                                       // group of 64: earlier candidates that overlap
    __shared__ unsigned long long s_dead;                                // group of 64: suppressed by kept boxes
    __shared__ uint32_t s_some;                                          // classes with a score above the threshold
    __shared__ int s_count, s_nk;
    constexpr int NWV = SELC_THREADS / 64, JW = 64 / NWV;                // a wavefront's share of a group's overlap words
    const int NC = Kc - 1, c0 = blockIdx.x * group, f = blockIdx.y, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    int nr = roi_n[f];
    nr = nr < post ? nr : post;
    const float* sc = scores + (size_t)f * post * Kc;
    const float* bx = boxes + (size_t)f * post * Kc * 4;
    int32_t* counts = reinterpret_cast<int32_t*>(gkeys + (size_t)f * key_cap + (size_t)NC * Dc);
    auto as_box = [](const float4& v) { return Box{v.x, v.y, v.z, v.w}; };
    uint32_t todo = 1u;                                                  // (uniform)
    if constexpr (GROUPED) {
        if (t == 0) s_some = 0u;
        __syncthreads();
        const int gc = NC - c0 < group ? NC - c0 : group;
        uint32_t some = 0u;
        for (int i = t; i < nr * gc; i += SELC_THREADS) {
            const int roi = i / gc, g = i - roi * gc;
            if (sc[roi * Kc + c0 + g + 1] > score_thr) some |= 1u << g;
        }
        if (some) atomicOr(&s_some, some);
        __syncthreads();
        todo = s_some;
        if (t < gc && ((todo >> t) & 1u) == 0u) counts[c0 + t] = 0;
    }
    for (; todo != 0u; todo &= todo - 1u) {
        const int c = c0 + (GROUPED ? __builtin_ctz(todo) : 0);
        uint64_t* out = gkeys + (size_t)f * key_cap + (size_t)c * Dc;
        if (t == 0) { s_count = 0; s_nk = 0; s_dead = 0ull; }
        __syncthreads();
        for (int r0 = 0; r0 < nr; r0 += SELC_THREADS) {
            const int roi = r0 + t;
            uint64_t key = 0ull;
            if (roi < nr) {
                const int j = roi * Kc + c + 1;
                const float s = sc[j];
                const float4 b = *reinterpret_cast<const float4*>(bx + 4 * (size_t)j);
                if (s > score_thr && (b.z - b.x >= 1e-3f) && (b.w - b.y >= 1e-3f)) key = ((uint64_t)score_key(s) << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)j);
            }
            const uint64_t has = __ballot(key != 0ull);
            int base = 0;
            if (lane == 0 && has != 0ull) base = atomicAdd(&s_count, (int)__popcll(has));
            base = __shfl(base, 0);
            if (key != 0ull) lkeys[base + __popcll(has & ((1ull << lane) - 1ull))] = key;
        }
        __syncthreads();
        const int nc = s_count;
        int nk = 0;
        if (nc > 0) {
            int n2 = 64;
            while (n2 < nc) n2 <<= 1;
            for (int i = nc + t; i < n2; i += SELC_THREADS) lkeys[i] = 0ull;
            const uint64_t* keys = block_sort_desc(lkeys, lkeys + SELC_MAX_POST, n2);
            for (int i = t; i < nc; i += SELC_THREADS) {
                const uint32_t j = 0xFFFFFFFFu - (uint32_t)(keys[i] & 0xFFFFFFFFull);
                sbox[i] = *reinterpret_cast<const float4*>(bx + 4 * (size_t)j);
            }
            __syncthreads();
            for (int s0 = 0; s0 < nc && nk < Dc; s0 += 64) {
                const int i = s0 + lane;
                const bool valid = i < nc;
                const Box me = valid ? as_box(sbox[i]) : Box{0.f, 0.f, 0.f, 0.f};
                // every wavefront: its share of the kept boxes against the group's 64, one candidate per lane
                bool hit = false;
                for (int q = wv; q < nk; q += NWV) hit = iou_over(as_box(kbox[q]), me, nms_thr) || hit;
                const uint64_t dead = __ballot(hit);
                if (lane == 0 && dead != 0ull) atomicOr(&s_dead, (unsigned long long)dead);
                // and JW earlier candidates of the group against every later one
                uint32_t bits = 0u;
#pragma unroll
                for (int u = 0; u < JW; ++u) {
                    const int j = wv * JW + u;
                    if (j < lane && valid && iou_over(as_box(sbox[s0 + j]), me, nms_thr)) bits |= 1u << u;
                }
                static_assert(JW == 8, "one byte of a row's word per wavefront");
                reinterpret_cast<unsigned char*>(early)[lane * 8 + wv] = (unsigned char)bits;
                __syncthreads();
                if (wv == 0) {
                    const uint64_t in_group = nc - s0 < 64 ? (1ull << (nc - s0)) - 1ull : ~0ull;
                    const uint64_t kept = greedy_keep(in_group & ~s_dead, early[lane]);
                    const int pos = nk + __popcll(kept & ((1ull << lane) - 1ull));
                    const bool mine = ((kept >> lane) & 1ull) != 0ull && pos < Dc;
                    if (mine) { kbox[pos] = sbox[i]; out[pos] = keys[i]; }
                    if (lane == 0) { s_nk = nk + __popcll(kept) < Dc ? nk + __popcll(kept) : Dc; s_dead = 0ull; }
                }
                __syncthreads();
                nk = s_nk;
            }
        }
        if (t == 0) counts[c] = nk;
        if constexpr (GROUPED) __syncthreads();   // (the next class reuses the lists; s_nk and s_count are read above)
    }
}

// The D largest of a frame's kept keys.  A key's place is the number of larger keys.  Up to SELC_FEW classes: its place in its
// own class's list plus, found by binary search, the number of larger keys in every other list.  That grows with the square
// of the classes (19 of 50 kept boxes 11 to 18 us, 90 of 50 145 to 295), so with more of them only keys not below a bound are
// counted: among the first p of every class, p as small as leaves at least D of them, the D-th largest is a lower bound of
// the D-th largest of all (19 of 50 6 to 7 us, 90 of 50 9 to 11; 4 of 50 4.2 by searching, 5.0 by counting).
__global__ __launch_bounds__(1024) void select_merge_kernel(const uint64_t* __restrict__ gkeys, int key_cap, const float* __restrict__ boxes,
                                                            int post, int Kc, int Dc, int D, float* __restrict__ out_boxes,
                                                            float* __restrict__ out_scores, int32_t* __restrict__ out_labels,
                                                            int32_t* __restrict__ out_n) {
    extern __shared__ __align__(16) unsigned char sel_smem[];
    __shared__ uint64_t s_bound;
    __shared__ int s_n[2];
    const int NC = Kc - 1, f = blockIdx.x, t = threadIdx.x, lane = t & 63;
    const bool few = NC <= SELC_FEW;
    uint64_t* kkey = reinterpret_cast<uint64_t*>(sel_smem);              // [NC][Dc]
    uint64_t* list = kkey + (size_t)NC * Dc;                             // more classes: [NC * Dc] keys to be counted, in any order
    int* kcount = reinterpret_cast<int*>(few ? list : list + (size_t)NC * Dc);   // [NC]
    const uint64_t* gk = gkeys + (size_t)f * key_cap;
    const int32_t* gn = reinterpret_cast<const int32_t*>(gk + (size_t)NC * Dc);
    if (t < 2) s_n[t] = 0;
    if (t == 0) s_bound = 0ull;
    for (int c = t; c < NC; c += 1024) kcount[c] = gn[c];
    for (int e = t; e < NC * Dc; e += 1024) kkey[e] = gk[e];             // (entries behind a class's count are never used)
    __syncthreads();
    auto put = [&](uint64_t key, int rank) {
        const uint32_t j = 0xFFFFFFFFu - (uint32_t)(key & 0xFFFFFFFFull);
        *reinterpret_cast<float4*>(out_boxes + ((size_t)f * D + rank) * 4) = *reinterpret_cast<const float4*>(boxes + ((size_t)f * post * Kc + j) * 4);
        out_scores[(size_t)f * D + rank] = key_score((uint32_t)(key >> 32));
        out_labels[(size_t)f * D + rank] = (int)(j % (uint32_t)Kc);
    };
    auto first = [&](int p) {                                            // keys among the first p of every class
        int sum = 0;
        for (int c = lane; c < NC; c += 64) sum += kcount[c] < p ? kcount[c] : p;
        for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
        return sum;
    };
    const int total = first(Dc), want = total < D ? total : D;
    // the first p keys of every class that are not below `bound`, put behind list[0 .. count)
    auto collect = [&](int p, uint64_t bound, int* count) {
        for (int e0 = 0; e0 < NC * p; e0 += 1024) {                      // (whole wavefronts)
            const int e = e0 + t, c = e / p, q = e - c * p;
            const bool in = e < NC * p && q < kcount[c < NC ? c : 0] && kkey[(size_t)(c < NC ? c : 0) * Dc + q] >= bound;
            const uint64_t has = __ballot(in);
            int base = 0;
            if (lane == 0 && has != 0ull) base = atomicAdd(count, (int)__popcll(has));
            base = __shfl(base, 0);
            if (in) list[base + __popcll(has & ((1ull << lane) - 1ull))] = kkey[(size_t)c * Dc + q];
        }
        __syncthreads();
        return *count;
    };
    // visit(key, number of larger keys) for list[0 .. m), by one lane per key: 16 lanes count a key together; in the rare longer
    // list a thread counts alone and stops at `most`
    auto ranked = [&](int m, int most, auto&& visit) {
        if (m <= 1024) {
            const int part = lane & 15;
            for (int i = t >> 4; i < m; i += 64) {                       // (16 lanes in step: i is theirs)
                const uint64_t key = list[i];
                int cnt = 0;
                for (int j = part; j < m; j += 16) cnt += list[j] > key ? 1 : 0;
                for (int d = 8; d > 0; d >>= 1) cnt += __shfl_xor(cnt, d);
                if (part == 0) visit(key, cnt);
            }
        } else {
            for (int i = t; i < m; i += 1024) {
                const uint64_t key = list[i];
                int cnt = 0;
                for (int j = 0; j < m && cnt < most; ++j) cnt += list[j] > key ? 1 : 0;
                visit(key, cnt);
            }
        }
    };
    if (few) {
        for (int e = t; e < NC * Dc; e += 1024) {
            const int c = e / Dc, q = e - c * Dc;
            if (q >= kcount[c]) continue;
            const uint64_t key = kkey[e];
            int rank = q;
            for (int c2 = 0; c2 < NC && rank < D; ++c2) {
                if (c2 == c) continue;
                const uint64_t* l = kkey + (size_t)c2 * Dc;
                int lo = 0, hi = kcount[c2];                             // first position whose key is smaller
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (l[mid] > key) lo = mid + 1; else hi = mid;
                }
                rank += lo;
            }
            if (rank < D) put(key, rank);
        }
    } else {
        if (total > 2 * D) {
            int p = (want + NC - 1) / NC;
            while (first(p) < want) p *= 2;                                  // (first(Dc) = total: ends)
            p = p < Dc ? p : Dc;
            const int m = collect(p, 0ull, &s_n[0]);
            ranked(m, want, [&](uint64_t key, int rank) { if (rank == want - 1) s_bound = key; });   // (keys are unique: one key)
            __syncthreads();
        }
        const int m = collect(Dc, s_bound, &s_n[1]);
        ranked(m, D, [&](uint64_t key, int rank) { if (rank < D) put(key, rank); });
    }
    for (int d = want + t; d < D; d += 1024) {
        *reinterpret_cast<float4*>(out_boxes + ((size_t)f * D + d) * 4) = make_float4(0.f, 0.f, 0.f, 0.f);
        out_scores[(size_t)f * D + d] = 0.f;
        out_labels[(size_t)f * D + d] = -1;
    }
    if (t == 0 && out_n) out_n[f] = want;
}

hipError_t launch_select(const float* scores, const float* boxes, const int32_t* roi_n, int n, int post, int Kc,
                         float score_thr, float nms_thr, int D, uint64_t* keys, int key_cap, float* out_boxes,
                         float* out_scores, int32_t* out_labels, int32_t* out_n, hipStream_t s) {
    if (n <= 0 || D <= 0 || D > SEL_MAX_D || key_cap < post * Kc) return hipErrorInvalidValue;
    const int NC = Kc - 1, Dc = D < post ? D : post;   // a class keeps at most Dc
    if (post <= SELC_MAX_POST && NC >= 1 && NC <= 2 * post && (long)NC * Dc <= SELC_MAX_KEPT && n <= 65535) {
        // (key_cap >= post * Kc holds the NC * Dc kept keys and, in the post that are left, the NC counts)
        hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(select_merge_kernel), (size_t)SELC_MAX_KEPT * 16 + 2 * SELC_MAX_POST * 4);
        if (e != hipSuccess) return e;
        const long long blocks = (long long)n * NC;
        const long long g = (blocks + SELC_RESIDENT - 1) / SELC_RESIDENT;
        const int group = NC <= 32 ? 1 : g > SELC_MAX_GROUP ? SELC_MAX_GROUP : (int)g;
        hipLaunchKernelGGL(group > 1 ? select_class_kernel<true> : select_class_kernel<false>, dim3((NC + group - 1) / group, n), dim3(SELC_THREADS),
                           0, s, scores, boxes, roi_n, post, Kc, group, score_thr, nms_thr, Dc, keys, key_cap);
        const size_t lds = (size_t)NC * Dc * (NC <= SELC_FEW ? 8 : 16) + (size_t)NC * 4;
        hipLaunchKernelGGL(select_merge_kernel, dim3(n), dim3(1024), lds, s, keys, key_cap, boxes, post, Kc, Dc, D,
                           out_boxes, out_scores, out_labels, out_n);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(select_kernel, dim3(n), dim3(1024), 0, s, scores, boxes, roi_n, post, Kc, score_thr, nms_thr, D, keys,
                       key_cap, out_boxes, out_scores, out_labels, out_n);
    return hipGetLastError();
}

__global__ void fill_empty_kernel(int total, float* __restrict__ out_boxes, float* __restrict__ out_scores,
                                  int32_t* __restrict__ out_labels) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    *reinterpret_cast<float4*>(out_boxes + 4 * (size_t)i) = make_float4(0.f, 0.f, 0.f, 0.f);
    out_scores[i] = 0.f;
    out_labels[i] = -1;
}

hipError_t launch_fill_empty(int n, int D, float* out_boxes, float* out_scores, int32_t* out_labels, hipStream_t s) {
    const int total = n * D;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_empty_kernel, dim3((total + 255) / 256), dim3(256), 0, s, total, out_boxes, out_scores, out_labels);
    return hipGetLastError();
}

}  // namespace thia
