// Host-side arithmetic of the layer kernels against plain loops (no GPU, no HIP call): the division by multiplication, the tap
// mask in closed form, and the 32-bit offsets of the large tiles' buffer loads.  Built and run by tests/test_layer_rules.py, not part of
// libthia.so; prints "layer_rules_driver: ok" or what failed.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "conv_common.h"

using namespace thia;

static int failures = 0;
#define CHECK(ok, ...)                                        \
    do {                                                      \
        if (!(ok) && ++failures <= 20) std::printf(__VA_ARGS__); \
    } while (0)

static void check_division(std::mt19937_64& rng) {
    auto one = [&](int d) {
        const FastDiv by(d);
        const long long top = 0x7fffffffll;
        for (long long q : {0ll, 1ll, 2ll, (long long)(rng() % 1000), top / d / 2, top / d - 1, top / d})
            for (long long n : {q * d - 1, q * d, q * d + d / 2, q * d + d - 1})
                if (n >= 0 && n <= top) CHECK(by((int)n) == (int)(n / d), "FastDiv: %lld / %d = %d\n", n, d, by((int)n));
    };
    for (int d = 1; d <= 70000; ++d) one(d);
    for (int l = 17; l < 31; ++l)
        for (int e = -2; e <= 2; ++e) one((1 << l) + e);
    for (int i = 0; i < 100000; ++i) one((int)(rng() % 0x7fffffff) + 1);
    one(0x7fffffff);
}

static void check_tap_mask() {
    for (int kh = 1; kh <= 32; ++kh)
        for (int kw = 1; kh * kw <= 32; ++kw) {
            uint32_t every_row = 0;
            for (int ky = 0; ky < kh; ++ky) every_row |= 1u << (ky * kw);
            for (int H : {1, 2, 3, 7, 40})
                for (int W : {1, 2, 5, 40})
                    for (int y = -kh - 2; y <= H + 2; ++y)
                        for (int x = -kw - 2; x <= W + 2; ++x) {
                            uint32_t want = 0;
                            for (int t = 0; t < kh * kw; ++t) {
                                const int iy = y + t / kw, ix = x + t % kw;
                                if (iy >= 0 && iy < H && ix >= 0 && ix < W) want |= 1u << t;
                            }
                            const uint32_t got = tap_mask(y, x, H, W, kh, kw, every_row);
                            CHECK(got == want, "tap_mask: %d x %d filter at (%d, %d) of %d x %d: %08x, not %08x\n", kh, kw, y, x, H, W, got, want);
                        }
        }
}

// Byte offsets that the blocks of a bm-pixel tile load input pixels at: (least, largest) over the taps inside the image.  The
// least is that of the first tap, inside the image or not: the part of the offset that a pixel's register holds.
static void large_offsets(const ConvArgs& a, int bm, long long& least, long long& largest) {
    least = 1ll << 62, largest = -(1ll << 62);
    const long long HoWo = (long long)a.Ho * a.Wo, M = a.N * HoWo;
    for (long long m0 = 0; m0 < M; m0 += bm) {
        const long long img0 = m0 / HoWo;
        const long long oy0 = m0 % HoWo / a.Wo, base = (img0 * a.H + large_first_row((int)oy0, a.stride, a.H) - a.pad) * a.W - a.pad;
        for (long long m = m0; m < std::min(M, m0 + bm); ++m) {
            const long long img = m / HoWo, oy = m % HoWo / a.Wo, ox = m % a.Wo;
            // the first and the last tap inside the image (none: nothing is read)
            const long long ky0 = std::max(0ll, a.pad - oy * a.stride), ky1 = std::min<long long>(a.kh, a.H + a.pad - oy * a.stride) - 1;
            const long long kx0 = std::max(0ll, a.pad - ox * a.stride), kx1 = std::min<long long>(a.kw, a.W + a.pad - ox * a.stride) - 1;
            if (ky0 > ky1 || kx0 > kx1) continue;
            auto at = [&](long long ky, long long kx) {
                return ((img * a.H + oy * a.stride - a.pad + ky) * a.W + ox * a.stride - a.pad + kx - base) * a.Cin * 2;
            };
            least = std::min(least, at(0, 0));
            largest = std::max(largest, at(ky1, kx1) + (a.Cin - 8) * 2 + 16);
        }
    }
}

static ConvArgs layer(int N, int H, int W, int Cin, int Cout, int k, int stride, int pad) {
    ConvArgs a{};
    a.N = N; a.H = H; a.W = W; a.Cin = Cin; a.Cout = Cout; a.kh = a.kw = k; a.stride = stride; a.pad = pad;
    a.Ho = (H + 2 * pad - k) / stride + 1; a.Wo = (W + 2 * pad - k) / stride + 1;
    a.ld0 = a.n_split = Cout;
    a.relu = 1;
    return a;
}

static const int TILES[4][2] = {{256, 256}, {192, 256}, {256, 128}, {192, 128}};

static void check_large_offsets(std::mt19937_64& rng) {
    auto pick = [&](int low, int high) { return low + (int)(rng() % (uint64_t)(high - low + 1)); };
    int taken = 0, refused = 0;
    auto one = [&](const ConvArgs& a) {
        for (auto& t : TILES) {
            if (!conv_large_supported(a, 1, t[0], t[1])) { ++refused; continue; }
            ++taken;
            long long least, largest;
            large_offsets(a, t[0], least, largest);
            CHECK(least >= 0 && largest <= 1ll << 31, "%d x %d tile: %d images of %d x %d x %d, filter %d stride %d pad %d: offsets %lld .. %lld\n", t[0],
                  t[1], a.N, a.H, a.W, a.Cin, a.kh, a.stride, a.pad, least, largest);
        }
    };
    // maps of 2 GiB and more
    for (const ConvArgs& a : {layer(1, 4096, 4096, 64, 256, 3, 1, 1), layer(3, 2048, 2048, 256, 256, 3, 1, 1), layer(1, 16384, 16384, 64, 256, 3, 1, 1),
                              layer(2, 8191, 8193, 128, 512, 1, 2, 0)})
        for (auto& t : TILES) {
            CHECK(conv_large_supported(a, 1, t[0], t[1]), "%d x %d tile: %d images of %d x %d x %d refused\n", t[0], t[1], a.N, a.H, a.W, a.Cin);
            ConvArgs few = a;   // (block by block: the first rows)
            few.N = 1, few.Ho = std::min(a.Ho, 40);
            long long least, largest;
            large_offsets(few, t[0], least, largest);
            CHECK(least >= 0 && largest <= 1ll << 31, "%d x %d tile: %d x %d x %d: offsets %lld .. %lld\n", t[0], t[1], a.H, a.W, a.Cin, least, largest);
        }
    for (int i = 0; i < 20000; ++i) {
        const int k = pick(1, 5), pad = pick(0, rng() % 4 ? k / 2 : 3 * k), stride = rng() % 3 ? pick(1, 3) : pick(4, 300);
        const int H = (pick(1, 20) - 1) * stride + std::max(1, k - 2 * pad) + pick(0, stride - 1);
        const int W = (pick(1, 20) - 1) * stride + std::max(1, k - 2 * pad) + pick(0, stride - 1);
        const long long rows = std::min<long long>(8 * H, pick(1, 300) * (long long)stride + k);   // about 2 GiB in so many rows
        const long long cin = (1ll << 31) / (rows * W * 2) / 64 * 64;
        if (cin < 64 || cin > 1 << 22) continue;
        one(layer(pick(1, 8), H, W, (int)cin, 256, k, stride, pad));
    }
    CHECK(taken > 10000 && refused > 1000, "offsets: %d layers taken, %d refused\n", taken, refused);
}

int main() {
    std::mt19937_64 rng(20481);
    check_division(rng);
    check_tap_mask();
    check_large_offsets(rng);
    if (failures) {
        std::printf("layer_rules_driver: %d failures\n", failures);
        return 1;
    }
    std::printf("layer_rules_driver: ok\n");
    return 0;
}
