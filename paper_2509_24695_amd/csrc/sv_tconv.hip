// C ABI of the temporal convolution (include/sv_tconv.h): argument checks and launches.
#include "../../include/sv_tconv.h"
#include "../../include/sv_measure.h"

#include <mutex>
#include <type_traits>

#include "tconv_mfma.hpp"

namespace {

using namespace sv;

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

bool overlaps(const void *a, size_t na, const void *b, size_t nb)
{
    const auto pa = reinterpret_cast<uintptr_t>(a), pb = reinterpret_cast<uintptr_t>(b);
    return pa < pb + nb && pb < pa + na;
}

using TconvKernel = void (*)(TconvArgs);

// The tile kernels, and the measurement variants of the 256 x 256 one (0 = the library's own).
struct TconvForm {
    int bm, bn, lds;
    TconvKernel kernel;
};
template <int BM, int BN> TconvForm form()
{
    using P = TcTile<BM, BN>;
    return TconvForm{BM, BN, P::kLdsBytes, tconv_mfma<P>};
}
enum { kForm256, kForm256x128, kForm128, kForm64, kForm256Long, kForm256LongTail };   // Long: the 32 x 32 x 16 kernel
const TconvForm kForms[] = {form<256, 256>(), form<256, 128>(), form<128, 128>(), form<64, 64>(),
                            {kTcBM, kTcBN, kTcLdsBytes, tconv_mfma32<false>}, {kTcBM, kTcBN, kTcLdsBytes, tconv_mfma32<true>}};
TconvKernel variant_kernel(int variant)
{
    using P = TcTile<256, 256>;
    switch (variant) {
    case 1: return tconv_mfma<P, 1>;
    case 2: return tconv_mfma<P, 2>;
    case 3: return tconv_mfma<P, 3>;
    default: return tconv_mfma<P>;
    }
}

// The kernels need their dynamic LDS allowed once per device.
bool tconv_kernels_ready()
{
    static bool ready[64] = {};
    static std::mutex mu;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
    std::lock_guard<std::mutex> lock(mu);
    if (!ready[dev]) {
        auto allow = [](TconvKernel k, int lds) {
            return hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, lds) == hipSuccess;
        };
        for (const TconvForm &f : kForms)
            if (!allow(f.kernel, f.lds)) return false;
        for (int v = 1; v < 4; ++v)
            if (!allow(variant_kernel(v), kForms[0].lds)) return false;
        ready[dev] = true;
    }
    return true;
}

// Which tile.  A large one reads less per product, but has to fill 256 compute units: what is compared is the time in us per K-step,
// over the rounds that the tiles take (two of 128 x 128 or five of 64 x 64 share a compute unit), as measured.  256 x 128 pays
// where rows do not start on 64-byte boundaries, which costs loads more than products.  Measured per call, 256 / 256 long / 256 x 128 /
// 128 / 64 wide: one frame of 1 560 tokens, 2 240 channels 74 / 120 / - / 42 / 60 us; 4 680 tokens, 2 240 channels 137 / 142 / 250 /
// 194 / 319; 7 800 tokens, 1 024 channels 68 / 63 / 64 / 64 / 97; 4 200 tokens, 1 800 channels 134 / 133 / 111 / 137; 9 360 tokens, 640
// channels 47 / 44 / 44 / 36 / 46; 530 tokens, 328 channels 36 / 31 / - / 19 / 12.
int tconv_form(int64_t M, int D)
{
    constexpr int64_t kCus = 256;
    auto tiles = [&](int f) { return ((M + kForms[f].bm - 1) / kForms[f].bm) * ((D + kForms[f].bn - 1) / kForms[f].bn); };
    auto rounds = [&](int64_t n, int64_t at_once) { return (double)((n + at_once - 1) / at_once); };
    const int64_t t256 = tiles(kForm256), t256x128 = tiles(kForm256x128), t128 = tiles(kForm128), t64 = tiles(kForm64);
    int best = kForm256;
    double least = 0.62 * rounds(t256, kCus);
    auto offer = [&](int f, double us) {
        if (us < least) { least = us; best = f; }
    };
    if (t256 <= 160 || D < 16 * kTcBK) offer(D % kTcBK == 0 ? kForm256Long : kForm256LongTail, 0.56 * rounds(t256, kCus));
    if (D % kTcBK != 0) offer(kForm256x128, 0.42 * rounds(t256x128, kCus));
    offer(kForm128, t128 <= 2 * kCus ? 0.30 * (t128 > 290 ? (double)t128 / kCus : 1.13) : 0.60 * rounds(t128, 2 * kCus));
    const int64_t k64 = (t64 + kCus - 1) / kCus;
    offer(kForm64, 0.05 * (double)((k64 + 4) / 5) + 0.145 * (double)k64);
    return best;
}

sv_status tconv_enqueue(int variant, const void *x, const void *W, const void *cache_in, void *y, void *cache_out,
                        int32_t B, int32_t T, int32_t HW, int32_t D, int32_t dtype, void *stream)
{
    if (!x || !W || !y) return SV_ERR_NULL;
    if (B <= 0 || T <= 0 || HW <= 0 || D <= 0) return SV_ERR_SHAPE;
    if (dtype != SV_BF16) return SV_ERR_UNSUPPORTED;
    if (D % 8 != 0) return SV_ERR_UNSUPPORTED;
    const int64_t M = (int64_t)B * T * HW;
    if (M >= (int64_t)1 << 31 || (int64_t)3 * D * D >= (int64_t)1 << 31 || D > kTcMaxD) return SV_ERR_SHAPE;
    if (!aligned16(x) || !aligned16(W) || !aligned16(y) || !aligned16(cache_in) || !aligned16(cache_out))
        return SV_ERR_ALIGN;
    const size_t tok_bytes = (size_t)M * D * 2, w_bytes = (size_t)3 * D * D * 2, cache_bytes = (size_t)B * HW * D * 2;
    if (overlaps(y, tok_bytes, x, tok_bytes) || overlaps(y, tok_bytes, W, w_bytes) ||
        (cache_in && overlaps(y, tok_bytes, cache_in, cache_bytes)))
        return SV_ERR_SHAPE;
    // the new cache is copied out of x after y is complete: it may replace cache_in, nothing else
    if (cache_out && (overlaps(cache_out, cache_bytes, y, tok_bytes) || overlaps(cache_out, cache_bytes, x, tok_bytes) ||
                      overlaps(cache_out, cache_bytes, W, w_bytes)))
        return SV_ERR_SHAPE;
    if (variant != 0 && D % kTcBK != 0) return SV_ERR_UNSUPPORTED;
    if (!tconv_kernels_ready()) return SV_ERR_LAUNCH;

    TconvArgs a;
    a.x = static_cast<const uint16_t *>(x);
    a.W = static_cast<const uint16_t *>(W);
    a.cache = static_cast<const uint16_t *>(cache_in);
    a.y = static_cast<uint16_t *>(y);
    a.B = B; a.T = T; a.HW = HW; a.D = D;
    const TconvForm &f = kForms[variant != 0 ? 0 : tconv_form(M, D)];
    a.tiles_m = (int)((M + f.bm - 1) / f.bm);
    a.tiles_n = (D + f.bn - 1) / f.bn;
    const int64_t wgs = tc_grid_size((int64_t)a.tiles_m * a.tiles_n);
    if (wgs >= (int64_t)1 << 31) return SV_ERR_SHAPE;
    auto hs = static_cast<hipStream_t>(stream);
    const TconvKernel kernel = variant != 0 ? variant_kernel(variant) : f.kernel;
    kernel<<<dim3((unsigned)wgs), kThreads, f.lds, hs>>>(a);
    if (hipGetLastError() != hipSuccess) return SV_ERR_LAUNCH;
    if (cache_out) {
        const int64_t vecs = (int64_t)B * HW * D / 8;
        const int blocks = (int)((vecs + kThreads - 1) / kThreads < 2048 ? (vecs + kThreads - 1) / kThreads : 2048);
        tconv_cache_store<<<blocks, kThreads, 0, hs>>>(a.x, static_cast<uint16_t *>(cache_out), B, T, HW, D);
        if (hipGetLastError() != hipSuccess) return SV_ERR_LAUNCH;
    }
    return SV_OK;
}

}  // namespace

extern "C" sv_status sv_tconv_block_step(const void *x, const void *W, const void *cache_in, void *y, void *cache_out,
                                         int32_t B, int32_t T, int32_t HW, int32_t D, int32_t dtype, void *stream)
{
    return tconv_enqueue(0, x, W, cache_in, y, cache_out, B, T, HW, D, dtype, stream);
}

extern "C" sv_status sv_measure_tconv_variant(int32_t variant, const void *x, const void *W, const void *cache_in, void *y,
                                              int32_t B, int32_t T, int32_t HW, int32_t D, void *stream)
{
    if (variant < 0 || variant > 3) return SV_ERR_RANGE;
    return tconv_enqueue(variant, x, W, cache_in, y, nullptr, B, T, HW, D, SV_BF16, stream);
}
