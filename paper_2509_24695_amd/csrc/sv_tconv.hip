// C ABI of the temporal convolution (include/sv_tconv.h): argument checks and launches.
#include "../../include/sv_tconv.h"
#include "../../include/sv_measure.h"

#include <mutex>
#include <type_traits>

#include "tconv_frames.hpp"
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

// The kernels on row tiles in the order of TconvFormId; the long kernel's second form is for channels that are no multiple of the K-step.
struct TconvForm {
    int lds;
    TconvKernel kernel;
};
template <int F> TconvForm form()
{
    using P = TcTile<kTconvTile[F].bm, kTconvTile[F].bn>;
    return TconvForm{P::kLdsBytes, tconv_mfma<P>};
}
const TconvForm kForms[kRowForms + 1] = {form<kForm256>(), form<kForm256x128>(), form<kForm128>(), form<kForm64>(),
                                         {kTcLdsBytes, tconv_mfma32<false>}, {kTcLdsBytes, tconv_mfma32<true>}};

// The kernels on tiles of frames x positions, from kFrames3 on and by whether the call has a cache.
template <int F> TconvForm frame_form_of(bool front)
{
    constexpr FrameShape f = kFrameShape[F - kFrames3];
    using C = FrameTile<f.frames, f.blocks, f.channels / 64, true, f.back>;
    using N = FrameTile<f.frames, f.blocks, f.channels / 64, f.back, f.back>;      // of several groups all but the first have a frame in front
    return front ? TconvForm{C::kLdsBytes, tconv_frames<C>} : TconvForm{N::kLdsBytes, tconv_frames<N>};
}
const TconvForm kFrameForms[kTconvForms - kFrames3][2] = {{frame_form_of<kFrames3>(false), frame_form_of<kFrames3>(true)},
                                                          {frame_form_of<kFrames5>(false), frame_form_of<kFrames5>(true)},
                                                          {frame_form_of<kFrames7>(false), frame_form_of<kFrames7>(true)}};

// The measurement variants of the 256 x 256 kernel (sv_measure_tconv_variant; 0: the kernel itself).
constexpr int kVariants = 4;
const TconvKernel kVariantKernels[kVariants] = {tconv_mfma<TcTile<256, 256>>, tconv_mfma<TcTile<256, 256>, 1>,
                                                tconv_mfma<TcTile<256, 256>, 2>, tconv_mfma<TcTile<256, 256>, 3>};
constexpr int kByRule = -1;        // "variant" of the library's own calls: the form that tconv_form chooses

// Compute units of the current device; 0 on failure.  The kernels need their dynamic LDS allowed once per device.
int tconv_ready()
{
    static int num_cu[64] = {};
    static std::mutex mu;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    std::lock_guard<std::mutex> lock(mu);
    if (num_cu[dev] <= 0) {
        auto allow = [](TconvKernel k, int lds) {
            return hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, lds) == hipSuccess;
        };
        for (const TconvForm &f : kForms)
            if (!allow(f.kernel, f.lds)) return 0;
        for (const auto &forms : kFrameForms)
            for (const TconvForm &f : forms)
                if (!allow(f.kernel, f.lds)) return 0;
        for (const TconvKernel k : kVariantKernels)
            if (!allow(k, kForms[kForm256].lds)) return 0;
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        num_cu[dev] = n;
    }
    return num_cu[dev];
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
    if (variant > 0 && D % kTcBK != 0) return SV_ERR_UNSUPPORTED;
    const int num_cu = tconv_ready();
    if (num_cu <= 0) return SV_ERR_LAUNCH;

    TconvArgs a;
    a.x = static_cast<const uint16_t *>(x);
    a.W = static_cast<const uint16_t *>(W);
    a.cache = static_cast<const uint16_t *>(cache_in);
    a.y = static_cast<uint16_t *>(y);
    a.B = B; a.T = T; a.HW = HW; a.D = D;
    const TconvFormId id = variant == kByRule ? tconv_form(B, T, HW, D, cache_in != nullptr, num_cu) : kForm256;
    const TconvForm &f = id >= kFrames3 ? kFrameForms[id - kFrames3][cache_in != nullptr] : kForms[id + (id == kForm256Long && D % kTcBK != 0)];
    const int64_t tiles_m = tconv_tiles_m(id, B, T, HW);
    a.tiles_m = (int)tiles_m;
    a.tiles_n = tconv_tiles_n(id, D);
    const int64_t wgs = tc_grid_size(tiles_m * a.tiles_n);
    if (wgs >= (int64_t)1 << 31) return SV_ERR_SHAPE;
    auto hs = static_cast<hipStream_t>(stream);
    const TconvKernel kernel = variant == kByRule ? f.kernel : kVariantKernels[variant];
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
    return tconv_enqueue(kByRule, x, W, cache_in, y, cache_out, B, T, HW, D, dtype, stream);
}

extern "C" sv_status sv_measure_tconv_variant(int32_t variant, const void *x, const void *W, const void *cache_in, void *y,
                                              int32_t B, int32_t T, int32_t HW, int32_t D, void *stream)
{
    if (variant < 0 || variant >= kVariants) return SV_ERR_RANGE;
    return tconv_enqueue(variant, x, W, cache_in, y, nullptr, B, T, HW, D, SV_BF16, stream);
}
