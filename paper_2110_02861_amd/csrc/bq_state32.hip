// Optimizer step with 32-bit states, for tensors whose states stay in fp32
// (Section 3.3: the embedding layer keeps 32-bit optimizer states).  The same
// update as the 8-bit step (Eq. 1, Eq. 2, AdamW, AdaGrad) without quantization: the
// states m, r are fp32 arrays updated in place.  One 256-thread workgroup per
// tile of 1024 elements, 4 contiguous elements per thread; the workgroup finds
// its tensor by a binary search over the launch's descriptors.
#include "bq_device.h"

namespace bq {
namespace {

using namespace dev;

constexpr int kThreads32 = 256;
constexpr int kTile32 = kThreads32 * 4;

// How a launch streams.  HBM bounds the step (26 B per param for Adam with fp16
// grads), but a launch whose arrays the memory-side cache (256 MB) holds reads and
// writes them there, and stores by st_stream, which go on to HBM, cost it up to
// 40 %.  For longer ones they are the faster, and so are fewer workgroups than the
// 8 per CU that fit by registers, whose 4 input and 3 output streams get in each
// other's way: a launch then asks for LDS that it does not use, 52 or 32 KB of a
// CU's 160 (3 or 5 workgroups per CU).  Medians of 7 interleaved rounds of HIP
// graphs, us (st_nt, 8 per CU | st_stream, 5 per CU | st_stream, 3 per CU):
//   params (10^6)     Adam, fp16 grads     momentum, fp16       momentum, fp32
//     1               4.29  5.34  6.04     3.39  4.48  4.78     3.38  4.39  4.75
//     3               11.9  13.2  13.2     8.17  9.44  9.76     8.40  9.50  9.68
//     5               21.3  20.6  20.4     13.7  14.2  14.9     15.3  14.5  14.9
//     8               34.5  31.5  31.1     23.2  21.7  22.5     24.4  24.7  24.9
//    20               84.3  85.6  84.6     56.7  55.7  57.6     61.8  64.3  63.8
//    40                184   174   161      113   111   113      129   130   127
//    80                361   336   327      231   227   234      266   252   247
//   160                718   705   693      460   443   461      526   512   531
// (Adam with fp32 grads: as with fp16.  AdaGrad: as momentum.)
struct Streaming {
    bool stream;   // st_stream stores
    unsigned lds;  // bytes asked for
};
constexpr Streaming streaming(bool two_states, int grad, int tiles)
{
    if (two_states)
        return tiles >= 4096 ? Streaming{true, 52 * 1024} : Streaming{false, 0};
    if (grad != kF32)
        return tiles >= 6144 ? Streaming{true, 32 * 1024} : Streaming{false, 0};
    return tiles >= 32768 ? Streaming{true, 52 * 1024} : Streaming{false, 0};
}

template <int OPT, int GRAD, bool STREAM>
__global__ __launch_bounds__(kThreads32) void step32_kernel(const State32Args a)
{
    // tensor of this tile: the last descriptor with tile_begin <= tile
    const int tile = blockIdx.x;
    int lo = 0, hi = a.ntensors - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.d[mid].tile_begin <= tile)
            lo = mid;
        else
            hi = mid - 1;
    }
    const Desc32 &D = a.d[lo];
    const int64_t t0 = (int64_t)(tile - D.tile_begin) * kTile32;
    const int64_t e0 = t0 + threadIdx.x * 4;
    if (e0 >= D.numel)
        return;
    const int nv = D.numel - e0 >= 4 ? 4 : (int)(D.numel - e0);
    constexpr bool kTwo = has_two_states(OPT);
    const StepScalars &sc = a.sc;

    float w[4], g[4], m[4], v[4];
    if (nv == 4) {
        const vf4 wv = ld_nt(reinterpret_cast<const vf4 *>(D.param + e0));
        const vf4 mv = ld_nt(reinterpret_cast<const vf4 *>(D.m + e0));
        w[0] = wv.x; w[1] = wv.y; w[2] = wv.z; w[3] = wv.w;
        m[0] = mv.x; m[1] = mv.y; m[2] = mv.z; m[3] = mv.w;
        if constexpr (kTwo) {
            const vf4 vv = ld_nt(reinterpret_cast<const vf4 *>(D.v + e0));
            v[0] = vv.x; v[1] = vv.y; v[2] = vv.z; v[3] = vv.w;
        }
        if constexpr (GRAD != kF32) {
            const vu2 gv = ld_nt(reinterpret_cast<const vu2 *>(
                static_cast<const uint16_t *>(D.grad) + e0));
            g[0] = g16_lo<GRAD>(gv.x); g[1] = g16_hi<GRAD>(gv.x);
            g[2] = g16_lo<GRAD>(gv.y); g[3] = g16_hi<GRAD>(gv.y);
        } else {
            const vf4 gv =
                ld_nt(reinterpret_cast<const vf4 *>(static_cast<const float *>(D.grad) + e0));
            g[0] = gv.x; g[1] = gv.y; g[2] = gv.z; g[3] = gv.w;
        }
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool ok = r < nv;
            w[r] = ok ? G(D.param)[e0 + r] : 0.0f;
            m[r] = ok ? G(D.m)[e0 + r] : 0.0f;
            v[r] = (kTwo && ok) ? G(D.v)[e0 + r] : 0.0f;
            g[r] = ok ? grad_at<GRAD>(D.grad, e0 + r) : 0.0f;
        }
    }

#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float gi = g[r];
        if (a.use_wd)
            gi = gi + sc.wd * w[r];
        if constexpr (OPT == kMomentum) {
            m[r] = sc.b1 * m[r] + gi;
            w[r] = w[r] - sc.lr * m[r];
        } else if constexpr (OPT == kAdaGrad) {
            m[r] = m[r] + gi * gi;
            const float denom =
                __builtin_fmaf(__builtin_amdgcn_sqrtf(m[r]), sc.sdiv_c, sc.sdiv_eps);
            w[r] = __builtin_fmaf(-gi, __builtin_amdgcn_rcpf(denom), w[r]);
        } else {
            if constexpr (OPT == kAdamW)
                w[r] = w[r] * sc.decay;
            m[r] = sc.b1 * m[r] + sc.omb1 * gi;
            v[r] = sc.b2 * v[r] + sc.omb2 * (gi * gi);
            const float denom =
                __builtin_fmaf(__builtin_amdgcn_sqrtf(v[r]), sc.sdiv_c, sc.sdiv_eps);
            w[r] = __builtin_fmaf(-m[r], __builtin_amdgcn_rcpf(denom), w[r]);
        }
    }

    if (nv == 4) {
        const auto store = [&](float *p, const float (&x)[4]) {
            const vf4 v4 = {x[0], x[1], x[2], x[3]};
            if constexpr (STREAM)
                st_stream(stream_range(p + t0, kTile32 * 4), threadIdx.x * 16, v4);
            else
                st_nt(reinterpret_cast<vf4 *>(p + e0), v4);
        };
        store(D.param, w);
        store(D.m, m);
        if constexpr (kTwo)
            store(D.v, v);
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (r < nv) {
                G(D.param)[e0 + r] = w[r];
                G(D.m)[e0 + r] = m[r];
                if constexpr (kTwo)
                    G(D.v)[e0 + r] = v[r];
            }
        }
    }
}

template <int OPT, int GRAD>
hipError_t launch32(const State32Args &a, hipStream_t stream)
{
    const dim3 grid((unsigned)a.total_tiles), block(kThreads32);
    const Streaming how = streaming(has_two_states(OPT), GRAD, a.total_tiles);
    if (how.stream)
        hipLaunchKernelGGL((step32_kernel<OPT, GRAD, true>), grid, block, how.lds, stream, a);
    else
        hipLaunchKernelGGL((step32_kernel<OPT, GRAD, false>), grid, block, how.lds, stream, a);
    return hipGetLastError();
}

template <int OPT>
hipError_t launch32_g(int grad_dtype, const State32Args &a, hipStream_t stream)
{
    if (grad_dtype == kF16)
        return launch32<OPT, kF16>(a, stream);
    if (grad_dtype == kBF16)
        return launch32<OPT, kBF16>(a, stream);
    return launch32<OPT, kF32>(a, stream);
}

}  // namespace

hipError_t launch_step32(int opt, int grad_dtype, const State32Args &a, hipStream_t stream)
{
    switch (opt) {
    case kAdam: return launch32_g<kAdam>(grad_dtype, a, stream);
    case kAdamW: return launch32_g<kAdamW>(grad_dtype, a, stream);
    case kMomentum: return launch32_g<kMomentum>(grad_dtype, a, stream);
    case kAdaGrad: return launch32_g<kAdaGrad>(grad_dtype, a, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace bq
