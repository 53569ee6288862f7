// The residual sum and RMSNorm of a row, a template that two sources instantiate:
// rowops.hip for the rounds, score.hip with the check of a forward's last norm.
// (The check's kernels beside the others made a cached-AR rollout of B 0.2%
// longer without being launched: kernels of a few microseconds feel where their
// code lies.)
#pragma once
#include <type_traits>

#include "common.h"
#include "launch.h"

namespace hbsjd {

// One 64-lane block per row. Lane l holds dims 4 l + 256 k .. + 3 for k < NV4,
// read as float4 (d is a multiple of 4; chunks past d are clamped on load and
// never stored). Bad is empty, or a volatile int32_t* (host memory) that takes a 1
// from a row whose squares sum to NaN or infinity: a pack, so that the launches of
// the rounds stay without the argument (0.3% of the same rollout).
template <typename T, int NV4, typename... Bad>
__global__ __launch_bounds__(64) void k_reduce_norm(const float* __restrict__ part, int splits,
                                                    int m_cap, float* __restrict__ h,
                                                    const int* nrows_dev,
                                                    const float* __restrict__ g, float eps, int d,
                                                    T* __restrict__ hb, Bad... bad) {
    constexpr int kSplitMax = 4;
    const int r = blockIdx.x, lane = threadIdx.x;
    if (r >= m_cap) return;
    // the row count first: the grid covers the capacity, and rows at or past
    // the count (most of them in the last rounds) load and store nothing.
    // Then one phase of loads: every split's partial (splits = 0: the
    // projection has already added its sum into h), the residual and the gain.
    const int nrows = *nrows_dev;
    if (r >= nrows) return;
    const int nv = d >> 2;
    float4 pz[kSplitMax][NV4], hv[NV4], gv[NV4];
#pragma unroll
    for (int k = 0; k < NV4; ++k) {
        const int c = min(lane + 64 * k, nv - 1);
        if (splits > 0) {
#pragma unroll
            for (int z = 0; z < kSplitMax; ++z) {
                const int zz = min(z, splits - 1);
                pz[z][k] = reinterpret_cast<const float4*>(part + ((size_t)zz * m_cap + r) * d)[c];
            }
        }
        hv[k] = reinterpret_cast<const float4*>(h + (size_t)r * d)[c];
        gv[k] = reinterpret_cast<const float4*>(g)[c];
    }
    float4 x[NV4];
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < NV4; ++k) {
        const bool in = lane + 64 * k < nv;
        if (splits > 0) {
            float4 acc = pz[0][k];
#pragma unroll
            for (int z = 1; z < kSplitMax; ++z)
                if (z < splits) {   // split order
                    acc.x += pz[z][k].x;
                    acc.y += pz[z][k].y;
                    acc.z += pz[z][k].z;
                    acc.w += pz[z][k].w;
                }
            x[k] = make_float4(hv[k].x + acc.x, hv[k].y + acc.y, hv[k].z + acc.z, hv[k].w + acc.w);
        } else {
            x[k] = hv[k];
        }
        if (in) {
            ss = fmaf(x[k].x, x[k].x, ss);
            ss = fmaf(x[k].y, x[k].y, ss);
            ss = fmaf(x[k].z, x[k].z, ss);
            ss = fmaf(x[k].w, x[k].w, ss);
        }
    }
    if (splits > 0) {
#pragma unroll
        for (int k = 0; k < NV4; ++k)
            if (lane + 64 * k < nv) reinterpret_cast<float4*>(h + (size_t)r * d)[lane + 64 * k] = x[k];
    }
    if (!hb) return;
    ss = wave_sum(ss);
    if constexpr (sizeof...(Bad) > 0)
        if (lane == 0 && !(ss < INFINITY)) ((*bad = 1), ...);
    const float rn = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
    for (int k = 0; k < NV4; ++k) {
        const int i = 4 * (lane + 64 * k);
        if (i < d) {
            Elem<T>::store(hb + (size_t)r * d + i + 0, (x[k].x * rn) * gv[k].x);
            Elem<T>::store(hb + (size_t)r * d + i + 1, (x[k].y * rn) * gv[k].y);
            Elem<T>::store(hb + (size_t)r * d + i + 2, (x[k].z * rn) * gv[k].z);
            Elem<T>::store(hb + (size_t)r * d + i + 3, (x[k].w * rn) * gv[k].w);
        }
    }
}

// launches it for a row width d; bad: nothing, or the check's flag
template <typename T, typename... Bad>
void reduce_norm_dispatch(const float* part, int splits, int m_cap, float* h, const int* nrows_dev,
                          const float* gain, float eps, int d, void* hb, hipStream_t s,
                          Bad... bad) {
    auto go = [&](auto nv4) {
        launch(k_reduce_norm<T, decltype(nv4)::value, Bad...>, dim3(m_cap), dim3(64), 0, s, part,
               splits, m_cap, h, nrows_dev, gain, eps, d, (T*)hb, bad...);
    };
    switch ((d + 255) / 256) {
        case 1: go(std::integral_constant<int, 1>{}); break;
        case 2: go(std::integral_constant<int, 2>{}); break;
        case 3: go(std::integral_constant<int, 3>{}); break;
        case 4: go(std::integral_constant<int, 4>{}); break;
        case 5: go(std::integral_constant<int, 5>{}); break;
        default: go(std::integral_constant<int, 6>{}); break;
    }
}

}  // namespace hbsjd
