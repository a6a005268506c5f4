// Test-time register construction (Algorithm 1, "redirect sinks to r"; Appendix
// Eq. register_redirect_appendix): for each listed MLP channel k of the vision
// encoder, the register row of a sample takes the max of channel k over the
// sample's visual rows, and the visual rows' values of channel k become 0.
//
// register_redirect  grid (listed channel, sample), one workgroup each, the channels of a
//                    sample on one XCD (some share the lines of its rows): its threads stride
//                    over the visual rows, eight 2- or 4-byte reads in flight per thread,
//                    and clear each element behind its read; a wave and an LDS reduction
//                    give the maximum, which thread 0 writes to the register.  A
//                    workgroup skips an index outside [0, width) and a repeat of an
//                    earlier list entry, so distinct workgroups never touch the same
//                    element.  A maximum of zero is written as +0.
//                    Bound by the lines touched (each element sits in a row of its own)
//                    and, with few of them in flight, by latency: one wave per (channel,
//                    sample) with one read in flight took 55 to 57 us for ten channels of the
//                    LLaVA-NeXT activation (32 x 2884 rows of 8 KB), this form 46 to 48 (inputs
//                    the caches do not hold).  With a sample's channels dealt over the XCDs 64
//                    channels of 32 x 581 rows took 54 us, on one XCD 38.
#include "occam_internal.hpp"

namespace occam {

template <bool BF16>
__device__ __forceinline__ float load_act(const char* p) {
    if (BF16) return __uint_as_float(static_cast<uint32_t>(*reinterpret_cast<const uint16_t*>(p)) << 16);
    return *reinterpret_cast<const float*>(p);
}
template <bool BF16>
__device__ __forceinline__ void store_act(char* p, float v) {
    // A value read from the tensor converts back exactly (bf16 -> f32 -> bf16).
    if (BF16) *reinterpret_cast<uint16_t*>(p) = static_cast<uint16_t>(__float_as_uint(v) >> 16);
    else *reinterpret_cast<float*>(p) = v;
}

template <bool BF16, int NT>
__global__ __launch_bounds__(NT) void register_redirect_kernel(
    Prob p, char* __restrict__ h, int width, long long stride, const int* __restrict__ channels,
    int reg_slot)
{
    __shared__ float red[NT / kWave];
    int j = blockIdx.x, b = blockIdx.y;                        // list entry, sample
    const int n = (int)gridDim.x;
    if (n * p.B >= kXcds * 32) {             // (fewer find a CU of their own, line or not)
        const int task = xcd_remap(b * n + j, n * p.B);
        j = task % n;
        b = task / n;
    }
    const int k = channels[j];
    int repeat = 0;
    for (int i = threadIdx.x; i < j; i += NT) repeat |= channels[i] == k;
    if (__syncthreads_or(repeat) || k < 0 || k >= width) return;   // a repeat acts once
    const int N = keys_of(p, b) - p.R;
    if (N <= 0) return;
    constexpr int E = BF16 ? 2 : 4, U = 8;
    char* base = h + (long long)k_begin(p, b) * stride + (long long)k * E;
    char* vis = base + (long long)p.R * stride;
    float m = -INFINITY;
    for (int v0 = threadIdx.x; v0 < N; v0 += U * NT) {
        float x[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            x[u] = v0 + u * NT < N ? load_act<BF16>(vis + (long long)(v0 + u * NT) * stride) : -INFINITY;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            m = fmaxf(m, x[u]);
            if (v0 + u * NT < N) store_act<BF16>(vis + (long long)(v0 + u * NT) * stride, 0.f);
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x != 0) return;
#pragma unroll
    for (int w = 1; w < NT / kWave; ++w) m = fmaxf(m, red[w]);
    if (m == 0.f) m = 0.f;                                     // +0 for a zero maximum
    store_act<BF16>(base + (long long)reg_slot * stride, m);
}

template <bool BF16>
static hipError_t redirect(const Prob& p, char* h, int width, long long stride,
                           const int* channels, int n_channels, int reg_slot, hipStream_t s) {
    const dim3 grid(n_channels, p.B);
    // Threads for about one read per row and round; more of them idle on short samples, fewer
    // hold too few reads.  64 channels of 32 x 577 rows, 256 / 512 / 1024 threads: 44, 37 and
    // 38 us; 10 of 16 x 1024 9.1, 9.3 and 9.3; 30 of 32 x 1100 43, 43 and 40; 64 of 64 x 64
    // 10, 10 and 23.
    if (p.max_cands > 1024)
        return launch(register_redirect_kernel<BF16, 1024>, grid, dim3(1024), 0, s, p, h, width,
                      stride, channels, reg_slot);
    if (p.max_cands > 512 && (long long)p.B * n_channels >= 512)
        return launch(register_redirect_kernel<BF16, 512>, grid, dim3(512), 0, s, p, h, width,
                      stride, channels, reg_slot);
    return launch(register_redirect_kernel<BF16, 256>, grid, dim3(256), 0, s, p, h, width, stride,
                  channels, reg_slot);
}

hipError_t launch_register_redirect(const Prob& p, int bf16, void* h, int width, long long stride,
                                    const int* channels, int n_channels, int reg_slot,
                                    hipStream_t s)
{
    if (n_channels == 0) return hipSuccess;
    char* hc = static_cast<char*>(h);
    return bf16 ? redirect<true>(p, hc, width, stride, channels, n_channels, reg_slot, s)
                : redirect<false>(p, hc, width, stride, channels, n_channels, reg_slot, s);
}

}  // namespace occam
