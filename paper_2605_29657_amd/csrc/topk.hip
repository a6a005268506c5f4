// Fixed-budget selection, the component ablation's alternative to the relative test
// (Appendix, Table tab:qwen_compact_component_ablation): per sample, the K visual tokens
// with the largest scores, the lower index first among equal scores.
//
// select_topk   one workgroup per sample.  The float-ordered score keys of a sample of up to
//               kTopkLds candidates are kept in LDS (longer ones are formed again from the
//               scores in every pass).  A radix select over them (8 bits per pass from the
//               top, LDS histogram, a scan over the first four waves picks the digit) finds
//               the K-th largest key t and how many keys equal to t are kept (q).  Every
//               wave then owns a contiguous range of candidates and walks it 64 at a time:
//               ballots count the keys above and equal to t, scans of the wave totals give
//               each wave its share of the equal keys (the first q in index order) and its
//               output position, and a second walk writes the survivors in ascending order
//               into the same per-sample slot list that the threshold selection fills, so
//               the packing and the gathers are shared with it.
//               Bound by latency (16 KB per sample): 64 samples of 256-4096 candidates took
//               21.5 us with 256 threads that read the scores from memory in each of six
//               walks, 10.8 us now.
#include "occam_internal.hpp"

namespace occam {

constexpr int kTopkThreads = 1024, kTopkWaves = kTopkThreads / kWave;
constexpr int kTopkLds = 12288;                          // keys held in LDS (48 KB)
constexpr int kTopkCopies = 4, kTopkStride = 256 + 16;   // histogram copies on different banks

// Sum of x over the waves before this one; `total` gets the sum over all.  x is uniform in
// a wave.  wsum: kTopkWaves ints of LDS.
__device__ __forceinline__ int waves_before(int x, int* wsum, int& total) {
    const int wave = threadIdx.x >> 6;
    __syncthreads();                              // wsum is free
    if ((threadIdx.x & 63) == 0) wsum[wave] = x;
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kTopkWaves; ++w) {
        before += w < wave ? wsum[w] : 0;
        total += wsum[w];
    }
    return before;
}
__device__ __forceinline__ int below_lane(unsigned long long m) {
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                          __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

__global__ __launch_bounds__(kTopkThreads) void select_topk_kernel(
    Prob p, const float* __restrict__ scores, int k_keep, int* __restrict__ slot,
    int* __restrict__ count)
{
    __shared__ uint32_t held[kTopkLds];
    __shared__ uint32_t hist[kTopkCopies * kTopkStride];
    __shared__ uint32_t wave_sum[4];
    __shared__ uint32_t sh_prefix, sh_rank;
    __shared__ int wsum[kTopkWaves];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int N = keys_of(p, b) - p.R;
    const int co = cand_begin(p, b);
    const float* sv = scores + k_begin(p, b) + p.R;
    const int K = min(k_keep, N);
    if (tid == 0) count[b] = K;
    if (K == 0) return;
    const bool in_lds = N <= kTopkLds;
    if (in_lds)
        for (int v = tid; v < N; v += kTopkThreads) held[v] = order_key(sv[v]);
    auto key_of = [&](int v) { return in_lds ? held[v] : order_key(sv[v]); };

    // The K-th largest key t and the rank q of the target among the keys equal to t.
    uint32_t prefix = 0, mask = 0, rank = (uint32_t)K;
    uint32_t* mine = hist + (tid % kTopkCopies) * kTopkStride;
    for (int shift = 24; shift >= 0; shift -= 8) {
        for (int i = tid; i < kTopkCopies * kTopkStride; i += kTopkThreads) hist[i] = 0;
        __syncthreads();
        for (int v = tid; v < N; v += kTopkThreads) {
            const uint32_t key = key_of(v);
            if ((key & mask) == prefix) atomicAdd(&mine[(key >> shift) & 255u], 1u);
        }
        __syncthreads();
        // Thread t of the first four waves holds digit 255 - t: the number of keys with a
        // digit at or above its own is a prefix sum over threads.
        uint32_t n = 0, inc = 0;
        if (tid < 256) {
#pragma unroll
            for (int c = 0; c < kTopkCopies; ++c) n += hist[c * kTopkStride + 255 - tid];
            inc = n;
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const uint32_t o = __shfl_up(inc, off);
                if (lane >= off) inc += o;
            }
            if (lane == 63) wave_sum[wave] = inc;
        }
        __syncthreads();
        if (tid < 256) {
            for (int w = 0; w < wave; ++w) inc += wave_sum[w];
            if (inc - n < rank && rank <= inc) {
                sh_prefix = prefix | ((uint32_t)(255 - tid) << shift);
                sh_rank = rank - (inc - n);
            }
        }
        __syncthreads();
        prefix = sh_prefix;
        rank = sh_rank;
        mask |= 255u << shift;
    }
    const uint32_t t = prefix;
    const int q = (int)rank;                      // keys equal to t that are kept

    // Contiguous ranges per wave: counts above t and equal to t, then positions.
    const int Q = ((N + kTopkWaves - 1) / kTopkWaves + kWave - 1) & ~(kWave - 1);
    const int v0 = min(N, wave * Q), v1 = min(N, v0 + Q);
    int gt = 0, eq = 0;
    for (int vb = v0; vb < v1; vb += kWave) {
        const uint32_t key = vb + lane < v1 ? key_of(vb + lane) : 0u;
        gt += (int)__popcll(__ballot(vb + lane < v1 && key > t));
        eq += (int)__popcll(__ballot(vb + lane < v1 && key == t));
    }
    int total;
    const int eq_before = waves_before(eq, wsum, total);
    int eq_left = min(max(q - eq_before, 0), eq);
    int pos = waves_before(gt + eq_left, wsum, total);
    for (int vb = v0; vb < v1; vb += kWave) {
        const bool in = vb + lane < v1;
        const uint32_t key = in ? key_of(vb + lane) : 0u;
        const unsigned long long me = __ballot(in && key == t);
        const bool keep = in && (key > t || (key == t && below_lane(me) < eq_left));
        const unsigned long long mk = __ballot(keep);
        if (keep) slot[co + pos + below_lane(mk)] = vb + lane;
        pos += (int)__popcll(mk);
        eq_left = max(0, eq_left - (int)__popcll(me));
    }
}

hipError_t launch_select_topk(const Prob& p, const float* scores, int k_keep, int* slot,
                              int* count, hipStream_t s)
{
    return launch(select_topk_kernel, dim3(p.B), dim3(kTopkThreads), 0, s, p, scores, k_keep, slot,
                  count);
}

}  // namespace occam
