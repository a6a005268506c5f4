// Budget matching (Appendix Eq. lambda2_budget_matching_appendix) on the device: the
// lambda whose mean kept count over the batch is closest to a target.
//
// The count #{v : s_b(v) >= lambda s_b(r)} summed over samples is a step function of
// lambda that drops at each ratio s_b(v) / s_b(r).  With T = k_target * B and
// c = T rounded half down (clamped to [1, M], M candidates), the best level is either
// the level of the c-th largest ratio v1 (count #{r >= v1}) or the level just above it
// (count #{r > v1}, value = the smallest ratio above v1): every other level's count is
// farther from T.  Ties take the smaller count.  lambda is the geometric midpoint of
// the chosen level's value and the next smaller distinct ratio (half the value if
// there is no positive one; 0 if the level itself is not positive).
//
// Ratios are mapped to unsigned keys that order like the floats, and the c-th largest
// key is found by a radix select, 8 bits per pass from the top:
//   match_init   one workgroup: clears the selection state, counts M, sets c.
//   match_hist   grid (B, candidate chunks of 4096): the first pass forms the keys and
//                leaves them in the workspace; every pass takes an LDS histogram of its
//                digit over the keys that match the prefix chosen so far, added into one
//                global histogram; the last workgroup to finish picks the digit and
//                the rank left inside it.
//   match_count  same grid: #{key >= v1}, #{key > v1}, the nearest keys above and
//                below v1; the last workgroup chooses the level and writes lambda.
// The first pass's workgroups form their sample's reference (s_b(r), or the mean visual
// score of the ablation) with the same reduction as the threshold kernels.
//
// Every pass moves under a megabyte at calibration sizes, so it is bound by latency: the
// loads, the atomics (the top digit of a batch's ratios takes two or three values, so
// they meet on a few addresses: 1024-thread workgroups add once per bin for 4096 keys, and
// an LDS bin has eight copies on different banks) and the hand-over to the last workgroup
// (relaxed device-scope atomics behind a wait, no cache-wide fence).  64 samples of 2880
// candidates: 90.3 us in six launches with 256-thread workgroups, fences and the keys
// formed in every pass, 29.0 us now.
#include "occam_internal.hpp"

namespace occam {

constexpr int kMatchThreads = 1024;
constexpr int kMatchCopies = 8, kMatchStride = 256 + 8;   // LDS histogram copies
constexpr int kMatchPer = 4;                              // keys per thread per chunk
constexpr int kMatchChunk = kMatchThreads * kMatchPer;

struct MatchState {
    uint32_t hist[4][256];
    uint32_t prefix[4];       // key bits chosen up to and including pass i
    uint32_t rank[5];         // rank of the target inside the prefix group (rank[0] = c)
    uint32_t done[5];         // finished workgroups per pass (4 histograms + count)
    uint32_t M;
    uint32_t c_hi, c_lo, v_above, v_below;
};
static_assert(sizeof(MatchState) <= kMatchStateBytes, "match state exceeds its workspace");

__device__ __forceinline__ uint32_t load_cc(const uint32_t* a) {  // coherent across workgroups
    return __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The chunk's keys: out-of-range slots get `valid` cleared.  FORM: from the scores, left in
// keys[b * max_cands + v]; otherwise read from there.
struct ChunkKeys {
    uint32_t key[kMatchPer];
    bool valid[kMatchPer];
};
template <bool FORM>
__device__ __forceinline__ ChunkKeys chunk_keys(const Prob& p, const float* scores, int reduce,
                                                uint32_t* keys) {
    __shared__ float red[kSelThreads / kWave];
    const int b = blockIdx.x;
    const int N = keys_of(p, b) - p.R;
    uint32_t* kb = keys + (size_t)b * p.max_cands;
    ChunkKeys ck;
    if (FORM) {
        const float* sv = scores + k_begin(p, b) + p.R;
        float x[kMatchPer];
#pragma unroll
        for (int j = 0; j < kMatchPer; ++j) {
            const int v = blockIdx.y * kMatchChunk + j * kMatchThreads + threadIdx.x;
            x[j] = v < N ? sv[v] : 0.f;
        }
        // The reference sum runs in the order of kSelThreads threads: occam_threshold's bits.
        const float sr = sample_reference<kSelThreads>(p, scores, b, reduce, red);
#pragma unroll
        for (int j = 0; j < kMatchPer; ++j) {
            const int v = blockIdx.y * kMatchChunk + j * kMatchThreads + threadIdx.x;
            ck.valid[j] = v < N;
            ck.key[j] = ck.valid[j] ? order_key(x[j] / sr) : 0u;
            if (ck.valid[j]) kb[v] = ck.key[j];
        }
        return ck;
    }
#pragma unroll
    for (int j = 0; j < kMatchPer; ++j) {
        const int v = blockIdx.y * kMatchChunk + j * kMatchThreads + threadIdx.x;
        ck.valid[j] = v < N;
        ck.key[j] = ck.valid[j] ? kb[v] : 0u;
    }
    return ck;
}

// True in every thread of the workgroup that finished last among the grid.  The values
// handed over are device-scope atomics: each wave waits until its own have completed.
__device__ __forceinline__ bool last_workgroup(uint32_t* done) {
    __shared__ bool last;
    __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0)
    __syncthreads();
    if (threadIdx.x == 0)
        last = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
               gridDim.x * gridDim.y - 1;
    __syncthreads();
    return last;
}

// Relaxed device-scope atomics (performed where every XCD sees them).
__device__ __forceinline__ void add_cc(uint32_t* a, uint32_t v) {
    __hip_atomic_fetch_add(a, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(kMatchThreads) void match_init_kernel(Prob p, float k_target,
                                                                   MatchState* st)
{
    __shared__ uint32_t m_sh;
    const int tid = threadIdx.x;
    uint32_t* w = reinterpret_cast<uint32_t*>(st);
    for (int i = tid; i < (int)(sizeof(MatchState) / 4); i += kMatchThreads) w[i] = 0u;
    if (tid == 0) m_sh = 0;
    __syncthreads();
    uint32_t m = 0;
    for (int b = tid; b < p.B; b += kMatchThreads) m += (uint32_t)(keys_of(p, b) - p.R);
    atomicAdd(&m_sh, m);
    __syncthreads();
    if (tid == 0) {
        const uint32_t M = m_sh;
        double c = ceil((double)k_target * (double)p.B - 0.5);   // T rounded half down
        c = c < 1.0 ? 1.0 : (c > (double)M ? (double)M : c);
        st->M = M;
        st->rank[0] = (uint32_t)c;
        st->v_above = 0xFFFFFFFFu;
    }
}

template <int PASS>
__global__ __launch_bounds__(kMatchThreads) void match_hist_kernel(
    Prob p, const float* __restrict__ scores, int reduce, uint32_t* __restrict__ keys, MatchState* st)
{
    __shared__ uint32_t hist[kMatchCopies * kMatchStride];
    __shared__ uint32_t wave_sum[4];
    constexpr int shift = 24 - 8 * PASS;
    const int tid = threadIdx.x;
    for (int i = tid; i < kMatchCopies * kMatchStride; i += kMatchThreads) hist[i] = 0;
    const uint32_t mask = PASS == 0 ? 0u : ~0u << (32 - 8 * PASS);
    const uint32_t prefix = PASS == 0 ? 0u : st->prefix[PASS - 1];
    __syncthreads();
    const ChunkKeys ck = chunk_keys<PASS == 0>(p, scores, reduce, keys);
    uint32_t* mine = hist + (tid % kMatchCopies) * kMatchStride;
#pragma unroll
    for (int j = 0; j < kMatchPer; ++j)
        if (ck.valid[j] && (ck.key[j] & mask) == prefix)
            atomicAdd(&mine[(ck.key[j] >> shift) & 255u], 1u);
    __syncthreads();
    if (tid < 256) {
        uint32_t n = 0;
#pragma unroll
        for (int c = 0; c < kMatchCopies; ++c) n += hist[c * kMatchStride + tid];
        if (n) add_cc(&st->hist[PASS][tid], n);
    }
    if (!last_workgroup(&st->done[PASS])) return;

    // Pick the digit: suffix(d) = keys in the group with digit >= d; the target of rank
    // k (1 = largest) has the digit d with suffix(d + 1) < k <= suffix(d).  Thread t of the
    // first four waves holds digit 255 - t, so that its suffix is a prefix over threads.
    const uint32_t k = load_cc(&st->rank[PASS]);
    const uint32_t n = tid < 256 ? load_cc(&st->hist[PASS][255 - tid]) : 0u;
    uint32_t inc = n;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t o = __shfl_up(inc, off);
        if ((tid & 63) >= off) inc += o;
    }
    if (tid < 256 && (tid & 63) == 63) wave_sum[tid >> 6] = inc;
    __syncthreads();
    if (tid >= 256) return;
    for (int w = 0; w < (tid >> 6); ++w) inc += wave_sum[w];
    if (inc - n < k && k <= inc) {
        st->prefix[PASS] = prefix | ((uint32_t)(255 - tid) << shift);
        st->rank[PASS + 1] = k - (inc - n);
    }
}

__global__ __launch_bounds__(kMatchThreads) void match_count_kernel(
    Prob p, uint32_t* __restrict__ keys, float k_target, MatchState* st,
    float* __restrict__ lambda, float* __restrict__ mean_kept)
{
    __shared__ uint32_t s_hi, s_lo, s_above, s_below;
    const int tid = threadIdx.x;
    if (tid == 0) { s_hi = 0; s_lo = 0; s_above = 0xFFFFFFFFu; s_below = 0u; }
    const uint32_t v1 = st->prefix[3];
    __syncthreads();
    const ChunkKeys ck = chunk_keys<false>(p, nullptr, 0, keys);
    uint32_t hi = 0, lo = 0, above = 0xFFFFFFFFu, below = 0u;    // below holds key + 1
#pragma unroll
    for (int j = 0; j < kMatchPer; ++j) {
        if (!ck.valid[j]) continue;
        const uint32_t key = ck.key[j];
        hi += key >= v1;
        lo += key > v1;
        if (key > v1) above = min(above, key);
        if (key < v1) below = max(below, key + 1u);
    }
    // One LDS atomic per wave.
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        hi += __shfl_xor(hi, off);
        lo += __shfl_xor(lo, off);
        above = min(above, (uint32_t)__shfl_xor(above, off));
        below = max(below, (uint32_t)__shfl_xor(below, off));
    }
    if ((tid & 63) == 0) {
        if (hi) atomicAdd(&s_hi, hi);
        if (lo) atomicAdd(&s_lo, lo);
        if (above != 0xFFFFFFFFu) atomicMin(&s_above, above);
        if (below) atomicMax(&s_below, below);
    }
    __syncthreads();
    if (tid == 0) {
        if (s_hi) add_cc(&st->c_hi, s_hi);
        if (s_lo) add_cc(&st->c_lo, s_lo);
        if (s_above != 0xFFFFFFFFu)
            __hip_atomic_fetch_min(&st->v_above, s_above, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (s_below)
            __hip_atomic_fetch_max(&st->v_below, s_below, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!last_workgroup(&st->done[4]) || tid != 0) return;

    const uint32_t M = load_cc(&st->M);
    if (M == 0) {                                  // no candidates: nothing to match
        lambda[0] = 1.f;
        if (mean_kept) mean_kept[0] = 0.f;
        return;
    }
    const uint32_t c_hi = load_cc(&st->c_hi), c_lo = load_cc(&st->c_lo);
    const uint32_t v_above = load_cc(&st->v_above), v_below = load_cc(&st->v_below);
    const double T = (double)k_target * (double)p.B;
    uint32_t level, count;
    bool has_next;
    uint32_t next;
    if (c_lo >= 1 && fabs((double)c_lo - T) <= fabs((double)c_hi - T)) {
        level = v_above; count = c_lo; has_next = true; next = v1;
    } else {
        level = v1; count = c_hi; has_next = v_below != 0u; next = v_below - 1u;
    }
    const double lv = (double)key_value(level);
    const double nv = has_next ? (double)key_value(next) : 0.0;
    const double lam = (lv > 0.0 && nv > 0.0) ? sqrt(lv * nv) : (lv > 0.0 ? 0.5 * lv : 0.0);
    lambda[0] = (float)lam;
    if (mean_kept) mean_kept[0] = (float)((double)count / (double)p.B);
}

hipError_t launch_match_lambda(const Prob& p, const float* scores, int reduce, float k_target,
                               void* state, void* keys, float* lambda, float* mean_kept, hipStream_t s)
{
    MatchState* st = static_cast<MatchState*>(state);
    uint32_t* kk = static_cast<uint32_t*>(keys);
    const int chunks = (p.max_cands + kMatchChunk - 1) / kMatchChunk;
    const dim3 grid(p.B, chunks > 0 ? chunks : 1);
    const dim3 block(kMatchThreads);
    hipError_t e = launch(match_init_kernel, dim3(1), block, 0, s, p, k_target, st);
    if (e != hipSuccess) return e;
    if (chunks > 0) {
        if ((e = launch(match_hist_kernel<0>, grid, block, 0, s, p, scores, reduce, kk, st)) != hipSuccess ||
            (e = launch(match_hist_kernel<1>, grid, block, 0, s, p, scores, reduce, kk, st)) != hipSuccess ||
            (e = launch(match_hist_kernel<2>, grid, block, 0, s, p, scores, reduce, kk, st)) != hipSuccess ||
            (e = launch(match_hist_kernel<3>, grid, block, 0, s, p, scores, reduce, kk, st)) != hipSuccess)
            return e;
    }
    return launch(match_count_kernel, grid, block, 0, s, p, kk, k_target, st, lambda,
                  mean_kept);
}

}  // namespace occam
