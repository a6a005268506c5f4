// Internal definitions shared by the HIP kernels and the host entry points of
// liboccam (gfx950 / CDNA4, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <tuple>
#include <utility>

namespace occam {

// Launch `kernel` and return the status of this launch alone (hipLaunchKernel reports
// its own result; hipGetLastError would also report an unrelated earlier failure).
// The arguments are converted to the kernel's parameter types before their addresses
// are taken.
template <typename... KArgs, typename... Args>
inline hipError_t launch(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t smem,
                         hipStream_t s, Args&&... args) {
    static_assert(sizeof...(KArgs) == sizeof...(Args), "kernel argument count");
    std::tuple<KArgs...> vals(std::forward<Args>(args)...);
    return std::apply(
        [&](auto&... v) {
            void* ptrs[] = {static_cast<void*>(&v)...};
            return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, ptrs,
                                   smem, s);
        },
        vals);
}

// Raise the dynamic LDS limit of `kernel` to `bytes` on the current device, once per
// device: `done` holds one bit per device ordinal (0..63) whose call succeeded.  A
// failure is returned and the call is tried again next time.
inline hipError_t allow_lds(const void* kernel, int bytes, std::atomic<uint64_t>& done) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = (dev >= 0 && dev < 64) ? (uint64_t(1) << dev) : 0;
    if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess && bit) done.fetch_or(bit, std::memory_order_acq_rel);
    return e;
}

constexpr int kWave = 64;
constexpr int kMaxGridY = 65535;   // launch limit of grid.y (the sample index of several kernels)

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr float kLog2e = 1.4426950408889634f;

// Loads and stores of values that other workgroups of the same launch write or read
// (possibly on other XCDs, each with its own L2): device-coherent when CC, i.e. they
// bypass the non-coherent caches instead of needing a cache-wide write-back or
// invalidation.
template <bool CC, typename T>
__device__ __forceinline__ T ld(const T* p) {
    if constexpr (CC) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return *p;
}
template <typename T>
__device__ __forceinline__ void st_cc(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Problem view passed by value to every kernel.  Offsets are device pointers
// or null (uniform batch).
struct Prob {
    int B, H, Hkv, d, R;
    int rows, cands;          // uniform T and N (used when the offsets are null)
    const int* q_off;         // [B+1] prefix of T_b, or null
    const int* k_off;         // [B+1] prefix of R + N_b, or null
    int max_rows, max_cands;  // bounds of T_b and N_b
    float scale;              // softmax temperature of Eq. (1)
    int mean_rows;            // visual keys: mean over anchor rows (1) or max (0)
    int lse_splits;           // key ranges of the statistics pass (0 or 1: one)
    long long lse_stride;     // floats between the ranges' normaliser tables
};

__device__ __forceinline__ int q_begin(const Prob& p, int b) {
    return p.q_off ? p.q_off[b] : b * p.rows;
}
__device__ __forceinline__ int rows_of(const Prob& p, int b) {
    if (!p.q_off) return p.rows;
    int t = p.q_off[b + 1] - p.q_off[b];
    return t < p.max_rows ? t : p.max_rows;
}
__device__ __forceinline__ int k_begin(const Prob& p, int b) {
    return p.k_off ? p.k_off[b] : b * (p.R + p.cands);
}
// Keys of sample b (registers + visual), clamped to the launch bounds.
__device__ __forceinline__ int keys_of(const Prob& p, int b) {
    if (!p.k_off) return p.R + p.cands;
    int s = p.k_off[b + 1] - p.k_off[b];
    int hi = p.R + p.max_cands;
    s = s < hi ? s : hi;
    return s > p.R ? s : p.R;
}
// Visual tokens of the samples before b (indexes index_map and gather sources).
__device__ __forceinline__ int cand_begin(const Prob& p, int b) {
    return k_begin(p, b) - p.R * b;
}

// s_b(r): the register scores of one sample reduced by mean, max or sum.
template <bool CC = false>
__device__ __forceinline__ float reg_reduce(const float* s, int R, int reduce) {
    if (reduce == 1) {                     // OCCAM_REG_MAX
        float m = ld<CC>(s);
        for (int r = 1; r < R; ++r) m = fmaxf(m, ld<CC>(s + r));
        return m;
    }
    float acc = 0.f;
    for (int r = 0; r < R; ++r) acc += ld<CC>(s + r);
    return reduce == 0 ? acc / (float)R : acc;   // MEAN : SUM
}

constexpr int kRefCandMean = 3;            // OCCAM_REF_CAND_MEAN

// Reference score of one sample from its R + N scores s[0 .. R + N) (registers first),
// returned to every thread of a workgroup of at least NT threads (all of them must call
// it).  Register reductions read the R register scores; the candidate mean sums the visual
// scores in a fixed order (strided over the first NT threads, a fixed shuffle tree per
// wave, the waves in order; threads past NT take no part), so every kernel that calls it
// with the same NT gets the same bits, whatever its workgroup size and wherever the scores
// are held.  `red` is NT / 64 floats of LDS.
template <int NT, bool CC = false>
__device__ __forceinline__ float reference_of(const float* s, int R, int N, int reduce,
                                              float* red) {
    if (reduce != kRefCandMean) return reg_reduce<CC>(s, R, reduce);
    const float* sv = s + R;
    const bool part = threadIdx.x < NT;
    float acc = 0.f;
    if (part) {
        // Eight loads in flight per thread; the sum still runs over v in order.
        constexpr int U = 8;
        for (int v0 = threadIdx.x; v0 < N; v0 += U * NT) {
            float x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = v0 + u * NT < N ? ld<CC>(sv + v0 + u * NT) : 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (v0 + u * NT < N) acc += x[u];
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    __syncthreads();                          // `red` may still be read by a previous call
    if (part && (threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) sum += red[w];
    return N > 0 ? sum / (float)N : 0.f;
}

// The reference of sample b read from the packed score array.
template <int NT, bool CC = false>
__device__ __forceinline__ float sample_reference(const Prob& p, const float* scores, int b,
                                                  int reduce, float* red) {
    return reference_of<NT, CC>(scores + k_begin(p, b), p.R, keys_of(p, b) - p.R, reduce, red);
}

// Ascending compaction of a sample's survivors (sv[v] >= tau over its N visual scores)
// into out[i] and *count, by a workgroup of NT threads (all must call it).  Wave w owns the
// contiguous range [w*Q, w*Q + Q) of the candidates (Q a multiple of 64) and walks it 64
// candidates at a time: a ballot of the keep flags, its population count for the wave's
// total, and in the second pass mbcnt (the set bits below the lane) for each survivor's
// position; an LDS scan of the NT/64 wave totals places the waves' ranges.  The result
// does not depend on NT.  `wsum` is NT / 64 ints of LDS.
template <int NT>
__device__ __forceinline__ void compact_of(const float* sv, int N, float tau, int* out,
                                           int* count, int* wsum) {
    constexpr int NW = NT / kWave;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int Q = (((N + NW - 1) / NW) + kWave - 1) & ~(kWave - 1);
    const int v0 = min(N, wave * Q), v1 = min(N, v0 + Q);
    // Both walks load U groups of 64 candidates before testing them, so that U loads are in
    // flight per lane (the scores may sit in global memory); the groups are taken in order.
    constexpr int U = 8;
    int cnt = 0;
    for (int vb = v0; vb < v1; vb += U * kWave) {
        float x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = vb + u * kWave + lane;
            x[u] = v < v1 ? sv[v] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            cnt += __popcll(__ballot(vb + u * kWave + lane < v1 && x[u] >= tau));
    }
    __syncthreads();                          // `wsum` may still be read by a previous call
    if (lane == 0) wsum[wave] = cnt;
    __syncthreads();
    int base = 0, total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        base += w < wave ? wsum[w] : 0;
        total += wsum[w];
    }
    for (int vb = v0; vb < v1; vb += U * kWave) {
        float x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = vb + u * kWave + lane;
            x[u] = v < v1 ? sv[v] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = vb + u * kWave + lane;
            const bool keep = v < v1 && x[u] >= tau;
            const unsigned long long m = __ballot(keep);
            const int below = (int)__builtin_amdgcn_mbcnt_hi(
                (unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
            if (keep) out[base + below] = v;
            base += __popcll(m);
        }
    }
    if (threadIdx.x == 0) *count = total;
}

// The compaction of sample b from the packed score array into slot[co_b + i], count[b].
template <int NT>
__device__ __forceinline__ void compact_sample(const Prob& p, const float* scores, int b,
                                               float tau, int* slot, int* count, int* wsum) {
    compact_of<NT>(scores + k_begin(p, b) + p.R, keys_of(p, b) - p.R, tau,
                   slot + cand_begin(p, b), count + b, wsum);
}

// Floats as unsigned keys with the same order: -0 folds into +0, non-negative values
// set the top bit, negative values are bit-inverted.
__device__ __forceinline__ uint32_t order_key(float x) {
    const uint32_t u = x == 0.f ? 0u : __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_value(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// bf16 <-> f32 on raw 16-bit patterns.
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Row tensors gathered with the survivors (host struct occam_rows, by value).
constexpr int kMaxRowTensors = 8;
struct RowTensor {
    const char* src;
    char* dst;
    long long src_pad_rows, src_row0, src_stride, dst_stride, row_bytes;
};
struct RowTensors {
    RowTensor t[kMaxRowTensors];
    int n;
    int vec16;  // every pointer, stride and row length is a multiple of 16 bytes
};

// ---------------------------------------------------------------------------
// Tiling constants.
// Anchor (T = 1) path: VALU dot products, KPW keys per workgroup.
constexpr int kClsThreads = 256;
constexpr int kClsPartials = 8192;   // LDS floats of per-chunk partial dot products
// Text (T > 1) path: MFMA 32x32x16 bf16; statistics on blocks of 128 anchor rows (4 waves
// of 32), scoring on 32 keys per wave (score_form).
constexpr int kStatsThreads = 256;
constexpr int kTxtRows = 128;
constexpr int kTxtKeysPerWave = 32;
constexpr int kSelThreads = 256;    // threshold; the order of every reference sum
constexpr int kSelectThreads = 512; // the select kernel (its reference sum uses kSelThreads)
constexpr int kGatherThreads = 256;

// The chip dispatches consecutive workgroups of a launch round-robin over its 8
// XCDs, each with its own L2.  xcd_remap turns a linear workgroup id into a task
// index such that each XCD receives one contiguous range of tasks (XCD x gets
// ranges of q+1 tasks for x < r, q otherwise, with total = 8 q + r), so tasks that
// share data (the key chunks of one sample share its query tiles) meet in one L2.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_remap(int id, int total) {
    const int q = total / kXcds, r = total % kXcds;
    const int x = id % kXcds, j = id / kXcds;
    return x < r ? x * (q + 1) + j : r * (q + 1) + (x - r) * q + j;
}

// Forms of the text-row scoring kernel: waves per workgroup (32 keys each), anchor rows per
// workgroup, and whether the keys reach LDS before the registers.  LDS: two query tiles (rows
// x d bf16), the waves' keys and the [H][rows] float normaliser table; at most kScoreSmemMax.
constexpr size_t kScoreSmemMax = 160 * 1024;
struct ScoreForm {
    int waves, rows;
    bool keys_lds;
};
constexpr int kScoreNarrow = 0, kScoreWide = 1, kScoreTall = 2;
constexpr ScoreForm kScoreForms[] = {{4, 64, true}, {8, 128, true}, {4, 128, false}};
inline size_t score_smem(const ScoreForm& f, int H, int d16) {
    return (2 * (size_t)f.rows + (f.keys_lds ? (size_t)f.waves * kTxtKeysPerWave : 0)) * d16 * 2 +
           (size_t)H * f.rows * 4;
}
// The forms of 128 rows read the keys half as often as the narrow one; they want (nearly)
// whole row blocks, at most one 32-row sub-block past the rows, or one to six, and tasks for
// most CUs.  Row blocks that are not quite full (whole calls, 128-row form / narrow, 32 heads of 128
// unless said): 32 samples of 2880 keys x 100 rows 347 and 354 us, 8 of 4096 x 330 312 and
// 338, 1 of 4096 x 2000 255 and 268, 40 of 3000 x 80 406 and 440 (d = 96 345 and 385); past
// the line 16 of 4096 x 190 397 and 375.  Elsewhere the narrow form's finer tasks win: ragged
// grouped-query batch (64 samples of 256-4096 keys and 16-512 rows), scoring pass, narrow
// 427 us, wide 449, tall 470; one image (2880 keys x 128 rows) 47, 79 and 63.
// d > 112: wide, whose waves share a query tile among 256 keys (one workgroup per CU at 32
// heads).  Video batch (8 x 16384 keys x 256 rows, 1040 wide tasks) 465 us, narrow 549, tall
// 522; LLaVA-NeXT (384) 219, 221 and 220.  From 128 wide tasks narrow needs a second round of
// two workgroups per CU (whole calls, wide / narrow: 4 samples of 8000 keys x 128 rows, 128
// tasks, 159 and 145 us; 2 of 16384, 130, 158 and 181; 20 of 2880, 240, 213 and 242), and just
// past 256 the wide form's own second round is nearly empty (4 of 4096 x 512, 272, 258 and 240;
// with the caller's normaliser 174 and 158).
// With key offsets the tasks are counted by the bound max_cands, which a batch of mixed lengths fills about half, so the line lies higher.
// Whole call, samples of 64-1100 keys x 128 rows with the caller's normaliser, wide / narrow /
// tall: 40 samples (200 tasks by the bound) 103, 82 and 91 us; 52 (260) 106, 86 and 94; 64
// (320) 110, 138 and 133.
// d <= 112: tall.  A head has less matrix work, so what a head step costs beside it weighs
// more (the keys' way through LDS, fewer waves per SIMD beside the larger tiles).  Whole call,
// 32 samples of 2880 keys x 128 rows, tall / narrow / wide: d = 40 (8 heads) 65, 73 and 77 us;
// 64 (16) 114, 121 and 129; 80 (16) 142, 150 and 150; 96 (32) 302, 320 and 310; 112 (32) 347,
// 379 and 370.  From d = 72 wide is faster where its last round over the CUs is more than half
// full (d = 96, 32 heads, wide / tall: 13 samples, 156 tasks, 156 and 164 us; 24, 288, 281 and
// 264; 34, 408, 339 and 360; 42, 504, 378 and 404), and with key offsets above the same line
// as at d > 112 (64 samples of 256-4096 keys 407 and 422 us).
// Below a task of 128 x 128 per CU narrow is the faster one from d = 64 (one image: d = 64 46
// against 49, d = 96 68 against 82), at d = 40 the slower one (4 samples of 4096 keys: 45
// against 43).
inline long long score_tasks(const Prob& p, const ScoreForm& f) {
    const long long kpw = (long long)f.waves * kTxtKeysPerWave;
    return (long long)p.B * ((p.R + (long long)p.max_cands + kpw - 1) / kpw) *
           ((p.max_rows + f.rows - 1) / f.rows);
}
inline int score_form(const Prob& p) {
    const int d16 = (p.d + 15) / 16 * 16;
    constexpr int rows = kScoreForms[kScoreWide].rows;
    static_assert(rows == kScoreForms[kScoreTall].rows, "row blocks");
    const int subs = (p.rows + 31) / 32, idle = (p.rows + rows - 1) / rows * (rows / 32) - subs;
    if (p.q_off || (idle > 1 ? 6 * idle > subs : subs < 3)) return kScoreNarrow;
    const long long wide = score_tasks(p, kScoreForms[kScoreWide]), last = wide % 256;
    const bool enough = p.k_off ? wide >= 300
                        : d16 > 112 ? wide > 128 && (wide <= 256 || wide >= 300)
                                    : last == 0 || last >= 150;
    if (d16 > 64 && enough && score_smem(kScoreForms[kScoreWide], p.H, d16) <= kScoreSmemMax)
        return kScoreWide;
    if (d16 > 112) return kScoreNarrow;
    return d16 < 64 || score_tasks(p, kScoreForms[kScoreTall]) >= (p.k_off ? 512 : 256)
               ? kScoreTall
               : kScoreNarrow;
}

// LDS a scoring workgroup may take for the copy of its sample's scores: what it has, or up to
// an equal share of the CU among the workgroups that fit there (registers: at most four).  More
// would cost workgroups per CU: with half a CU's LDS for every copy, 8 samples of 20000 keys x
// 100 rows (8 heads of 40) took 165 us, 2 of 16384 x 100 (16 of 64) 106; with the select in
// a launch of its own 123 and 80.
inline size_t score_room(const ScoreForm& f, int H, int d16) {
    const size_t smem = score_smem(f, H, d16), per = kScoreSmemMax / smem;
    const size_t share = kScoreSmemMax / (per < 1 ? 1 : per > 4 ? 4 : per) / 2048 * 2048;
    return smem > share ? smem : share;
}
// Whether one workgroup per sample combines its row blocks (the last scoring workgroup, or the
// select with a caller normaliser) instead of text_rows_combine, whose launch it saves: up to
// 8192 partials, which it reads a few thousand at a time.  Whole calls, in the sample's
// workgroup / launch of its own: one sample of 2000 keys x 128 rows (2 blocks) 67 and 67 us,
// with the caller's normaliser 50 and 52; 1000 x 160 (3) 66 and 68; 4096 x 128 (2) 70 and 68;
// 4096 x 500 (8) 91 and 84; 16384 x 2000 (16) 736 and 710, 16 heads of 64 302 and 247, with the
// caller's normaliser 188 and 147.
inline bool combine_in_sample(const Prob& p, const ScoreForm& f) {
    return (p.max_rows + f.rows - 1) / f.rows * ((long long)p.R + p.max_cands) <= 8192;
}

// Dynamic LDS of the text-row statistics kernel: a ring of kStatsRing key blocks
// (32 keys x d bf16), plus the (max, sum) merge arrays.  Two stages (one
// block in flight while the other is used) and four workgroups per CU read
// the head slices faster than deeper rings at fewer workgroups per CU: the scattered
// 256-byte slices stream better with fewer requests outstanding per CU.
constexpr int kStatsRing = 2;
// Row blocks per statistics workgroup, for nrb 128-row blocks per sample (at most) and `heads`
// (sample, head) pairs.  Two share each key block's copy where both are there and the halved
// launch still fills the chip: always for two or four of a uniform batch (which the key ranges
// fill, but for mutual scoring); an even uniform count, or from 16 blocks any, with 448 or more
// workgroups; ragged rows from 32.  Otherwise the idle half, or the CUs without a workgroup,
// cost more than the shared copies save.  Whole calls, one / two: ragged grouped-query batch
// (64 samples of 16-512 rows) statistics 394 and 443 us; mutual scoring, 16 heads of 72, 8
// samples of 1028 rows (9 blocks) 97 and 101, 1 of 4100 (33, 272 workgroups) 202 and 216, 4 of
// 1404 (11) 88 and 92, 16 of 1704 (14) 358 and 352, 8 of 2884 (23) 496 and 487, 32 ragged of
// 132-2004 325 and 350, 16 of 260-4100 915 and 903; text, 8 samples of 4096 keys x 700 rows
// (6) 579 and 569.
inline int stats_row_blocks(int nrb, bool uniform, long long heads) {
    if (!uniform) return nrb >= 32 ? 2 : 1;
    if (nrb <= 4) return nrb % 2 == 0 ? 2 : 1;
    return heads * ((nrb + 1) / 2) >= 448 && (nrb % 2 == 0 || nrb >= 16) ? 2 : 1;
}
// Key ranges of the statistics pass: a batch with fewer than kStatsMinWorkgroups
// (sample, head, row-block group) tasks splits each task's keys into up to kStatsMaxSplits
// ranges of at least kStatsMinSplitBlocks 32-key blocks; each range writes its own base-2
// log-sum-exp table, and the scoring pass merges them.
constexpr int kStatsMinWorkgroups = 1024;
constexpr int kStatsMaxSplits = 8;
constexpr int kStatsMinSplitBlocks = 16;
inline int stats_splits(long long tasks, long long keys) {
    if (tasks <= 0 || tasks >= kStatsMinWorkgroups) return 1;
    long long ks = (kStatsMinWorkgroups + tasks - 1) / tasks;
    const long long by_keys = ((keys + 31) / 32) / kStatsMinSplitBlocks;
    if (ks > by_keys) ks = by_keys;
    if (ks > kStatsMaxSplits) ks = kStatsMaxSplits;
    return ks < 1 ? 1 : (int)ks;
}
// rbw: row blocks per workgroup.
inline size_t text_stats_smem(int d16, int rbw) {
    return (size_t)kStatsRing * 32 * d16 * 2 + 2 * (size_t)rbw * kTxtRows * 4;
}

// Anchor-path keys per workgroup for a given row geometry.
// Streaming form of the one-row logits (cls_stream_kernel): every query head has its
// own key head, a head is NC 16-byte chunks with NC a power of two up to 16, and a key
// row is 1 to 4 whole 64-lane loads.  Returns NC when the form applies, else 0.
// Lanes per head of the streaming one-row form: the head's 16-byte chunk count rounded
// up to a power of two (at most 16; lanes past the real chunks contribute zero), or 0
// when the form does not apply.
inline int cls_stream_nc(int H, int Hkv, int d, int elem_bytes) {
    if (H != Hkv || (d * elem_bytes) % 16 != 0) return 0;
    const int nc = d * elem_bytes / 16;
    if (nc < 1 || nc > 16) return 0;
    int ncp = 1;
    while (ncp < nc) ncp *= 2;
    const int cpk = ncp * Hkv;
    if (cpk % 64 != 0 || cpk / 64 > 4) return 0;
    return ncp;
}
// Key rows per wave step of the contiguous-run form (cls_stream_run_kernel; bf16, every
// query head with its own key head), or 0 when it does not apply: a step fills whole 1 KB
// wave loads and one lane serves each (row, head).  16 heads of 5-7 or 9 chunks (padding
// would idle lanes; ten chunks gain 7 % on large batches but lose 10 % on one image, and stay
// with the padded form), and 12 or 20 heads of 64 (their padded slots fill
// no whole wave loads, so they had only the LDS-partials kernel).
inline int cls_run_rows(int H, int Hkv, int d, int elem_bytes) {
    if (elem_bytes != 2 || H != Hkv) return 0;
    if (H == 16 && (d == 40 || d == 48 || d == 56 || d == 72)) return 4;
    if (d == 64 && H == 12) return 4;
    if (d == 64 && H == 20) return 2;
    return 0;
}
constexpr int kClsStreamKeys = 128;    // keys per workgroup of the streaming form
// Small batches: the streaming form halves its keys per workgroup (down to 16) until the
// launch has this many workgroups (two per CU), so that a single image is read by many
// CUs at once instead of a handful.
constexpr int kClsMinWorkgroups = 512;

inline int cls_keys_per_wg(int H, int Hkv, int d, int elem_bytes, int B = 0, long long keys = 0) {
    if (cls_stream_nc(H, Hkv, d, elem_bytes) || cls_run_rows(H, Hkv, d, elem_bytes)) {
        int kpw = kClsStreamKeys;
        while (kpw > 16 && (long long)B * ((keys + kpw - 1) / kpw) < kClsMinWorkgroups) kpw /= 2;
        return kpw;
    }
    int chunks_per_head = d * elem_bytes / 16;
    int kpw = kClsPartials / (H * chunks_per_head);
    if (kpw > 64) kpw = 64;
    if (kpw < 1) kpw = 1;
    return kpw;
}

// Per-sample epilogue of occam_prune, run inside the scoring kernels by the last
// workgroup to finish each sample (so that no separate threshold / select or row-block
// combine launch is needed).  done[B] counts the finished workgroups of every sample; the
// kernel that runs just before the scoring kernel in the same call clears it.  done ==
// null: no epilogue.
struct Finish {
    unsigned* done;
    int select;            // threshold + compaction (else only the row-block combine)
    float lambda;
    int reduce;
    float* tau;            // [B], tau_b
    int* slot;             // survivors, slot[co_b + i]
    int* count;            // [B]
    // One-row path instead (chunk_cnt != null): every scoring workgroup thresholds and
    // compacts its own chunk of kpw keys into chunk_slot[b * (R + max_cands) + c * kpw + i],
    // writes chunk_cnt[b * nchunks + c] and adds it to count[b] (cleared by the logits
    // kernel); pack_gather places the chunk lists.
    int* chunk_slot;
    int* chunk_cnt;
};

// Zero the counters the scoring kernel accumulates into (one workgroup of the kernel that
// precedes it in the call): done[0 .. B), or count[0 .. B) for the per-chunk compaction.
__device__ __forceinline__ void clear_done(const Finish& f, int B) {
    if (f.done)
        for (int i = threadIdx.x; i < B; i += blockDim.x) f.done[i] = 0u;
    if (f.chunk_cnt)
        for (int i = threadIdx.x; i < B; i += blockDim.x) f.count[i] = 0;
}

// Most chunks per sample of the per-chunk compaction (pack_gather scans their counts in LDS).
constexpr int kMaxChunkLists = 1024;

// Every thread of the workgroup calls this after writing its share of sample b's scores
// (or row-block partials) with device-coherent stores (st_cc).  Each wave waits until its
// stores have completed, the workgroup counts itself, and the one that completes the
// sample's ntask workgroups gets true; it then reads the other workgroups' values with
// device-coherent loads (ld<true>).  No cache-wide write-back or invalidation is needed
// (measured: an agent-scope release/acquire fence pair in every workgroup of the Stage II
// scoring kernel cost ~90 us per launch).  flag: one int of LDS.
__device__ __forceinline__ bool last_of_sample(unsigned* done, int b, unsigned ntask, int* flag) {
    __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0): this wave's stores are done
    __syncthreads();
    if (threadIdx.x == 0)
        *flag = __hip_atomic_fetch_add(done + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u ==
                ntask;
    __syncthreads();
    return *flag != 0;
}

// LDS the per-sample epilogue needs: its scratch words and a copy of the sample's scores.
constexpr size_t kSelectScratch = 128;
inline size_t select_lds_bytes(int R, int max_cands) {
    return kSelectScratch + 4 * ((size_t)R + (size_t)max_cands);
}

// Where select_sample keeps its copy of the sample's scores (lds as passed to it).
__device__ __forceinline__ float* select_scores_lds(char* lds) {
    return reinterpret_cast<float*>(lds + kSelectScratch);
}

// Threshold (tau_b = lambda * reference, the fused threshold of select_kernel) and
// compaction of sample b by one workgroup of NT threads (kSelThreads or more).  The
// sample's scores, written by other workgroups of the launch, are first copied into LDS
// with device-coherent loads (eight in flight per thread), unless the caller has already
// put them there (in_lds, followed by a barrier); the reference and the compaction then
// read the copy, with select_kernel's arithmetic.  lds: select_lds_bytes(R, N_b).
template <int NT>
__device__ __forceinline__ void select_sample(const Prob& p, const float* scores, int b,
                                              const Finish& f, char* lds, bool in_lds) {
    float* red = reinterpret_cast<float*>(lds);              // kSelThreads / 64 floats
    float* tau_s = reinterpret_cast<float*>(lds + 16);
    int* wsum = reinterpret_cast<int*>(lds + 32);            // NT / 64 ints
    static_assert(NT >= kSelThreads && NT / kWave <= 16, "scratch layout");
    float* sl = select_scores_lds(lds);
    const int S = keys_of(p, b);
    const float* src = scores + k_begin(p, b);
    constexpr int U = 8;
    for (int i0 = threadIdx.x; i0 < S && !in_lds; i0 += U * NT) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * NT;
            v[u] = i < S ? ld<true>(src + i) : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * NT;
            if (i < S) sl[i] = v[u];
        }
    }
    __syncthreads();
    const float t = f.lambda * reference_of<kSelThreads>(sl, p.R, S - p.R, f.reduce, red);
    if (threadIdx.x == 0) {
        if (f.tau) f.tau[b] = t;
        *tau_s = t;
    }
    __syncthreads();
    compact_of<NT>(sl + p.R, S - p.R, *tau_s, f.slot + cand_begin(p, b), f.count + b,
                            wsum);
}

// ---------------------------------------------------------------------------
// Launchers (defined in the .hip files).  Each returns the status of its own launches.
hipError_t launch_select_topk(const Prob& p, const float* scores, int k_keep, int* slot,
                              int* count, hipStream_t s);
// Selection state of budget matching, in the workspace; `keys` takes the ratios' order keys,
// B * max_cands words.
constexpr size_t kMatchStateBytes = 8192;
hipError_t launch_match_lambda(const Prob& p, const float* scores, int reduce, float k_target,
                               void* state, void* keys, float* lambda, float* mean_kept, hipStream_t s);
hipError_t launch_register_redirect(const Prob& p, int bf16, void* h, int width, long long stride,
                                    const int* channels, int n_channels, int reg_slot,
                                    hipStream_t s);
// fin.done (nullable) is cleared by launch_cls_logits / launch_text_stats and used by the
// scoring launch that follows them in the same call.
hipError_t launch_cls_logits(const Prob& p, int bf16, const void* q, const void* k,
                             float* logits, float2* stats, int kpw, const Finish& fin,
                             hipStream_t s);
hipError_t launch_cls_scores(const Prob& p, int bf16, const float* logits, const float2* stats,
                             const float* row_lse, float* scores, int kpw, const Finish& fin,
                             hipStream_t s);
hipError_t launch_text_stats(const Prob& p, const void* q, const void* k, float* lse2,
                             const Finish& fin, hipStream_t s);
// Mutual scoring (every key: mean over rows): column sums per (row block, head) into
// part [B][ceil(max_rows/128)][H][R + max_cands], then their fixed-order mean.
hipError_t launch_text_colsum(const Prob& p, const void* q, const void* k, const float* lse,
                              int lse_natural, float* part, float* scores, hipStream_t s);
// Max-over-rows scoring; with several row blocks of the form's rows (score_form), per-block
// partials go to part [B][ceil(max_rows / rows)][R + max_cands] and a combine forms the scores.
// With fin.done the row-block combine (and with fin.select the threshold and the
// compaction) run in each sample's last workgroup; without it text_rows_combine follows,
// unless leave_blocks (launch_select then combines them).
hipError_t launch_text_score(const Prob& p, const void* q, const void* k, const float* lse,
                             int lse_natural, float* scores, float* part, const Finish& fin,
                             bool leave_blocks, hipStream_t s);
hipError_t launch_threshold(const Prob& p, const float* scores, float lambda, int reduce,
                            float* tau, hipStream_t s);
// part (nullable): row blocks of rb_rows rows left by launch_text_score, from which the
// scores are formed (and stored) first.
hipError_t launch_select(const Prob& p, float* scores, const float* part, int rb_rows,
                         const float* tau, int fuse_tau, float lambda, int reduce, float* tau_out,
                         int* slot, int* count, hipStream_t s);
// Survivors from the per-chunk lists of the one-row scoring kernel (chunk_cnt != null)
// or from slot[co_b + i] (select); counts per sample in count[B] either way.
struct ChunkLists {
    const int* slot;       // [B][R + max_cands], chunk c from c * kpw on
    const int* cnt;        // [B][nchunks]
    int nchunks, kpw;
};
hipError_t launch_pack_gather(const Prob& p, const int* slot, const int* count,
                              const int* index_map, int* kept_idx, int* kept_offsets,
                              const int* packed_idx, const int* packed_offsets,
                              const RowTensors& rows, hipStream_t s,
                              const ChunkLists& lists = ChunkLists{});

}  // namespace occam
