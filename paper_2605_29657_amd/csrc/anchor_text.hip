// Anchor path for several anchor rows per sample (the text rows of Stage II,
// Eq. text_scoring), steps 1-2, on the gfx950 matrix cores.
//
// For T text rows, H heads and R+N keys the logits are a T x (R+N) x d
// contraction per head, done with v_mfma_f32_32x32x16_bf16.  The MFMA's A
// operand is a block of 32 keys and its B operand a block of 32 text rows, so
// each lane of the accumulator holds 16 keys of ONE text row: reductions over
// keys (the softmax statistics) stay inside a lane, and the head sum is an
// element-wise accumulation in registers.  (The column-sum form below swaps the
// operands, so that a lane holds 16 rows of one key.)
//
// Every (row, head) softmax needs its normaliser before the head mean can be
// formed, so the path has two passes over the keys:
//
// text_stats  task (sample, head, group of one or two row blocks of 128[, key range]),
//             XCD-aware; a batch with few such tasks splits their keys into ranges whose tables
//             text_lse_merge combines.
//             The keys are consumed by four waves of 32 rows per row block, so each
//             key block is copied once for every row block of the group; the
//             query rows of the head sit in
//             registers as MFMA B fragments, and a (reference, sum 2^(x - reference))
//             pair is kept per row: the reference is the first key block's maximum
//             and moves only when a block's sum would exceed 2^64, so a logit costs
//             a multiply-add, an exponential and an add (no running maximum); pairs
//             are merged across the two lane halves
//             in a fixed order.  Key blocks reach LDS through direct global -> LDS
//             copies (a 2-stage ring per stream).  Writes the base-2
//             log-sum-exp lse2[row, head] of x = logit * log2(e).  Its COLSUM
//             form streams the keys the same way with the normalisers known and
//             writes per-(row block, head) column sums for mutual scoring (Eq.
//             mutual_scoring, every key takes the mean over rows);
//             text_colsum_reduce adds them in a fixed order.
// text_score  one workgroup per (sample, block of keys, row block): four waves and 64 or 128
//             rows, or eight waves and 128 rows (score_form).  Each wave owns 32 keys.  For
//             every head the query tile (double-buffered) and the wave's keys are copied
//             global -> LDS in whole lines one head ahead, and the key fragments then go
//             to registers (or the keys are loaded into them directly), while
//             p = 2^(x - lse2) of the
//             current head is accumulated over heads per (key, row); the workgroups
//             of one XCD walk the heads from the same start.  Afterwards the row
//             reduction of Eq. text_scoring is applied: max over rows for visual
//             keys, mean for registers, both over the head mean (1/H); with several
//             row blocks the per-block maxima and sums are combined by the sample's
//             last workgroup (or text_rows_combine), which with a threshold also
//             selects the survivors.  Rows beyond T_b carry lse2 = +inf and so
//             contribute exactly 0.
//
// The LDS copies are issued as inline global_load_lds so that the compiler does
// not fold them into its own memory-counter waits; each kernel waits for them
// explicitly (s_waitcnt vmcnt, then a barrier) before the stage is read.
//
// When the caller supplies its own natural-log normaliser (row_lse), text_stats
// is skipped and the second pass reads lse2 = row_lse * log2(e).
#include "occam_internal.hpp"

#include <algorithm>

namespace occam {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ u32x4 load16(const uint16_t* p) {
    return *reinterpret_cast<const u32x4*>(p);
}
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Row (key) index, inside a 32-key block, of accumulator element r of a lane
// whose upper-half flag is hi (lanes 32..63): 8*(r/4) + 4*hi + r%4.
__device__ __forceinline__ int acc_key(int r, int hi) { return 8 * (r >> 2) + 4 * hi + (r & 3); }

// Merge two online-softmax pairs (max, sum 2^(x - max)).
__device__ __forceinline__ void merge_pair(float& m, float& z, float mo, float zo) {
    const float mn = fmaxf(m, mo);
    if (mn == -INFINITY) return;
    z = z * __builtin_amdgcn_exp2f(m - mn) + zo * __builtin_amdgcn_exp2f(mo - mn);
    m = mn;
}

// Loads are unconditional so that the compiler can count outstanding loads and
// keep prefetches in flight: key and row indices are clamped into range (a
// clamped key's logits are never used, a clamped row's results are never
// written or carry zero weight), and when d % 16 == 8 (HALF) the upper lane
// half of the last 16-wide step reads a valid address and is zeroed by select.
template <int DS, bool HALF>
__device__ __forceinline__ u32x4 frag16(const uint16_t* row, int kk, int hi) {
    const bool pad = HALF && kk == DS - 1 && hi;
    u32x4 v = load16(row + kk * 16 + (pad ? 0 : hi * 8));
    const u32x4 zero = {0u, 0u, 0u, 0u};
    return pad ? zero : v;
}

// The same copy with a wave-uniform base address and a 32-bit per-lane byte offset,
// issued as inline assembly: the compiler does not see it, so it neither counts it
// among the wave's outstanding loads nor makes later LDS reads wait for it.  The
// caller orders it explicitly (wait_vmem + barrier before the copied data is read).
// lds is the wave-uniform LDS byte address of lane 0's 16 bytes.
__device__ __forceinline__ void dma16_async(const void* base, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds)) : "memory");
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)p);
}
// Make the compiler treat v as produced here: a load into v must be complete before
// this point (the compiler inserts the wait), and no later code waits for it again.
__device__ __forceinline__ void settle(u32x4& v) { asm volatile("" : "+v"(v)); }
// Wait until every global load of this wave (including LDS copies) has landed.
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// vmcnt(n) wait with expcnt / lgkmcnt left unconstrained (gfx9 encoding).
template <int N>
__device__ __forceinline__ void wait_vmem_le() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// COLSUM = false: the base-2 log-sum-exp of every (row, head) over the sample's keys
// (lse2).  COLSUM = true (mutual scoring, Eq. mutual_scoring): with the normalisers
// given (lse_in), the sum over this workgroup's 128 rows of p = 2^(x - lse2) for every
// key, written to part[b][row block][h][key]; the mean over rows and heads is then a
// fixed-order sum over the partials (text_colsum_reduce).  Both modes stream the keys
// the same way; the column sums use the MFMA the other way round (rows as the A
// operand), so that a lane holds 16 rows of one key and sums them in registers.
template <int DS, bool HALF, bool COLSUM, int RING, int RBW>
__device__ __forceinline__ void stats_task(
    const Prob& p, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
    float* __restrict__ lse2, const float* __restrict__ lse_in, int lse_natural,
    float* __restrict__ part, int b, int h, int tblk, int split, int nsplit, char* smem_raw)
{
    // Keys: range split of nsplit (32-key blocks [kb_lo, kb_lo + nkb_s) of the sample);
    // the base-2 log-sum-exp over that range goes to table split of lse2.
    // RBW row blocks (tblk * RBW + rbl, rbl < RBW) of RG = 4 waves each: wave rg of a row
    // block owns its 32 rows [32 rg, +32).  All NW waves consume the same key blocks, so each
    // block is copied once, global -> LDS, into a ring of RING stages: RING - 1 blocks are in
    // flight while one is used.
    // A row block past T_b computes nothing but still copies its share of the blocks and
    // meets every barrier.
    // A block is 32 keys x NCH 16-byte chunks; chunk c of key j sits in LDS unit
    // j*NCH + (c ^ (j & SW)), SW = NCH - 1 when NCH is a power of two (else 0), so a
    // copy writes whole 256-byte key slices and the MFMA fragment reads of 32
    // consecutive keys spread over the banks.
    static_assert(RBW == 1 || !COLSUM, "column sums take one row block per workgroup");
    constexpr int RG = kStatsThreads / kWave;        // waves of a row block
    constexpr int RPW = kTxtRows / RG;               // rows per wave
    constexpr int NSBW = RPW / 32;                   // 32-row sub-blocks per wave
    constexpr int NW = RG * RBW;                     // waves of the workgroup
    constexpr int NCH = 2 * DS;                      // 16-byte chunks per key row
    constexpr int UNITS = 32 * NCH;                  // 16-byte units per block
    constexpr int COPIES = UNITS / kWave;            // = DS copies of 64 lanes per block
    constexpr int MINE = (COPIES + NW - 1) / NW;     // most copies a wave issues
    constexpr int MINE_MIN = COPIES / NW;            // fewest copies a wave issues
    constexpr int SW = (NCH & (NCH - 1)) == 0 ? NCH - 1 : 0;
    u32x4* ring = reinterpret_cast<u32x4*>(smem_raw);              // [stage][UNITS]
    float* red_m = reinterpret_cast<float*>(ring + RING * UNITS);
    float* red_z = red_m + RBW * kTxtRows;
    const int nrb = (p.max_rows + kTxtRows - 1) / kTxtRows;
    const int T = rows_of(p, b);
    if (tblk * RBW * kTxtRows >= T) return;
    const int S = keys_of(p, b);
    const int lane = threadIdx.x & 63;
    const int mi = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);         // wave-uniform
    const int rbl = mi / RG, rg = mi % RG;
    const int t0 = (tblk * RBW + rbl) * kTxtRows;
    const int hi = lane >> 5, lo = lane & 31;
    const int H = p.H, Hkv = p.Hkv, d = p.d;
    const int g = h / (H / Hkv);
    const int tw = t0 + rg * RPW;                      // first row of this wave
    const int nsb = max(0, min(NSBW, (T - tw + 31) >> 5));
    const int qb = q_begin(p, b), kb0 = k_begin(p, b);
    const float c2 = p.scale * kLog2e;

    bf16x8 qf[NSBW][DS];
#pragma unroll
    for (int sb = 0; sb < NSBW; ++sb) {
        const int t = min(tw + sb * 32 + lo, T - 1);
        const uint16_t* qrow = q + ((size_t)(qb + t) * H + h) * d;
#pragma unroll
        for (int kk = 0; kk < DS; ++kk) qf[sb][kk] = as_bf16x8(frag16<DS, HALF>(qrow, kk, hi));
    }

    float m[NSBW], z[NSBW];
#pragma unroll
    for (int sb = 0; sb < NSBW; ++sb) { m[sb] = -INFINITY; z[sb] = 0.f; }
    // COLSUM: base-2 normaliser of the 16 rows this lane holds in each sub-block (row
    // 8*(r/4) + 4*hi + r%4 of the sub-block); rows past T_b get +inf and weigh 0.
    float lsev[COLSUM ? NSBW : 1][16];
    if (COLSUM) {
#pragma unroll
        for (int sb = 0; sb < NSBW; ++sb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int t = tw + sb * 32 + acc_key(r, hi);
                float v = INFINITY;
                if (t < T) {
                    v = lse_in[(size_t)(qb + t) * H + h];
                    if (lse_natural) v *= kLog2e;
                }
                lsev[sb][r] = v;
            }
    }

    const int nkb = (S + 31) >> 5;
    const int kb_lo = __builtin_amdgcn_readfirstlane(nkb * split / nsplit);   // wave-uniform
    const int nkb_s = __builtin_amdgcn_readfirstlane(nkb * (split + 1) / nsplit) - kb_lo;
    const char* kbase = reinterpret_cast<const char*>(k + ((size_t)kb0 * Hkv + g) * d);
    const int kstride = Hkv * d;                      // elements per key row
    const uint32_t ring_lds = lds_addr(ring);

    // Copy block j of the range (clamped to its last block) into its stage.
    // Copy c of the block fills units 64c .. 64c+63; this wave issues c = mi, mi+NW, ...
    // Lane offsets inside a block are fixed (key kc = u / NCH of the block, chunk
    // (u % NCH) ^ (kc & SW)); only a block running past S_b clamps its keys.  The pad
    // chunk past d (HALF) reads chunk 0 of the key: its fragment is zeroed below.
    uint32_t coff[MINE];
#pragma unroll
    for (int i = 0; i < MINE; ++i) {
        const int u = min(mi + NW * i, COPIES - 1) * kWave + lane;
        const int kc = u / NCH, ch = (u % NCH) ^ (kc & SW);
        const int e = (HALF && ch == NCH - 1) ? 0 : ch * 8;
        coff[i] = (uint32_t)(kc * kstride + e) * 2u;
    }
    auto issue = [&](int j) {
        const int jj = min(j, max(nkb_s - 1, 0));
        // An empty range copies the sample's last block at most: every copy stays inside the
        // sample's keys, and the stage is never read.
        const int kbi = min(kb_lo + jj, nkb - 1);
        const char* bbase = kbase + (size_t)kbi * 32 * kstride * 2;
        const uint32_t dst = ring_lds + (uint32_t)((jj % RING) * UNITS * 16);
        const bool full = kbi * 32 + 32 <= S;
#pragma unroll
        for (int i = 0; i < MINE; ++i) {
            const int c = mi + NW * i;
            if (c >= COPIES) break;
            uint32_t off = coff[i];
            if (!full) {
                const int u = c * kWave + lane;
                const int kc = u / NCH, ch = (u % NCH) ^ (kc & SW);
                const int e = (HALF && ch == NCH - 1) ? 0 : ch * 8;
                off = (uint32_t)(min(kc, S - 1 - kbi * 32) * kstride + e) * 2u;
            }
            dma16_async(bbase, off, dst + (uint32_t)(c * kWave * 16));
        }
    };
    // Byte offset in a block of fragment (key lo, chunk hi) for k-step 0; k-step kk
    // reads (kfrag ^ kk*32) with SW, (kfrag + kk*32) without.
    const uint32_t kfrag = (uint32_t)(lo * NCH + (hi ^ (lo & SW))) * 16u;

    // One key block: MFMA logits from the LDS stage, then the (reference, sum) update.
    // The reference m of a row is the largest logit of the wave's first block (all later
    // blocks see a full first block, so m is finite there).  Later blocks add
    // 2^(x - m) with m fixed; x may exceed m, and a block whose sum passes 2^64 (or
    // overflows) is redone with its own maximum, which also moves m.  Terms below
    // 2^-126 relative to m are below float32 resolution of z >= 1.
    auto block = [&](int kbi, const u32x4* blk, bool first) -> float {
        const int nvalid = S - kbi * 32;
        u32x4 kf[DS];
#pragma unroll
        for (int kk = 0; kk < DS; ++kk) {
            const uint32_t fo = SW ? (kfrag ^ (uint32_t)(kk * 32)) : kfrag + kk * 32;
            const u32x4 v = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(blk) + fo);
            const u32x4 zero = {0u, 0u, 0u, 0u};
            kf[kk] = (HALF && kk == DS - 1 && hi) ? zero : v;
        }
        f32x16 acc[NSBW];
#pragma unroll
        for (int sb = 0; sb < NSBW; ++sb) acc[sb] = f32x16{};
        if (COLSUM) {
            // Rows as the A operand: lane (key lo, half hi) holds rows acc_key(r, hi).
            // Both sub-blocks always: a branch between the MFMAs costs more than the
            // clamped rows of a partial second sub-block (whose terms are skipped below).
#pragma unroll
            for (int kk = 0; kk < DS; ++kk)
#pragma unroll
                for (int sb = 0; sb < NSBW; ++sb)
                    acc[sb] = mfma32(qf[sb][kk], as_bf16x8(kf[kk]), acc[sb]);
            // Four partial sums (r mod 4) keep the dependent add chains short.
            float c4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int sb = 0; sb < NSBW; ++sb) {
                if (sb >= nsb) break;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    c4[r & 3] += __builtin_amdgcn_exp2f(fmaf(acc[sb][r], c2, -lsev[sb][r]));
            }
            const float cs = (c4[0] + c4[1]) + (c4[2] + c4[3]);
            return cs + __shfl_xor(cs, 32);
        }
#pragma unroll
        for (int kk = 0; kk < DS; ++kk)
#pragma unroll
            for (int sb = 0; sb < NSBW; ++sb)
                acc[sb] = mfma32(as_bf16x8(kf[kk]), qf[sb][kk], acc[sb]);
#pragma unroll
        for (int sb = 0; sb < NSBW; ++sb) {
            if (sb >= nsb) break;
            if (!first) {
                // Sum against the fixed reference in four partial chains (r mod 4).
                float a4[4] = {0.f, 0.f, 0.f, 0.f};
                if (nvalid >= 32) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        a4[r & 3] += __builtin_amdgcn_exp2f(fmaf(acc[sb][r], c2, -m[sb]));
                } else {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (acc_key(r, hi) < nvalid)
                            a4[r & 3] += __builtin_amdgcn_exp2f(fmaf(acc[sb][r], c2, -m[sb]));
                }
                const float asum = (a4[0] + a4[1]) + (a4[2] + a4[3]);
                if (asum <= 0x1p64f) { z[sb] += asum; continue; }
            }
            // Maximum and sum over the lane's 16 keys in four partial chains (r mod 4).
            float m4[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
            if (nvalid >= 32) {
#pragma unroll
                for (int r = 0; r < 16; ++r) m4[r & 3] = fmaxf(m4[r & 3], acc[sb][r]);
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (acc_key(r, hi) < nvalid) m4[r & 3] = fmaxf(m4[r & 3], acc[sb][r]);
            }
            const float mx = fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3]));
            if (mx == -INFINITY) continue;
            const float mn = fmaxf(m[sb], mx * c2);
            float s4[4] = {0.f, 0.f, 0.f, 0.f};
            if (nvalid >= 32) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    s4[r & 3] += __builtin_amdgcn_exp2f(fmaf(acc[sb][r], c2, -mn));
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (acc_key(r, hi) < nvalid)
                        s4[r & 3] += __builtin_amdgcn_exp2f(fmaf(acc[sb][r], c2, -mn));
            }
            const float sum = (s4[0] + s4[1]) + (s4[2] + s4[3]);
            z[sb] = z[sb] * __builtin_amdgcn_exp2f(m[sb] - mn) + sum;
            m[sb] = mn;
        }
        return 0.f;
    };

    // COLSUM: the RG waves leave their column sums of block j in
    // sums[j & 1][rg][key] (red_m and red_z together); after the next barrier the
    // rg = 0 wave adds them in order of rg and stores the workgroup's partial.
    float* sums = red_m;
    float* prow = part + (((size_t)b * nrb + tblk) * H + h) * (size_t)(p.R + p.max_cands);
    auto store_sums = [&](int j) {
        const float* sp = sums + (j & 1) * (RG * 32);
        const int key = j * 32 + lane;
        if (lane < 32 && key < S) {
            float v = sp[lane];
#pragma unroll
            for (int w = 1; w < RG; ++w) v += sp[w * 32 + lane];
            prow[key] = v;
        }
    };
#pragma unroll
    for (int j = 0; j < RING - 1; ++j) issue(j);
    for (int i = 0; i < nkb_s; ++i) {
        // Own copies of block i have landed once at most RING-2 later blocks remain
        // (counted with the fewest copies a wave issues: a stronger wait for the others).
        wait_vmem_le<(RING - 2) * MINE_MIN>();
        __syncthreads();                 // partner's copies landed; stage (i-1) is free
        issue(i + RING - 1);
        if (COLSUM && rg == 0 && i >= 1) store_sums(i - 1);
        float cs = 0.f;
        if (nsb > 0) cs = block(kb_lo + i, ring + (i % RING) * UNITS, i == 0);
        if (COLSUM && hi == 0) sums[(i & 1) * (RG * 32) + rg * 32 + lo] = cs;
    }
    wait_vmem_le<0>();
    if (COLSUM) {
        __syncthreads();
        if (rg == 0 && nkb_s >= 1) store_sums(nkb_s - 1);
        return;
    }

    // Merge the two lane halves (same rows, different keys).
#pragma unroll
    for (int sb = 0; sb < NSBW; ++sb) {
        const float mo = __shfl_xor(m[sb], 32);
        const float zo = __shfl_xor(z[sb], 32);
        merge_pair(m[sb], z[sb], mo, zo);
        if (hi == 0) {
            red_m[rbl * kTxtRows + rg * RPW + sb * 32 + lo] = m[sb];
            red_z[rbl * kTxtRows + rg * RPW + sb * 32 + lo] = z[sb];
        }
    }
    __syncthreads();
    if (threadIdx.x < RBW * kTxtRows) {
        const int rr = threadIdx.x / kTxtRows, i = threadIdx.x % kTxtRows;
        const int t = (tblk * RBW + rr) * kTxtRows + i;
        if (t < T) lse2[(size_t)split * p.lse_stride + (size_t)(qb + t) * H + h] =
            red_m[threadIdx.x] + __builtin_amdgcn_logf(red_z[threadIdx.x]);
    }
}

// Whether the statistics tasks are dealt to the XCDs by units (below) instead of as eight
// contiguous ranges.  A contiguous range holds whole samples, so with ragged samples the XCD
// with the longest ones finished last while the others idled (mutual scoring of 16 samples of
// 256-4096 keys, work ~ keys^2: statistics 697 -> 435 us, column sums 730 -> 470 us; ragged
// grouped-query batch: statistics 493 -> 430 us).  The ranges stay (whole calls, units /
// ranges)
//  * on uniform batches, and with fewer than eight units per XCD, whose remainder would leave
//    XCDs idle;
//  * where a unit is one workgroup (`per`), which shares nothing, and there are samples
//    enough to even out: 64 samples of 256-4096 keys x 128 rows, 16 heads of 72 204 and 200
//    us, 32 of 96 406 and 390, 32 of 112 492 and 466, 32 of 128 468 and 459; 20 of 100-2000
//    keys, 32 of 112 114 and 109; but 16 samples of 500-4096 keys x 200 rows 200 and 229;
//  * on short samples whose key slices are no whole 128-byte lines, which the heads side by
//    side on one XCD share: mutual scoring, 16 heads of 72, 32 samples of 31-250 tokens 43 and
//    40 us (62-500: 77 and 73, 125-1000: 150 and 166; text rows, 32 heads of 128, 8 samples of
//    37-300 keys x 250 rows: 62 and 64).
static bool stats_by_unit(const Prob& p, int ns, int per, int rbw) {
    return (p.k_off || p.q_off) && (long long)p.B * p.Hkv * ns >= 8 * kXcds &&
           (per > 1 || p.B <= 16 * rbw) && (p.d % 64 == 0 || p.R + p.max_cands >= 384);
}

// One statistics task per workgroup.  Task = (sample, head, group of RBW row blocks),
// groups fastest, XCD-aware: the groups of one (sample, head) read the same keys and
// meet in one L2; the RBW row blocks of a group share one copy of every key block.
// per > 0: the tasks are dealt by units of that many (stats_by_unit).  Workgroup 0 also clears the per-sample counters of the scoring kernel that follows.
template <int DS, bool HALF, bool COLSUM, int RBW>
__global__ __launch_bounds__(kStatsThreads * RBW, 1) void text_stats_kernel(
    Prob p, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
    float* __restrict__ lse2, const float* __restrict__ lse_in, int lse_natural,
    float* __restrict__ part, int per, Finish fin)
{
    extern __shared__ __attribute__((aligned(16))) char smem_raw[];
    if (blockIdx.x == 0) clear_done(fin, p.B);
    const int nrb = (p.max_rows + kTxtRows - 1) / kTxtRows;
    const int ngrp = (nrb + RBW - 1) / RBW;
    const int ns = COLSUM || p.lse_splits < 1 ? 1 : p.lse_splits;
    int b, h, tblk, split;
    if (per) {
        // Unit = (sample, key head, key range): the row-block groups of the query heads that
        // read the same keys, `per` workgroups.  Units are dealt to the XCDs in turn.
        const int j = (int)blockIdx.x / kXcds;
        const int unit = j / per * kXcds + (int)blockIdx.x % kXcds, in = j % per;
        if (unit >= p.B * p.Hkv * ns) return;
        split = unit % ns;
        tblk = in % ngrp;
        h = (unit / ns) % p.Hkv * (p.H / p.Hkv) + in / ngrp;
        b = unit / (ns * p.Hkv);
    } else {
        const int task = xcd_remap((int)blockIdx.x, ngrp * p.H * p.B * ns);
        const int rest = task / ns;
        split = task % ns;
        tblk = rest % ngrp;
        h = (rest / ngrp) % p.H;
        b = rest / (ngrp * p.H);
    }
    // Wave-uniform (the key copies take a scalar base address).
    b = __builtin_amdgcn_readfirstlane(b);
    h = __builtin_amdgcn_readfirstlane(h);
    tblk = __builtin_amdgcn_readfirstlane(tblk);
    split = __builtin_amdgcn_readfirstlane(split);
    stats_task<DS, HALF, COLSUM, kStatsRing, RBW>(p, q, k, lse2, lse_in, lse_natural, part, b,
                                                  h, tblk, split, ns, smem_raw);
}

// Ragged launches: workgroup id -> the id-th non-empty (sample, key chunk, row block)
// task of the scoring pass, so that the active tasks take the lowest ids and spread over
// the CUs in dispatch order, instead of sitting among the empty chunks of short samples
// (where two of them can share a CU while other CUs idle).  Samples in reverse order,
// chunks then row blocks, as in the uniform mapping; xcd_remap over the A active tasks
// keeps a sample's tasks on one XCD.  Called by wave 0: each lane counts the tasks of a
// run of consecutive samples, a scan finds the lane and sample holding the task, which
// leaves (b, c, rb) in sh[0..2], or b = -1 past the last task.
__device__ void ragged_score_task(const Prob& p, int id, int kpw, int rb, int* sh) {
    const int lane = threadIdx.x;
    const int per = (p.B + kWave - 1) / kWave;
    const int i0 = min(lane * per, p.B), i1 = min(i0 + per, p.B);
    auto ntask = [&](int b) {
        const int T = rows_of(p, b), S = keys_of(p, b);
        if (T <= 0 || S <= 0) return 0;
        return ((S + kpw - 1) / kpw) * ((T + rb - 1) / rb);
    };
    int cnt = 0;
    for (int i = i0; i < i1; ++i) cnt += ntask(p.B - 1 - i);
    int incl = cnt;
    for (int off = 1; off < kWave; off <<= 1) {
        const int v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    const int A = __shfl(incl, kWave - 1);
    if (id >= A) {
        if (lane == 0) sh[0] = -1;
        return;
    }
    const int t = xcd_remap(id, A);
    int acc = incl - cnt;
    if (t < acc || t >= incl) return;
    for (int i = i0; i < i1; ++i) {
        const int b = p.B - 1 - i, n = ntask(b);
        if (t < acc + n) {
            const int nrb_b = (rows_of(p, b) + rb - 1) / rb;
            sh[0] = b;
            sh[1] = (t - acc) / nrb_b;
            sh[2] = (t - acc) % nrb_b;
            return;
        }
        acc += n;
    }
}

// One scoring task: keys [KPW c, KPW c + KPW) of sample b (KPW = 32 NW) against its row
// block rb, by NW waves.  cc_out: the scores / partials are read later in the same launch
// by another workgroup, so they are written with device-coherent stores.  rot_id picks the
// starting head (rot_id % 8 of 8 heads spread over H).  KLDS: the keys reach LDS first.
template <int DS, bool HALF, int NW, int NSB, bool KLDS>
__device__ __forceinline__ void score_task(
    const Prob& p, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
    const float* __restrict__ lse, int lse_natural, float* __restrict__ scores,
    float* __restrict__ part, int b, int c, int rb, int rot_id, char* smem_raw, bool cc_out)
{
    // Wave w owns the 32 keys [s_lo + 32 w, +32) and the RB rows of the workgroup's row
    // block (NSB sub-blocks of 32 rows, one MFMA accumulator chain each).
    //
    // Bound at full load by the matrix and vector work per logit (8 MFMAs and 48 vector
    // operations per 32 x 32 x 128 block): a probe of that block with operands from LDS
    // takes ~250 ns per SIMD on random data (206-219 ns without the LDS reads, 160 ns on
    // constant data, i.e. the card's power limit shows); the video batch's 1025 blocks per
    // SIMD take 440 ns each here, 500 with the keys loaded straight into the MFMA layout
    // (32 lines touched per 1 KB load, ~58 cycles each; whole-line copies take 16).
    //
    // Both operands of a head reach LDS by whole-line global -> LDS copies, row-major with
    // an XOR swizzle: chunk c of row t sits in unit t*NCH + (c ^ (t & SW)), SW = NCH - 1
    // when NCH is a power of two (else 0).  The query tile is shared by the waves and
    // double-buffered (one barrier per head); a wave's 32 keys go to an area of its own,
    // from which it takes its fragments into registers before the next head's copy starts,
    // so one buffer is enough.  Without KLDS the fragments of the next head are loaded into
    // a second set of registers instead.
    constexpr bool FULL = NSB == 4;              // all sub-blocks, rows past T_b weigh 0
    constexpr int KPW = kTxtKeysPerWave * NW, RB = 32 * NSB;
    constexpr int NCH = 2 * DS;                                   // 16-byte chunks per row
    constexpr int QTILE = RB * NCH;                         // 16-byte units per tile
    constexpr int KTILE = KLDS ? kTxtKeysPerWave * NCH : 0;       // units of one wave's keys
    constexpr int QCOPIES = (QTILE / kWave + NW - 1) / NW;        // per wave per head
    constexpr int KCOPIES = KTILE / kWave;                        // = DS
    constexpr int SW = (NCH & (NCH - 1)) == 0 ? NCH - 1 : 0;
    const int nrb = (p.max_rows + RB - 1) / RB;
    const int S = keys_of(p, b);
    const int s_lo = c * KPW;
    const int t0 = rb * RB;
    if (s_lo >= S || t0 >= rows_of(p, b)) return;
    const int T = rows_of(p, b);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hi = lane >> 5, lo = lane & 31;
    const int H = p.H, Hkv = p.Hkv, d = p.d, group = H / Hkv;
    const int qb = q_begin(p, b), kb0 = k_begin(p, b);
    const float c2 = p.scale * kLog2e;
    const int wkey0 = s_lo + wave * kTxtKeysPerWave;
    const bool wactive = wkey0 < S;
    const int R = p.R;
    u32x4* qt = reinterpret_cast<u32x4*>(smem_raw);                         // [2][QTILE]
    u32x4* kt = qt + 2 * QTILE + wave * KTILE;                              // this wave's keys
    float* l2t = reinterpret_cast<float*>(smem_raw + (2 * QTILE + NW * KTILE) * 16);  // [H][RB]
    // Loop step h works on head (h + rot) mod H: a key row's head slices all sit at
    // the same offset within 8 KB rows, so workgroups moving through the heads in step
    // would load the same memory channels at the same time.  Eight starting heads,
    // spread over the H heads, balance the channels as well as H of them do; with one
    // start per XCD (rot_id % 8 is the XCD), the workgroups that share an L2 also share
    // the query tile and key slices they are reading.
    const int nrot = H < 8 ? H : 8;
    const int rot = (int)((unsigned)rot_id % (unsigned)nrot) * (H / nrot);
    // The head of the current step and its key head, followed without a division per step.
    int head = rot, kv = rot / group, in_group = rot % group;
    auto advance = [&]() {
        ++head;
        if (++in_group == group) {
            in_group = 0;
            ++kv;
        }
        if (head == H) head = kv = in_group = 0;
    };

    // Copy the head's query tile (rows t0 .. t0 + RB - 1) into buffer buf.  Copy j of this
    // wave fills units U = (wave + NW*j)*64 + lane: row t = U / NCH, the chunk
    // stored there is (U % NCH) ^ (t & SW).  Rows past T_b are clamped (their lse2 is
    // +inf, so they weigh exactly 0); the pad chunk past d (HALF) reads chunk 0
    // instead, harmless because the matching key chunk is zero.  The per-lane byte
    // offsets are fixed; a head only moves the base.  The wave's keys likewise (keys past
    // S_b are clamped and never written).
    uint32_t qoff[QCOPIES], koff[KLDS ? KCOPIES : 1];
#pragma unroll
    for (int j = 0; j < QCOPIES; ++j) {
        const int U = (wave + NW * j) * kWave + lane;
        const int t = min(U / NCH, T - t0 - 1), ch = (U % NCH) ^ ((U / NCH) & SW);
        const int e = (HALF && ch == NCH - 1) ? 0 : ch * 8;
        qoff[j] = (uint32_t)(t * H * d + e) * 2u;
    }
    if constexpr (KLDS) {
#pragma unroll
        for (int j = 0; j < KCOPIES; ++j) {
            const int U = j * kWave + lane;
            const int kc = U / NCH, ch = (U % NCH) ^ (kc & SW);
            const int e = (HALF && ch == NCH - 1) ? 0 : ch * 8;
            koff[j] = (uint32_t)(min(wkey0 + kc, S - 1) * Hkv * d + e) * 2u;
        }
    } else {
        koff[0] = (uint32_t)(min(wkey0 + lo, S - 1) * Hkv * d) * 2u;
    }
    const char* qrows = reinterpret_cast<const char*>(q + ((size_t)qb + t0) * H * d);
    const char* ksample = reinterpret_cast<const char*>(k + (size_t)kb0 * Hkv * d);
    const uint32_t qt_lds = lds_addr(qt), kt_lds = lds_addr(kt);
    auto copy_q = [&](int buf) {
        const char* base = qrows + (size_t)head * d * 2;
#pragma unroll
        for (int j = 0; j < QCOPIES; ++j)
            if ((QTILE / kWave) % NW == 0 || wave + NW * j < QTILE / kWave)
                dma16_async(base, qoff[j],
                            qt_lds + (uint32_t)((buf * QTILE + (wave + NW * j) * kWave) * 16));
    };
    auto copy_k = [&]() {
        const char* base = ksample + (size_t)kv * d * 2;
#pragma unroll
        for (int j = 0; j < KCOPIES; ++j)
            dma16_async(base, koff[j], kt_lds + (uint32_t)(j * kWave * 16));
    };
    // Byte offset of fragment (row lo of a 32-row block, chunk hi) for k-step 0; k-step kk
    // reads (frag ^ kk*32) with SW, (frag + kk*32) without.
    const uint32_t frag = (uint32_t)(lo * NCH + (hi ^ (lo & SW))) * 16u;
    u32x4 k0[DS], k1[KLDS ? 1 : DS];
    auto read_k = [&](u32x4 (&kf)[DS]) {
#pragma unroll
        for (int kk = 0; kk < DS; ++kk) {
            const uint32_t fo = SW ? (frag ^ (uint32_t)(kk * 32)) : frag + kk * 32;
            const u32x4 v = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(kt) + fo);
            const u32x4 zero = {0u, 0u, 0u, 0u};
            kf[kk] = (HALF && kk == DS - 1 && hi) ? zero : v;
        }
#pragma unroll
        for (int kk = 0; kk < DS; ++kk) settle(kf[kk]);
    };
    auto load_k = [&](u32x4 (&kf)[DS]) {
        const char* base = ksample + (size_t)kv * d * 2 + koff[0];
#pragma unroll
        for (int kk = 0; kk < DS; ++kk)
            kf[kk] = frag16<DS, HALF>(reinterpret_cast<const uint16_t*>(base), kk, hi);
    };

    if constexpr (KLDS) copy_k();
    else load_k(k0);
    copy_q(0);
    const int nsb = min(NSB, (T - t0 + 31) >> 5);
    for (int i = tid; i < H * RB; i += kWave * NW) {
        const int hh = i / RB, t = t0 + (i % RB);
        float v = INFINITY;
        if (t < T) {
            v = lse[(size_t)(qb + t) * H + hh];
            if (lse_natural) v *= kLog2e;
        }
        l2t[i] = v;
    }
    float abar[NSB][16];
#pragma unroll
    for (int sb = 0; sb < NSB; ++sb)
#pragma unroll
        for (int r = 0; r < 16; ++r) abar[sb][r] = 0.f;
    wait_vmem();
    if constexpr (KLDS) {
        read_k(k0);
    } else {
#pragma unroll
        for (int kk = 0; kk < DS; ++kk) settle(k0[kk]);
    }
    __syncthreads();

    // One head: start the copies (or loads) of head h+1, then the MFMA logits of the wave's
    // 32 keys (kf) x RB rows, p = 2^(x - lse2) and the head sum; then wait for the copies,
    // take the next key fragments (kn) and synchronise.
    auto step = [&](int h, const u32x4 (&kf)[DS], u32x4 (&kn)[DS]) {
        const int buf = h & 1;
        const bool more = h + 1 < H;
        const float* l2h = l2t + head * RB + lo;
        const int kv_now = kv;
        advance();
        // Grouped-query heads share their keys.
        const bool nk = more && (group == 1 || kv != kv_now);
        // Nothing of this wave is in flight here except compiler reloads; waiting for them
        // now keeps the compiler from waiting inside the head, where that wait would also
        // cover the loads issued next.
        if constexpr (!KLDS) wait_vmem();
        if (more) copy_q(buf ^ 1);
        if constexpr (KLDS) {
            if (nk) copy_k();
        } else {
            load_k(kn);                          // past the last head: the first one again
        }
        if (wactive) {
            const char* qtile = reinterpret_cast<const char*>(qt) + buf * QTILE * 16;
            auto chain = [&](int sp) {
                f32x16 acc = {};
#pragma unroll
                for (int kk = 0; kk < DS; ++kk) {
                    const uint32_t fo = SW ? (frag ^ (uint32_t)(kk * 32)) : frag + kk * 32;
                    const u32x4 qv = *reinterpret_cast<const u32x4*>(qtile + sp * 32 * NCH * 16 + fo);
                    acc = mfma32(as_bf16x8(kf[kk]), as_bf16x8(qv), acc);
                }
                return acc;
            };
            auto soft = [&](int sp, const f32x16& acc) {
                const float l2 = l2h[sp * 32];
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    abar[sp][r] += __builtin_amdgcn_exp2f(fmaf(acc[r], c2, -l2));
            };
            // The chain of sub-block sp+1 is issued next to the exponentials of
            // sub-block sp (scheduling barriers keep each pair together), so the wave
            // keeps the matrix core and the vector unit busy at once; left to itself
            // the compiler issues all 32 MFMAs first.
            if (FULL || nsb == NSB) {
                f32x16 a[2] = {};
                // The first chain has nothing beside it: all its reads go out before it
                // (the order the scheduler picked by itself cost one image 0.7 us of 46).
                u32x4 q0[DS];
#pragma unroll
                for (int kk = 0; kk < DS; ++kk) {
                    const uint32_t fo = SW ? (frag ^ (uint32_t)(kk * 32)) : frag + kk * 32;
                    q0[kk] = *reinterpret_cast<const u32x4*>(qtile + fo);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int kk = 0; kk < DS; ++kk)
                    a[0] = mfma32(as_bf16x8(kf[kk]), as_bf16x8(q0[kk]), a[0]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int sp = 1; sp < NSB; ++sp) {
                    a[sp & 1] = chain(sp);
                    soft(sp - 1, a[(sp - 1) & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                soft(NSB - 1, a[(NSB - 1) & 1]);
            } else {
#pragma unroll
                for (int sp = 0; sp < NSB; ++sp) {
                    if (sp >= nsb) break;
                    soft(sp, chain(sp));
                }
            }
        }
        wait_vmem();
        if constexpr (KLDS)
            if (nk) read_k(kn);
        __syncthreads();
    };
    if constexpr (KLDS) {
        for (int h = 0; h < H; ++h) step(h, k0, k0);
    } else {
        for (int h = 0; h < H; h += 2) {
            step(h, k0, k1);
            if (h + 1 >= H) break;
            step(h + 1, k1, k0);
        }
    }

    // Row reduction of Eq. text_scoring (visual keys: max over rows, registers: mean):
    // over the lane's sub-blocks, then across the 32 lanes of a lane half (fixed
    // order).  Rows past T_b hold exact zeros.
    const bool regs = wactive && wkey0 < R;              // keys whose row sum is needed
    float mx[16], sm[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        mx[r] = abar[0][r];
        sm[r] = abar[0][r];
#pragma unroll
        for (int sb = 1; sb < NSB; ++sb) {
            mx[r] = fmaxf(mx[r], abar[sb][r]);
            sm[r] += abar[sb][r];
        }
#pragma unroll
        for (int off = 16; off >= 1; off >>= 1) {
            mx[r] = fmaxf(mx[r], __shfl_xor(mx[r], off));
            if (regs) sm[r] += __shfl_xor(sm[r], off);
        }
    }
    if (wactive && lo == 0) {
        const float invH = 1.f / (float)H;
        const float invHT = 1.f / ((float)H * (float)T);
        float* prow = part ? part + ((size_t)b * nrb + rb) * (size_t)(p.R + p.max_cands) : nullptr;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int key = wkey0 + acc_key(r, hi);
            if (key >= S) continue;
            float* dst = prow ? prow + key : scores + kb0 + key;
            const float v = prow ? (key < R ? sm[r] : mx[r]) : (key < R ? sm[r] * invHT : mx[r] * invH);
            if (cc_out) st_cc(dst, v);
            else *dst = v;
        }
    }
}

// One scoring task per workgroup.  Task = (sample, key chunk, row block), row blocks
// fastest, XCD-aware: the chunks of one sample run on one XCD and share its L2 for the
// query tiles, and the row blocks of one chunk read the same keys there.  Samples in
// reverse order: the statistics pass streamed sample B-1 last, so its keys are the
// likeliest to still sit in the memory-side cache.
// With fin.done, the last workgroup of each sample forms its scores from the row blocks'
// partials (text_rows_combine's arithmetic) and, with fin.select, applies the threshold
// and the compaction (select_kernel's arithmetic).
// FORM: the workgroup's shape (score_form).  Waves per SIMD that the registers are held to:
// the tall form needs three at d <= 80 (d = 80 otherwise takes 169 registers: 155 against 143
// us for 32 samples of 2880 keys x 128 rows), and exactly two from d = 88 (three, at d = 96,
// 330 against 302 us: the loads are then issued late).
template <int DS, bool HALF, int FORM>
__global__ __launch_bounds__(kScoreForms[FORM].waves* kWave)
    __attribute__((amdgpu_waves_per_eu(FORM == kScoreTall && DS <= 5 ? 3 : 2,
                                       FORM == kScoreTall && DS >= 6 ? 2 : 8)))
void text_score_kernel(
    Prob p, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
    const float* __restrict__ lse, int lse_natural, float* __restrict__ scores,
    float* __restrict__ part, Finish fin)
{
    extern __shared__ __attribute__((aligned(16))) char smem_raw[];
    constexpr int NW = kScoreForms[FORM].waves, RB = kScoreForms[FORM].rows, NSB = RB / 32;
    constexpr int KPW = kTxtKeysPerWave * NW, NT = NW * kWave;
    const int nchunk = (p.R + p.max_cands + KPW - 1) / KPW;
    const int nrb = (p.max_rows + RB - 1) / RB;
    int b, c, rb;
    if (p.k_off || p.q_off) {
        // The decoded task passes through the start of query buffer 1 (after the first
        // RB x d tile), which is first written (head 1's copy) after the barrier that
        // ends the task's prologue.
        int* sh = reinterpret_cast<int*>(smem_raw + (size_t)RB * 2 * DS * 16);
        if (threadIdx.x < kWave) ragged_score_task(p, (int)blockIdx.x, KPW, RB, sh);
        __syncthreads();
        b = sh[0];
        if (b < 0) return;
        c = sh[1];
        rb = sh[2];
    } else {
        const int task = xcd_remap((int)blockIdx.x, nchunk * nrb * p.B);
        rb = task % nrb;
        c = (task / nrb) % nchunk;
        b = p.B - 1 - task / (nrb * nchunk);
    }
    // The starting head follows the XCD (workgroups are dealt to the 8 XCDs round-robin,
    // and each XCD runs one contiguous range of tasks): every workgroup of an XCD walks the
    // heads in the same order, so the chunks of a sample read its query tiles, and the row
    // blocks of a chunk its key slices, at about the same time, and share them in that
    // XCD's L2: 816 MB fetched per launch at the LLaVA-NeXT shape (790 MB of keys, queries
    // and scores), 1159 MB on the video batch (1092).  A start per key chunk, measured on 128 x
    // 128 tasks, fetched 1062 MB where this order fetched 807, ~1 % slower.
    score_task<DS, HALF, NW, NSB, kScoreForms[FORM].keys_lds>(
        p, q, k, lse, lse_natural, scores, part, b, c, rb, (int)blockIdx.x, smem_raw, fin.done != nullptr);
    if (!fin.done) return;
    const int S = keys_of(p, b), T = rows_of(p, b);
    const int nrb_b = (T + RB - 1) / RB;
    const unsigned ntask = (unsigned)(((S + KPW - 1) / KPW) * nrb_b);
    if (!last_of_sample(fin.done, b, ntask, reinterpret_cast<int*>(smem_raw + 64))) return;
    if (part) {
        // Row maxima (visual keys) / row sums (registers) over the row blocks in order,
        // then the head (and row) mean: text_rows_combine's arithmetic.  Each thread takes
        // U keys at a time, so that U coherent loads per row block are in flight (one at a
        // time cost ~40 us on the video batch's 16384-key samples).  With the threshold to
        // follow, the scores also go straight into the LDS copy that it reads.
        constexpr int U = 16;
        const size_t smax = (size_t)(p.R + p.max_cands);
        const float* pb = part + (size_t)b * nrb * smax;
        float* out = scores + k_begin(p, b);
        float* sl = fin.select ? select_scores_lds(smem_raw + 128) : nullptr;
        const float inv_reg = 1.f / ((float)p.H * (float)T), inv_vis = 1.f / (float)p.H;
        for (int s0 = threadIdx.x; s0 < S; s0 += U * NT) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = 0.f;
            for (int r = 0; r < nrb_b; ++r) {
                float x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int s = s0 + u * NT;
                    x[u] = s < S ? ld<true>(pb + (size_t)r * smax + s) : 0.f;
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    v[u] = s0 + u * NT < p.R ? v[u] + x[u] : fmaxf(v[u], x[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int s = s0 + u * NT;
                if (s < S) {
                    const float w = v[u] * (s < p.R ? inv_reg : inv_vis);
                    st_cc(out + s, w);
                    if (sl) sl[s] = w;
                }
            }
        }
        if (fin.select) {
            __syncthreads();
            select_sample<NT>(p, scores, b, fin, smem_raw + 128, true);
        }
        return;
    }
    if (fin.select) select_sample<NT>(p, scores, b, fin, smem_raw + 128, false);
}

// Scores from the row blocks' partials: the maximum over row blocks (visual keys) or
// the sum in row-block order (registers), then the head mean (and row mean).
__global__ __launch_bounds__(256) void text_rows_combine_kernel(Prob p, int rb_rows,
                                                                const float* __restrict__ part,
                                                                float* __restrict__ scores)
{
    const int b = blockIdx.y, s = blockIdx.x * 256 + threadIdx.x;
    const int S = keys_of(p, b), T = rows_of(p, b);
    if (s >= S) return;
    const int nrb_max = (p.max_rows + rb_rows - 1) / rb_rows, nrb = (T + rb_rows - 1) / rb_rows;
    const size_t smax = (size_t)(p.R + p.max_cands);
    const float* pb = part + (size_t)b * nrb_max * smax + s;
    float v = 0.f;
    if (s < p.R) {
        for (int rb = 0; rb < nrb; ++rb) v += pb[(size_t)rb * smax];
        v *= 1.f / ((float)p.H * (float)T);
    } else {
        for (int rb = 0; rb < nrb; ++rb) v = fmaxf(v, pb[(size_t)rb * smax]);
        v *= 1.f / (float)p.H;
    }
    scores[k_begin(p, b) + s] = v;
}

// Key ranges of the statistics pass: merge the ranges' base-2 log-sum-exps, in range
// order, into the first table (every (row, head) entry of the workspace's tables; entries
// of rows past a sample's T_b are never read).
__global__ __launch_bounds__(256) void text_lse_merge_kernel(Prob p, float* __restrict__ lse2,
                                                             long long n)
{
    const int ns = min(p.lse_splits, kStatsMaxSplits);
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) {
        float l[kStatsMaxSplits];
        float mx = -INFINITY;
        for (int r = 0; r < ns; ++r) {
            l[r] = lse2[(size_t)r * p.lse_stride + i];
            mx = fmaxf(mx, l[r]);
        }
        float z = 0.f;
        for (int r = 0; r < ns; ++r) z += __builtin_amdgcn_exp2f(l[r] - mx);
        lse2[i] = mx == -INFINITY ? mx : mx + __builtin_amdgcn_logf(z);
    }
}

template <int DS, bool HALF, bool COLSUM, int RBW>
static hipError_t stats_launch_rbw(const Prob& p, const void* q, const void* k, float* lse2,
                                  const float* lse_in, int lse_natural, float* part,
                                  const Finish& fin, hipStream_t s) {
    const size_t smem = text_stats_smem(DS * 16, RBW);
    static std::atomic<uint64_t> lds_set{0};
    const hipError_t attr = allow_lds(
        reinterpret_cast<const void*>(&text_stats_kernel<DS, HALF, COLSUM, RBW>),
        (int)kScoreSmemMax, lds_set);
    if (attr != hipSuccess) return attr;
    const int nrb = (p.max_rows + kTxtRows - 1) / kTxtRows;
    const int ns = COLSUM || p.lse_splits < 1 ? 1 : p.lse_splits;
    const int ngrp = (nrb + RBW - 1) / RBW;
    const int units = p.B * p.Hkv * ns, per = p.H / p.Hkv * ngrp;
    const bool deal = stats_by_unit(p, ns, per, RBW);
    dim3 grid(deal ? (units + kXcds - 1) / kXcds * kXcds * per : per * units);
    const hipError_t e = launch(text_stats_kernel<DS, HALF, COLSUM, RBW>, grid,
                                dim3(kStatsThreads * RBW), smem, s, p,
                                static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(k),
                                lse2, lse_in, lse_natural, part, deal ? per : 0, fin);
    if (e != hipSuccess || ns == 1) return e;
    const long long n = p.lse_stride;
    const long long nblk = (n + 255) / 256;
    return launch(text_lse_merge_kernel, dim3((unsigned)(nblk < 2048 ? nblk : 2048)), dim3(256), 0,
                  s, p, lse2, n);
}

template <int DS, bool HALF, bool COLSUM>
static hipError_t stats_launch(const Prob& p, const void* q, const void* k, float* lse2,
                               const float* lse_in, int lse_natural, float* part,
                               const Finish& fin, hipStream_t s) {
    // The column sums keep one row block per workgroup (their partials are per row block).
    if constexpr (!COLSUM)
        if (stats_row_blocks((p.max_rows + kTxtRows - 1) / kTxtRows, !p.q_off,
                             (long long)p.B * p.H) == 2)
            return stats_launch_rbw<DS, HALF, COLSUM, 2>(p, q, k, lse2, lse_in, lse_natural, part,
                                                           fin, s);
    return stats_launch_rbw<DS, HALF, COLSUM, 1>(p, q, k, lse2, lse_in, lse_natural, part, fin, s);
}

template <int DS, bool HALF>
static hipError_t stats_ds(const Prob& p, const void* q, const void* k, float* lse2,
                           const Finish& fin, hipStream_t s) {
    return stats_launch<DS, HALF, false>(p, q, k, lse2, nullptr, 0, nullptr, fin, s);
}

template <int DS, bool HALF>
static hipError_t colsum_ds(const Prob& p, const void* q, const void* k, const float* lse,
                            int lse_natural, float* part, hipStream_t s) {
    return stats_launch<DS, HALF, true>(p, q, k, nullptr, lse, lse_natural, part, Finish{}, s);
}

// Mutual scores: the mean over rows and heads of p, from the per-(row block, head)
// column sums, added in a fixed order (row blocks outer, heads inner).
__global__ __launch_bounds__(256) void text_colsum_reduce_kernel(Prob p, const float* __restrict__ part,
                                                                 float* __restrict__ scores)
{
    const int b = blockIdx.y, s = blockIdx.x * 256 + threadIdx.x;
    const int S = keys_of(p, b), T = rows_of(p, b);
    if (s >= S) return;
    const int nrb_max = (p.max_rows + kTxtRows - 1) / kTxtRows, nrb = (T + kTxtRows - 1) / kTxtRows;
    const size_t smax = (size_t)(p.R + p.max_cands);
    const float* pb = part + (size_t)b * nrb_max * p.H * smax + s;
    // Up to 16 partials are loaded before they are added (in order): the loads do not
    // depend on the running sum, so they are in flight together.
    const int n = nrb * p.H;
    float acc = 0.f;
    int i = 0;
    for (; i + 16 <= n; i += 16) {
        float v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = pb[(size_t)(i + j) * smax];
#pragma unroll
        for (int j = 0; j < 16; ++j) acc += v[j];
    }
    for (; i < n; ++i) acc += pb[(size_t)i * smax];
    scores[k_begin(p, b) + s] = T > 0 ? acc * (1.f / ((float)p.H * (float)T)) : 0.f;
}

template <int DS, bool HALF, int FORM>
static hipError_t score_launch(const Prob& p, const void* q, const void* k, const float* lse,
                               int lse_natural, float* scores, float* part, const Finish& fin,
                               bool leave_blocks, hipStream_t s) {
    constexpr ScoreForm f = kScoreForms[FORM];
    constexpr int RB = f.rows, KPW = kTxtKeysPerWave * f.waves;
    size_t smem = score_smem(f, p.H, DS * 16);
    if (fin.select) smem = std::max(smem, 128 + select_lds_bytes(p.R, p.max_cands));
    // The tiles need more than the default 64 KB of dynamic LDS: raise the limit (once per
    // device).
    static std::atomic<uint64_t> lds_set{0};
    const hipError_t attr = allow_lds(
        reinterpret_cast<const void*>(&text_score_kernel<DS, HALF, FORM>), (int)kScoreSmemMax,
        lds_set);
    if (attr != hipSuccess) return attr;
    const int nrb = (p.max_rows + RB - 1) / RB;
    dim3 grid((p.R + p.max_cands + KPW - 1) / KPW * nrb * p.B);
    const hipError_t e = launch(text_score_kernel<DS, HALF, FORM>, grid, dim3(f.waves * kWave),
                                smem, s, p, static_cast<const uint16_t*>(q),
                                static_cast<const uint16_t*>(k), lse, lse_natural, scores,
                                nrb > 1 ? part : nullptr, fin);
    if (e != hipSuccess || nrb == 1 || fin.done || leave_blocks) return e;
    dim3 cgrid((p.R + p.max_cands + 255) / 256, p.B);
    return launch(text_rows_combine_kernel, cgrid, dim3(256), 0, s, p, RB, part, scores);
}

// (score_form takes no wide form up to d = 64 and no tall one from d = 120.)
template <int DS, bool HALF>
static hipError_t score_ds(const Prob& p, const void* q, const void* k, const float* lse,
                           int lse_natural, float* scores, float* part, const Finish& fin,
                           bool leave_blocks, hipStream_t s) {
    const int form = score_form(p);
    if constexpr (DS >= 5)
        if (form == kScoreWide)
            return score_launch<DS, HALF, kScoreWide>(p, q, k, lse, lse_natural, scores, part, fin,
                                                      leave_blocks, s);
    if constexpr (DS <= 7)
        if (form == kScoreTall)
            return score_launch<DS, HALF, kScoreTall>(p, q, k, lse, lse_natural, scores, part, fin,
                                                      leave_blocks, s);
    return score_launch<DS, HALF, kScoreNarrow>(p, q, k, lse, lse_natural, scores, part, fin,
                                                leave_blocks, s);
}

// d = 16*DS (HALF = false) or 16*DS - 8 (HALF = true), d <= 128.
#define OCCAM_D_SWITCH(FN, ...)                                                  \
    switch (p.d) {                                                               \
        case 8: return FN<1, true>(__VA_ARGS__);    case 16: return FN<1, false>(__VA_ARGS__);  \
        case 24: return FN<2, true>(__VA_ARGS__);   case 32: return FN<2, false>(__VA_ARGS__);  \
        case 40: return FN<3, true>(__VA_ARGS__);   case 48: return FN<3, false>(__VA_ARGS__);  \
        case 56: return FN<4, true>(__VA_ARGS__);   case 64: return FN<4, false>(__VA_ARGS__);  \
        case 72: return FN<5, true>(__VA_ARGS__);   case 80: return FN<5, false>(__VA_ARGS__);  \
        case 88: return FN<6, true>(__VA_ARGS__);   case 96: return FN<6, false>(__VA_ARGS__);  \
        case 104: return FN<7, true>(__VA_ARGS__);  case 112: return FN<7, false>(__VA_ARGS__); \
        case 120: return FN<8, true>(__VA_ARGS__);  case 128: return FN<8, false>(__VA_ARGS__); \
        default: return hipErrorInvalidValue;                                    \
    }

hipError_t launch_text_stats(const Prob& p, const void* q, const void* k, float* lse2,
                             const Finish& fin, hipStream_t s) {
    OCCAM_D_SWITCH(stats_ds, p, q, k, lse2, fin, s)
}

hipError_t launch_text_score(const Prob& p, const void* q, const void* k, const float* lse,
                             int lse_natural, float* scores, float* part, const Finish& fin,
                             bool leave_blocks, hipStream_t s) {
    OCCAM_D_SWITCH(score_ds, p, q, k, lse, lse_natural, scores, part, fin, leave_blocks, s)
}

static hipError_t colsum_any(const Prob& p, const void* q, const void* k, const float* lse,
                             int lse_natural, float* part, hipStream_t s) {
    OCCAM_D_SWITCH(colsum_ds, p, q, k, lse, lse_natural, part, s)
}

hipError_t launch_text_colsum(const Prob& p, const void* q, const void* k, const float* lse,
                              int lse_natural, float* part, float* scores, hipStream_t s) {
    const hipError_t e = colsum_any(p, q, k, lse, lse_natural, part, s);
    if (e != hipSuccess) return e;
    dim3 grid((p.R + p.max_cands + 255) / 256, p.B);
    return launch(text_colsum_reduce_kernel, grid, dim3(256), 0, s, p, part, scores);
}

}  // namespace occam
