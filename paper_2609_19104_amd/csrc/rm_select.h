// Device helpers shared by the kernels that rank float32 scores: an exactly rounded product, a workgroup prefix
// sum, and the top-K selection of a workgroup of 256 or 1024 threads (group_mask.hip, context_cache.hip).
//
// Top K is an MSB-first radix select over the scores' bit patterns (non-negative floats order like their bits), taken
// relative to the smallest key and from the highest bit in which the keys differ: passes of 8 bits, each a histogram
// (per-wave LDS histograms with integer atomics, so the counts are exact, then added) and a suffix scan that finds the
// digit of the K-th largest key, until every key of that digit is taken (mostly after two passes) or the bits end;
// then, of keys equal to the K-th largest, the lowest-index ones, by ballots and a prefix sum of their counts.  Digits
// from bit 31 on would put nearly all keys of one magnitude into a few counters, whose atomics then run one by one.
#pragma once

#include "rm_internal.h"

namespace rm_sel {

constexpr int kSelThreads = 1024;      // the largest workgroup: 16384 keys
constexpr int kSelThreadsSmall = 256;  // up to 4096 keys: a quarter of the waves at each barrier
constexpr int kSelPerThread = 16;      // keys per thread

// a * b rounded to float32 on its own: the empty asm statement hides the product from the optimizer, so it
// cannot be fused with the sum it feeds into one multiply-add (HIP compiles with contraction allowed).
__device__ __forceinline__ float mul_rounded(float a, float b) {
    float p = a * b;
    asm volatile("" : "+v"(p));
    return p;
}

template <int kThreads>
struct SelLds {
    static constexpr int kWaves = kThreads / 64;
    // One histogram per wave (atomics only contend within a wave), two sets: a pass counts into one while the
    // other is cleared for the next pass.
    uint32_t whist[2][kWaves][256];
    uint32_t wave_lo[kWaves], wave_hi[kWaves];
    int wave_sum[kWaves];
    int eq_before[kSelPerThread * kWaves];  // items equal to the K-th largest before each run of 64 items
    int digit, need, in_digit;
};

// Inclusive prefix sum over the 64 lanes of a wave (every lane active), with DPP moves instead of LDS
// permutes: scans within rows of 16 lanes (row_shr 1, 2, 4, 8, a source outside the row adding 0), then row 0's
// total into row 1 and row 2's into row 3 (row_bcast:15), then rows 0-1's into rows 2-3 (row_bcast:31).
__device__ __forceinline__ int wave_incl_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);
    return x;
}

// Exclusive prefix sum of v over the workgroup, in thread order.
template <int kThreads>
__device__ __forceinline__ int block_excl_scan(int v, SelLds<kThreads> &l) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int incl = wave_incl_scan(v);
    __syncthreads();  // wave_sum may still be read by a previous call
    if (lane == 63) l.wave_sum[wave] = incl;
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wave; ++w) before += l.wave_sum[w];
    return before + incl - v;
}

// Items are dealt to the threads in turn: item i * kThreads + tid is the thread's i-th, so that a wave's loads and
// stores of one i are consecutive.  Selection bits (bit i: the thread's i-th item) of the k largest keys among the
// valid ones (bit i of `valid`), ties to the lower item index; all valid ones where they are k or fewer.  n_most: at
// least the number of valid items in the workgroup (k >= n_most saves the passes).  0 <= k; every thread of the
// workgroup calls it.
template <int kThreads>
__device__ inline uint32_t select_top_k(const uint32_t (&key)[kSelPerThread], uint32_t valid, int k, int n_most,
                                        SelLds<kThreads> &l) {
    static_assert(kThreads >= 256, "wave 0 finds the digit while at least three other waves clear histograms");
    if (k <= 0) return 0u;
    if (k >= n_most) return valid;
    constexpr int kWaves = kThreads / 64;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
    for (int i = 0; i < kSelPerThread; ++i)
        if ((valid >> i) & 1u) {
            lo = min(lo, key[i]);
            hi = max(hi, key[i]);
        }
    for (int off = 1; off < 64; off <<= 1) {
        lo = min(lo, static_cast<uint32_t>(__shfl_xor(static_cast<int>(lo), off)));
        hi = max(hi, static_cast<uint32_t>(__shfl_xor(static_cast<int>(hi), off)));
    }
    if (lane == 0) {
        l.wave_lo[wave] = lo;
        l.wave_hi[wave] = hi;
    }
    for (int b = lane; b < 256; b += 64) l.whist[0][wave][b] = 0u;
    if (tid == 0) l.digit = l.need = l.in_digit = 0;  // stays so if fewer than k are valid: every digit from 0 on is taken
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        lo = min(lo, l.wave_lo[w]);
        hi = max(hi, l.wave_hi[w]);
    }
    // Keys relative to lo, `bits` bits wide.  A pass splits the keys whose bits above `shift + width` equal prefix.
    const int bits = hi > lo ? 32 - __clz(hi - lo) : 1;
    int shift = bits, need = k;
    uint32_t prefix = 0;
    bool all = false;  // every key with the prefix is taken
    // Two barriers per pass: after the counts, and after wave 0 has found the digit (meanwhile the other waves
    // clear the other histogram set for the next pass).
    for (int pass = 0; shift > 0 && !all; ++pass) {
        const int width = min(8, shift), buf = pass & 1;
        shift -= width;
#pragma unroll
        for (int i = 0; i < kSelPerThread; ++i) {
            const uint32_t q = (key[i] - lo) >> shift;
            if (((valid >> i) & 1u) && (q >> width) == prefix)
                atomicAdd(&l.whist[buf][wave][q & ((1u << width) - 1u)], 1u);
        }
        __syncthreads();
        if (wave == 0) {  // lane j holds digits 4j .. 4j+3; find the digit holding the need-th largest key
            uint32_t b[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int w = 0; w < kWaves; ++w)
#pragma unroll
                for (int q = 0; q < 4; ++q) b[q] += l.whist[buf][w][4 * lane + q];
            const int own = static_cast<int>(b[0] + b[1] + b[2] + b[3]);
            const int incl = wave_incl_scan(own);
            const int above = __builtin_amdgcn_readlane(incl, 63) - incl;  // keys in digits above 4j + 3
            int cum = above;
#pragma unroll
            for (int q = 3; q >= 0; --q) {
                const int c = static_cast<int>(b[q]);
                if (cum < need && cum + c >= need) {
                    l.digit = 4 * lane + q;
                    l.need = need - cum;
                    l.in_digit = c;
                }
                cum += c;
            }
        } else {
            for (int w = wave - 1; w < kWaves; w += kWaves - 1)
                for (int b = lane; b < 256; b += 64) l.whist[buf ^ 1][w][b] = 0u;
        }
        __syncthreads();  // l.digit and the rest are rewritten by wave 0 only after the next pass's first barrier
        prefix = (prefix << width) | static_cast<uint32_t>(l.digit);
        need = l.need;
        all = l.in_digit == need;
    }
    // Take every key above the prefix, and those with it: all, or the `need` lowest-index ones.
    uint32_t sel = 0, eq = 0;
#pragma unroll
    for (int i = 0; i < kSelPerThread; ++i) {
        if (!((valid >> i) & 1u)) continue;
        const uint32_t q = (key[i] - lo) >> shift;
        if (q > prefix) sel |= 1u << i;
        if (q == prefix) eq |= 1u << i;
    }
    if (all) return sel | eq;
#pragma unroll
    for (int i = 0; i < kSelPerThread; ++i) {
        const unsigned long long b = __ballot((eq >> i) & 1u);
        if (lane == 0) l.eq_before[i * kWaves + wave] = __popcll(b);
    }
    __syncthreads();
    if (wave == 0) {  // their exclusive prefix sum, in item order
        constexpr int kEach = kSelPerThread * kWaves / 64;
        int c[kEach], own = 0;
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            c[j] = l.eq_before[lane * kEach + j];
            own += c[j];
        }
        int before = wave_incl_scan(own) - own;
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            l.eq_before[lane * kEach + j] = before;
            before += c[j];
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSelPerThread; ++i) {
        const unsigned long long b = __ballot((eq >> i) & 1u);
        const int rank = l.eq_before[i * kWaves + wave] + __popcll(b & ((1ull << lane) - 1ull));
        if (((eq >> i) & 1u) && rank < need) sel |= 1u << i;
    }
    return sel;
}

}  // namespace rm_sel
