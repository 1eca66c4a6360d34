// float32 masked SwiGLU FFN (for float32 weights; float32 end to end) on the float32 matrix cores
// (v_mfma_f32_16x16x4_f32: full float32 products and sums).
//
// A fragment of that instruction holds one float per lane: row (or column) lane % 16, K value lane / 16.  Both
// kernels load float4s instead and let component j of every lane be call j's fragment: lane group g = lane / 16
// then carries the K values 4 g + j (j = 0..3) of a 16-wide step, in the same order for both operands, so a
// 16-byte load feeds four calls and no lane permutation is needed.
//
// gate/up (gateup_f32_kernel), 512 threads = 8 waves, NG groups of 8 listed neurons x one block of up to 32 tokens.
//   A = 8 gate + 8 up weight rows per group; B = the FFN input, NT (1 or 2) tiles of 16 tokens.  The waves split d in units of
//   32 columns (a 128-byte line of every row), unit w, w + 8, ...: a wave copies a unit of the weight and token rows
//   into its own LDS region, 8 lanes per line, and reads the fragments there.  (A fragment loaded straight from memory
//   has 16 rows in 16 neighbouring lanes, and the L1 looks up a line per row and 16 lanes: 64 lookups for the kilobyte
//   that whole lines bring with 8.)  On the way it multiplies the input by the norm gain and adds up the tokens'
//   squares, so the kernel reads the layer's input itself: no launch prepares it.  The 8 waves' tiles
//   are added in wave order through LDS, then h = act(r g) * (r u) goes to H [slot / 16][token][slot % 16].
// down (down_f32_kernel), 512 threads, 16 CW columns x 16 NT tokens; A = H (tokens x slots), B = the listed W_down
//   rows: lane n of a group loads CW contiguous columns of a row, call q takes column q of each lane, so the 16
//   output columns of call q are CW n + q and no transpose is needed.  The waves take interleaved chunks of 16 slots,
//   PD chunks in flight; their tiles are added in wave order through LDS.  One slice: the kernel adds the residual
//   itself (kFused); several: float32 partials that the epilogue kernel adds in slice order.
//
// Rounding.  One chain of sums per wave over all its columns (d / 8) or slots (list / 8) loses more than the 8-lane dot
// products and short slices that these kernels replaced.  So gate/up starts at zero for every 8 columns and the down
// kernel for every chunk of 16 slots, and those sums are added up: error of an FFN output against 64 bits (2-norm, units of
// 2^-24; before the matrix cores, one chain, now) 6.2, 6.8, 3.9 at d = 1024 and 1229 neurons, 6.4, 8.8, 4.1 at 4096, 8.5,
// 10.6, 4.6 at d = 2048 and 5000, 3.0, 3.5, 2.8 at d = 256 and 256; the time stays (18.4 -> 18.3 us for the layer below).
//
// What bounds them.  At T = 51 a listed neuron is 12 KB of weights and 0.31 MFLOP at d = 1024: 26 FLOP per byte
// against a ridge of 28 (145 TFLOP/s measured from these instructions over a 5.2 TB/s copy), so the matrix cores have
// to be used: a vector-ALU product of 8 tokens at a time, one wave per 8 neurons, read every weight 7 times.  One
// layer of d = 1024, 1229 of 4096 neurons, 51 tokens, a norm: gate/up 136 -> 11.2 us (3.4 us of it matrix-core
// work, 7.0 the launch, the first loads' two round trips and the sum over the waves), down and epilogue 44 -> 8 us;
// the call 183 -> 18.3 us.  Four samples of it 296 -> 43 us.  More loads in flight per wave were slower in both
// kernels (that layer with one, two and three units ahead in gate/up: 19.0, 19.8, 20.1 us; with 6, 4 and 3 chunks
// in the down kernel 19.0, 18.5, 18.2, but at 2 samples of d = 1568 41.0, 41.2, 42.9).
#include <algorithm>

#include "rm_internal.h"

namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kUnit = 32;                // gate/up: columns per unit
constexpr int kPitch = kUnit * 4 + 16;   // bytes per token row in LDS (16 bytes of padding against bank conflicts)
constexpr int kChunk = rm::kF32Chunk;    // down: slots per step

__device__ __forceinline__ int clamp_neuron(int n, int d_ff) { return n < 0 ? 0 : (n >= d_ff ? d_ff - 1 : n); }
__device__ __forceinline__ int clamp_count(int c, int m) { return c < 0 ? 0 : (c > m ? m : c); }

template <int N>
using f32v = float __attribute__((ext_vector_type(N)));

__device__ __forceinline__ rm_f32x4 mfma_f32(float a, float b, rm_f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ rm_f32x4 ld16(const float *p) { return *reinterpret_cast<const rm_f32x4 *>(p); }

struct GuArgs {
    const float *wg, *wu, *x;
    const float *norm_g;  // [d], or null (no norm)
    const int32_t *idx, *count;
    float eps;
    int max_count, d_ff, d, T, kcap, act;
    int t_first, tblocks; // the launch's first token, and its token blocks
    float *H;             // [B][kcap / 16][T][16]
    // Eq. 4 (optional, [B][max_count][T]): h_anchor is subtracted from h (delta step); with h_out the kernel writes
    // h there instead of writing H (anchor step).
    const float *h_anchor;
    float *h_out;
};

template <int NT, int NG, bool kNorm>
__global__ __launch_bounds__(kThreads, 4) void gateup_f32_kernel(GuArgs a) {
    constexpr int kRows = 16 * NT;                    // token rows staged per unit
    constexpr int kPieces = kRows * kUnit / 4 / 64;   // float4 of them per lane and unit (8 lanes per row, 8 rows per load)
    constexpr int kRegion = (kRows + 16 * NG) * kPitch;  // LDS bytes per wave: token rows, then weight rows
    static_assert(NT * NG * 1024 <= kRegion, "a wave's tiles fit its region");
    const int b = blockIdx.y;
    // The token blocks of 8 neuron blocks (one per XCD) come one after the other, so that a block's weight rows are
    // read again while its XCD's L2 holds them.
    const int per = 8 * a.tblocks;
    const int within = static_cast<int>(blockIdx.x) % per;
    const int slot0 = (static_cast<int>(blockIdx.x) / per * 8 + within % 8) * 8 * NG;
    const int t0 = a.t_first + within / 8 * 16 * NT;
    const int raw_cnt = a.count[b];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // known uniform: scalar branches on it
    const int r = lane & 15;    // A row (0-7 gate, 8-15 up) and B column (token within the tile)
    const int grp = lane >> 4;  // K values 4 grp .. 4 grp + 3 of a 16-wide step
    // The block's first token row; the lane's rows below it as 32-bit offsets (rows past T repeat the last token).
    const float *xb = a.x + (static_cast<size_t>(b) * a.T + t0) * a.d;

    __shared__ __attribute__((aligned(16))) unsigned char lds[kWaves * kRegion];
    __shared__ float ssq[kWaves][kRows];
    unsigned char *region = lds + wave * kRegion;

    // With the count, the first loads out.  A slot past the list gives any neuron: its sums are not stored.
    int raw_n[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g)
        raw_n[g] = a.idx[static_cast<size_t>(b) * a.d_ff + min(slot0 + g * 8 + (lane >> 3), a.d_ff - 1)];
    __builtin_amdgcn_sched_barrier(0);
    const int units = a.d / kUnit;
    const int mine = (units - wave + kWaves - 1) / kWaves;  // units wave, wave + 8, ...
    // First column of the wave's unit k (past the end: the last unit again).
    auto col_of = [&](int k) { return min(wave + k * kWaves, units - 1) * kUnit; };
    uint32_t xoff[kPieces];
#pragma unroll
    for (int j = 0; j < kPieces; ++j) xoff[j] = min((lane >> 3) + 8 * j, a.T - 1 - t0) * a.d + (lane & 7) * 4;

    // One unit in flight beside the one in LDS (two or three were slower, see above).
    rm_f32x4 xv[kPieces], gv, w[NG][2];
    auto load_x = [&](int k) {
        const int col = col_of(k);
#pragma unroll
        for (int j = 0; j < kPieces; ++j) xv[j] = ld16(xb + col + xoff[j]);
        if constexpr (kNorm) gv = ld16(a.norm_g + col + (lane & 7) * 4);
    };
    load_x(0);
    __builtin_amdgcn_sched_barrier(0);  // the input goes out before the wait for the indices
    const int cnt = clamp_count(raw_cnt, a.max_count);
    if (slot0 >= cnt) return;  // the down projection reads no slot past the list
    size_t wrow[NG];           // neuron lane / 8 of each group: its gate and its up row
#pragma unroll
    for (int g = 0; g < NG; ++g) wrow[g] = static_cast<size_t>(clamp_neuron(raw_n[g], a.d_ff)) * a.d + (lane & 7) * 4;
    auto load_w = [&](int k) {
        const int col = col_of(k);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            w[g][0] = ld16(a.wg + wrow[g] + col);
            w[g][1] = ld16(a.wu + wrow[g] + col);
        }
    };
    load_w(0);
    __builtin_amdgcn_sched_barrier(0);

    rm_f32x4 acc[NG][NT];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) acc[g][tt] = rm_f32x4{0.f, 0.f, 0.f, 0.f};
    float ss[kPieces];
#pragma unroll
    for (int j = 0; j < kPieces; ++j) ss[j] = 0.0f;

    unsigned char *wregion = region + kRows * kPitch;
    const int piece = (lane >> 3) * kPitch + (lane & 7) * 16;  // where this lane's 16 bytes of 8 rows go
    for (int k = 0; k < mine; ++k) {
#pragma unroll
        for (int j = 0; j < kPieces; ++j) {
            rm_f32x4 v = xv[j];
            if constexpr (kNorm) {
                ss[j] = fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, fmaf(v.w, v.w, ss[j]))));
                v.x *= gv.x;
                v.y *= gv.y;
                v.z *= gv.z;
                v.w *= gv.w;
            }
            *reinterpret_cast<rm_f32x4 *>(region + 8 * j * kPitch + piece) = v;
        }
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int i = 0; i < 2; ++i)
                *reinterpret_cast<rm_f32x4 *>(wregion + (g * 16 + i * 8) * kPitch + piece) = w[g][i];
        load_x(k + 1);  // a wave's LDS operations run in order: the region is read before it is refilled
        load_w(k + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int frag = r * kPitch + i * 64 + grp * 16;
            rm_f32x4 bx[NT], aw[NG];
#pragma unroll
            for (int g = 0; g < NG; ++g)
                aw[g] = *reinterpret_cast<const rm_f32x4 *>(wregion + g * 16 * kPitch + frag);
#pragma unroll
            for (int tt = 0; tt < NT; ++tt)
                bx[tt] = *reinterpret_cast<const rm_f32x4 *>(region + tt * 16 * kPitch + frag);
#pragma unroll
            for (int j = 0; j < 4; j += 2)  // 8 columns' own sums, see above
#pragma unroll
                for (int tt = 0; tt < NT; ++tt)
#pragma unroll
                    for (int g = 0; g < NG; ++g)
                        acc[g][tt] += mfma_f32(aw[g][j + 1], bx[tt][j + 1],
                                               mfma_f32(aw[g][j], bx[tt][j], rm_f32x4{0.f, 0.f, 0.f, 0.f}));
        }
    }
    // The wave's tiles and its share of the tokens' squares.
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
            *reinterpret_cast<rm_f32x4 *>(region + ((g * NT + tt) * 64 + lane) * 16) = acc[g][tt];
    if constexpr (kNorm) {
#pragma unroll
        for (int off = 1; off < 8; off <<= 1)
#pragma unroll
            for (int j = 0; j < kPieces; ++j) ss[j] += __shfl_xor(ss[j], off);
        if ((lane & 7) == 0)
#pragma unroll
            for (int j = 0; j < kPieces; ++j) ssq[wave][(lane >> 3) + 8 * j] = ss[j];
    }
    __syncthreads();

    // Thread tid forms h for neuron tid % 8 of each group and token tid / 8.
    const int j = tid & 7, tok = tid >> 3;
    const int t = t0 + tok;
    if (tok >= kRows || t >= a.T) return;
    float rn = 1.0f;
    if constexpr (kNorm) {
        float s = ssq[0][tok];
#pragma unroll
        for (int w2 = 1; w2 < kWaves; ++w2) s += ssq[w2][tok];
        rn = rm_rnorm_from_ssq(s, a.d, a.eps);
    }
    // Gate row j of a tile: lane 16 (j / 4) + token, register j % 4; its up row is 8 further.
    const int lg = (j >> 2) * 16 + (tok & 15), lu = lg + 32, reg = j & 3;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int slot = slot0 + g * 8 + j;
        float gs = 0.f, us = 0.f;
#pragma unroll
        for (int w2 = 0; w2 < kWaves; ++w2) {
            const float *tile = reinterpret_cast<const float *>(lds + w2 * kRegion) + (g * NT + (tok >> 4)) * 256;
            gs = w2 == 0 ? tile[lg * 4 + reg] : gs + tile[lg * 4 + reg];
            us = w2 == 0 ? tile[lu * 4 + reg] : us + tile[lu * 4 + reg];
        }
        if (slot >= cnt) continue;
        float h = rm_glu_act(a.act, gs * rn) * (us * rn);
        const size_t ai = (static_cast<size_t>(b) * a.max_count + slot) * a.T + t;
        if (a.h_out != nullptr) {
            a.h_out[ai] = h;
        } else {
            if (a.h_anchor != nullptr) h -= a.h_anchor[ai];
            a.H[(static_cast<size_t>(b) * (a.kcap / kChunk) + slot / kChunk) * a.T * kChunk +
                static_cast<size_t>(t) * kChunk + slot % kChunk] = h;
        }
    }
}

struct DnArgs {
    const float *H, *wd;
    const int32_t *idx, *count;
    int max_count, d_ff, d, T, kcap;
    int slices, slice_chunks, ncol;
    int t_first;          // the launch's first token
    float *part;          // [B][slices][T][d] (several slices)
    // kFused (one slice): y = x + out_gate (ya_in + sum), ya_out = sum; all but x and y optional.
    const float *x;
    float *y;
    const float *ya_in;
    float *ya_out;
    const float *out_gate;
};

// PD: chunks in flight per wave (their registers: 4 NT + 4 CW each).
template <int NT, int CW, int PD, bool kFused>
__global__ __launch_bounds__(kThreads, 4) void down_f32_kernel(DnArgs a) {
    using vec = f32v<CW>;
    constexpr int kIdxRound = 2048;  // slots whose indices are staged in LDS at a time
    constexpr int kRoundChunks = kIdxRound / kChunk;
    static_assert(kRoundChunks % kWaves == 0, "every round starts at wave 0's chunk");
    const int ct = blockIdx.x % a.ncol;
    const int s = blockIdx.x / a.ncol % a.slices;
    const int t0 = a.t_first + static_cast<int>(blockIdx.x) / (a.ncol * a.slices) * 16 * NT;
    const int b = blockIdx.y;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // known uniform: scalar branches on it
    const int grp = lane >> 4;  // slots 4 grp .. 4 grp + 3 of a chunk
    const int nn = lane & 15;   // A row (token in tile) and B column group (columns CW nn + q)
    const int raw_cnt = a.count[b];
    const int colw = (ct * 16 + nn) * CW;
    const bool colok = colw < a.d;
    const int col = min(colw, a.d - CW);  // columns past d re-read the last ones; those outputs are not stored
    const int c_begin = s * a.slice_chunks;
    const int c_cap = min(c_begin + a.slice_chunks, a.kcap / kChunk);  // the slice's end for a list of max_count
    const float *Hb = a.H + static_cast<size_t>(b) * a.kcap * a.T;
    const int32_t *idxb = a.idx + static_cast<size_t>(b) * a.d_ff;

    __shared__ __attribute__((aligned(16))) int sidx[kIdxRound];
    __shared__ rm_f32x4 red[kWaves][CW][64];
    rm_f32x4 acc[NT][CW];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
        for (int q = 0; q < CW; ++q) acc[tt][q] = rm_f32x4{0.f, 0.f, 0.f, 0.f};

    // Everything that depends on nothing goes out first: the first round's indices, the first chunks of H, the
    // residual's inputs.  (A slot past the list has any neuron's weights; they are dropped below.)
    constexpr int kIdxPer = kIdxRound / kThreads;
    int iv[kIdxPer];
    auto load_idx = [&](int c0) {
#pragma unroll
        for (int i = 0; i < kIdxPer; ++i) iv[i] = idxb[min(c0 * kChunk + tid + i * kThreads, a.d_ff - 1)];
    };
    rm_f32x4 hv[PD][NT];
    vec wv[PD][4];
    auto load_h = [&](int p, int k, int c0) {  // chunk wave + 8 k of the round from c0 (clamped to the slice)
        const int c = min(c0 + wave + k * kWaves, c_cap - 1);
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
            hv[p][tt] = ld16(Hb + (static_cast<size_t>(c) * a.T + min(t0 + tt * 16 + nn, a.T - 1)) * kChunk + grp * 4);
    };
    load_idx(c_begin);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < PD; ++p) load_h(p, p, c_begin);
    vec xin[NT];
    if constexpr (kFused) {
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
            xin[tt] = *reinterpret_cast<const vec *>(
                a.x + (static_cast<size_t>(b) * a.T + min(t0 + tt * 16 + grp * 4 + (wave & 3), a.T - 1)) * a.d + col);
    }
    __builtin_amdgcn_sched_barrier(0);
    const int cnt = clamp_count(raw_cnt, a.max_count);
    const int c_end = min(c_cap, (cnt + kChunk - 1) / kChunk);
    if (!kFused && c_begin >= c_end) return;  // the epilogue skips the slice

    for (int c0 = c_begin; c0 < c_end; c0 += kRoundChunks) {
        const int n = min(kRoundChunks, c_end - c0);  // chunks of this round
        if (c0 > c_begin) {
            load_idx(c0);
#pragma unroll
            for (int p = 0; p < PD; ++p) load_h(p, p, c0);
            __syncthreads();  // every wave is done with the last round's indices
        }
#pragma unroll
        for (int i = 0; i < kIdxPer; ++i) sidx[tid + i * kThreads] = clamp_neuron(iv[i], a.d_ff);
        __syncthreads();
        auto load_w = [&](int p, int k) {
            const int c = min(wave + k * kWaves, n - 1);
            const int4 ni = *reinterpret_cast<const int4 *>(sidx + c * kChunk + grp * 4);
            const int row[4] = {ni.x, ni.y, ni.z, ni.w};
#pragma unroll
            for (int j = 0; j < 4; ++j)
                wv[p][j] = *reinterpret_cast<const vec *>(a.wd + static_cast<size_t>(row[j]) * a.d + col);
        };
#pragma unroll
        for (int p = 0; p < PD; ++p) load_w(p, p);
        __builtin_amdgcn_sched_barrier(0);
        for (int k0 = 0; wave + k0 * kWaves < n; k0 += PD) {
#pragma unroll
            for (int p = 0; p < PD; ++p) {
                const int c = wave + (k0 + p) * kWaves;
                if (c >= n) break;
                const int live = cnt - (c0 + c) * kChunk;  // listed slots from this chunk's first on
                if (live < kChunk) {  // the list's last chunk: nothing of a slot past the list may enter (H is unset
                                      // there, and its weights could be infinite)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const bool in = grp * 4 + j < live;
#pragma unroll
                        for (int tt = 0; tt < NT; ++tt) hv[p][tt][j] = in ? hv[p][tt][j] : 0.0f;
#pragma unroll
                        for (int q = 0; q < CW; ++q) wv[p][j][q] = in ? wv[p][j][q] : 0.0f;
                    }
                }
#pragma unroll
                for (int q = 0; q < CW; ++q) {
                    rm_f32x4 chunk[NT];  // the chunk's own sums, see above
#pragma unroll
                    for (int tt = 0; tt < NT; ++tt) chunk[tt] = rm_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int tt = 0; tt < NT; ++tt) chunk[tt] = mfma_f32(hv[p][tt][j], wv[p][j][q], chunk[tt]);
#pragma unroll
                    for (int tt = 0; tt < NT; ++tt) acc[tt][q] += chunk[tt];
                    if constexpr (NT * CW > 4) __builtin_amdgcn_sched_barrier(0);  // one column's sums at a time
                }
                load_h(p, k0 + p + PD, c0);
                load_w(p, k0 + p + PD);
            }
        }
    }

    // One token tile at a time: wave i < 4 finishes token 4 grp + i (lane L, register i of a tile: token 4 (L / 16) +
    // i, column CW (L % 16) + q of call q), the 8 waves' sums in wave order.
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
        if (tt > 0) __syncthreads();
#pragma unroll
        for (int q = 0; q < CW; ++q) red[wave][q][lane] = acc[tt][q];
        __syncthreads();
        const int t = t0 + tt * 16 + grp * 4 + (wave & 3);
        if (wave >= 4 || t >= a.T || !colok) continue;
        vec v;
#pragma unroll
        for (int q = 0; q < CW; ++q) {
            float sum = red[0][q][lane][wave];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) sum += red[w][q][lane][wave];
            v[q] = sum;
        }
        if constexpr (!kFused) {
            *reinterpret_cast<vec *>(a.part + ((static_cast<size_t>(b) * a.slices + s) * a.T + t) * a.d + colw) = v;
        } else {
            const size_t o = (static_cast<size_t>(b) * a.T + t) * a.d + colw;
            vec out = xin[tt];
            if (a.ya_in != nullptr || cnt > 0) {  // an empty list without an anchor leaves y = x bit for bit
                vec f = v;
                if (a.ya_in != nullptr) f = *reinterpret_cast<const vec *>(a.ya_in + o) + v;
                if (a.out_gate != nullptr)
                    f = f * *reinterpret_cast<const vec *>(a.out_gate + static_cast<size_t>(b) * a.d + colw);
                out = out + f;
            }
            *reinterpret_cast<vec *>(a.y + o) = out;
            if (a.ya_out != nullptr) *reinterpret_cast<vec *>(a.ya_out + o) = v;
        }
    }
}

// launch(first, n) for token blocks first .. first + n - 1: as many at a time as one grid dimension of 512-thread
// workgroups takes, `per` workgroups each.
template <typename F>
hipError_t by_token_blocks(int blocks, long long per, F launch) {
    const int most = static_cast<int>(std::max<long long>(1, (0xffffffffLL / kThreads) / per));
    for (int first = 0; first < blocks; first += most) {
        hipError_t e = launch(first, std::min(most, blocks - first));
        if (e == hipSuccess) e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

namespace rm {

hipError_t launch_gateup_f32(const Plan &p, const void *w_gate, const void *w_up, const int32_t *idx,
                             const int32_t *count, const float *x, const float *norm_g, const float *h_anchor,
                             float *h_out, void *ws, hipStream_t st) {
    GuArgs a{};
    a.wg = static_cast<const float *>(w_gate);
    a.wu = static_cast<const float *>(w_up);
    a.x = x;
    a.norm_g = norm_g;
    a.idx = idx;
    a.count = count;
    a.eps = p.eps;
    a.max_count = p.max_count;
    a.d_ff = p.d_ff;
    a.d = p.d;
    a.T = p.T;
    a.kcap = p.kcap;
    a.act = p.act;
    a.H = reinterpret_cast<float *>(static_cast<char *>(ws) + p.off_h);
    a.h_anchor = h_anchor;
    a.h_out = h_out;
    return by_token_blocks(p.f32_tblocks, p.gate_blocks, [&](int first, int n) {
        a.t_first = first * 16 * p.f32_nt;
        a.tblocks = n;
        const dim3 grid(p.gate_blocks * n, p.B), block(kThreads);
#define RM_GU(NT)                                                                                                   \
    {                                                                                                               \
        if (p.gate_groups == 2)                                                                                     \
            return a.norm_g ? launch_timed(RM_KERNEL_GATEUP, gateup_f32_kernel<NT, 2, true>, grid, block, st, a)    \
                            : launch_timed(RM_KERNEL_GATEUP, gateup_f32_kernel<NT, 2, false>, grid, block, st, a);  \
        return a.norm_g ? launch_timed(RM_KERNEL_GATEUP, gateup_f32_kernel<NT, 1, true>, grid, block, st, a)        \
                        : launch_timed(RM_KERNEL_GATEUP, gateup_f32_kernel<NT, 1, false>, grid, block, st, a);      \
    }
        switch (p.f32_nt) {
            case 1: RM_GU(1)
            default: RM_GU(2)
        }
#undef RM_GU
    });
}

hipError_t launch_down_f32(const Plan &p, const void *w_down, const int32_t *idx, const int32_t *count,
                           const float *x, float *y, const float *ya_in, float *ya_out, const float *out_gate, void *ws,
                           hipStream_t st) {
    char *base = static_cast<char *>(ws);
    DnArgs a{};
    a.H = reinterpret_cast<const float *>(base + p.off_h);
    a.wd = static_cast<const float *>(w_down);
    a.idx = idx;
    a.count = count;
    a.max_count = p.max_count;
    a.d_ff = p.d_ff;
    a.d = p.d;
    a.T = p.T;
    a.kcap = p.kcap;
    a.slices = p.slices;
    a.slice_chunks = p.slice_units / kChunk;
    a.ncol = p.ncol;
    a.part = reinterpret_cast<float *>(base + p.off_part);
    a.x = x;
    a.y = y;
    a.ya_in = ya_in;
    a.ya_out = ya_out;
    a.out_gate = out_gate;
    return by_token_blocks((p.T + 16 * p.df_nt - 1) / (16 * p.df_nt), p.ncol * p.slices, [&](int first, int n) {
        a.t_first = first * 16 * p.df_nt;
        const dim3 grid(p.ncol * p.slices * n, p.B), block(kThreads);
        if (p.df_nt == 1 && p.df_cw == 2)
            return p.fused_down ? launch_timed(RM_KERNEL_DOWN, down_f32_kernel<1, 2, 4, true>, grid, block, st, a)
                                : launch_timed(RM_KERNEL_DOWN, down_f32_kernel<1, 2, 4, false>, grid, block, st, a);
        if (p.df_nt == 2 && p.df_cw == 4)
            return p.fused_down ? launch_timed(RM_KERNEL_DOWN, down_f32_kernel<2, 4, 2, true>, grid, block, st, a)
                                : launch_timed(RM_KERNEL_DOWN, down_f32_kernel<2, 4, 2, false>, grid, block, st, a);
        return hipErrorInvalidValue;
    });
}

}  // namespace rm
