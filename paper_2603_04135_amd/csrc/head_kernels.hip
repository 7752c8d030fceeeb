// HBM-bound kernels around the vocabulary GEMMs of the LM-head path: row gather and
// transposes, target logits, combination of per-tile softmax partials, the per-token
// surrogate + KL terms of Eq. 1 and their derivative, the row scales that turn a chunk of stored
// exponentials into softmax gradients (bf16 path) or the softmax-gradient pass over a stored logits
// chunk (float32 path), and the segmented (per packed sequence) loss reduction.
// All global accesses are coalesced 16-byte (or full-wave contiguous) transactions; the
// transposes go through padded LDS tiles.
#include <type_traits>

#include "token_rows.h"

namespace dppo {
namespace {

// ------------------------------------------------------------------------------------
__global__ void fill_zero_kernel(uint4* p, size_t n16, unsigned char* tail, size_t ntail, int32_t* word, int32_t* word2) {
    if (word && blockIdx.x == 0 && threadIdx.x == 0) *word = 0;
    if (word2 && blockIdx.x == 0 && threadIdx.x == 0) *word2 = 0;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
    if (blockIdx.x == 0 && threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

// ------------------------------------------------------------------------------------
// One wavefront per row of the chunk: target id and (clamped) row of H of the loss token, a copy of that row
// to Hc (zero beyond n_c), and for bfloat16 the target logit zy = H[row] . W[y] from the same registers. An id
// outside [0, V) or a position outside [0, T) is clamped into the range and reported in *status, so that every
// later gather and scatter of the call stays in bounds.
// Bound by HBM: 3 rows of D elements per token. One launch instead of three (targets, copy, dot product), the copy
// is not read back.
template <typename E>
__global__ __launch_bounds__(256) void gather_rows_kernel(GatherArgs a, int64_t n0, int32_t n_c, int32_t n_cp, int vec) {
    const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (a.flag && blockIdx.x == 0 && threadIdx.x == 0) *a.flag = 0;
    if (n >= n_cp) return;
    int64_t row = 0;
    int32_t t = 0;
    const bool valid = n < n_c;
    if (valid) {
        const int flags = locate_token(a.ids, a.loss_pos, a.T, a.V, n0 + n, row, t);
        if (flags != 0 && a.status != nullptr && lane == 0) atomicOr(a.status, flags);
    }
    if (lane == 0) {
        a.y[n] = t;
        a.rowc[n] = (int32_t)row;
    }
    const E* src = reinterpret_cast<const E*>(a.H) + (size_t)row * a.D;
    E* dst = reinterpret_cast<E*>(a.Hc) + (size_t)n * a.D;
    float s = 0.0f;
    if (vec) {                                   // rows of whole 16-byte vectors, 16-byte aligned
        constexpr int PER = 16 / (int)sizeof(E);
        const uint4* h = reinterpret_cast<const uint4*>(src);
        const uint4* w = reinterpret_cast<const uint4*>(reinterpret_cast<const E*>(a.W) + (size_t)t * a.D);
        // all loads of up to 8 vectors first: one by one, few tokens wait for memory D / 512 times over (33 tokens of D = 2560
        // 8.2 -> 5.0 us, 333 of D = 4096 12.4 -> 6.6, 8600 of D = 2560 30 -> 25.5)
        constexpr int U = 8;
        const int vectors = a.D / PER;
        for (int c0 = lane; c0 < vectors; c0 += 64 * U) {
            uint4 x[U], b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = c0 + u * 64;
                x[u] = valid && c < vectors ? h[c] : make_uint4(0, 0, 0, 0);
                if (sizeof(E) == 2) b[u] = c < vectors ? w[c] : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = c0 + u * 64;
                if (c >= vectors) break;
                reinterpret_cast<uint4*>(dst)[c] = x[u];
                if (sizeof(E) == 2) s = dot_bf16x8(x[u], b[u], s);
            }
        }
    } else {
        for (int d = lane; d < a.D; d += 64) dst[d] = valid ? src[d] : (E)0;
    }
    if (sizeof(E) == 4) return;
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) {
        a.zy[n] = s;
        if (a.bref) a.bref[n] = s;
    }
}

// ------------------------------------------------------------------------------------
// Per-tile softmax partials part[tile][n] of TOK tokens per workgroup -> lse and log-prob. The tiles are split over
// COMBINE_THREADS / TOK lane groups, eight loads in flight per thread; the groups meet by shuffles and in LDS, in a fixed
// order. Bound by HBM for many tokens (8 bytes per tile and token) and by latency for few: with 64 tokens and 4 groups per
// workgroup, a thread walked 149 dependent loads and 256 tokens kept four workgroups busy (V = 151936, 33 tokens:
// 68 us of a 276 us call; 16 tokens and 32 groups 8.6 us, 64 groups 9.5).
// From COMBINE_WIDE_TOKENS on, where 32 tokens a workgroup still give every compute unit one, 256 bytes in a row are read
// instead of 128: 32768 tokens of V = 151936 30 us (16 tokens and 32 groups 35, 64 groups 44), 18688 of V = 32000
// 6.2 us (8.5, 13.4); 4096 tokens of V = 151936 8.6 against 7.7 us with 16.
constexpr int COMBINE_THREADS = 512, COMBINE_WAVES = COMBINE_THREADS / 64;
constexpr int COMBINE_WIDE_TOKENS = 8192;
constexpr int COMBINE_UNROLL = 8;

// (max, sum exp(z - max)) of the union of two sets.
__device__ __forceinline__ float2 join_softmax(float2 a, float2 b) {
    const float m = fmaxf(a.x, b.x);
    if (m == -__builtin_inff()) return make_float2(m, 0.0f);
    return make_float2(m, a.y * expf(a.x - m) + b.y * expf(b.x - m));
}
// (max z, sum exp(z - reference)) with one reference per token: the sums just add up.
__device__ __forceinline__ float2 join_referenced(float2 a, float2 b) { return make_float2(fmaxf(a.x, b.x), a.y + b.y); }

// The token's joined pair, valid in the first TOK threads of the workgroup.
template <bool REFERENCED, int TOK>
__device__ __forceinline__ float2 combine_tiles(const float2* __restrict__ part, int32_t n_tiles, int32_t pitch, int32_t n_c, int n) {
    constexpr int GROUPS = COMBINE_THREADS / TOK;
    __shared__ float2 red[COMBINE_WAVES][TOK];
    const int group = threadIdx.x / TOK, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto join = [](float2 a, float2 b) { return REFERENCED ? join_referenced(a, b) : join_softmax(a, b); };
    const float2 none = make_float2(-__builtin_inff(), 0.0f);
    float2 r = none;
    if (n < n_c) {
        for (int t0 = group; t0 < n_tiles; t0 += GROUPS * COMBINE_UNROLL) {
            float2 p[COMBINE_UNROLL];
#pragma unroll
            for (int u = 0; u < COMBINE_UNROLL; ++u) {
                const int t = t0 + u * GROUPS;
                p[u] = t < n_tiles ? part[(size_t)t * pitch + n] : none;
            }
            float m = r.x, s = 0.0f;
#pragma unroll
            for (int u = 0; u < COMBINE_UNROLL; ++u) m = fmaxf(m, p[u].x);
            const bool any = m != none.x;
#pragma unroll
            for (int u = 0; u < COMBINE_UNROLL; ++u) s += REFERENCED ? p[u].y : any ? p[u].y * expf(p[u].x - m) : 0.0f;
            r = make_float2(m, s + (REFERENCED ? r.y : any ? r.y * expf(r.x - m) : 0.0f));
        }
    }
#pragma unroll
    for (int off = TOK; off < 64; off <<= 1)
        r = join(r, make_float2(__shfl_xor(r.x, off, 64), __shfl_xor(r.y, off, 64)));
    if (lane < TOK) red[wave][lane] = r;
    __syncthreads();
    if (threadIdx.x < TOK) {
        r = red[0][threadIdx.x];
        for (int w = 1; w < COMBINE_WAVES; ++w) r = join(r, red[w][threadIdx.x]);
    }
    return r;
}

template <int TOK>
__global__ __launch_bounds__(COMBINE_THREADS) void combine_logprob_kernel(
    const float2* __restrict__ part, int32_t n_tiles, int32_t pitch, const float* __restrict__ zy, int64_t n0, int32_t n_c,
    int32_t n_cp, float* __restrict__ lse_chunk, float* __restrict__ logp_out, float* __restrict__ lse_out) {
    const int n = blockIdx.x * TOK + threadIdx.x % TOK;
    const float2 r = combine_tiles<false, TOK>(part, n_tiles, pitch, n_c, n);
    if (threadIdx.x >= TOK || n >= n_cp) return;
    if (n >= n_c) { lse_chunk[n] = 0.0f; return; }
    const float lse = r.x + logf(r.y);
    lse_chunk[n] = lse;
    logp_out[n0 + n] = zy[n] - lse;
    if (lse_out) lse_out[n0 + n] = lse;
}

// The same for the GEMM that stores exponentials: part[tile][n] = (max z, sum of exp(z - bref[n])),
// lse = bref + log(sum). With the target logit as reference the sum is 1 / p(target), the stored
// exponentials reach that size and the row scale c p(target) shrinks by it; beyond 1e15 (a target
// token with log-prob below about -34.5) the scaled hidden-state rows of the dW operand would
// approach the bottom of the bf16 range for small loss weights, so the token goes on the redo
// list instead and is redone against its row maximum.
constexpr float EXP_SUM_LIMIT = 1e15f;
template <int TOK>
__global__ __launch_bounds__(COMBINE_THREADS) void combine_exp_kernel(
    const float2* __restrict__ part, int32_t n_tiles, const float* __restrict__ zy, const float* __restrict__ bref, int64_t n0,
    int32_t n_c, int32_t n_cp, float* __restrict__ lse_chunk, float* __restrict__ logp_out, float* __restrict__ mx,
    int32_t* redo_count, int32_t* __restrict__ redo_list, float* __restrict__ redo_sum) {
    const int n = blockIdx.x * TOK + threadIdx.x % TOK;
    const float2 r = combine_tiles<true, TOK>(part, n_tiles, n_cp, n_c, n);
    if (threadIdx.x >= TOK || n >= n_cp) return;
    mx[n] = r.x;
    if (n >= n_c) { lse_chunk[n] = 0.0f; return; }
    if (!(r.y < EXP_SUM_LIMIT)) {
        redo_list[atomicAdd(redo_count, 1)] = n;
        redo_sum[n] = 0.0f;
        return;
    }
    const float lse = bref[n] + logf(r.y);
    lse_chunk[n] = lse;
    logp_out[n0 + n] = zy[n] - lse;
}

// Slow exact path for the tokens on the redo list: E[n, v] = exp(Hc[n] . W[v] - mx[n]) with fp32
// dot products, 8 listed tokens x 256 vocabulary entries per workgroup pass (one thread per
// vocabulary entry, the token rows in LDS in slabs of REDO_SLAB columns), row sums by atomic adds.
constexpr int REDO_TOK = 8, REDO_SLAB = 2048;
__global__ __launch_bounds__(256) void exp_redo_rows_kernel(const int32_t* redo_count,
                                                            const int32_t* __restrict__ redo_list,
                                                            const uint16_t* __restrict__ Hc,
                                                            const uint16_t* __restrict__ W, int32_t V, int32_t D,
                                                            const float* __restrict__ mx, uint16_t* __restrict__ E,
                                                            int64_t lde, float* redo_sum) {
    __shared__ uint4 hs[REDO_TOK][REDO_SLAB / 8];
    const int cnt = *reinterpret_cast<const volatile int32_t*>(redo_count);
    const int v = blockIdx.x * 256 + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const int vr = v < V ? v : V - 1;
    for (int g = blockIdx.y; g * REDO_TOK < cnt; g += gridDim.y) {
        const int nt = (cnt - g * REDO_TOK) < REDO_TOK ? (cnt - g * REDO_TOK) : REDO_TOK;
        float acc[REDO_TOK];
#pragma unroll
        for (int t = 0; t < REDO_TOK; ++t) acc[t] = 0.0f;
        for (int d0 = 0; d0 < D; d0 += REDO_SLAB) {
            const int dw = ((D - d0) < REDO_SLAB ? (D - d0) : REDO_SLAB) / 8;   // 16-byte pieces of the slab
            __syncthreads();
            for (int i = threadIdx.x; i < REDO_TOK * dw; i += 256) {
                const int t = i / dw, c = i % dw;
                uint4 x = make_uint4(0, 0, 0, 0);
                if (t < nt) x = *reinterpret_cast<const uint4*>(Hc + (size_t)redo_list[g * REDO_TOK + t] * D + d0 + c * 8);
                hs[t][c] = x;
            }
            __syncthreads();
            const uint4* wr = reinterpret_cast<const uint4*>(W + (size_t)vr * D + d0);
            for (int c = 0; c < dw; ++c) {
                const uint4 w8 = wr[c];
                const uint32_t ww[4] = {w8.x, w8.y, w8.z, w8.w};
#pragma unroll
                for (int t = 0; t < REDO_TOK; ++t) {
                    const uint4 h8 = hs[t][c];
                    const uint32_t hh[4] = {h8.x, h8.y, h8.z, h8.w};
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        acc[t] = fmaf(__uint_as_float(ww[k] << 16), __uint_as_float(hh[k] << 16), acc[t]);
                        acc[t] = fmaf(__uint_as_float(ww[k] & 0xffff0000u), __uint_as_float(hh[k] & 0xffff0000u), acc[t]);
                    }
                }
            }
        }
#pragma unroll
        for (int t = 0; t < REDO_TOK; ++t) {
            if (t >= nt) break;                                  // uniform over the workgroup
            const int64_t n = redo_list[g * REDO_TOK + t];
            float e = v < V ? expf(acc[t] - mx[n]) : 0.0f;
            const __bf16 eb = (__bf16)e;
            constexpr int64_t BR = 64, BC = 256;                 // blocked chunk layout; v < lde by the grid
            E[(size_t)(n / BR) * BR * lde + (size_t)(v / BC) * (BR * BC) + (n % BR) * BC + v % BC] =
                __builtin_bit_cast(uint16_t, eb);
            for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off, 64);
            if (lane == 0) atomicAdd(redo_sum + n, e);
        }
    }
}

__global__ void exp_redo_finish_kernel(const int32_t* redo_count, const int32_t* __restrict__ redo_list,
                                       const float* __restrict__ redo_sum, const float* __restrict__ zy,
                                       const float* __restrict__ mx, int64_t n0, float* __restrict__ bref,
                                       float* __restrict__ lse_chunk, float* __restrict__ logp_out) {
    const int cnt = *reinterpret_cast<const volatile int32_t*>(redo_count);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += gridDim.x * blockDim.x) {
        const int n = redo_list[i];
        const float lse = mx[n] + logf(redo_sum[n]);
        bref[n] = mx[n];
        lse_chunk[n] = lse;
        logp_out[n0 + n] = zy[n] - lse;
    }
}

// Row scale of the stored exponentials and their entry at the target: with E[n, v] = exp(z - b[n]),
// c[n] (1[v = y] - p[n, v]) = s[n] E'[n, v] for s[n] = -c[n] exp(b[n] - lse[n]) and E' = E except
// E'[n, y[n]] = exp(zy[n] - b[n]) - exp(lse[n] - b[n]). Rows beyond n_c get s = 0.
__global__ void softmax_scale_kernel(const int32_t* __restrict__ y, const float* __restrict__ zy,
                                     const float* __restrict__ bref, const float* __restrict__ lse,
                                     const float* __restrict__ cvec, int32_t n_c, int32_t n_cp,
                                     uint16_t* __restrict__ E, int64_t lde, float* __restrict__ scale) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= n_cp) return;
    if (n >= n_c) { scale[n] = 0.0f; return; }
    const float b = bref[n], l = lse[n];
    scale[n] = -cvec[n] * expf(b - l);
    const __bf16 e = (__bf16)(expf(zy[n] - b) - expf(l - b));
    const int64_t v = y[n];
    constexpr int64_t BR = 64, BC = 256;   // blocked chunk layout
    E[(size_t)(n / BR) * BR * lde + (size_t)(v / BC) * (BR * BC) + (n % BR) * BC + v % BC] =
        __builtin_bit_cast(uint16_t, e);
}

// bf16 transpose by 16-byte accesses: dstT[c, r] = scale[r] * src[r, c] (scale NULL = 1) for
// r < rows_out, c < cols; source rows >= rows_valid read as zero. cols and rows_out are
// multiples of 64, all pointers and pitches multiples of 8 elements. A 64 x 64 tile goes through
// LDS; every thread loads and stores whole 8-element vectors. dstT has the blocked B-operand layout of the
// MFMA GEMMs: blocks of GEMM_B_BLOCK_ROWS rows x GEMM_B_BLOCK_K columns, block (i, j) at
// (i * rows_out / GEMM_B_BLOCK_K + j) blocks from the start (a 64 x 64 tile is then one contiguous 8 KB run).
__global__ __launch_bounds__(256) void transpose_bf16_kernel(const uint16_t* __restrict__ src, int64_t ld_src,
                                                             int32_t rows_valid, const float* __restrict__ scale,
                                                             uint16_t* __restrict__ dstT, int64_t rows_out) {
    __shared__ uint16_t tile[64][64 + 2];
    const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
    const int vec = threadIdx.x & 7, line = threadIdx.x >> 3;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        const int rr = line + pass * 32, r = r0 + rr;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (r < rows_valid) v = *reinterpret_cast<const uint4*>(src + (int64_t)r * ld_src + c0 + vec * 8);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        if (scale && r < rows_valid) {
            const float sc = scale[r];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const __bf16 lo = (__bf16)(sc * __uint_as_float(w[k] << 16));
                const __bf16 hi = (__bf16)(sc * __uint_as_float(w[k] & 0xffff0000u));
                tile[rr][vec * 8 + 2 * k] = __builtin_bit_cast(uint16_t, lo);
                tile[rr][vec * 8 + 2 * k + 1] = __builtin_bit_cast(uint16_t, hi);
            }
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                tile[rr][vec * 8 + 2 * k] = (uint16_t)(w[k] & 0xffffu);
                tile[rr][vec * 8 + 2 * k + 1] = (uint16_t)(w[k] >> 16);
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        const int cc = line + pass * 32;
        uint32_t w[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            w[k] = (uint32_t)tile[vec * 8 + 2 * k][cc] | ((uint32_t)tile[vec * 8 + 2 * k + 1][cc] << 16);
        static_assert(GEMM_B_BLOCK_K == 64, "a 64-column tile = one block column");
        const int64_t drow = c0 + cc;
        const int64_t off = ((drow / GEMM_B_BLOCK_ROWS) * (rows_out / GEMM_B_BLOCK_K) + r0 / GEMM_B_BLOCK_K) *
                                (int64_t)(GEMM_B_BLOCK_ROWS * GEMM_B_BLOCK_K) +
                            (drow % GEMM_B_BLOCK_ROWS) * GEMM_B_BLOCK_K + vec * 8;
        *reinterpret_cast<uint4*>(dstT + off) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// fp32 path: one workgroup per token over the stored logits row (pitch a multiple of 256 columns, those beyond V hold
// anything), which is read once, eight 16-byte vectors in flight per thread; up to V = 16384 that is the whole row, and the sums are
// formed against each thread's maximum with one rescaling when the threads meet. NaN entries reach the result.
// Bound by HBM, 4 bytes per logit. As two passes of single dependent loads it took 227 us for 2400 tokens of V = 32000 (309 MB);
// the call of 4.73 ms is 0.15 ms shorter.
constexpr int ROW_THREADS = 512, ROW_UNROLL = 8;
__device__ __forceinline__ float2 join_row(float2 a, float2 b) {
    const float m = fmaxf(a.x, b.x), ref = m == -__builtin_inff() ? 0.0f : m;
    return make_float2(m, a.y * expf(a.x - ref) + b.y * expf(b.x - ref));
}
__global__ __launch_bounds__(ROW_THREADS) void row_stats_kernel(const float* __restrict__ Z, int64_t ldz, int32_t V,
                                                                const int32_t* __restrict__ y, TokenArgs a, int64_t n0, int32_t n_c,
                                                                float* __restrict__ lse_chunk, float* __restrict__ logp_out,
                                                                float* __restrict__ lse_out) {
    __shared__ float2 red[ROW_THREADS / 64];
    const int n = blockIdx.x;
    if (n >= n_c) { if (threadIdx.x == 0) lse_chunk[n] = 0.0f; return; }
    const float* z = Z + (size_t)n * ldz;
    int32_t target;                               // (y NULL: the token was not gathered)
    if (y != nullptr) {
        target = y[n];
    } else {
        int64_t row;
        const int flags = locate_token(a.ids, a.loss_pos, a.T, a.V, n0 + n, row, target);
        if (flags != 0 && a.status != nullptr && threadIdx.x == 0) atomicOr(a.status, flags);
    }
    const float NONE = -__builtin_inff();
    float2 r = make_float2(NONE, 0.0f);
    const int vectors = (V + 3) / 4;
    for (int i0 = threadIdx.x; i0 < vectors; i0 += ROW_THREADS * ROW_UNROLL) {
        float p[ROW_UNROLL][4];
#pragma unroll
        for (int u = 0; u < ROW_UNROLL; ++u) {
            const int i = i0 + u * ROW_THREADS;
            float4 x = make_float4(NONE, NONE, NONE, NONE);
            if (i < vectors) x = reinterpret_cast<const float4*>(z)[i];
            const float xx[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) p[u][q] = i * 4 + q < V ? xx[q] : NONE;
        }
        float m = NONE, s = 0.0f;
#pragma unroll
        for (int u = 0; u < ROW_UNROLL; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) m = fmaxf(m, p[u][q]);
        const float ref = m == NONE ? 0.0f : m;
#pragma unroll
        for (int u = 0; u < ROW_UNROLL; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) s += expf(p[u][q] - ref);
        r = join_row(r, make_float2(m, s));
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) r = join_row(r, make_float2(__shfl_xor(r.x, off, 64), __shfl_xor(r.y, off, 64)));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < ROW_THREADS / 64; ++w) r = join_row(r, red[w]);
        const float lse = r.x + logf(r.x == NONE ? __builtin_nanf("") : r.y);
        if (lse_chunk) lse_chunk[n] = lse;
        logp_out[n0 + n] = z[target] - lse;
        if (lse_out) lse_out[n0 + n] = lse;
    }
}

// ------------------------------------------------------------------------------------
// Per-token terms of Eq. 1 and d(loss)/d(logp), weighted by seq_coef / C_s (token-sum aggregation:
// by seq_coef). With a sequence-level ratio every token of a sequence uses the same rho.
__device__ __forceinline__ int packed_sequence(const TokenLossArgs& a, int64_t gi) {
    int lo = 0, hi = a.S;          // largest s with loss_cu[s] <= gi
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((int64_t)a.loss_cu[mid] <= gi) lo = mid; else hi = mid;
    }
    return lo;
}
// Terms of loss token gi of sequence s with log-prob lp; returns d(loss)/d(logp).
__device__ __forceinline__ float token_terms(const TokenLossArgs& a, int64_t gi, int s, float lp) {
    const float A = a.seq_adv[s];
    const float w = a.aggregation == DPPO_AGG_TOKEN_SUM ? a.seq_coef[s]
                                                       : a.seq_coef[s] / (float)(a.loss_cu[s + 1] - a.loss_cu[s]);
    const float d_old = lp - a.logp_old[gi];
    const float d_ref = a.logp_ref[gi] - lp;
    const float rho = a.ratio_level == DPPO_RATIO_SEQUENCE ? a.seq_ratio[s] : expf(d_old);
    const float unclipped = rho * A;
    const float clipped = fminf(fmaxf(rho, a.lo), a.hi) * A;
    const float sur = fminf(unclipped, clipped);
    const float em1 = expm1f(d_ref);             // rho_hat - 1
    const float kl = em1 - d_ref;                // rho_hat - log rho_hat - 1
    const bool away = (A > 0.0f && rho > a.hi) || (A < 0.0f && rho < a.lo);
    const float g = (away ? 0.0f : -A * rho) - a.beta * em1;
    a.ell[gi] = -sur + a.beta * kl;
    a.kl[gi] = kl;
    a.clipped[gi] = away ? 1.0f : 0.0f;
    return w * g;
}
__global__ void token_loss_kernel(TokenLossArgs a, int64_t n0, int32_t n_c, int32_t n_cp) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= n_cp) return;
    if (n >= n_c) { a.c_chunk[n] = 0.0f; return; }
    const int64_t gi = n0 + n;
    a.c_chunk[n] = token_terms(a, gi, packed_sequence(a, gi), a.logp[gi]);
}

// ------------------------------------------------------------------------------------
// float32 path: softmax-gradient pass over the stored logits, in place, one 16-byte vector per thread (the pitch is
// a multiple of 256 columns). Bound by HBM: 8 bytes per logit.
__global__ __launch_bounds__(256) void grad_logits_kernel(float* __restrict__ ZG, int32_t V, int32_t Vp,
                                                          const int32_t* __restrict__ y, const float* __restrict__ lse,
                                                          const float* __restrict__ cvec) {
    const int n = blockIdx.x;
    const float l = lse[n], cn = cvec[n];
    const int yt = y[n];
    float4* row = reinterpret_cast<float4*>(ZG + (size_t)n * Vp);
    for (int i = blockIdx.y * 256 + threadIdx.x; i < Vp / 4; i += gridDim.y * 256) {
        const float4 z = row[i];
        const float zz[4] = {z.x, z.y, z.z, z.w};
        float g[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int v = i * 4 + q;
            const float gv = cn * ((v == yt ? 1.0f : 0.0f) - expf(zz[q] - l));
            g[q] = v < V ? gv : 0.0f;
        }
        row[i] = make_float4(g[0], g[1], g[2], g[3]);
    }
}

// float32 path with a token-level ratio: everything between the logits GEMM and the backward GEMMs, one workgroup per loss
// token: row statistics as in row_stats_kernel, log-prob, the token's terms of Eq. 1, and the row's logits turned into
// softmax-gradient entries in place. Up to THREADS * NV vectors the row stays in registers in between; a longer one (LONG) is
// read again, from the L2 (128 KB and more). Bound by HBM: 8 bytes per logit instead of 12, and one launch instead of three:
// 2400 tokens of V = 32000 92 + 70 + 5 us -> 124 us (5.0 TB/s); 100 tokens of V = 512, whole step 41.6 -> 33.5 us.
template <int THREADS, int NV, bool LONG>
__global__ __launch_bounds__(THREADS) void loss_rows_kernel(float* __restrict__ ZG, int32_t V, int32_t Vp,
                                                            const int32_t* __restrict__ y, TokenLossArgs a, float* __restrict__ logp,
                                                            int64_t n0) {
    __shared__ float2 red[THREADS / 64];
    __shared__ float s_c;
    const int n = blockIdx.x;
    const int64_t gi = n0 + n;
    float* z = ZG + (size_t)n * Vp;
    const int yt = y[n];
    const float NONE = -__builtin_inff();
    const int vectors = (V + 3) / 4;
    float p[NV][4];
    auto load = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int i = i0 + u * THREADS;
            float4 x = make_float4(NONE, NONE, NONE, NONE);
            if (i < vectors) x = reinterpret_cast<const float4*>(z)[i];
            const float xx[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) p[u][q] = i * 4 + q < V ? xx[q] : NONE;
        }
    };
    float2 r = make_float2(NONE, 0.0f);
    const float zy = z[yt];
    for (int i0 = threadIdx.x; i0 < (LONG ? vectors : THREADS); i0 += THREADS * NV) {
        load(i0);
        float m = NONE, s = 0.0f;
#pragma unroll
        for (int u = 0; u < NV; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) m = fmaxf(m, p[u][q]);
        const float ref = m == NONE ? 0.0f : m;
#pragma unroll
        for (int u = 0; u < NV; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) s += expf(p[u][q] - ref);
        r = join_row(r, make_float2(m, s));
    }
    const int sequence = packed_sequence(a, gi);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) r = join_row(r, make_float2(__shfl_xor(r.x, off, 64), __shfl_xor(r.y, off, 64)));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = r;
    __syncthreads();
    r = red[0];
#pragma unroll
    for (int w = 1; w < THREADS / 64; ++w) r = join_row(r, red[w]);
    const float lse = r.x + logf(r.x == NONE ? __builtin_nanf("") : r.y);
    if (threadIdx.x == 0) {
        const float lp = zy - lse, c = token_terms(a, gi, sequence, lp);
        logp[gi] = lp;
        s_c = c;
    }
    __syncthreads();                              // (zy has been read by every thread before the row is overwritten)
    const float c = s_c;
    for (int i0 = threadIdx.x; i0 < (LONG ? Vp / 4 : THREADS); i0 += THREADS * NV) {
        if (LONG) load(i0);
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int i = i0 + u * THREADS;
            if (i >= Vp / 4) break;
            float g[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int v = i * 4 + q;
                const float gv = c * ((v == yt ? 1.0f : 0.0f) - expf(p[u][q] - lse));
                g[q] = v < V ? gv : 0.0f;
            }
            reinterpret_cast<float4*>(z)[i] = make_float4(g[0], g[1], g[2], g[3]);
        }
    }
}

// One workgroup per packed sequence: exp of the mean log-ratio over its tokens, for the sequences
// that end in the token range (n_lo, n_hi] (all their log-probs are known once the tokens below
// n_hi are). A sequence that starts below n_lo and ends beyond n_hi is longer than the caller
// promised: it is flagged in `status` (its ratio is not written by this launch).
__global__ __launch_bounds__(256) void seq_ratio_kernel(const int32_t* __restrict__ loss_cu, int32_t S,
                                                        const float* __restrict__ logp,
                                                        const float* __restrict__ logp_old,
                                                        float* __restrict__ seq_ratio, int64_t n_lo, int64_t n_hi,
                                                        int32_t* __restrict__ status) {
    __shared__ float r0[256];
    for (int s = blockIdx.x; s < S; s += gridDim.x) {
        const int b = loss_cu[s], e = loss_cu[s + 1];
        if (e > n_hi) {
            if (b < n_lo && status && threadIdx.x == 0) atomicOr(status, DPPO_HEAD_SEQ_TOO_LONG);
            continue;
        }
        if (e <= n_lo) continue;
        float x = 0.0f;
        for (int i = b + threadIdx.x; i < e; i += 256) x += logp[i] - logp_old[i];
        r0[threadIdx.x] = x;
        __syncthreads();
        for (int st = 128; st > 0; st >>= 1) {
            if (threadIdx.x < st) r0[threadIdx.x] += r0[threadIdx.x + st];
            __syncthreads();
        }
        if (threadIdx.x == 0) seq_ratio[s] = e > b ? expf(r0[0] / (float)(e - b)) : 1.0f;
        __syncthreads();
    }
}

// One wavefront per prompt group: coef * G / (completion tokens of the whole group). Bound by latency: 256 groups of 16, one
// thread per group with a chain of loads and stores, 6.5 us; 2.6 us.
__global__ __launch_bounds__(256) void token_norm_coef_kernel(int32_t Q, int32_t G, const int32_t* __restrict__ comp_len,
                                                              const float* coef, float* coef_out) {
    const int q = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (q >= Q) return;
    int64_t tot = 0;
    for (int i = lane; i < G; i += 64) tot += comp_len[(size_t)q * G + i];
    for (int off = 32; off > 0; off >>= 1) tot += __shfl_xor(tot, off, 64);
    const float f = tot > 0 ? (float)((double)G / (double)tot) : 0.0f;
    for (int i = lane; i < G; i += 64) coef_out[(size_t)q * G + i] = coef[(size_t)q * G + i] * f;
}

// ------------------------------------------------------------------------------------
// Weighted sum over the sequences in fp64 by one workgroup of 256 threads, fixed order.
__device__ __forceinline__ void final_reduce(const SeqReduceArgs& a) {
    __shared__ double r0[256], r1[256], r2[256];
    double x0 = 0.0, x1 = 0.0, x2 = 0.0;
    for (int s = threadIdx.x; s < a.S; s += 256) {
        x0 += (double)a.seq_coef[s] * (double)a.seq_mean[s];
        x1 += (double)a.seq_kl[s];
        x2 += (double)a.seq_clip[s];
    }
    r0[threadIdx.x] = x0; r1[threadIdx.x] = x1; r2[threadIdx.x] = x2;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (threadIdx.x < st) {
            r0[threadIdx.x] += r0[threadIdx.x + st];
            r1[threadIdx.x] += r1[threadIdx.x + st];
            r2[threadIdx.x] += r2[threadIdx.x + st];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        a.loss_out[0] = (float)r0[0];
        if (a.stats_out) {
            const double n = a.N > 0 ? (double)a.N : 1.0;
            a.stats_out[0] = (float)(r1[0] / n);
            a.stats_out[1] = (float)(r2[0] / n);
            a.stats_out[2] = (float)a.N;
            a.stats_out[3] = 0.0f;
        }
    }
}

// One workgroup per packed sequence: token-mean (or token-sum) loss, KL sum, clipped count. The last workgroup to finish also
// forms the totals: a launch less, 104 -> 100 us for the smallest step (which workgroup that is does not change the order of any sum).
// *done counts them; it is zero when the launch starts.
__global__ __launch_bounds__(256) void seq_reduce_kernel(SeqReduceArgs a) {
    __shared__ float r0[256], r1[256], r2[256];
    __shared__ int s_last;
    for (int s = blockIdx.x; s < a.S; s += gridDim.x) {
        const int b = a.loss_cu[s], e = a.loss_cu[s + 1];
        float x0 = 0.0f, x1 = 0.0f, x2 = 0.0f;
        for (int i = b + threadIdx.x; i < e; i += 256) { x0 += a.ell[i]; x1 += a.kl[i]; x2 += a.clipped[i]; }
        r0[threadIdx.x] = x0; r1[threadIdx.x] = x1; r2[threadIdx.x] = x2;
        __syncthreads();
        for (int st = 128; st > 0; st >>= 1) {
            if (threadIdx.x < st) {
                r0[threadIdx.x] += r0[threadIdx.x + st];
                r1[threadIdx.x] += r1[threadIdx.x + st];
                r2[threadIdx.x] += r2[threadIdx.x + st];
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            // an empty segment contributes nothing (its sums are 0)
            const float mean = (a.aggregation == DPPO_AGG_TOKEN_SUM || e <= b) ? r0[0] : r0[0] / (float)(e - b);
            a.seq_mean[s] = mean;
            a.seq_kl[s] = r1[0];
            a.seq_clip[s] = r2[0];
            if (a.seq_loss_out) a.seq_loss_out[s] = mean;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        __threadfence();             // this workgroup's sums before its count
        s_last = atomicAdd(a.done, 1) == (int)gridDim.x - 1;
        __threadfence();             // the others' sums behind theirs
    }
    __syncthreads();
    if (s_last) final_reduce(a);
}

__global__ __launch_bounds__(256) void no_sequences_kernel(SeqReduceArgs a) { final_reduce(a); }

}  // namespace

// ======================================================================================
void launch_fill_zero(void* p, size_t bytes, int32_t* word, hipStream_t st, int32_t* word2) {
    if (bytes == 0 && !word && !word2) return;
    const size_t n16 = bytes / 16, ntail = bytes % 16;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks == 0) blocks = 1;
    fill_zero_kernel<<<(unsigned)blocks, 256, 0, st>>>(reinterpret_cast<uint4*>(p), n16,
                                                       reinterpret_cast<unsigned char*>(p) + n16 * 16, ntail, word, word2);
}

void launch_gather_rows(int dtype, const GatherArgs& a, ChunkView cv, hipStream_t st) {
    const unsigned blocks = (unsigned)ceil_div(cv.n_cp, 4);
    if (dtype == 1) {                            // D is a multiple of 64, H and W are 16-byte aligned
        gather_rows_kernel<uint16_t><<<blocks, 256, 0, st>>>(a, cv.n0, cv.n_c, cv.n_cp, 1);
    } else {
        const int vec = a.D % 4 == 0 && (reinterpret_cast<uintptr_t>(a.H) & 15u) == 0 ? 1 : 0;
        gather_rows_kernel<float><<<blocks, 256, 0, st>>>(a, cv.n0, cv.n_c, cv.n_cp, vec);
    }
}

void launch_transpose_w(const void* W, int32_t V, int32_t D, int32_t Vp, void* WT, hipStream_t st) {
    dim3 grid((unsigned)(D / 64), (unsigned)(Vp / 64));      // D and Vp are multiples of 64 on the bf16 path
    transpose_bf16_kernel<<<grid, 256, 0, st>>>(reinterpret_cast<const uint16_t*>(W), D, V, nullptr,
                                                reinterpret_cast<uint16_t*>(WT), Vp);
}

void launch_combine_exp(const float2* part, int32_t n_tiles, const float* zy, const float* bref, ChunkView cv,
                        float* lse_chunk, float* logp_out, float* mx, int32_t* redo_count, int32_t* redo_list,
                        float* redo_sum, hipStream_t st) {
    auto run = [&](auto tok) {
        constexpr int TOK = decltype(tok)::value;
        combine_exp_kernel<TOK><<<(unsigned)ceil_div(cv.n_cp, TOK), COMBINE_THREADS, 0, st>>>(
            part, n_tiles, zy, bref, cv.n0, cv.n_c, cv.n_cp, lse_chunk, logp_out, mx, redo_count, redo_list, redo_sum);
    };
    if (cv.n_cp >= COMBINE_WIDE_TOKENS) run(std::integral_constant<int, 32>{});
    else run(std::integral_constant<int, 16>{});
}

void launch_exp_redo_rows(const int32_t* redo_count, const int32_t* redo_list, float* redo_sum, const void* Hc,
                          const void* W, int32_t V, int32_t Vp, int32_t D, const float* zy, const float* mx,
                          ChunkView cv, void* E, int64_t lde, float* bref, float* lse_chunk, float* logp_out,
                          hipStream_t st) {
    dim3 grid((unsigned)(Vp / 256), 4);
    exp_redo_rows_kernel<<<grid, 256, 0, st>>>(redo_count, redo_list, reinterpret_cast<const uint16_t*>(Hc),
                                               reinterpret_cast<const uint16_t*>(W), V, D, mx,
                                               reinterpret_cast<uint16_t*>(E), lde, redo_sum);
    exp_redo_finish_kernel<<<4, 256, 0, st>>>(redo_count, redo_list, redo_sum, zy, mx, cv.n0, bref, lse_chunk,
                                              logp_out);
}

void launch_softmax_scale(const int32_t* y, const float* zy, const float* bref, const float* lse, const float* c,
                          ChunkView cv, void* E, int64_t lde, float* scale, hipStream_t st) {
    softmax_scale_kernel<<<(unsigned)ceil_div(cv.n_cp, 256), 256, 0, st>>>(y, zy, bref, lse, c, cv.n_c, cv.n_cp,
                                                                           reinterpret_cast<uint16_t*>(E), lde, scale);
}

void launch_scale_transpose_bf16(const void* Hc, const float* scale, int32_t n_cp, int32_t D, void* HcT, hipStream_t st) {
    dim3 grid((unsigned)(D / 64), (unsigned)(n_cp / 64));
    transpose_bf16_kernel<<<grid, 256, 0, st>>>(reinterpret_cast<const uint16_t*>(Hc), D, n_cp, scale,
                                                reinterpret_cast<uint16_t*>(HcT), n_cp);
}

void launch_combine_logprob(const float2* part, LogitsPart lp, const float* zy, ChunkView cv, float* lse_chunk,
                            float* logp_out, float* lse_out, hipStream_t st) {
    auto run = [&](auto tok) {
        constexpr int TOK = decltype(tok)::value;
        combine_logprob_kernel<TOK><<<(unsigned)ceil_div(cv.n_cp, TOK), COMBINE_THREADS, 0, st>>>(
            part, lp.tiles, lp.pitch, zy, cv.n0, cv.n_c, cv.n_cp, lse_chunk, logp_out, lse_out);
    };
    if (cv.n_cp >= COMBINE_WIDE_TOKENS) run(std::integral_constant<int, 32>{});
    else run(std::integral_constant<int, 16>{});
}

void launch_row_stats_f32(const float* Z, int64_t ldz, int32_t V, const int32_t* y, ChunkView cv, float* lse_chunk,
                          float* logp_out, float* lse_out, hipStream_t st) {
    row_stats_kernel<<<(unsigned)cv.n_cp, ROW_THREADS, 0, st>>>(Z, ldz, V, y, TokenArgs{}, cv.n0, cv.n_c, lse_chunk, logp_out, lse_out);
}

void launch_score_rows_f32(const float* Z, int64_t ldz, const TokenArgs& a, ChunkView cv, float* logp_out, float* lse_out,
                           hipStream_t st) {
    row_stats_kernel<<<(unsigned)cv.n_c, ROW_THREADS, 0, st>>>(Z, ldz, a.V, nullptr, a, cv.n0, cv.n_c, nullptr, logp_out, lse_out);
}

void launch_token_loss(const TokenLossArgs& a, ChunkView cv, hipStream_t st) {
    token_loss_kernel<<<(unsigned)ceil_div(cv.n_cp, 256), 256, 0, st>>>(a, cv.n0, cv.n_c, cv.n_cp);
}

void launch_seq_ratio(const int32_t* loss_cu, int32_t S, const float* logp, const float* logp_old,
                      float* seq_ratio, int64_t n_lo, int64_t n_hi, int32_t* status, hipStream_t st) {
    if (S <= 0) return;
    const unsigned blocks = S < 4096 ? (unsigned)S : 4096u;
    seq_ratio_kernel<<<blocks, 256, 0, st>>>(loss_cu, S, logp, logp_old, seq_ratio, n_lo, n_hi, status);
}

void launch_token_norm_coef(int32_t Q, int32_t G, const int32_t* comp_len, const float* coef, float* coef_out,
                            hipStream_t st) {
    token_norm_coef_kernel<<<(unsigned)ceil_div(Q, 4), 256, 0, st>>>(Q, G, comp_len, coef, coef_out);
}

void launch_grad_logits_f32(float* ZG, int32_t V, int32_t Vp, const int32_t* y, const float* lse, const float* c,
                            int32_t n_c, hipStream_t st) {
    const int64_t per_row = ceil_div(Vp / 4, 256);
    dim3 grid((unsigned)n_c, (unsigned)(per_row < 64 ? per_row : 64));
    grad_logits_kernel<<<grid, 256, 0, st>>>(ZG, V, Vp, y, lse, c);
}

void launch_loss_rows_f32(float* ZG, int32_t V, int32_t Vp, const int32_t* y, const TokenLossArgs& a, float* logp, ChunkView cv,
                          hipStream_t st) {
    const unsigned rows = (unsigned)cv.n_c;
    if (Vp <= 4 * 256 * 4) loss_rows_kernel<256, 4, false><<<rows, 256, 0, st>>>(ZG, V, Vp, y, a, logp, cv.n0);
    else if (Vp <= 4 * 512 * 8) loss_rows_kernel<512, 8, false><<<rows, 512, 0, st>>>(ZG, V, Vp, y, a, logp, cv.n0);
    else if (Vp <= 4 * 512 * 16) loss_rows_kernel<512, 16, false><<<rows, 512, 0, st>>>(ZG, V, Vp, y, a, logp, cv.n0);
    else loss_rows_kernel<512, 8, true><<<rows, 512, 0, st>>>(ZG, V, Vp, y, a, logp, cv.n0);
}

void launch_seq_reduce(const SeqReduceArgs& a, hipStream_t st) {
    if (a.S > 0) seq_reduce_kernel<<<a.S < 4096 ? (unsigned)a.S : 4096u, 256, 0, st>>>(a);
    else no_sequences_kernel<<<1, 256, 0, st>>>(a);
}

}  // namespace dppo
