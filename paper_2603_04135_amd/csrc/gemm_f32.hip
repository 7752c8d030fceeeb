// fp32 GEMMs of the float32 data type, C[M,N] = A[M,K] * B[N,K]^T for any M, N, K and any 4-byte aligned operands.
// Each operand is K-contiguous ([rows, K]) or k-major ([K, rows]), so that the three GEMMs of the path read W, the
// chunk's hidden states and its logits / gradient entries as they lie: nothing is transposed in memory.
//
// The fp32 matrix instructions run at a sixteenth of the bf16 rate, so every operand element is split on its way
// into LDS into three bf16 values, x = h + m + l (each the rounded remainder of the ones before: 8 + 8 + 8 significand
// bits, the sum is x exactly; all are scaled by 2^24, see SCALE), and a product takes six bf16 MFMAs into the fp32 accumulators:
//     x y = l h' + m h' + m m' + h m' + h l' + h h',      dropped: m l' + l m' + l l' <= 2^-24 |x y| (2^-26.5 rms),
// at most the rounding of one fp32 product. K = 32 costs 96 matrix cycles per 16 x 16 block instead of 256, and the
// accumulator is rounded 6 times instead of 8. The instruction cuts off the bits of an accumulator that lie below the new
// product's last place (-1 to +1/2 ulp, 0.39 ulp rms, measured; fp32 rounding 0.29), so the order matters where few products make up
// the sum: with h h' last only its addition errs at full magnitude. Error of a sum of K products of normally distributed factors
// (2-norm; in brackets the fp32 instruction's): K = 1 3.4e-8 (2.5e-8; at worst 2^-22.7, 2^-24), 2 3.30e-8 (3.13e-8), 3 3.31e-8 (3.55e-8),
// 32 3.8e-8 (1.0e-7), 1024 4.8e-7 (5.7e-7), 8192 1.44e-6 (1.64e-6); with h h' fourth K = 1 to 4 4.8e-8. Below FEW_K products, where
// storing the result takes longer, the fp32 instruction (v_mfma_f32_16x16x4_f32) makes the sums. Slices that hold a value of BIG or
// more (where an infinity times a part of the other factor would be a NaN, or a part's product could overflow) are multiplied by it, too.
// Measured against those instructions throughout (2400 tokens, D = 1024, V = 32000, kernel trace): logits 1407 -> 774 us
// (203 TFLOP/s), dH 1464 -> 912, dW 1476 -> 792; relative error of the logits 5.7e-7 -> 4.9e-7, of dH 1.0e-6 -> 0.8e-6. What bounds it: the
// matrix pipes are busy half of the time at 2.1 GHz, the splitting (13 VALU instructions per pair) takes most of the rest,
// only partly under other wavefronts' products. Splitting the next slice between the products of the present one, with the
// parts in registers and two workgroups per compute unit, was slower (928 / 999 / 880 us against 801 / 851 / 774 in the same runs).
#include "dppo_internal.h"
#include "gemm_f32_plan.h"

namespace dppo {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Elements are split as 2^24 x, so that every part of any float32 value, subnormals among them, is a normal bf16 number or zero (a
// multiple of 2^-125) and no part of a product that reaches the result underflows; the accumulators are scaled back by 2^-48.
// Unscaled, a gradient entry below 2^-110 (a token suppressed by e^-76) lost its low parts: 1.5e-2 of a row of dW at e^-80. The
// two multiplications per pair cost nothing: the largest magnitude, taken of their results, needs no maximum that quiets
// signalling NaNs (2400 tokens, D = 1024, V = 32000: 2.70 ms without the scale; 2.69 with it, 2.78 with the maximum of the unscaled values).
// Values below BIG keep the sum of 2^31 products finite: (2^48)^2 2^31 = 2^127.
constexpr float SCALE = 16777216.0f, UNSCALE = 1.0f / 281474976710656.0f, BIG = 16777216.0f;
constexpr int FEW_K = 3;

template <int BM_, int BN_, int BK_, int WGM_, int WGN_>
struct F32Cfg {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WGM = WGM_, WGN = WGN_;
    static constexpr int NT = WGM * WGN * 64;
    static constexpr int MI = BM / WGM / 16, NI = BN / WGN / 16;
};
typedef F32Cfg<128, 128, 32, 2, 2> F32Big;
typedef F32Cfg<64, 64, 32, 2, 2> F32Mid;

struct F32Args {
    const float* A; int64_t lda;
    const float* B; int64_t ldb;
    int M, N, K;
    int tiles_n, k_parts, slices_per_part;
    float* C; int64_t ldc; int accumulate;
    const int32_t* row_map;      // output row = row_map[m] if not NULL
    const int32_t* a_map;        // K-contiguous A: row m of it is row a_map[m] (clamped to the a_rows there are) if not NULL
    int a_rows;
    float* partial;              // k_parts > 1: part p of the sums goes to partial + p * M * N, row-major
};

// Row r of an operand of `rows` rows (beyond them: the last one, for outputs that are not stored), through its map.
__device__ __forceinline__ int operand_row(int r, int rows, const int32_t* map, int map_rows) {
    r = r < rows ? r : rows - 1;
    if (map) {
        r = map[r];
        r = r < 0 ? 0 : r < map_rows ? r : map_rows - 1;
    }
    return r;
}

// x = h + m + l (x scaled), element pairs packed into 32-bit words.
__device__ __forceinline__ uint32_t pack_bf16(f32x2 v) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2)); }
__device__ __forceinline__ f32x2 unpack_bf16(uint32_t w) {
    return f32x2{__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u)};
}
__device__ __forceinline__ void split_pair(f32x2 x, uint32_t& h, uint32_t& m, uint32_t& l) {
    h = pack_bf16(x);
    f32x2 r = x - unpack_bf16(h);
    m = pack_bf16(r);
    r -= unpack_bf16(m);
    l = pack_bf16(r);
}

// One operand of a tile: ROWS x BK elements, loaded by one half of the workgroup's wavefronts (the other half loads the
// other operand). A wavefront's W = 16 BLOCKS rows are dealt out to its BLOCKS MFMA blocks in turn: block i holds the rows
// i, BLOCKS + i, 2 BLOCKS + i, ... (so a lane's accumulators of one output row are BLOCKS neighbouring columns), and lies in
// LDS at the positions 16 i .. 16 i + 15 of the W, which makes all blocks of a plane immediate offsets of one address. A plane
// (h, m or l) consists of 16-byte chunks of 8 k-values:
//   K-contiguous source: [position][chunk], chunk XOR-swizzled by the position; a thread loads two 16-byte vectors of a
//                        row per chunk;
//   k-major source:      [chunk][position]; a thread loads 8 k-rows of RPL neighbouring rows, which are RPL chunks once
//                        transposed in its registers.
// Either way the 16 lanes that a ds_write_b128 or ds_read_b128 serves at a time (reads: {0-7, 24-31}, ...: positions 0-7 at
// chunk c, 8-15 at chunk c ^ 1) fall into different banks.
template <class Cfg, int ROWS, int BLOCKS, bool KM>
struct Operand {
    static constexpr int BK = Cfg::BK, CPR = BK / 8, NT = Cfg::NT / 2;
    static constexpr int PLANE = ROWS * BK * 2;                  // bytes
    static constexpr int LDS_BYTES = 3 * PLANE;
    static constexpr int UNITS = ROWS * CPR / NT;                // chunks per thread
    static constexpr int RPL = UNITS < 4 ? UNITS : 4;            // k-major: rows per lane
    static constexpr int GROUPS = KM ? UNITS / RPL : UNITS;
    static_assert(ROWS * CPR % NT == 0 && UNITS % RPL == 0 && ROWS % RPL == 0 && ROWS % 16 == 0, "chunks of a tile per thread");
    typedef float Vec __attribute__((ext_vector_type(RPL), aligned(4)));
    typedef float Vec4 __attribute__((ext_vector_type(4), aligned(4)));

    static constexpr int W = 16 * BLOCKS, BLOCK_BYTES = KM ? 256 : 256 * CPR;
    static_assert(ROWS % W == 0, "whole wavefront rows");

    static __device__ __forceinline__ int lds_at(int pos, int chunk) {
        if (KM) return (chunk * ROWS + pos) * 16;
        constexpr int SHIFT = CPR == 4 ? 2 : 0;
        return (pos * CPR + (chunk ^ ((pos >> SHIFT) & (CPR - 1)))) * 16;
    }
    static __device__ __forceinline__ int position(int row) { return row / W * W + row % BLOCKS * 16 + row % W / BLOCKS; }
    static __device__ __forceinline__ int row_at(int pos) { return pos / W * W + pos % 16 * BLOCKS + pos % W / 16; }
    static __device__ __forceinline__ int row_of(int g, int t) {
        return KM ? (t + g * NT) % (ROWS / RPL) * RPL : row_at((t + g * NT) / CPR);
    }
    static __device__ __forceinline__ int chunk_of(int g, int t) { return KM ? (t + g * NT) / (ROWS / RPL) : (t + g * NT) % CPR; }

    // Start of the thread's chunks in a whole slice at k = 0 of the tile at row0. Rows are clamped: those beyond the matrix only
    // reach outputs that are not stored.
    static __device__ __forceinline__ void source(const float* (&x)[UNITS], const float* X, int64_t ld, int row0, int rows, int t,
                                                  const int32_t* map, int map_rows) {
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            const int r = operand_row(row0 + row_of(g, t), rows, map, map_rows);
            const int k = chunk_of(g, t) * 8;
            x[g] = KM ? X + (size_t)k * ld + r : X + (size_t)r * ld + k;
        }
    }
    // The thread's values v[unit][k] of the slice at k0, in vectors of four (RPL) elements.
    static __device__ __forceinline__ void load(float (&v)[UNITS][8], const float* const (&src)[UNITS], int64_t ld, int k0) {
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            if (!KM) {
                const float* x = src[g] + k0;
                const Vec4 a = *reinterpret_cast<const Vec4*>(x), b = *reinterpret_cast<const Vec4*>(x + 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) { v[g][j] = a[j]; v[g][4 + j] = b[j]; }
            } else {
                const float* x = src[g] + (size_t)k0 * ld;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const Vec a = *reinterpret_cast<const Vec*>(x + (size_t)j * ld);
#pragma unroll
                    for (int i = 0; i < RPL; ++i) v[g * RPL + i][j] = a[i];
                }
            }
        }
    }
    // The same element by element, with k-values beyond K read as zero.
    static __device__ __forceinline__ void load_tail(float (&v)[UNITS][8], const float* __restrict__ X, int64_t ld, int row0, int rows,
                                                     int k0, int K, int tid, int first, const int32_t* map, int map_rows) {
        asm volatile("" : "+v"(tid));   // this one slice's addresses are formed here, not kept in registers over the K loop
        const int t = tid - first;
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            const int r = operand_row(row0 + unit_row(u, t), rows, map, map_rows);
            const int k = k0 + unit_chunk(u, t) * 8;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int kc = k + j < K ? k + j : K - 1;
                const float x = KM ? X[(size_t)kc * ld + r] : X[(size_t)r * ld + kc];
                v[u][j] = k + j < K ? x : 0.0f;
            }
        }
    }
    // Whether the vectors of the slice at k0 stay inside the operand's memory: the slice is whole, and k-major vectors that run
    // over the end of a k-row, by up to RPL - 1 elements that are not used, end in one of the rows behind the slice.
    static __device__ __forceinline__ bool safe(int64_t ld, int row0, int rows, int k0, int K) {
        return k0 + BK <= K && (!KM || row0 + ROWS <= rows || (int64_t)(K - k0 - BK) * ld >= RPL - 1);
    }
    static __device__ __forceinline__ int unit_row(int u, int t) { return row_of(KM ? u / RPL : u, t) + (KM ? u % RPL : 0); }
    static __device__ __forceinline__ int unit_chunk(int u, int t) { return chunk_of(KM ? u / RPL : u, t); }
    // Where the thread's chunks go in the operand's LDS planes.
    static __device__ __forceinline__ void places(int (&at)[UNITS], int t) {
#pragma unroll
        for (int u = 0; u < UNITS; ++u) at[u] = lds_at(position(unit_row(u, t)), unit_chunk(u, t));
    }
    // Operand of this lane (position pos in block 0) for block i.
    static __device__ __forceinline__ bf16x8 read(const char* lds, int pos, int chunk, int plane, int i) {
        return *reinterpret_cast<const bf16x8*>(lds + lds_at(pos, chunk) + plane * PLANE + i * BLOCK_BYTES);
    }
};

template <class Cfg, bool A_KM, bool B_KM>
__global__ __launch_bounds__(Cfg::NT, 3) void gemm_f32_kernel(F32Args g) {
    typedef Operand<Cfg, Cfg::BM, Cfg::MI, A_KM> OA;
    typedef Operand<Cfg, Cfg::BN, Cfg::NI, B_KM> OB;
    constexpr int MI = Cfg::MI, NI = Cfg::NI, BK = Cfg::BK, HALF = Cfg::NT / 2;
    __shared__ __attribute__((aligned(16))) char smem[OA::LDS_BYTES + OB::LDS_BYTES];
    char *s_a = smem, *s_b = smem + OA::LDS_BYTES;
    __shared__ int s_big;                        // k0 of the last slice with a value of BIG or more
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_m = wave % Cfg::WGM, wave_n = wave / Cfg::WGM;
    const int part = blockIdx.x % g.k_parts, tile = blockIdx.x / g.k_parts;
    const int m0 = tile / g.tiles_n * Cfg::BM, n0 = tile % g.tiles_n * Cfg::BN;
    const int k_lo = part * g.slices_per_part * BK;
    const int k_end = k_lo + g.slices_per_part * BK < g.K ? k_lo + g.slices_per_part * BK : g.K;

    f32x4 acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // The wavefronts of the first half load A, the others B. Where both lie the same way one body serves either.
    static_assert(OA::UNITS == OB::UNITS && Cfg::BM == Cfg::BN, "one set of registers for either operand");
    constexpr int UNITS = OA::UNITS;
    constexpr bool ALIKE = A_KM == B_KM;
    float v[UNITS][8];
    const bool for_a = wave < Cfg::NT / 128;
    const int first = for_a ? 0 : HALF, t = tid - first;
    const float* X = for_a ? g.A : g.B;
    const int64_t ld = for_a ? g.lda : g.ldb;
    const int row0 = for_a ? m0 : n0, rows = for_a ? g.M : g.N;
    char* s_x = for_a ? s_a : s_b;
    const float* src[UNITS];
    int at[UNITS];
    const int32_t* map = !A_KM && for_a ? g.a_map : nullptr;
    if (ALIKE || for_a) { OA::source(src, X, ld, row0, rows, t, map, g.a_rows); OA::places(at, t); }
    else { OB::source(src, X, ld, row0, rows, t, nullptr, 0); OB::places(at, t); }
    auto load = [&](int k0) __attribute__((always_inline)) {
        if (ALIKE || for_a) {
            if (OA::safe(ld, row0, rows, k0, g.K)) OA::load(v, src, ld, k0);
            else OA::load_tail(v, X, ld, row0, rows, k0, g.K, tid, first, map, g.a_rows);
        } else {
            if (OB::safe(ld, row0, rows, k0, g.K)) OB::load(v, src, ld, k0);
            else OB::load_tail(v, X, ld, row0, rows, k0, g.K, tid, first, nullptr, 0);
        }
    };
    if (tid == 0) s_big = -1;
    const int lane = tid & 63, ra = wave_m * (MI * 16) + (lane & 15), rb = wave_n * (NI * 16) + (lane & 15), kq = lane >> 4;
    int k0 = k_lo;
    const bool few = g.K < FEW_K;
    if (k_lo < k_end) load(k_lo);
    for (; !few && k0 < k_end; k0 += BK) {
        __syncthreads();                         // the slice before has been read
        float top = 0.0f;                        // largest magnitude (a NaN is left out: it spoils all six products)
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            uint32_t h[4], m[4], l[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x2 x = f32x2{v[u][2 * j], v[u][2 * j + 1]} * SCALE;
                top = fmaxf(fmaxf(top, __builtin_fabsf(x[0])), __builtin_fabsf(x[1]));
                split_pair(x, h[j], m[j], l[j]);
            }
            *reinterpret_cast<u32x4*>(s_x + at[u]) = u32x4{h[0], h[1], h[2], h[3]};
            *reinterpret_cast<u32x4*>(s_x + at[u] + OA::PLANE) = u32x4{m[0], m[1], m[2], m[3]};
            *reinterpret_cast<u32x4*>(s_x + at[u] + 2 * OA::PLANE) = u32x4{l[0], l[1], l[2], l[3]};
        }
        if (__any(top >= SCALE * BIG)) s_big = k0;
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(s_big) == k0) break;
        if (k0 + BK < k_end) load(k0 + BK);
        // Six products of one plane of A with one of B, row by row or column by column of blocks. A plane is replaced in its
        // registers by the next one as the product before is done with it, so that two planes are live and three
        // workgroups fit a compute unit: one's splitting falls into the others' products. h h' comes last (see above).
#pragma unroll
        for (int kk = 0; kk < BK / 32; ++kk) {
            const int chunk = kk * 4 + kq;
            bf16x8 x[MI], y[NI];
            auto by_rows = [&](int next_a) __attribute__((always_inline)) {
#pragma unroll
                for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[mi], y[ni], acc[mi][ni], 0, 0, 0);
                    if (next_a >= 0) x[mi] = OA::read(s_a, ra, chunk, next_a, mi);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            auto by_columns = [&](int next_b) __attribute__((always_inline)) {
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi)
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[mi], y[ni], acc[mi][ni], 0, 0, 0);
                    if (next_b >= 0) y[ni] = OB::read(s_b, rb, chunk, next_b, ni);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            constexpr int H = 0, M = 1, L = 2;
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) y[ni] = OB::read(s_b, rb, chunk, H, ni);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) x[mi] = OA::read(s_a, ra, chunk, L, mi);
            __builtin_amdgcn_sched_barrier(0);
            by_rows(M);            // l h'
            by_columns(M);         // m h'
            by_rows(H);            // m m'
            by_columns(L);         // h m'
            by_columns(H);         // h l'
            by_columns(-1);        // h h'
        }
    }
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) acc[mi][ni] *= UNSCALE;
    // From the first slice with a BIG value on, or for few products: fp32 products of the values themselves; v holds the slice
    // at k0. (A loop of its own: as a branch of the one above it costs that one the accumulators' registers a second time.) Bound by the
    // instruction: 2400 tokens, D = 1024, V = 32000 with a BIG value in an early slice of every row 1.46 to 1.53 ms for the scoring (without the
    // next slice's loads under the products 1.53 to 1.55; all slices through the instruction, without a split, 1.48) and 3.76 to
    // 3.87 ms for the loss (4.55), of which one to three GEMMs meet such values.
    for (; k0 < k_end; k0 += BK) {
        constexpr int PITCH = BK + 1;
        static_assert((Cfg::BM + Cfg::BN) * PITCH * 4 <= OA::LDS_BYTES + OB::LDS_BYTES, "fp32 slices fit the planes' LDS");
        float* raw = reinterpret_cast<float*>(smem);
        int et = tid;
        asm volatile("" : "+v"(et));             // these addresses are formed here, not kept in registers over the loop above
        const int el = et & 15, eq = (et & 63) >> 4;
        et -= first;
        __syncthreads();                         // the slice before has been read
#pragma unroll
        for (int u = 0; u < UNITS; ++u)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int row = for_a ? OA::unit_row(u, et) : OB::unit_row(u, et), c = for_a ? OA::unit_chunk(u, et) : OB::unit_chunk(u, et);
                raw[((for_a ? 0 : Cfg::BM) + row) * PITCH + c * 8 + j] = v[u][j];
            }
        __syncthreads();
        if (k0 + BK < k_end) load(k0 + BK);
        const int k_top = g.K - k0 < BK ? g.K - k0 : BK;      // (zeros beyond: not multiplied where there are few products)
#pragma unroll 1
        for (int k = 0; k < k_top; k += 4) {
            float x[MI], y[NI];
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) x[mi] = raw[(wave_m * (MI * 16) + el * MI + mi) * PITCH + k + eq];
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) y[ni] = raw[(Cfg::BM + wave_n * (NI * 16) + el * NI + ni) * PITCH + k + eq];
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[mi], y[ni], acc[mi][ni], 0, 0, 0);
        }
    }

    // accumulator lane: of block (mi, ni) column NI (lane % 16) + ni, rows MI (4 (lane / 16) + j) + mi
    typedef float VecN __attribute__((ext_vector_type(NI), aligned(4)));
    int last_tid = tid;
    asm volatile("" : "+v"(last_tid));           // (likewise)
    const int cq = (last_tid & 63) >> 4, col = n0 + wave_n * (NI * 16) + (last_tid & 15) * NI;
    const bool add = g.k_parts == 1 && g.accumulate;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = m0 + wave_m * (MI * 16) + (4 * cq + j) * MI + mi;
            if (row >= g.M) continue;
            float* out = (g.k_parts > 1 ? g.partial + ((size_t)part * g.M + row) * g.N
                                        : g.C + (size_t)(g.row_map ? (int64_t)g.row_map[row] : (int64_t)row) * g.ldc) + col;
            if (NI > 1 && col + NI <= g.N) {
                VecN x;
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) x[ni] = acc[mi][ni][j];
                if (add) x += *reinterpret_cast<const VecN*>(out);
                *reinterpret_cast<VecN*>(out) = x;
            } else {
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) {
                    if (col + ni >= g.N) break;
                    out[ni] = add ? out[ni] + acc[mi][ni][j] : acc[mi][ni][j];
                }
            }
        }
}

// Small products: 32 x 32 tiles, NW wavefronts that share nothing until the end. Each takes every NW-th slice of 32
// k-values, straight from memory into its MFMA operand registers (DEPTH slices in flight, no LDS, no barrier), and the
// tile is the sum of the wavefronts' accumulators, added up in order through LDS. What bounds these products is the
// latency of a slice, which this divides by NW x DEPTH.
// Lane l holds rows 2 (l % 16) + i of an operand in block i, k-values 8 (l / 16) .. + 7.
template <bool KM>
struct Direct {
    typedef float Vec2 __attribute__((ext_vector_type(2), aligned(4)));
    typedef float Vec4 __attribute__((ext_vector_type(4), aligned(4)));
    static __device__ __forceinline__ void load(float (&v)[2][8], const float* __restrict__ X, int64_t ld, int row0, int rows,
                                                const int (&r)[2], int k0, int K, int lane) {
        const int k = k0 + 8 * (lane >> 4);
        const bool whole = k0 + 32 <= K;
        if (KM && whole && (row0 + 32 <= rows || (int64_t)(K - k0 - 32) * ld >= 1)) {     // (as in Operand::safe)
            const float* x = X + (size_t)k * ld + r[0];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const Vec2 a = *reinterpret_cast<const Vec2*>(x + (size_t)j * ld);
                v[0][j] = a[0];
                v[1][j] = a[1];
            }
        } else if (!KM && whole) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float* x = X + (size_t)r[i] * ld + k;
                const Vec4 a = *reinterpret_cast<const Vec4*>(x), b = *reinterpret_cast<const Vec4*>(x + 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) { v[i][j] = a[j]; v[i][4 + j] = b[j]; }
            }
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int kc = k + j < K ? k + j : K - 1;
                    const float x = KM ? X[(size_t)kc * ld + r[i]] : X[(size_t)r[i] * ld + kc];
                    v[i][j] = k + j < K ? x : 0.0f;
                }
            }
        }
    }
};
constexpr int DIRECT_EDGE = 32, DIRECT_DEPTH = 2;

template <int NW, bool A_KM, bool B_KM>
__global__ __launch_bounds__(NW * 64, 2) void gemm_f32_direct_kernel(F32Args g) {
    constexpr int DEPTH = DIRECT_DEPTH, PER_THREAD = 16 / NW;
    __shared__ float s_acc[NW][16][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int part = blockIdx.x % g.k_parts, tile = blockIdx.x / g.k_parts;
    const int m0 = tile / g.tiles_n * DIRECT_EDGE, n0 = tile % g.tiles_n * DIRECT_EDGE;
    const int k_lo = part * g.slices_per_part * 32;
    const int k_end = k_lo + g.slices_per_part * 32 < g.K ? k_lo + g.slices_per_part * 32 : g.K;
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i / 2][i % 2] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float a[DEPTH][2][8], b[DEPTH][2][8];
    int ra[2], rb[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        ra[i] = operand_row(m0 + 2 * (lane & 15) + i, g.M, A_KM ? nullptr : g.a_map, g.a_rows);
        rb[i] = operand_row(n0 + 2 * (lane & 15) + i, g.N, nullptr, 0);
    }
    auto load = [&](int d, int k0) __attribute__((always_inline)) {
        Direct<A_KM>::load(a[d], g.A, g.lda, m0, g.M, ra, k0, g.K, lane);
        Direct<B_KM>::load(b[d], g.B, g.ldb, n0, g.N, rb, k0, g.K, lane);
    };
    bool split = g.K >= FEW_K;                   // (until the wavefront's first slice with a BIG value)
    auto unscale = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i / 2][i % 2] *= UNSCALE;
    };
    auto products = [&](int d) __attribute__((always_inline)) {
        float top = 0.0f;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) top = fmaxf(fmaxf(top, __builtin_fabsf(a[d][i][j] * SCALE)), __builtin_fabsf(b[d][i][j] * SCALE));
        if (split && __any(top >= SCALE * BIG)) {
            split = false;
            unscale();
        }
        if (!split) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (j >= g.K) break;             // (k-values 8 (lane / 16) + j: zeros where there are few products)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    acc[i / 2][i % 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[d][i / 2][j], b[d][i % 2][j], acc[i / 2][i % 2], 0, 0, 0);
            }
            return;
        }
        bf16x8 x[2][3], y[2][3];
        auto parts_of = [&](const float (&v)[8], bf16x8 (&p)[3]) __attribute__((always_inline)) {
            uint32_t w[3][4];
#pragma unroll
            for (int j = 0; j < 4; ++j) split_pair(f32x2{v[2 * j], v[2 * j + 1]} * SCALE, w[0][j], w[1][j], w[2][j]);
#pragma unroll
            for (int q = 0; q < 3; ++q) p[q] = __builtin_bit_cast(bf16x8, u32x4{w[q][0], w[q][1], w[q][2], w[q][3]});
        };
#pragma unroll
        for (int i = 0; i < 2; ++i) { parts_of(a[d][i], x[i]); parts_of(b[d][i], y[i]); }
        constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int p = 0; p < 6; ++p)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc[i / 2][i % 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[i / 2][PA[p]], y[i % 2][PB[p]], acc[i / 2][i % 2], 0, 0, 0);
    };
    int k0 = k_lo + wave * 32;
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        if (k0 + d * (NW * 32) < k_end) load(d, k0 + d * (NW * 32));
    while (k0 < k_end) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            if (k0 >= k_end) break;
            products(d);
            const int next = k0 + DEPTH * (NW * 32);
            if (next < k_end) load(d, next);
            k0 += NW * 32;
        }
    }
    if (split) unscale();
    // element e = 8 mi + 2 j + ni of lane l: row m0 + 2 (4 (l / 16) + j) + mi, column n0 + 2 (l % 16) + ni
#pragma unroll
    for (int e = 0; e < 16; ++e) s_acc[wave][e][lane] = acc[e / 8][e % 2][e / 2 % 4];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER_THREAD; i += 2) {
        const int e = wave * PER_THREAD + i;
        float v[2];
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
            v[ni] = s_acc[0][e + ni][lane];
#pragma unroll
            for (int w = 1; w < NW; ++w) v[ni] += s_acc[w][e + ni][lane];
        }
        const int row = m0 + 2 * (4 * (lane >> 4) + e / 2 % 4) + e / 8, col = n0 + 2 * (lane & 15);
        if (row >= g.M) continue;
        float* out = (g.k_parts > 1 ? g.partial + ((size_t)part * g.M + row) * g.N
                                    : g.C + (size_t)(g.row_map ? (int64_t)g.row_map[row] : (int64_t)row) * g.ldc) + col;
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
            if (col + ni < g.N) out[ni] = g.k_parts == 1 && g.accumulate ? out[ni] + v[ni] : v[ni];
    }
}

// Adds the k_parts partial results up, in part order, into the (mapped) rows of C.
__global__ __launch_bounds__(256) void sum_parts_f32_kernel(const float* __restrict__ partial, int k_parts, int M, int N,
                                                            float* __restrict__ C, int64_t ldc, int accumulate,
                                                            const int32_t* __restrict__ row_map) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, total = (int64_t)M * N;
    if (i >= total) return;
    float v = partial[i];
#pragma unroll 8
    for (int p = 1; p < k_parts; ++p) v += partial[(size_t)p * total + i];
    const int row = (int)(i / N), col = (int)(i % N);
    float* out = C + (size_t)(row_map ? (int64_t)row_map[row] : (int64_t)row) * ldc + col;
    *out = accumulate ? *out + v : v;
}

F32Args args_of(const GemmF32& p, int edge, int bk, int parts) {
    F32Args g;
    g.A = p.A; g.lda = p.lda; g.B = p.B; g.ldb = p.ldb; g.M = p.M; g.N = p.N; g.K = p.K;
    g.tiles_n = (int)ceil_div(p.N, edge);
    g.k_parts = parts;
    g.slices_per_part = (int)ceil_div(ceil_div(p.K, bk), parts);
    g.C = p.C; g.ldc = p.ldc; g.accumulate = p.accumulate; g.row_map = p.row_map; g.partial = p.partial;
    g.a_map = p.a_map; g.a_rows = p.a_rows;
    return g;
}

template <class Cfg>
void launch_cfg(const GemmF32& p, int parts, hipStream_t st) {
    const F32Args g = args_of(p, Cfg::BM, Cfg::BK, parts);
    const unsigned grid = (unsigned)(ceil_div(p.M, Cfg::BM) * g.tiles_n * parts);
    if (p.a_km) gemm_f32_kernel<Cfg, true, true><<<grid, Cfg::NT, 0, st>>>(g);
    else if (p.b_km) gemm_f32_kernel<Cfg, false, true><<<grid, Cfg::NT, 0, st>>>(g);
    else gemm_f32_kernel<Cfg, false, false><<<grid, Cfg::NT, 0, st>>>(g);
}

template <int NW>
void launch_direct(const GemmF32& p, int parts, hipStream_t st) {
    const F32Args g = args_of(p, DIRECT_EDGE, 32, parts);
    const unsigned grid = (unsigned)(ceil_div(p.M, DIRECT_EDGE) * g.tiles_n * parts);
    if (p.a_km) gemm_f32_direct_kernel<NW, true, true><<<grid, NW * 64, 0, st>>>(g);
    else if (p.b_km) gemm_f32_direct_kernel<NW, false, true><<<grid, NW * 64, 0, st>>>(g);
    else gemm_f32_direct_kernel<NW, false, false><<<grid, NW * 64, 0, st>>>(g);
}

}  // namespace

void launch_gemm_f32(const GemmF32& p, int cus, hipStream_t st) {
    if (p.M <= 0 || p.N <= 0) return;
    static_assert(F32_EDGE[F32_BIG] == F32Big::BM && F32_EDGE[F32_MID] == F32Mid::BM && F32_EDGE[F32_DIRECT_4] == DIRECT_EDGE &&
                  F32_EDGE[F32_DIRECT_8] == DIRECT_EDGE && F32_STEP_K[F32_BIG] == F32Big::BK && F32_STEP_K[F32_MID] == F32Mid::BK,
                  "the plan knows the kernels' tiles");
    const F32Plan plan = plan_gemm_f32(p.M, p.N, p.K, p.partial ? p.partial_floats / ((int64_t)p.M * p.N) : 1, cus);
    const int parts = plan.parts;
    if (plan.kernel == F32_BIG) launch_cfg<F32Big>(p, parts, st);
    else if (plan.kernel == F32_MID) launch_cfg<F32Mid>(p, parts, st);
    else if (plan.kernel == F32_DIRECT_4) launch_direct<4>(p, parts, st);
    else launch_direct<8>(p, parts, st);
    if (parts > 1)
        sum_parts_f32_kernel<<<(unsigned)ceil_div((int64_t)p.M * p.N, 256), 256, 0, st>>>(p.partial, parts, p.M, p.N, p.C,
                                                                                          p.ldc, p.accumulate, p.row_map);
}

}  // namespace dppo
