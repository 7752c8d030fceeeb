// fp32 GEMMs of the float32 data type on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32: fp32 products,
// fp32 accumulation), C[M,N] = A[M,K] * B[N,K]^T for any M, N, K and any 4-byte aligned operands. Each operand
// is K-contiguous ([rows, K]) or k-major ([K, rows]), so that the three GEMMs of the path read W, the chunk's
// hidden states and its logits / gradient entries as they lie: nothing is transposed in memory.
//
// What bounds it is the fp32 matrix rate (256 flop per clock and compute unit, a sixteenth of bf16): a
// 128 x 128 x 32 slice keeps the matrix pipes busy for 4096 cycles and needs only 32 four-byte loads per
// thread, so operands go through registers (any alignment, zeros beyond K) into two LDS buffers, one barrier
// per slice, and two workgroups per compute unit cover each other's barriers.
// Measured (loss forward + backward, D = 1024, V = 32000): 1700 loss tokens 9.3 -> 3.6 ms, 100 tokens of D = 512 4.8 ->
// 0.27 ms (64-wide FMA tiles before, with transposed copies of W, H and the logits); the logits GEMM of 2400 tokens 103
// TFLOP/s of the 152 that a register-only loop of the instruction sustains.
#include "dppo_internal.h"

namespace dppo {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int BM_, int BN_, int BK_, int WGM_, int WGN_>
struct F32Cfg {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WGM = WGM_, WGN = WGN_;
    static constexpr int NT = WGM * WGN * 64;
    static constexpr int MI = BM / WGM / 16, NI = BN / WGN / 16;
};
typedef F32Cfg<128, 128, 32, 2, 2> F32Big;
typedef F32Cfg<64, 64, 32, 2, 2> F32Mid;
typedef F32Cfg<32, 32, 64, 2, 2> F32Small;

struct F32Args {
    const float* A; int64_t lda;
    const float* B; int64_t ldb;
    int M, N, K;
    int tiles_n, k_parts, slices_per_part;
    float* C; int64_t ldc; int accumulate;
    const int32_t* row_map;      // output row = row_map[m] if not NULL
    float* partial;              // k_parts > 1: part p of the sums goes to partial + p * M * N, row-major
};

// One operand of a tile: ROWS x BK elements, in LDS as
//   K-contiguous source: [row][k], the 16-byte chunks of a row XOR-swizzled so that the 16 lanes a ds_read_b128
//                        serves at a time ({0-7, 24-31}, ...: rows 0-7 at chunk c, rows 8-15 at chunk c ^ 1) fall
//                        into different banks;
//   k-major source:      [k][row], read by four 4-byte reads per 16 k-values; the lanes of a read sit in four k-rows
//                        4 apart, which the XOR (64 rows and more) or the pitch (32) moves to different banks.
// MFMA j of a 16-wide k-chunk takes k = 4 (lane / 16) + j from every lane: both operands use the same order,
// so it is a permutation of the chunk's k-values and a K-contiguous lane reads its four values at once.
template <class Cfg, int ROWS, bool KM>
struct Operand {
    static constexpr int BK = Cfg::BK, NT = Cfg::NT, CPR = BK / 4;
    static constexpr int PITCH = KM ? (ROWS >= 64 ? ROWS : ROWS + 4) : BK;
    static constexpr int LDS_FLOATS = KM ? BK * PITCH : ROWS * PITCH;
    static constexpr int PER_THREAD = ROWS * BK / NT;
    static constexpr int STEP = NT / (KM ? ROWS : BK);           // rows (k-rows) between a thread's elements
    static_assert(NT % (KM ? ROWS : BK) == 0 && ROWS * BK % NT == 0, "elements of a tile per thread");

    static __device__ __forceinline__ int lds_at(int row, int k) {
        if (KM) return k * PITCH + (ROWS >= 64 ? row ^ (((k >> 2) & 3) << 4) : row);
        return row * PITCH + (((k >> 2) ^ (row & (CPR - 1))) << 2) + (k & 3);
    }
    // Loads the thread's elements of the slice at k0 of the tile at row0: rows are clamped (rows beyond the
    // matrix only reach outputs that are not stored), k-values beyond K read as zero.
    template <bool TAIL>
    static __device__ __forceinline__ void load(float (&v)[PER_THREAD], const float* __restrict__ X, int64_t ld, int row0,
                                                int rows, int k0, int K, int tid) {
        if (KM) {
            int r = row0 + tid % ROWS;
            r = r < rows ? r : rows - 1;
            const int kb = k0 + tid / ROWS;
#pragma unroll
            for (int i = 0; i < PER_THREAD; ++i) {
                const int k = kb + i * STEP;
                const int kc = !TAIL || k < K ? k : K - 1;
                const float x = X[(size_t)kc * ld + r];
                v[i] = !TAIL || k < K ? x : 0.0f;
            }
        } else {
            const int k = k0 + tid % BK;
            const int rb = row0 + tid / BK;
            if (TAIL && PER_THREAD >= 16) {
                // 128 x 128 tiles: row offsets formed for every load, and kept from being moved out of the K loop: the
                // addresses of whole slices stay in registers there, a second set for this one slice would not fit (both
                // operands K-contiguous: 24 registers spilled and reloaded one by one; log-probs of 2000 tokens, V = 32000, D =
                // 1000 1.33 -> 1.27 ms, V = 30000, D = 300 0.515 -> 0.443). Forming them for every slice costs 2 % at D = 1024,
                // and in the smaller tiles' last slice 1 % (418 tokens, V = 1849, D = 709: 40.3 -> 40.9 us).
                const int kc = k < K ? k : K - 1;
                const int r0 = rb < rows ? rb : rows - 1;
                int last = rows - 1 - r0;
                asm volatile("" : "+v"(last));
                const float* x0 = X + (size_t)r0 * ld + kc;
#pragma unroll
                for (int i = 0; i < PER_THREAD; ++i) {
                    const int r = i * STEP < last ? i * STEP : last;
                    const float x = x0[(uint64_t)(uint32_t)r * (uint32_t)ld];   // (pitches are 32-bit)
                    v[i] = k < K ? x : 0.0f;
                }
                return;
            }
            const int kc = !TAIL || k < K ? k : K - 1;
#pragma unroll
            for (int i = 0; i < PER_THREAD; ++i) {
                int r = rb + i * STEP;
                r = r < rows ? r : rows - 1;
                const float x = X[(size_t)r * ld + kc];
                v[i] = !TAIL || k < K ? x : 0.0f;
            }
        }
    }
    static __device__ __forceinline__ void store(const float (&v)[PER_THREAD], float* lds, int tid) {
#pragma unroll
        for (int i = 0; i < PER_THREAD; ++i) {
            const int row = KM ? tid % ROWS : tid / BK + i * STEP;
            const int k = KM ? tid / ROWS + i * STEP : tid % BK;
            lds[lds_at(row, k)] = v[i];
        }
    }
    static __device__ __forceinline__ f32x4 read(const float* lds, int row, int k) {   // k multiple of 4
        if (!KM) return *reinterpret_cast<const f32x4*>(lds + lds_at(row, k));
        f32x4 v;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = lds[lds_at(row, k + j)];
        return v;
    }
};

template <class Cfg, bool A_KM, bool B_KM>
__global__ __launch_bounds__(Cfg::NT, 2) void gemm_f32_kernel(F32Args g) {
    typedef Operand<Cfg, Cfg::BM, A_KM> OA;
    typedef Operand<Cfg, Cfg::BN, B_KM> OB;
    constexpr int MI = Cfg::MI, NI = Cfg::NI, BK = Cfg::BK;
    __shared__ __attribute__((aligned(16))) float s_a[2][OA::LDS_FLOATS];
    __shared__ __attribute__((aligned(16))) float s_b[2][OB::LDS_FLOATS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
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

    float va[OA::PER_THREAD], vb[OB::PER_THREAD];
    auto load = [&](int k0) {
        if (k0 + BK <= g.K) {
            OA::template load<false>(va, g.A, g.lda, m0, g.M, k0, g.K, tid);
            OB::template load<false>(vb, g.B, g.ldb, n0, g.N, k0, g.K, tid);
        } else {
            OA::template load<true>(va, g.A, g.lda, m0, g.M, k0, g.K, tid);
            OB::template load<true>(vb, g.B, g.ldb, n0, g.N, k0, g.K, tid);
        }
    };
    int buf = 0;
    if (k_lo < k_end) {
        load(k_lo);
        OA::store(va, s_a[0], tid);
        OB::store(vb, s_b[0], tid);
    }
    __syncthreads();
    const int ra = wave_m * (MI * 16) + (lane & 15), rb = wave_n * (NI * 16) + (lane & 15), kq = 4 * (lane >> 4);
    for (int k0 = k_lo; k0 < k_end; k0 += BK) {
        const bool more = k0 + BK < k_end;
        if (more) load(k0 + BK);
#pragma unroll
        for (int c = 0; c < BK / 16; ++c) {
            f32x4 a[MI], b[NI];
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) a[mi] = OA::read(s_a[buf], ra + mi * 16, c * 16 + kq);
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) b[ni] = OB::read(s_b[buf], rb + ni * 16, c * 16 + kq);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[mi][j], b[ni][j], acc[mi][ni], 0, 0, 0);
        }
        if (more) {
            OA::store(va, s_a[buf ^ 1], tid);
            OB::store(vb, s_b[buf ^ 1], tid);
        }
        __syncthreads();
        buf ^= 1;
    }

    // accumulator lane: column lane % 16, rows 4 (lane / 16) .. + 3 of each 16 x 16 block
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = m0 + wave_m * (MI * 16) + mi * 16 + kq + j;
            if (row >= g.M) continue;
            float* out = g.k_parts > 1 ? g.partial + ((size_t)part * g.M + row) * g.N
                                       : g.C + (size_t)(g.row_map ? (int64_t)g.row_map[row] : (int64_t)row) * g.ldc;
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const int col = n0 + wave_n * (NI * 16) + ni * 16 + (lane & 15);
                if (col >= g.N) continue;
                out[col] = g.k_parts == 1 && g.accumulate ? out[col] + acc[mi][ni][j] : acc[mi][ni][j];
            }
        }
}

// Adds the k_parts partial results up, in part order, into the (mapped) rows of C.
__global__ __launch_bounds__(256) void sum_parts_f32_kernel(const float* __restrict__ partial, int k_parts, int M, int N,
                                                            float* __restrict__ C, int64_t ldc, int accumulate,
                                                            const int32_t* __restrict__ row_map) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, total = (int64_t)M * N;
    if (i >= total) return;
    float v = partial[i];
    for (int p = 1; p < k_parts; ++p) v += partial[(size_t)p * total + i];
    const int row = (int)(i / N), col = (int)(i % N);
    float* out = C + (size_t)(row_map ? (int64_t)row_map[row] : (int64_t)row) * ldc + col;
    *out = accumulate ? *out + v : v;
}

template <class Cfg>
void launch_cfg(const GemmF32& p, int parts, hipStream_t st) {
    F32Args g;
    g.A = p.A; g.lda = p.lda; g.B = p.B; g.ldb = p.ldb; g.M = p.M; g.N = p.N; g.K = p.K;
    g.tiles_n = (int)ceil_div(p.N, Cfg::BN);
    g.k_parts = parts;
    g.slices_per_part = (int)ceil_div(ceil_div(p.K, Cfg::BK), parts);
    g.C = p.C; g.ldc = p.ldc; g.accumulate = p.accumulate; g.row_map = p.row_map; g.partial = p.partial;
    const unsigned grid = (unsigned)(ceil_div(p.M, Cfg::BM) * g.tiles_n * parts);
    if (p.a_km) gemm_f32_kernel<Cfg, true, true><<<grid, Cfg::NT, 0, st>>>(g);
    else if (p.b_km) gemm_f32_kernel<Cfg, false, true><<<grid, Cfg::NT, 0, st>>>(g);
    else gemm_f32_kernel<Cfg, false, false><<<grid, Cfg::NT, 0, st>>>(g);
}

}  // namespace

// Most parts the K dimension of an [M, K] x [K, N] product is cut into (at least 256 k-values each).
int gemm_f32_max_parts(int64_t K) {
    const int64_t p = K / 256;
    return (int)(p < 1 ? 1 : p > 16 ? 16 : p);
}

// Tile and K split: the least estimated time of the compute unit with most work, tile area x K x a factor for what
// smaller tiles lose on loads and latency, plus 64 k-values for a tile's start and end and a constant for the
// summing launch of a split. Large products take 128 x 128 tiles; with 100 tokens of D = 64 and V = 512 the 32 x 32
// tiles spread the work over 64 compute units instead of 4.
void launch_gemm_f32(const GemmF32& p, int cus, hipStream_t st) {
    if (p.M <= 0 || p.N <= 0) return;
    static const struct { int edge; double cost; } tile[3] = {{128, 1.0}, {64, 1.25}, {32, 2.0}};
    const int max_parts = p.partial ? (p.max_parts < gemm_f32_max_parts(p.K) ? p.max_parts : gemm_f32_max_parts(p.K)) : 1;
    int best = 0, parts = 1;
    double best_t = -1.0;
    for (int c = 0; c < 3; ++c) {
        const int64_t tiles = ceil_div(p.M, tile[c].edge) * ceil_div(p.N, tile[c].edge);
        for (int q = 1; q <= max_parts; ++q) {
            const double t = (double)ceil_div(tiles * q, cus) * tile[c].edge * tile[c].edge * tile[c].cost *
                                 ((double)p.K / q + 64.0) + (q > 1 ? 4e6 : 0.0);
            if (best_t < 0.0 || t < best_t) { best_t = t; best = c; parts = q; }
        }
    }
    if (best == 0) launch_cfg<F32Big>(p, parts, st);
    else if (best == 1) launch_cfg<F32Mid>(p, parts, st);
    else launch_cfg<F32Small>(p, parts, st);
    if (parts > 1)
        sum_parts_f32_kernel<<<(unsigned)ceil_div((int64_t)p.M * p.N, 256), 256, 0, st>>>(p.partial, parts, p.M, p.N, p.C,
                                                                                          p.ldc, p.accumulate, p.row_map);
}

}  // namespace dppo
