// What a loss token is, shared by the kernels that gather its rows and those that read them where they lie.
#pragma once
#include "dppo_internal.h"

namespace dppo {

// Row of H and target id of loss token i, clamped into range; returns what had to be clamped.
__device__ __forceinline__ int locate_token(const int32_t* ids, const int32_t* loss_pos, int64_t T, int32_t V, int64_t i, int64_t& row,
                                            int32_t& target) {
    int flags = 0;
    row = loss_pos ? (int64_t)loss_pos[i] : i;
    int64_t pos = loss_pos ? row + 1 : row;
    if (row < 0 || pos >= T) flags |= DPPO_HEAD_BAD_POSITION;
    row = row < 0 ? 0 : (row >= T ? T - 1 : row);
    pos = pos < 0 ? 0 : (pos >= T ? T - 1 : pos);
    target = ids[pos];
    if (target < 0 || target >= V) flags |= DPPO_HEAD_BAD_TARGET;
    target = target < 0 ? 0 : (target >= V ? V - 1 : target);
    return flags;
}
// s + x . b of 8 bfloat16 values.
__device__ __forceinline__ float dot_bf16x8(uint4 x, uint4 b, float s) {
    const uint32_t aw[4] = {x.x, x.y, x.z, x.w}, bw[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        s = fmaf(__uint_as_float(aw[k] << 16), __uint_as_float(bw[k] << 16), s);
        s = fmaf(__uint_as_float(aw[k] & 0xffff0000u), __uint_as_float(bw[k] & 0xffff0000u), s);
    }
    return s;
}
// Dot product of the bfloat16 rows h and w of D elements (whole 16-byte vectors) by one wavefront, in every lane. All loads of
// up to 8 vectors first: one by one, the wavefront waits for memory D / 512 times over.
__device__ __forceinline__ float dot_bf16_rows(const uint16_t* h_, const uint16_t* w_, int32_t D, int lane) {
    constexpr int U = 8;
    const uint4 *h = reinterpret_cast<const uint4*>(h_), *w = reinterpret_cast<const uint4*>(w_);
    const int vectors = D / 8;
    float s = 0.0f;
    for (int c0 = lane; c0 < vectors; c0 += 64 * U) {
        uint4 x[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + u * 64;
            x[u] = c < vectors ? h[c] : make_uint4(0, 0, 0, 0);
            b[u] = c < vectors ? w[c] : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (c0 + u * 64 >= vectors) break;
            s = dot_bf16x8(x[u], b[u], s);
        }
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    return s;
}

}  // namespace dppo
