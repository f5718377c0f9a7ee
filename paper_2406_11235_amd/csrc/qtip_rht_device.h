// Device-side core of the random Hadamard transform (Section 2.1 of arXiv 2406.11235): a
// block-diagonal Walsh-Hadamard transform with +-1 signs, on the matrix cores.  Used by the
// stand-alone kernel and by the decode + matvec kernel that transforms its own input.
//
// A chunk of 4096 values, index (t, j, a) of four bits each, is H_16 (x) H_16 (x) H_16 applied to the
// three digits one after the other:
//   a: D1[j][a'] = sum_a X[j][a] H[a][a']     on the matrix cores, one tile t = 256 values at a time, X
//                                             the A operand: a lane holds four neighbouring inputs;
//   j: D2[j'][a'] = sum_j H[j'][j] D1[j][a']  D1 stays where it is: the result layout of the matrix
//                                             cores is the B operand layout with the contraction
//                                             index in the order (lane / 16, register);
//   t: after one exchange through LDS a lane holds four neighbouring values of one t, and the 16 lanes
//      of a row hold the 16 t: butterflies with DPP operands.
// Blocks of 2^p < 4096 values leave out the butterflies above bit p; below 256 the digit j takes
// butterflies too, so that a value meets nothing but its own block (a product with a matrix
// that has zeros would carry an infinity into the neighbours as 0 inf).  Blocks of 8192 and 16384 add
// one or two butterfly stages between chunks, which a lane has at the same places.
// Inputs, sums and results are binary32; the 1/sqrt(block) scale and the rounding to binary16 happen once, at the end.
//
// What bounds it at batch 1 is latency, and this form has little: one load, 4 + 4 matrix
// instructions, one barrier, 32 additions.  (16 values per thread through twelve butterfly stages
// in registers, with an exchange after every four of them, has three times as many instructions in a row.)
#pragma once
#include "qtip_device.h"

namespace qtip {

constexpr int RHT_CHUNK = 4096;
// LDS of the exchange: [t][j][a] with j apart by 20 and t by 324 floats, so that the 32 lanes of a pass
// fall on different banks where D2 is written (j = 4 (lane / 16) + register), and the 8 lanes of a pass
// where four neighbouring values are read at once (t = 0..7 in some order).
constexpr int RHT_LDS_J = 20, RHT_LDS_T = 324, RHT_LDS_FLOATS = 16 * RHT_LDS_T;

// 2^(-p/2) as an exact power of two times the correctly rounded 1/sqrt(2).
__device__ __forceinline__ float rht_scale(int p) {
    return ((p & 1) ? 0.70710678118654752440f : 1.0f) * __builtin_bit_cast(float, (uint32_t)(127 - (p >> 1)) << 23);
}

// The signs of four neighbouring values (four bytes of +-1, negative ones have bit 7 set) applied.
__device__ __forceinline__ half4_t rht_signed(half4_t v, uint32_t s) {
    const u32x2_t w = __builtin_bit_cast(u32x2_t, v);
    return __builtin_bit_cast(half4_t, u32x2_t{w.x ^ ((s << 8) & 0x8000u) ^ ((s << 16) & 0x80000000u),
                                               w.y ^ ((s >> 8) & 0x8000u) ^ (s & 0x80000000u)});
}
__device__ __forceinline__ float4_t rht_signed(float4_t v, uint32_t s) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 w = __builtin_bit_cast(u32x4, v);
    return __builtin_bit_cast(float4_t, w ^ u32x4{(s << 24) & 0x80000000u, (s << 16) & 0x80000000u,
                                                  (s << 8) & 0x80000000u, s & 0x80000000u});
}

// Entries (lane % 16, 4 (lane / 16) + r) of H, +-1: an A or B operand.
struct RhtMatrix {
    float4_t h;
    __device__ __forceinline__ void init(int lane) {
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const uint32_t bits = (uint32_t)(lane & 15) & (uint32_t)(4 * (lane >> 4) + r);
            h[r] = __builtin_bit_cast(float, 0x3F800000u | ((uint32_t)__builtin_popcount(bits) << 31));
        }
    }
};

__device__ __forceinline__ float4_t rht_digit_a(float4_t x, const RhtMatrix &M) {
    float4_t d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 4; r++) d = __builtin_amdgcn_mfma_f32_16x16x4f32(x[r], M.h[r], d, 0, 0, 0);
    return d;
}
// (binary16 inputs are converted: the binary16 matrix instruction, one in place of four, adds in another order,
// and a vector in either type has one transform.)
__device__ __forceinline__ float4_t rht_digit_a(half4_t x, const RhtMatrix &M) {
    return rht_digit_a(float4_t{(float)x[0], (float)x[1], (float)x[2], (float)x[3]}, M);
}
// Digit j of blocks of 2^p values: j = 4 (lane / 16) + register.
__device__ __forceinline__ float4_t rht_digit_j(float4_t d, const RhtMatrix &M, int p, int lane) {
    if (p >= 8) {
        float4_t e = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 4; r++) e = __builtin_amdgcn_mfma_f32_16x16x4f32(M.h[r], d[r], e, 0, 0, 0);
        return e;
    }
    if (p >= 5) d = float4_t{d[0] + d[1], d[0] - d[1], d[2] + d[3], d[2] - d[3]};
    if (p >= 6) d = float4_t{d[0] + d[2], d[1] + d[3], d[0] - d[2], d[1] - d[3]};
    if (p >= 7) {
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const float o = __shfl_xor(d[r], 16, 64);
            d[r] = lane & 16 ? o - d[r] : d[r] + o;
        }
    }
    return d;
}
// One butterfly stage over the lanes of a row of 16: CTRL is the DPP pattern that brings a lane its
// partner, `upper` says that the lane is the one that subtracts.
template <int CTRL>
__device__ __forceinline__ void rht_lane_stage(float4_t &v, bool upper) {
    const uint32_t flip = upper ? 0x80000000u : 0u;
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const float mine = v[r];  // (a value of its own: the compiler's bit cast of a vector element takes element 0)
        const float other = __builtin_bit_cast(
            float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, mine), CTRL, 0xF, 0xF, true));
        v[r] = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, mine) ^ flip) + other;
    }
}
// The t that lane l of a row of 16 holds.  DPP can exchange lanes l and l ^ 1, l ^ 2, l ^ 7 (mirrored halves
// of a row) and l ^ 15 (a mirrored row), but not l ^ 4: so t's bits are the coordinates of l in the
// basis 1, 2, 7, 15, and changing one bit of t is one of these exchanges.
__device__ __forceinline__ int rht_lane_t(int l) {
    const int b3 = (l >> 3) & 1, b2 = ((l >> 2) & 1) ^ b3, up = b2 ^ b3;
    return (b3 << 3) | (b2 << 2) | ((l & 3) ^ (up ? 3 : 0));
}
__device__ __forceinline__ void rht_digit_t(float4_t &v, int p, int t) {
    if (p >= 9) rht_lane_stage<0xB1>(v, t & 1);    // quad_perm [1, 0, 3, 2]
    if (p >= 10) rht_lane_stage<0x4E>(v, t & 2);   // quad_perm [2, 3, 0, 1]
    if (p >= 11) rht_lane_stage<0x141>(v, t & 4);  // row_half_mirror
    if (p >= 12) rht_lane_stage<0x140>(v, t & 8);  // row_mirror
}

// Where lane l's four results of tile number w (0..15) belong in the chunk.
__device__ __forceinline__ int rht_out_index(int w, int lane) {
    return 256 * rht_lane_t(lane & 15) + 16 * w + 4 * (lane >> 4);
}
// Where its four inputs are.
__device__ __forceinline__ int rht_in_index(int w, int lane) { return 256 * w + 16 * (lane & 15) + 4 * (lane >> 4); }

// One chunk by a workgroup of NW waves (a power of two, at most 16), every one of which makes the call.
// x[i]: the inputs of tile wave + NW i, signs applied; the chunk's first `tiles` tiles have values.  y[i]: the
// sums of tile number wave + NW i.
// s_v: RHT_LDS_FLOATS floats.  Between two calls on the same s_v the caller synchronizes the workgroup.
template <int NW, typename T4>
__device__ __forceinline__ void rht_chunk(const T4 (&x)[16 / NW], const RhtMatrix &M, int p, int tiles, float *s_v,
                                          int wave, int lane, float4_t (&y)[16 / NW]) {
    const int i16 = lane & 15, g = lane >> 4;
#pragma unroll
    for (int i = 0; i < 16 / NW; i++) {
        if (wave + NW * i >= tiles) break;
        const float4_t d = rht_digit_j(rht_digit_a(x[i], M), M, p, lane);
        float *at = s_v + (wave + NW * i) * RHT_LDS_T + 4 * g * RHT_LDS_J + i16;
#pragma unroll
        for (int r = 0; r < 4; r++) at[r * RHT_LDS_J] = d[r];
    }
    __syncthreads();
    const int t = rht_lane_t(i16);
#pragma unroll
    for (int i = 0; i < 16 / NW; i++) {
        y[i] = *reinterpret_cast<const float4_t *>(s_v + t * RHT_LDS_T + (wave + NW * i) * RHT_LDS_J + 4 * g);
        rht_digit_t(y[i], p, t);
    }
}

// Scale and round.  (The binary32 product and the rounding to binary16 are kept apart: left alone, the compiler
// merges them into one v_fma_mixlo_f16, a single rounding, in some instantiations and not in others.)
__device__ __forceinline__ half4_t rht_round(float4_t v, float scale) {
    half4_t h;
#pragma unroll
    for (int r = 0; r < 4; r++) {
        float t = v[r] * scale;
        asm volatile("" : "+v"(t));
        h[r] = (half_t)t;
    }
    return h;
}

// The butterfly stages between NCH chunks.
template <int NCH, int N>
__device__ __forceinline__ void rht_between_chunks(float4_t (&y)[NCH][N]) {
#pragma unroll
    for (int h = 1; h < NCH; h <<= 1)
#pragma unroll
        for (int c = 0; c < NCH; c++)
            if ((c & h) == 0) {
#pragma unroll
                for (int i = 0; i < N; i++) {
                    const float4_t a = y[c][i], b = y[c | h][i];
                    y[c][i] = a + b;
                    y[c | h][i] = a - b;
                }
            }
}

}  // namespace qtip
