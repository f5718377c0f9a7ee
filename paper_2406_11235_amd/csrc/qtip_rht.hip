// Random Hadamard transform of activations (Section 2.1 of arXiv 2406.11235):
// a block-diagonal Walsh-Hadamard transform with +-1 sign vectors.
//
// A workgroup transforms NCH chunks of 4096 values of one batch row (NCH = 1, or 2 and 4 for blocks
// of 8192 and 16384) with rht_chunk (qtip_rht_device.h).  At batch 1 a launch of next to nothing takes 2.0 us in
// a stream of dependent ones; this one takes 2.5 to 3.0 (28672 values), from binary32 2.5 to 3.1 (butterflies in
// registers, 16 values per thread, and the output's signs fetched at the end: 2.5 to 3.1 and 3.9 to 4.6).
#include "qtip_device.h"
#include "qtip_internal.h"
#include "qtip_rht_device.h"

namespace qtip {

// signs_n: the signs repeat after that many values.  It is n, except where the rows of a batch are
// taken as one long row.
template <typename TIN, int NW, int NCH>
__global__ __launch_bounds__(NW * 64) void rht_kernel(const TIN *__restrict__ x, const int8_t *__restrict__ signs,
                                                      uint32_t n, uint32_t signs_n, int p, int side,
                                                      half_t *__restrict__ out) {
    typedef TIN T4 __attribute__((ext_vector_type(4)));
    constexpr int N = 16 / NW;
    __shared__ __attribute__((aligned(16))) float s_v[RHT_LDS_FLOATS];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const uint32_t base = blockIdx.x * (uint32_t)(NCH * RHT_CHUNK);
    x += (size_t)blockIdx.y * n;
    out += (size_t)blockIdx.y * n;
    const uint32_t base_sign = signs_n == n ? base : base % signs_n;
    auto sign_word = [&](uint32_t idx) {
        uint32_t at = base_sign + (idx - base);
        if (signs_n != n) {  // (a chunk meets the end of a row at most once where a row is longer)
            if (signs_n >= RHT_CHUNK) at -= at >= signs_n ? signs_n : 0u;
            else at %= signs_n;
        }
        return *reinterpret_cast<const uint32_t *>(signs + at);
    };
    T4 v[NCH][N];
    uint32_t s_in[NCH][N], s_out[NCH][N];
#pragma unroll
    for (int c = 0; c < NCH; c++)
#pragma unroll
        for (int i = 0; i < N; i++) {
            // (beyond n: any values; no block in [0, n) has them)
            const uint32_t in = min(base + c * RHT_CHUNK + rht_in_index(wave + NW * i, lane), n - 4);
            const uint32_t to = min(base + c * RHT_CHUNK + rht_out_index(wave + NW * i, lane), n - 4);
            v[c][i] = *reinterpret_cast<const T4 *>(x + in);
            // (the signs of the output too are asked for here, not when the sums wait for them)
            if (side == 0) s_in[c][i] = sign_word(in);
            else s_out[c][i] = sign_word(to);
        }
    RhtMatrix M;
    M.init(lane);
    const float scale = rht_scale(p);
    float4_t y[NCH][N];
#pragma unroll
    for (int c = 0; c < NCH; c++) {
        if (side == 0) {
#pragma unroll
            for (int i = 0; i < N; i++) v[c][i] = rht_signed(v[c][i], s_in[c][i]);
        }
        if (c > 0) __syncthreads();
        rht_chunk<NW>(v[c], M, p, 16, s_v, wave, lane, y[c]);
    }
    rht_between_chunks<NCH, N>(y);
#pragma unroll
    for (int c = 0; c < NCH; c++)
#pragma unroll
        for (int i = 0; i < N; i++) {
            const uint32_t to = base + c * RHT_CHUNK + rht_out_index(wave + NW * i, lane);
            half4_t h = rht_round(y[c][i], scale);
            if (side != 0) h = rht_signed(h, s_out[c][i]);
            if (to < n) *reinterpret_cast<half4_t *>(out + to) = h;
        }
}

hipError_t launch_rht(const void *x, bool x_is_f32, const int8_t *signs, int n, int block,
                      int batch, int side, void *out, hipStream_t st) {
    int p = 0;
    while ((1 << p) < block) p++;
    const int nch = block > RHT_CHUNK ? block / RHT_CHUNK : 1;
    uint32_t row = (uint32_t)n, rows = (uint32_t)batch;
    // Rows that are not whole chunks: the batch is one long row, or its last chunks would stay part empty.
    // (Blocks lie one after the other in it as in the rows.)
    if (n % RHT_CHUNK != 0 && (uint64_t)n * batch < (1u << 31)) {
        row = (uint32_t)n * batch;
        rows = 1;
    }
    const uint32_t gx = (row + nch * RHT_CHUNK - 1) / (nch * RHT_CHUNK);
    // A wave per tile (16 waves) while there are no more workgroups than the chip runs at a time: the shortest
    // chain from load to store.  Beyond that 8 waves of two tiles (binary32, 997 x 14336 in blocks of 2048: 23.6 us
    // against 27.5 with 16 waves and 27.0 with 4).
    const bool wide = (uint64_t)gx * rows <= 512;
#define QTIP_RHT_LAUNCH(T, NW, NCH)                                                                            \
    hipLaunchKernelGGL((rht_kernel<T, NW, NCH>), dim3(gx, rows), dim3(NW * 64), 0, st, (const T *)x, signs, row, \
                       (uint32_t)n, p, side, (half_t *)out)
#define QTIP_RHT_BY_SIZE(T)                              \
    if (nch == 4) QTIP_RHT_LAUNCH(T, 16, 4);             \
    else if (nch == 2) QTIP_RHT_LAUNCH(T, 16, 2);        \
    else if (wide) QTIP_RHT_LAUNCH(T, 16, 1);            \
    else QTIP_RHT_LAUNCH(T, 8, 1);
    if (x_is_f32) {
        QTIP_RHT_BY_SIZE(float);
    } else {
        QTIP_RHT_BY_SIZE(half_t);
    }
    return hipGetLastError();
}

}  // namespace qtip
