// Decode kernels for gfx950: dequantize, fused decode + matrix-vector product on
// the vector ALUs, and fused decode + batched product on the matrix cores.
//
// Work split (all three): one workgroup owns one tile row I (16 output rows)
// and walks the tiles (I, J) along the input dimension, so outputs are written
// once by their owner and no atomics or zero-filled buffers are needed.  The
// waves of a workgroup take contiguous J ranges and their partial sums meet in
// LDS at the end.
#include <type_traits>

#include "qtip_device.h"
#include "qtip_internal.h"
#include "qtip_rht_device.h"

namespace qtip {

// The same plus the first word of the next lane of the same tile (cyclically: the
// tail-biting wrap of Section 3.2).
template <int K>
__device__ __forceinline__ void load_tile_words(const uint32_t *__restrict__ codes, size_t tile,
                                                int lane, uint32_t (&w)[Geo<K>::WPL + 1]) {
    constexpr int WPL = Geo<K>::WPL, LPT = Geo<K>::LPT;
    const int q = lane & (LPT - 1);
    const Words<K> r = load_words<K>(codes, tile, q);
#pragma unroll
    for (int i = 0; i < WPL; i++) w[i] = r.v[i];
    w[WPL] = __shfl(w[0], (lane & ~(LPT - 1)) | ((q + 1) & (LPT - 1)), 64);
}

// Decode tile row rr (0..RPL-1) of this lane: 16 fp16 weights as 8 pairs.
template <int K, int V, int CODE, int NWD>
__device__ __forceinline__ void decode_row(const uint32_t (&w)[NWD], int rr,
                                           const uint32_t *lut, half2_t (&out)[8]) {
#pragma unroll
    for (int c = 0; c < 8; c++) {
        if constexpr (V == 2) {
            uint32_t st = window16(w, rr * 16 * K + c * 2 * K);
            out[c] = CODE == CODE_HYB2 ? code_hyb2(st, lut) : code_hyb(st, lut);
        } else {
            uint32_t s0 = window16(w, rr * 16 * K + (2 * c) * K);
            uint32_t s1 = window16(w, rr * 16 * K + (2 * c + 1) * K);
            half2_t h;
            if constexpr (CODE == CODE_HYB1) {
                h.x = code_hyb1(s0, reinterpret_cast<const uint16_t *>(lut));
                h.y = code_hyb1(s1, reinterpret_cast<const uint16_t *>(lut));
            } else if constexpr (CODE == CODE_3INST) {
                h.x = code_3inst(s0);
                h.y = code_3inst(s1);
            } else {
                h.x = code_1mad(s0);
                h.y = code_1mad(s1);
            }
            out[c] = h;
        }
    }
}

__device__ __forceinline__ void stage_lut(const uint32_t *__restrict__ lut, uint32_t *s_lut) {
    for (int i = threadIdx.x; i < (1 << HYB_Q); i += blockDim.x) s_lut[i] = lut[i];
    __syncthreads();
}

// ---------------------------------------------------------------- dequantize

template <int K, int V, int CODE>
__global__ __launch_bounds__(256) void dequantize_kernel(const uint32_t *__restrict__ codes,
                                                         const uint32_t *__restrict__ lut,
                                                         int tn, long ntiles,
                                                         half_t *__restrict__ W) {
    constexpr int WPL = Geo<K>::WPL, LPT = Geo<K>::LPT, RPL = Geo<K>::RPL;
    constexpr int TPW = 64 / LPT;  // tiles per wave per step
    __shared__ uint32_t s_lut[1 << HYB_Q];
    if constexpr (code_is_hyb(CODE)) stage_lut(lut, s_lut);
    const int lane = threadIdx.x & 63;
    const long wave = (long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const long tile = wave * TPW + lane / LPT;
    const bool valid = tile < ntiles;
    uint32_t w[WPL + 1];
    load_tile_words<K>(codes, valid ? tile : ntiles - 1, lane, w);
    if (!valid) return;
    const long I = tile / tn, J = tile % tn;
    const int q = lane & (LPT - 1);
    const size_t n = (size_t)tn * 16;
#pragma unroll
    for (int rr = 0; rr < RPL; rr++) {
        half2_t h[8];
        decode_row<K, V, CODE>(w, rr, code_is_hyb(CODE) ? s_lut : lut, h);
        uint4 lo = {as_u32(h[0]), as_u32(h[1]), as_u32(h[2]), as_u32(h[3])};
        uint4 hi = {as_u32(h[4]), as_u32(h[5]), as_u32(h[6]), as_u32(h[7])};
        uint4 *dst = reinterpret_cast<uint4 *>(W + (size_t)(16 * I + q * RPL + rr) * n + 16 * J);
        dst[0] = lo;
        dst[1] = hi;
    }
}

// -------------------------------------------------------- decode one state each

template <int CODE>
__global__ void decode_states_kernel(const uint32_t *__restrict__ states, int count,
                                     const uint32_t *__restrict__ lut, half_t *__restrict__ out) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    uint32_t st = states[i] & 0xFFFFu;
    if constexpr (code_is_hyb(CODE)) {
        half2_t h = CODE == CODE_HYB2 ? code_hyb2(st, lut) : code_hyb(st, lut);
        out[2 * i] = h.x;
        out[2 * i + 1] = h.y;
    } else if constexpr (CODE == CODE_HYB1) {
        out[i] = code_hyb1(st, reinterpret_cast<const uint16_t *>(lut));
    } else if constexpr (CODE == CODE_3INST) {
        out[i] = code_3inst(st);
    } else {
        out[i] = code_1mad(st);
    }
}

// ------------------------------------------------------- decode + matvec (B = 1)

// A value of the lane `off` lanes away (lane ^ off), any off < 64.
__device__ __forceinline__ float lane_xor(float v, int lane, int off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((lane ^ off) << 2, __builtin_bit_cast(int, v)));
}
// v + the value of the lane N places further round this lane's row of 16 (a DPP row rotate).
template <int N> __device__ __forceinline__ float add_row_ror(float v) {
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + N, 0xF, 0xF, false));
}
// The end of the batch-1 kernels: lane = g * LPT + q holds RPL partial sums, rows q * RPL + rr
// of the tile row, and the 64 / LPT lanes with the same q are to be added up.  Over lane bits 5
// and 4 the lanes trade sums instead of each adding all of them: a lane hands the partner the
// rows the partner keeps and adds what it gets to the rows it keeps itself, so the number of
// sums per lane halves with every exchange (three cross-lane reads at RPL = 4, two at RPL = 2,
// where adding everything everywhere takes sixteen and six); the lane bits below 4 are summed
// with row rotates inside the vector ALU.  On return acc[0] is the whole sum for row
// q * RPL + (return value), the same in all lanes that differ only in the lane bits below 4
// that belong to g.
template <int LPT, int RPL>
__device__ __forceinline__ int reduce_over_tile_groups(float (&acc)[RPL], int lane) {
    static_assert((LPT <= 4 && RPL == 4) || (LPT == 8 && RPL == 2), "tile geometries of MvGeo");
    const bool b5 = lane & 32, b4 = lane & 16;
    float v;
    if constexpr (RPL == 4) {
        // bit 5 clear keeps rows 0 and 1, set keeps rows 2 and 3
        const float r0 = lane_xor(b5 ? acc[0] : acc[2], lane, 32), r1 = lane_xor(b5 ? acc[1] : acc[3], lane, 32);
        const float v0 = (b5 ? acc[2] : acc[0]) + r0, v1 = (b5 ? acc[3] : acc[1]) + r1;
        // bit 4 clear keeps the first of the two, set the second
        v = (b4 ? v1 : v0) + lane_xor(b4 ? v0 : v1, lane, 16);
        v = add_row_ror<8>(v);
        v = add_row_ror<4>(v);
        if constexpr (LPT <= 2) v = add_row_ror<2>(v);
        if constexpr (LPT <= 1) v = add_row_ror<1>(v);
        acc[0] = v;
        return (b5 ? 2 : 0) + (b4 ? 1 : 0);
    } else {
        v = (b5 ? acc[1] : acc[0]) + lane_xor(b5 ? acc[0] : acc[1], lane, 32);
        v += lane_xor(v, lane, 16);
        v = add_row_ror<8>(v);
        acc[0] = v;
        return b5 ? 1 : 0;
    }
}

// FUSED: x is the untransformed activation and the workgroup first computes the input-side
// random Hadamard transform V (S .* x) of Section 2.1 into LDS itself (every workgroup the
// whole vector, at most 8192 values, against a kernel launch and the gap to the next
// dependent kernel, which cost more for layers this small), with the device function
// of the stand-alone transform, so that the result is the same bit for bit.
constexpr int FUSED_MAX_N = 8192;

// SPREAD: the HYB codes' table in 16 copies (see RowDotHyb); it costs 64 KiB of LDS and their
// filling per workgroup, and pays on long rows.  (Eight waves per SIMD, i.e. at most 64
// registers: the loop needs no more, and a second workgroup per CU is worth more than the few
// values that spill around it.)
// (The V = 1 hash code keeps a whole tile's table reads in flight and needs more registers; the
// kernel that transforms its own input runs with at most one workgroup per CU, four waves per
// SIMD, and may take the registers that leaves it.)
// S: workgroups per tile row, 16 / S rows each (the launcher splits a tile row where whole ones leave CUs idle): this one
// does part `part` of tile row I.
template <int K, int V, int CODE, int S, int NW, bool FUSED, bool SPREAD, bool WIDE, bool ROUNDS = false>
__device__ __forceinline__ void matvec_tile_row(int I, int Iend, int part, bool staged, const uint32_t *__restrict__ codes,
                                                const uint32_t *__restrict__ lut, int tn, const half_t *__restrict__ x,
                                                const int8_t *__restrict__ signs, int log2_block,
                                                const half_t *__restrict__ scale, float *__restrict__ y,
                                                uint32_t *s_lut, float (*s_part)[16], half_t *s_x, float *s_v) {
    constexpr int WPL = MvGeo<K, WIDE>::WPL, LPT = MvGeo<K, WIDE>::LPT / S, RPL = MvGeo<K, WIDE>::RPL;
    constexpr int ROWS = 16 / S;
    constexpr int TPI = 64 / LPT;  // tiles per wave per iteration
    // the wave's number as a scalar: its tile range and the loop over it then live in scalar
    // registers and the loop control costs no vector instructions
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int g = lane / LPT, q = lane & (LPT - 1);
    const int chunk = ((tn + NW * TPI - 1) / (NW * TPI)) * TPI;
    const int J0 = wave * chunk;
    const int Jend = min(tn, J0 + chunk);
    // this tile row's words: a uniform base, so that a lane's address is base + 32-bit offset
    const uint32_t *row_codes = codes + (size_t)I * tn * (8 * K);
    struct Operands {
        WordsN<WPL> w;
        uint32_t next;  // S > 1: the word behind them
        uint4 xa, xb;
    };
    auto issue_words = [&](Operands &o, int Jb) {
        const uint32_t Jc = min(Jb + g, Jend - 1);  // lanes past the end re-read the last tile
        // (byte offsets in 32 bits from uniform bases: the loads take them as they are)
        o.w = load_words_at<WPL>(row_codes, Jc * (32 * K) + (part * LPT + q) * (4 * WPL));
        if constexpr (S > 1)
            o.next = stream_load(reinterpret_cast<const uint32_t *>(
                reinterpret_cast<const char *>(row_codes) + (size_t)(Jc * (32 * K) + ((part * LPT + q + 1) * WPL) % (8 * K) * 4)));
    };
    auto issue_x = [&](Operands &o, int Jb) {
        const uint32_t Jc = min(Jb + g, Jend - 1);
        if constexpr (FUSED) {
            const uint4 *xp = reinterpret_cast<const uint4 *>(s_x + 16 * Jc);
            o.xa = xp[0];
            o.xb = xp[1];
        } else {
            const uint4 *xp = reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(x) + (size_t)(Jc * 32u));
            o.xa = xp[0];
            o.xb = xp[1];
        }
    };
    auto issue = [&](Operands &o, int Jb) {
        issue_words(o, Jb);
        issue_x(o, Jb);
    };
    Operands opA, opB;
    if constexpr (FUSED) {
        constexpr int N = 16 / NW, NCH = NW == 16 || S > 1 ? 2 : 1;  // (else a row of less than 4096 values)
        const int n = 16 * tn;
        half4_t v[NCH][N];
        uint32_t sg[NCH][N];
#pragma unroll
        for (int c = 0; c < NCH; c++)
#pragma unroll
            for (int i = 0; i < N; i++) {
                const int at = min(c * RHT_CHUNK + rht_in_index(wave + NW * i, lane), n - 4);
                v[c][i] = *reinterpret_cast<const half4_t *>(x + at);
                sg[c][i] = *reinterpret_cast<const uint32_t *>(signs + at);
            }
        // the first step's words, from memory, arrive while the input is transformed
        if (J0 < Jend) issue_words(opA, J0);
        RhtMatrix M;
        M.init(lane);
        float4_t sum[NCH][N];
#pragma unroll
        for (int c = 0; c < NCH; c++) {
            if (c * RHT_CHUNK >= n) break;
#pragma unroll
            for (int i = 0; i < N; i++) v[c][i] = rht_signed(v[c][i], sg[c][i]);
            if (c > 0) __syncthreads();
            rht_chunk<NW>(v[c], M, log2_block, (n - c * RHT_CHUNK + 255) >> 8, s_v, wave, lane, sum[c]);
        }
        if (log2_block == 13) rht_between_chunks<NCH, N>(sum);
        const float unit = rht_scale(log2_block);
#pragma unroll
        for (int c = 0; c < NCH; c++)
#pragma unroll
            for (int i = 0; i < N; i++) {
                const int to = c * RHT_CHUNK + rht_out_index(wave + NW * i, lane);
                if (to < n) *reinterpret_cast<half4_t *>(s_x + to) = rht_round(sum[c][i], unit);
            }
        if constexpr (code_lds_words(CODE) == 1) __syncthreads();
    } else {
        // (ahead of the table, so that they are under way while it is filled)
        if (J0 < Jend) issue(opA, J0);
    }
    if (!staged) stage_code_table<CODE, SPREAD>(lut, s_lut, NW * 64);
    typename RowDotFor<K, CODE, SPREAD>::type rd;
    rd.init(s_lut);
    float acc[RPL];
#pragma unroll
    for (int rr = 0; rr < RPL; rr++) acc[rr] = 0.f;

    // Software pipeline: the loads of step i+1 are in flight while step i is decoded.
    // Two operand sets alternate (the loop body is two steps), so nothing is copied
    // (3-4 % on the computed codes, measured against the copying form on one box).
    auto compute = [&](const Operands &o, int Jb) {
        uint32_t w[WPL + 1];
#pragma unroll
        for (int i = 0; i < WPL; i++) w[i] = o.w.v[i];
        // first word of the next lane of the same tile, cyclically (tail-biting wrap)
        if constexpr (S > 1) w[WPL] = o.next;
        else w[WPL] = __shfl(w[0], (lane & ~(LPT - 1)) | ((q + 1) & (LPT - 1)), 64);
        if (Jb + g < Jend) {
            uint32_t xv[8] = {o.xa.x, o.xa.y, o.xa.z, o.xa.w, o.xb.x, o.xb.y, o.xb.z, o.xb.w};
            rd.prep_x(xv);
            rd.run_tile(w, xv, acc);
        }
    };
    if constexpr (FUSED) {
        if (J0 < Jend) issue_x(opA, J0);
    }
    auto finish_row = [&](int buf) {
        rd.finish(acc);
        const int rr_mine = reduce_over_tile_groups<LPT, RPL>(acc, lane);
        float(*const part_sums)[16] = s_part + buf * NW;
        if ((g & (16 / LPT - 1)) == 0) part_sums[wave][q * RPL + rr_mine] = acc[0];
        __syncthreads();
        if (threadIdx.x < ROWS) {
            float s = 0.f;
#pragma unroll
            for (int wv = 0; wv < NW; wv++) s += part_sums[wv][threadIdx.x];
            const int row = 16 * I + ROWS * part + threadIdx.x;
            if (scale) s *= (float)scale[row];
            y[row] = s;
        }
    };
    if constexpr (ROUNDS) {
        const int J1 = J0 + max(1, (Jend - J0 + TPI - 1) / TPI) * TPI;
        if (J0 >= Jend) issue(opA, J0);
        int Jb = J0, buf = 0;
        // one step: the next one's operands into `other`, decode, and the row's end; false after the last
        auto step = [&](Operands &o, Operands &other) {
            int Jn = Jb + TPI, In = I;
            if (Jn >= J1) {
                Jn = J0;
                In = I + (int)gridDim.x;
                row_codes = codes + (size_t)In * tn * (8 * K);
            }
            if (In < Iend) issue(other, Jn);
            compute(o, Jb);
            if (Jn == J0) {
                finish_row(buf);
                buf ^= 1;
#pragma unroll
                for (int rr = 0; rr < RPL; rr++) acc[rr] = 0.f;
                rd.init(s_lut);
            }
            Jb = Jn;
            I = In;
            return I < Iend;
        };
        while (step(opA, opB) && step(opB, opA)) {}
        return;
    }
    for (int Jb = J0; Jb < Jend; Jb += 2 * TPI) {
        if (Jb + TPI < Jend) issue(opB, Jb + TPI);
        compute(opA, Jb);
        if (Jb + TPI < Jend) {
            if (Jb + 2 * TPI < Jend) issue(opA, Jb + 2 * TPI);
            compute(opB, Jb + TPI);
        }
    }
    finish_row(0);
}
// TAIL 2 or 4: the tile rows from `whole` on are split into as many parts, by workgroups behind those of the whole ones (ahead
// of them, or the whole rows in a loop over at most 512 workgroups, is slower; in this order, on one card: 3INST 14336 x 4096
// 10.44, 10.85 and 10.52 us, 1MAD 5120 x 8192 8.45, 9.51 and 11.5).  ROUNDS, for the V = 1 hash code, of which one workgroup fits a CU, so that nothing is decoded
// while another one begins and ends: the whole rows in rounds over at most 256 workgroups that keep their table and
// have the next row's words under way, then the others' parts, if any (14336 x 4096 k = 4 19.1 -> 15.5 us, k = 2 16.7 -> 13.3).
// (The arguments are 64 bytes; with four more, for `whole`, a pass over a 1024 x 1024 layer, this launch and one other, took
// 8.05 us in place of 7.47.)
template <int K, int V, int CODE, int S, int NW, bool FUSED, bool SPREAD = false, bool WIDE = false, int TAIL = 0,
          bool ROUNDS = false>
__global__ __launch_bounds__(NW * 64, (CODE == CODE_HYB1 || FUSED) ? 4 : 8) void matvec_kernel(const uint32_t *__restrict__ codes,
                                                         const uint32_t *__restrict__ lut,
                                                         int tm, int tn, const half_t *__restrict__ x,
                                                         const int8_t *__restrict__ signs, int log2_block,
                                                         const half_t *__restrict__ scale,
                                                         float *__restrict__ y) {
    __shared__ __attribute__((aligned(16))) uint32_t s_lut[code_lds_words(CODE, SPREAD)];
    __shared__ float s_part[ROUNDS ? 2 * NW : NW][16];
    __shared__ __attribute__((aligned(16))) half_t s_x[FUSED ? FUSED_MAX_N : 8];
    __shared__ __attribute__((aligned(16))) float s_v[FUSED ? RHT_LDS_FLOATS : 1];
    // Workgroups go round the eight XCDs; those of one tile row, which read the same cache lines, stay on one.
    const int b = blockIdx.x, whole = TAIL ? tm / CUS * CUS : tm;
    auto tail_part = [&](int t, bool staged) {
        if constexpr (TAIL > 0) {
            const int I = whole + (t >> 3) / TAIL * 8 + (t & 7);
            if (I >= tm) return;
            if (staged) __syncthreads();
            matvec_tile_row<K, V, CODE, TAIL, NW, FUSED, SPREAD, K != 2>(I, I + 1, (t >> 3) % TAIL, staged, codes, lut, tn, x, signs,
                                                                         log2_block, scale, y, s_lut, s_part, s_x, s_v);
        }
    };
    if constexpr (ROUNDS) {
        if (b >= whole) return;  // (the grid has no more)
        matvec_tile_row<K, V, CODE, 1, NW, FUSED, SPREAD, WIDE, true>(b, whole, 0, false, codes, lut, tn, x, signs, log2_block, scale,
                                                                      y, s_lut, s_part, s_x, s_v);
        if constexpr (TAIL > 0) {
            for (int t = b; t < (tm - whole + 7) / 8 * 8 * TAIL; t += gridDim.x) tail_part(t, true);
        }
        return;
    }
    if constexpr (TAIL > 0) {
        if (b >= whole) return tail_part(b - whole, false);
    }
    const int I = S == 1 ? b : (b >> 3) / S * 8 + (b & 7);
    const int part = S == 1 ? 0 : (b >> 3) % S;
    if (S > 1 && I >= tm) return;
    matvec_tile_row<K, V, CODE, S, NW, FUSED, SPREAD, WIDE>(I, I + 1, part, false, codes, lut, tn, x, signs, log2_block, scale, y, s_lut,
                                                            s_part, s_x, s_v);
}

// ------------------------------------------- decode + batched product on MFMA
//
// v_mfma_f32_16x16x32_f16, D = A * B, with the decoded weights as A and the
// activations as B.  A wave step covers four tiles (I, J0..J0+3) of one tile row:
//   lane l = (row i = l % 16, slot s = l / 16) decodes the whole tile row i of tile
//   J0 + s: 16 weights = 8 packed registers, the A operands of two MFMAs (columns
//   0..7 and 8..15 of the tile);
//   the matching B operand of lane (j = l % 16, s) is X[b0 + j][16 (J0+s) + 8h .. +7],
//   one 16-byte load; A and B pair contraction slots by (s, element), so the order
//   in which the hardware numbers them does not matter;
//   D[4 (l / 16) + r][l % 16] = output row 16 I + 4 (l/16) + r for batch row b0 + l % 16.
// A wave owns R tile rows, two where there are enough, so that every B operand it loads
// feeds two MFMAs; NB groups of 16 batch rows share every decoded weight.  The waves of
// a workgroup split the tiles of the row band and meet in LDS.
// The B operand puts neighbouring lanes on different batch rows, that is on different
// cache lines, for each of which the texture units' address half takes cycles of its own.  With
// few distinct batch rows that rarely matters; otherwise (STAGE) a wave loads its
// activations line by line (8 lanes = the 128 bytes that one batch row has under the
// four tiles of a step) and transposes them through a private piece of LDS.

// The words that hold tile row i (16 K bits from bit 16 K i) and the 16 - K V bits after it, brought to bit offset 0;
// words behind a row's own wrap inside the tile (tail-biting).  At k = 2 and 4 a row is one or two whole words and
// the word behind it is the first one of the next row, which the next lane of a row of 16 lanes has: one load per row.
// (NEXT: where lane i has tile row i; else the word behind is a load of its own.)
template <int K, bool NEXT> struct RowWords {
    static constexpr int NWORDS = 8 * K;
    int row;
    uint32_t first, behind;  // byte offsets in a tile: of the row's words, of the word behind them
    __device__ __forceinline__ explicit RowWords(int row)
        : row(row), first(4 * (K * row / 2)), behind(4 * ((K * row / 2 + (K == 2 ? 1 : 2)) % NWORDS)) {}
    // from the tile `offset` bytes behind `base`, which all lanes share
    __device__ __forceinline__ void load(const uint32_t *__restrict__ base, uint32_t offset, uint32_t (&w)[3]) const {
        auto at = [&](uint32_t o) { return reinterpret_cast<const char *>(base) + (offset + o); };
        if constexpr (K == 2) {
            w[0] = stream_load(reinterpret_cast<const uint32_t *>(at(first)));
        } else {  // (at k = 3 on four bytes)
            typedef uint32_t two_words __attribute__((ext_vector_type(2), aligned(4)));
            const u32x2_t t = __builtin_nontemporal_load(reinterpret_cast<const two_words *>(at(first)));
            w[0] = t.x;
            w[1] = t.y;
        }
        if constexpr (K == 3 || !NEXT) w[K == 2 ? 1 : 2] = stream_load(reinterpret_cast<const uint32_t *>(at(behind)));
    }
    // (every lane of the wave makes the call)
    __device__ __forceinline__ void align(uint32_t (&w)[3]) const {
        if constexpr (K == 3) {
            if (row & 1) {  // odd rows start in the middle of a word
                w[0] = __builtin_amdgcn_alignbit(w[0], w[1], 16);
                w[1] = __builtin_amdgcn_alignbit(w[1], w[2], 16);
                w[2] <<= 16;
            }
        } else if constexpr (NEXT) {
            w[K / 2] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[0], 0x12F, 0xF, 0xF, false);  // row rotate by 15
        }
    }
};

// SPREAD: the HYB table in 16 copies, as in the batch-1 kernel (64 KiB: only next to the
// small partial-sum buffer of NB = 1).
//
// S = 2 (R = 1): the 16 rows of a tile row go to two workgroups, each of which still fills the A operand: lane row i is row
// i % 8 of the workgroup's own in one of twice as many tiles, J0 + 4 u + s with u = i / 8.  The B operand belongs to the tile,
// so there is one per u and twice as many MFMAs, of which each makes 8 rows of D that count; the decoding is no more than
// the rows'.  At the end a lane takes the rows it has from the u they belong to, and the two lanes with the same rows add up.
// (Four workgroups of four rows each, us, 8 batch rows, 2-bit 3INST: 1024 x 14336 8.9, two 8.4; whole 11.7.)
template <int K, int V, int CODE, int R, int NB, int NW, int SR, bool SPREAD = false, int S = 1>
__global__ __launch_bounds__(NW * 64) void matmat_kernel(const uint32_t *__restrict__ codes,
                                                         const uint32_t *__restrict__ lut,
                                                         int tm, int tn, const half_t *__restrict__ X,
                                                         int B, const half_t *__restrict__ scale,
                                                         float *__restrict__ Y) {
    constexpr int NWORDS = 8 * K;
    __shared__ __attribute__((aligned(16))) uint32_t s_lut[code_lds_words(CODE, SPREAD)];
    // one buffer, used twice: in the loop each wave's staging region (SR batch rows at a
    // time, 128 bytes each, padded to 144 so that the row-wise writes and the
    // column-wise reads both spread over the banks), after it the partial sums
    constexpr bool STAGE = SR > 0;
    constexpr int NH = NB == 1 ? 1 : 16 * NB / SR, XST = 144;  // staging rounds; bytes of a staged row
    constexpr int LOADS = !STAGE ? NB : NB == 1 ? SR / 8 : 2 * NB, NX = STAGE ? LOADS : 2 * NB;  // rows, pieces of X per lane
    constexpr int ROWS = 16 / S, TILES = 4 * S;  // rows of a workgroup's tile row, tiles of a wave's step
    static_assert(S == 1 || (S == 2 && R == 1), "halves of one tile row");
    constexpr int PART_FLOATS = NW * R * NB * 256;
    constexpr int STAGE_FLOATS = STAGE ? NW * SR * XST / 4 : 0;
    __shared__ __attribute__((aligned(16))) float s_buf[PART_FLOATS > STAGE_FLOATS ? PART_FLOATS : STAGE_FLOATS];
    float(*s_part)[R * NB * 4][64] = reinterpret_cast<float(*)[R * NB * 4][64]>(s_buf);
    // (workgroups go round the eight XCDs: those of one tile row, which read the same cache lines, stay on one)
    const int local = blockIdx.x >> 3;
    const int I0 = S == 1 ? blockIdx.x * R : local / S * 8 + (blockIdx.x & 7);
    if (S > 1 && I0 >= tm) return;
    const int b0 = blockIdx.y * (16 * NB);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = lane & 15, s = lane >> 4;
    const int row = S == 1 ? i : local % S * ROWS + i % ROWS, sub = 4 * (i / ROWS) + s;  // the lane's row, tile of a step
    const size_t n = (size_t)tn * 16;
    const int m = tm * 16;
    const int chunk = ((tn + NW * TILES - 1) / (NW * TILES)) * TILES;
    const int J0 = wave * chunk;
    const int tiles = max(min(tn, J0 + chunk) - J0, 0), steps = (tiles + TILES - 1) / TILES;

    // Addresses: a wave's step moves uniform bases (codes) and adds one uniform number per row of X; all that is the lane's is
    // made here.  Only the last step of a slice that is no whole number of them looks where its tiles end.
    const uint32_t *row_codes[R];
#pragma unroll
    for (int r = 0; r < R; r++) row_codes[r] = codes + ((size_t)min(I0 + r, tm - 1) * tn + J0) * NWORDS;
    const RowWords<K, S == 1> words(row);
    const int lr = lane >> 3, ch = lane & 7;  // STAGE: the lane loads piece ch of batch rows 8 q + lr
    const half_t *xrow[LOADS];
#pragma unroll
    for (int q = 0; q < LOADS; q++) {
        const int b = b0 + (STAGE ? 8 * q + lr : 16 * q + i);
        xrow[q] = X + (size_t)min(b, B - 1) * n + 16 * J0 + (STAGE ? 8 * ch : 16 * s);
    }
    char *const stage = reinterpret_cast<char *>(s_buf) + wave * (SR * XST);

    float4_t acc[R * S][NB];
#pragma unroll
    for (int r = 0; r < R * S; r++)
#pragma unroll
        for (int nb = 0; nb < NB; nb++) acc[r][nb] = float4_t{0.f, 0.f, 0.f, 0.f};

    // software pipeline: operands of step t + 1 are loaded while step t runs (code words two or three steps ahead: 8192 x
    // 8192 4-bit HYB, 8 rows, 10.7 us -> 12.1 and 12.9)
    struct Operands {
        uint32_t w[R][3];
        half8_t x[S][NX];
    };
    auto load = [&](Operands &o, int t, auto partial) {
        // (slots past the end re-read the last tile)
        const int last = tiles - 1 - t * TILES;
        const uint32_t back = partial ? (uint32_t)max(sub - last, 0) * (4 * NWORDS) : 0;
#pragma unroll
        for (int r = 0; r < R; r++)
            words.load(row_codes[r] + (size_t)t * (TILES * NWORDS), (uint32_t)sub * (4 * NWORDS) - back, o.w[r]);
#pragma unroll
        for (int u = 0; u < S; u++) {
            const int xback = partial ? max(4 * u + (STAGE ? ch >> 1 : s) - last, 0) : 0;
#pragma unroll
            for (int q = 0; q < LOADS; q++) {
                const half8_t *const x =
                    reinterpret_cast<const half8_t *>(xrow[q] + (size_t)t * (16 * TILES) + 64 * u - (partial ? 16 * xback : 0));
                if constexpr (STAGE) {
                    o.x[u][q] = x[0];
                } else {
                    o.x[u][2 * q] = x[0];
                    o.x[u][2 * q + 1] = x[1];
                }
            }
        }
    };
    auto issue = [&](Operands &o, int t) {
        if ((t + 1) * TILES <= tiles) load(o, t, std::false_type{});
        else load(o, t, std::true_type{});
    };
    RowDecode<K, CODE, SPREAD> rdec;
    auto compute = [&](Operands &o, int t) {
        half8_t xb[S][NB][2];
#pragma unroll
        for (int u = 0; u < S; u++) {
            if constexpr (STAGE) {
                // The lanes of the wave exchange data through LDS without a workgroup barrier:
                // the LDS operations of one wave complete in order, and the fences keep the
                // compiler from moving them across each other.
#pragma unroll
                for (int hf = 0; hf < NH; hf++) {
#pragma unroll
                    for (int qq = 0; qq < SR / 8; qq++)
                        *reinterpret_cast<half8_t *>(stage + (8 * qq + lr) * XST + 16 * ch) = o.x[u][hf * (SR / 8) + qq];
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
                    for (int nbb = 0; nbb < (SR + 15) / 16; nbb++)
#pragma unroll
                        for (int h = 0; h < 2; h++)
                            xb[u][hf * (SR / 16) + nbb][h] = *reinterpret_cast<const half8_t *>(
                                stage + (SR == 8 ? i & 7 : 16 * nbb + i) * XST + 16 * (2 * s + h));
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                }
            } else {
#pragma unroll
                for (int nb = 0; nb < NB; nb++)
#pragma unroll
                    for (int h = 0; h < 2; h++) xb[u][nb][h] = o.x[u][2 * nb + h];
            }
        }
        // (a batch row past the end is another column of D, which nobody takes: only dead slots are cleared)
        if ((t + 1) * TILES > tiles) {
            asm volatile("");  // (a branch, or every step would have the selects)
#pragma unroll
            for (int u = 0; u < S; u++)
#pragma unroll
                for (int nb = 0; nb < NB; nb++)
#pragma unroll
                    for (int h = 0; h < 2; h++)
                        if (t * TILES + 4 * u + s >= tiles) xb[u][nb][h] = half8_t{0, 0, 0, 0, 0, 0, 0, 0};
        }
#pragma unroll
        for (int r = 0; r < R; r++) {
            words.align(o.w[r]);
            uint32_t hrow[8];
            rdec.run(o.w[r], 0, hrow);
#pragma unroll
            for (int h = 0; h < 2; h++) {
                typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                const half8_t a = __builtin_bit_cast(
                    half8_t, u32x4{hrow[4 * h], hrow[4 * h + 1], hrow[4 * h + 2], hrow[4 * h + 3]});
#pragma unroll
                for (int u = 0; u < S; u++)
#pragma unroll
                    for (int nb = 0; nb < NB; nb++)
                        acc[r * S + u][nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, xb[u][nb][h], acc[r * S + u][nb], 0, 0, 0);
            }
        }
    };
    stage_code_table<CODE, SPREAD>(lut, s_lut, NW * 64);
    rdec.init(s_lut);
    // (one copy of the loop's body: with two, for alternating operand sets without moves, or with the first operands asked for
    // ahead of the table, small products take 0.2 to 0.5 us longer)
    Operands now, next;
    if (steps > 0) issue(next, 0);
    for (int t = 0; t < steps; t++) {
        now = next;
        if (t + 1 < steps) issue(next, t + 1);
        compute(now, t);
    }

    // (S = 2: D rows 4 s + e are rows (4 s + e) % 8 of the workgroup's, of sub-step u = s / 2)
    const int sum_row = S == 1 ? 4 * s : (local % S) * ROWS + 4 * (s & 1);
    if constexpr (S > 1) {
#pragma unroll
        for (int nb = 0; nb < NB; nb++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const float v = s < 2 ? acc[0][nb][e] : acc[S - 1][nb][e];
                acc[0][nb][e] = v + __shfl_xor(v, 32, 64);
            }
    }
    if constexpr (STAGE) __syncthreads();  // the staging regions become the partial sums
#pragma unroll
    for (int r = 0; r < R; r++)
#pragma unroll
        for (int nb = 0; nb < NB; nb++)
#pragma unroll
            for (int e = 0; e < 4; e++) s_part[wave][(r * NB + nb) * 4 + e][lane] = acc[S == 1 ? r : 0][nb][e];
    __syncthreads();
    // (the waves share the sums: one wave with all of them took 0.3 us longer at R = 2)
    for (int part = wave; part < R * NB * 4; part += NW) {
        float v = 0.f;
#pragma unroll
        for (int wv = 0; wv < NW; wv++) v += s_part[wv][part][lane];
        const int I = I0 + part / (4 * NB), b = b0 + 16 * (part / 4 % NB) + i, orow = 16 * I + sum_row + part % 4;
        if (I < tm && b < B && s < 4 / S) Y[(size_t)b * m + orow] = scale ? v * (float)scale[orow] : v;
    }
}

// ------------------------------------------------------------------ launchers

template <int K, int V, int CODE>
static hipError_t launch_dequantize_t(const uint32_t *codes, const uint32_t *lut, int m, int n,
                                      void *W, hipStream_t st) {
    const long ntiles = (long)(m / 16) * (n / 16);
    constexpr int TPW = 64 / Geo<K>::LPT;
    const long waves = (ntiles + TPW - 1) / TPW;
    const long blocks = (waves + 3) / 4;
    hipLaunchKernelGGL((dequantize_kernel<K, V, CODE>), dim3((unsigned)blocks), dim3(256), 0, st,
                       codes, lut, n / 16, ntiles, (half_t *)W);
    return hipGetLastError();
}

// Waves per workgroup for the batch-1 kernel.  A workgroup owns one tile row, so the
// grid has m/16 workgroups and NW decides both how many waves the chip gets and how
// many steps each wave runs: few steps leave a wave's start-up and reduction exposed,
// few waves leave SIMDs idle or the vector ALU short of waves to interleave.
// Measured by kernel durations from the profiler's trace (for kernels this short a loop
// of launches from the host times the host): as many waves as there are steps, up to 16,
// is best everywhere: 4096 x 4096 (16 steps) 6.0 us with 8 waves, 5.4 with 16; 14336 x 4096
// 11.6 -> 11.3.  The kernel that transforms its own input takes the same count, so that it
// adds its partial sums in the same order and gives the same bits as the two separate calls.
static int pick_matvec_waves(int steps_per_row) {
    if (steps_per_row >= 16) return 16;
    if (steps_per_row >= 8) return 8;
    if (steps_per_row >= 4) return 4;
    return 2;
}

// The 16-copy HYB table: from which row length on it pays for the 64 KiB each workgroup fills
// (measured: 8192 x 28672 29.9 -> 22.5 us at k = 2, 8192 x 8192 10.0 -> 9.6, 14336 x 4096 10.0 ->
// 12.0).  The two-sign-flip form is bound by its vector instructions and gains nothing.
static bool pick_hyb_spread(int code, int n) {
    return code == CODE_HYB && n >= 8192;
}

// Workgroups per tile row: the share of a CU, workgroups of about 0.8 us each and the time of their rows (0.5 us per
// 1000 inputs of a whole tile row), is smallest; a split leaves at least two steps.  (2-bit 3INST: 1280 x 26624
// 18.1 -> 12.1 us, 2048 x 8192 6.6 -> 4.4, 1024 x 4096 4.1 -> 3.0, with its transform 5.7 -> 4.7.  Matrices of 4096 rows
// and more gain nothing: a whole tile row per CU fills its issue slots.  The choice depends on the sizes alone, so
// that the kernel that transforms its own input makes the same one.)
// With more tile rows than CUs the ones behind the last whole round may be split alone, by the same measure, if the row is
// long enough for 16 waves (us, all rows whole and so, codes from memory: 1MAD k = 3 14336 x 4096 11.6 11.4, 6144 x 4096 6.7
// 6.0, 5120 x 8192 10.8 8.7, 2-bit 3INST 9216 x 4096 8.4 7.6, 4-bit HYB 10240 x 8192 21.6 16.5, HYB2 5120 x 28672 k = 2 25.5 21.0,
// k = 4 50.7 28.2) and their parts are one workgroup per CU at most.  More of them are slower than whole rows, of which a CU has two at a time (4-bit HYB,
// 14336 inputs, whole and split: 416 tile rows 13.3 23.1, 448 13.5 24.5, 704 19.9 29.6; 3-bit 1MAD 448 18.3 22.1), but for the
// 2-bit computed codes behind one round (1MAD, 416 rows: 17.7 16.5).  And where all rows in two halves were chosen before, halves
// stay for two kinds of product: the V = 1 hash code's with short rows, whose halves have 8 waves and so go two to a CU (us,
// last rows in parts and all in halves: k = 2 6144 x 4608 9.13 7.52, 6144 x 4096 7.20 6.55, 10240 x 7168 15.8 14.8, but with quarters
// 4128 x 6144 8.33 8.80; k = 3 5632 x 5120 10.76 10.04, but 6144 inputs 11.1 11.8; k = 4 5632 x 4608 9.71 9.15), and the 2-bit
// computed codes' behind one round (1MAD 6144 x 4096 5.49 5.19, 5120 inputs 6.98 7.30; 3INST 5.58 5.36, 6144 inputs 7.51 8.37, 14336
// 14.7 14.0, 28672 25.6 26.8).
// Over 15 codecs, 24 heights and 11 lengths, each split forced in turn, the pick takes 0.5 % more than the fastest, 20 % at
// worst (HYB1 k = 2, 13824 x 4608 in rounds, where halves are faster).
struct MatvecSplit {
    int s, whole, tail;  // rows from `whole`, the multiple of CUS, on: `tail` workgroups each
};
static MatvecSplit pick_matvec_split(int k, int code, int tm, int tn) {
    auto time = [&](int rows, int s) { return (float)((rows * (long)s + CUS - 1) / CUS) * (0.8f + (float)tn * (0.008f / (float)s)); };
    const int whole = tm / CUS * CUS, rest = tm - whole;
    const bool one_round_of_two_bits = k == 2 && (code == CODE_3INST || code == CODE_1MAD) && whole == CUS;
    // (of all rows, than parts of the last ones)
    auto halves_are_faster = [&](int s) {
        if (code == CODE_HYB1) return k == 2 ? tn < 384 || (tn < 512 && s == 2) : whole == CUS && tn <= 320;
        return one_round_of_two_bits && s == 2 && (tn < 320 || (code == CODE_3INST && tn >= 768 && tn < 1280));
    };
    MatvecSplit best{1, tm, 0};
    float least = time(tm, 1);
    for (int s = 2; s <= 4 && tn >= 2 * 16 * s; s *= 2) {
        if (time(tm, s) < least) best = {s, tm, 0}, least = time(tm, s);
        if (whole == 0 || rest == 0 || tn < 256) continue;
        if (rest * s > CUS && !(one_round_of_two_bits && rest > CUS / 2)) continue;
        if (best.s == 2 && halves_are_faster(s)) continue;
        const float t = time(whole, 1) + time(rest, s);
        if (t < least) best = {1, whole, s}, least = t;
    }
    return best;
}

template <int K, int V, int CODE>
static hipError_t launch_matvec_t(const uint32_t *codes, const uint32_t *lut, int m, int n,
                                  const void *x, const int8_t *signs, int log2_block, const void *scale,
                                  float *y, hipStream_t st) {
    constexpr int TPI = 64 / Geo<K>::LPT;
    const int tm = m / 16, tn = n / 16;
    const int steps = (tn + TPI - 1) / TPI;
    const int nw = pick_matvec_waves(steps);
    const bool spread = pick_hyb_spread(CODE, n);
    const MatvecSplit pick = pick_matvec_split(K, CODE, tm, tn);
    const int split = pick.s, tails = pick.tail ? (tm - pick.whole + 7) / 8 * 8 * pick.tail : 0;
    const bool rounds = CODE == CODE_HYB1 && split == 1 && tm > CUS && nw == 16;
    // (in rounds every workgroup begins with a whole row)
    const dim3 grid(split > 1 ? (tm + 7) / 8 * 8 * split : rounds ? std::min(CUS, pick.whole) : pick.whole + tails);
    // signs != null: x is untransformed and the kernel transforms it itself (n <= FUSED_MAX_N)
#define QTIP_MV_LAUNCH6(S, NW, FUSED, SPREAD, WIDE, TAIL, ROUNDS)                                                           \
    hipLaunchKernelGGL((matvec_kernel<K, V, CODE, S, NW, FUSED, SPREAD, WIDE, TAIL, ROUNDS>), grid, dim3(NW * 64), 0, st, codes, \
                       lut, tm, tn, (const half_t *)x, signs, log2_block, (const half_t *)scale, y)
#define QTIP_MV_LAUNCH4(S, NW, FUSED, SPREAD, WIDE) QTIP_MV_LAUNCH6(S, NW, FUSED, SPREAD, WIDE, 0, false)
// (more rows than one per CU, and so more than launch_rht_matvec takes: never with the transform)
#define QTIP_MV_LAUNCH_MANY(TAIL, WIDE)                                    \
    if (code_is_hyb(CODE) && spread)                                       \
        QTIP_MV_LAUNCH6(1, 16, false, code_is_hyb(CODE), WIDE, TAIL, false); \
    else                                                                   \
        QTIP_MV_LAUNCH6(1, 16, false, false, WIDE, TAIL, CODE == CODE_HYB1)
#define QTIP_MV_LAUNCH_WHOLE(WIDE)                    \
    if (pick.tail == 2) {                             \
        QTIP_MV_LAUNCH_MANY(2, WIDE);                 \
    } else if (pick.tail == 4) {                      \
        QTIP_MV_LAUNCH_MANY(4, WIDE);                 \
    } else if (rounds) {                              \
        if constexpr (CODE == CODE_HYB1) {            \
            QTIP_MV_LAUNCH_MANY(0, WIDE);             \
        }                                             \
    } else {                                          \
        QTIP_MV_LAUNCH(1, 16, WIDE);                  \
    }
#define QTIP_MV_LAUNCH(S, NW, WIDE)                                \
    if (signs)                                                     \
        QTIP_MV_LAUNCH4(S, NW, true, false, WIDE);                 \
    else if (code_is_hyb(CODE) && spread)                          \
        QTIP_MV_LAUNCH4(S, NW, false, code_is_hyb(CODE), WIDE);    \
    else                                                           \
        QTIP_MV_LAUNCH4(S, NW, false, false, WIDE)
    // (a lane has four tile rows of a tile at every k where a tile row is split)
    if (split > 1) {
        const int ssteps = (tn + 16 * split - 1) / (16 * split);
        constexpr bool WIDE = K != 2;
        if (split == 2) {
            if (ssteps >= 16) QTIP_MV_LAUNCH(2, 16, WIDE);
            else QTIP_MV_LAUNCH(2, 8, WIDE);
        } else {
            if (ssteps >= 16) QTIP_MV_LAUNCH(4, 16, WIDE);
            else QTIP_MV_LAUNCH(4, 8, WIDE);
        }
        return hipGetLastError();
    }
    // Four rows per lane at k = 3 and 4 (MvGeo<K, true>: steps of 16 tiles) where 16 waves still have a
    // step each and the row splits into such steps as evenly as into the narrow ones (measured, k = 4:
    // 14336 x 4096 12.44 -> 11.38 us, 8192 x 8192 HYB 10.64 -> 10.38; 4096 x 14336, 896 tiles = 3.5 wide
    // steps per wave, 11.76 -> 12.10 us, so it keeps the narrow form).  The choice depends on the row
    // length alone, so the kernel that transforms its own input makes the same one.
    if constexpr (K != 2) {
        constexpr int WTPI = 64 / MvGeo<K, true>::LPT;
        const int wsteps = (tn + WTPI - 1) / WTPI;
        if (wsteps >= 16 && 2 * ((wsteps + 15) / 16) <= (steps + nw - 1) / nw) {
            QTIP_MV_LAUNCH_WHOLE(true);
            return hipGetLastError();
        }
    }
    switch (nw) {
        case 2: QTIP_MV_LAUNCH(1, 2, false); break;
        case 4: QTIP_MV_LAUNCH(1, 4, false); break;
        case 16: QTIP_MV_LAUNCH_WHOLE(false); break;
        default: QTIP_MV_LAUNCH(1, 8, false); break;
    }
#undef QTIP_MV_LAUNCH
#undef QTIP_MV_LAUNCH_WHOLE
#undef QTIP_MV_LAUNCH_MANY
#undef QTIP_MV_LAUNCH4
#undef QTIP_MV_LAUNCH6
    return hipGetLastError();
}

template <int K, int V, int CODE>
static hipError_t launch_matmat_t(const uint32_t *codes, const uint32_t *lut, int m, int n,
                                  const void *X, int B, const void *scale, float *Y,
                                  hipStream_t st) {
    const int groups = (B + 15) / 16;  // more than one only where matmat_takes them or the large-batch kernel does not reach
    const int tm = m / 16, tn = n / 16;
    const half_t *Xh = (const half_t *)X, *sc = (const half_t *)scale;
    // Few outputs, where 16 batch rows at a time are more than one workgroup per CU and 32 are not.
    if (groups > 1 && n <= 1 << 22 && (long)tm * groups > CUS && (long)tm * ((groups + 1) / 2) <= CUS) {
        hipLaunchKernelGGL((matmat_kernel<K, V, CODE, 1, 2, 16, 32>), dim3(tm, (groups + 1) / 2), dim3(16 * 64), 0, st, codes, lut,
                           tm, tn, Xh, B, sc, Y);
        return hipGetLastError();
    }
    // Many outputs, 17 to 32 batch rows; and rows of more than 2^22 inputs: there a workgroup decodes a weight for 16 batch rows
    // while that makes at most two workgroups per CU, and for 32 or 64 otherwise (2^22 inputs, 2-bit 3INST, ms for 16 and for 32
    // or 64: 1024 outputs 64 rows 3.8 and 8.7, 128 rows 7.2 and 8.8, 200 rows 13.4 and 8.9; 4096 outputs 24 rows 6.8 and 6.8, 48
    // rows 10.0 and 8.7, 200 rows 39.8 and 21.7).
    if (groups > 1 && (long)tm * groups > 512) {
        if (groups == 2)
            hipLaunchKernelGGL((matmat_kernel<K, V, CODE, 2, 2, 8, 32>), dim3((tm + 1) / 2), dim3(8 * 64), 0, st, codes,
                               lut, tm, tn, Xh, B, sc, Y);
        else
            hipLaunchKernelGGL((matmat_kernel<K, V, CODE, 2, 4, 8, 32>), dim3((tm + 1) / 2, (groups + 3) / 4),
                               dim3(8 * 64), 0, st, codes, lut, tm, tn, Xh, B, sc, Y);
        return hipGetLastError();
    }
    // 16 batch rows.  Two tile rows per workgroup (R = 2) share what is loaded of X; a tile row by itself is for at most one
    // per CU, and half of one for at most half of that.  With 16 waves (NW) a workgroup has a CU's issue slots to itself, with 8
    // several share them.  Up to 8 rows a wave loads its activations as operands, in a half's kernel, which has twice as many,
    // and beyond that through LDS (SR).
    // Of those below, each forced in turn for ten codecs, 768 to 28672 outputs, 1024 to 28672 inputs and 2, 8, 9 and 16 rows, the
    // pick takes 1.0 % more than the fastest, 23 % at worst (a quarter of a tile row each, which is not kept: 768 x 28672).  us,
    // 8 rows, 2-bit 3INST: 1024 x 14336 whole 11.7, halves 8.4; 14336 x 4096 and 14336 x 1024 with 16 waves 11.2 and 5.03, with 8
    // 11.8 and 5.01; 10240 x 8192 (2.5 tile rows per CU) with single rows 16.5, with pairs 20.
    constexpr bool HYB = CODE == CODE_HYB, HASH = code_is_hyb(CODE);
    const bool big = B > 8;
    if (groups == 1 ? tm <= (HASH && K == 4 && big ? CUS / 4 : CUS / 2) && tn >= (HASH ? 256 : 64)
                    : n <= 1 << 22 && (long)tm * groups <= CUS / 2 && tn >= (HASH ? 256 : 64)) {
        // (at 4 bits table reads, not the decoding, take the time, and beyond 8 rows what is loaded of X: 2048 x 8192, 16 rows,
        // 9.1 us whole, 9.6 in halves)
        const dim3 grid((tm + 7) / 8 * 8 * 2, groups);
#define QTIP_MM_HALF(NW, SR) \
    hipLaunchKernelGGL((matmat_kernel<K, V, CODE, 1, 1, NW, SR, false, 2>), grid, dim3(NW * 64), 0, st, codes, lut, tm, tn, Xh, B, sc, Y)
        if (tn > 64) {
            if (big) QTIP_MM_HALF(16, 16);
            else QTIP_MM_HALF(16, 8);
        } else {
            if (big) QTIP_MM_HALF(8, 16);
            else QTIP_MM_HALF(8, 8);
        }
#undef QTIP_MM_HALF
        return hipGetLastError();
    }
    // The 16 copies of the HYB table: a step's 16 reads of one copy take the LDS 112 cycles, of 16 copies about 70, and filling
    // them 0.5 us (us, one copy and 16: 8 rows k = 2 8192 x 14336 16.2 13.3, 8192 x 4096 7.0 6.5, 8192 x 1024 4.1 4.5; 16 rows k = 2 4096 x
    // 28672 24.9 20.9).  At 3 and 4 bits it pays with the activations through LDS: the address half of the texture units, busy for
    // 58 400 of 80 000 cycles otherwise, then has 40 000 of 59 100 (k = 3 14336 x 14336, 8 rows; us, one copy, 16, 16 and so:
    // k = 3 8192 x 8192 12.3 12.9 11.1, 14336 x 14336 34.0 34.8 29.2, k = 4 14336 x 14336 27.2 26.7 25.3, 8192 x 28672 29.7 26.9
    // 26.2, but k = 2 14336 x 14336 26.7 21.9 25.8).
    const bool long_row = K == 2 ? n >= 4096 : K == 3 ? n >= (tm <= 2 * CUS ? 4096 : 8192) : n >= (tm <= 2 * CUS ? 12288 : 8192);
    const bool spread = HYB && (big ? n >= 8192 : tm > CUS && long_row);
#define QTIP_MM(R, NW, SR, SPREAD)                                                                              \
    hipLaunchKernelGGL((matmat_kernel<K, V, CODE, R, 1, NW, SR, SPREAD>), dim3((tm + R - 1) / R, groups),      \
                       dim3(NW * 64), 0, st, codes, lut, tm, tn, Xh, B, sc, Y)
    // (COPIES: where 16 copies can be picked: nowhere, beyond 8 batch rows alone, everywhere)
#define QTIP_MM_BATCH(R, NW, COPIES)                       \
    do {                                                   \
        if constexpr (HYB && COPIES > 0) {                 \
            if (big && spread) {                           \
                QTIP_MM(R, NW, 16, true);                  \
                break;                                     \
            }                                              \
        }                                                  \
        if constexpr (HYB && COPIES > 1) {                 \
            if (spread) {                                  \
                QTIP_MM(R, NW, (K == 2 ? 0 : 8), true);    \
                break;                                     \
            }                                              \
        }                                                  \
        if (big) QTIP_MM(R, NW, 16, false);                \
        else QTIP_MM(R, NW, 0, false);                     \
    } while (0)
    // Single rows at row counts between the rounds of pairs (beyond four rounds for the V = 1 hash code alone: single rows and
    // pairs, us, k = 3 28672 x 4096, 2 rows, 25.4 28.4; 3-bit 3INST 20480 x 14336, 8 rows, 64.5 54.9), but not where the table reads
    // of long rows count for more than an idle CU: HYB2 k = 4 12288 x 14336, 8 rows, 33.7 30.6; k = 3, 16 rows, 38.9 41.6.  With
    // 16 waves at 3 bits and up to 8 rows, where code words are two loads a lane (8 waves and 16: 3INST 10240 x 14336 42.5 37.7,
    // 1MAD 12288 x 28672 81.4 75.2; V = 1 hash code 12288 x 8192 28.5 27.4, but 4096 inputs 13.4 15.2).
    // And not for nearly 16 batch rows of 64 inputs in two cache lines each, where pairs read half of those: time over that of single
    // rows, more than 12 rows of inputs that are not whole lines, 2 bits, code words from memory: 3INST, HYB and HYB2 2048 to 8192
    // inputs 0.94, 3INST beyond 0.96, V = 1 hash code beyond 16384 0.86; 1MAD 1.12, whatever the code below 2048 inputs 1.06.
    const bool two_lines = K == 2 && B > 12 && n % 64 != 0 && n >= (CODE == CODE_HYB1 ? 16384 : 2048) && CODE != CODE_1MAD;
    const bool between = (tm <= 4 * CUS || (CODE == CODE_HYB1 && n >= 2048)) && !spread && !two_lines && !(HASH && n >= 8192 && !(K == 3 && big)) &&
                         (tm + 255) / 256 < 2 * (((tm + 1) / 2 + 255) / 256);
    const bool between_16 = between && K == 3 && !big && tm <= 4 * CUS && n >= (CODE == CODE_HYB1 ? 8192 : 4096);
    // Eight waves for more than two tile rows per CU where a row is short, and where code values and batch rows leave too few
    // registers for two workgroups of 16 (16 waves and 8, us: V = 1 hash code k = 3 14336 x 4096, 8 rows, 18.6 16.9; 16 rows, 2-bit 3INST
    // 16400 x 14336 54.2 48.7, HYB2 k = 3 14336 x 8192 27.0 25.3; but 8 rows, 2-bit 1MAD 14336 x 14336 36.8 39.1).  Over 15 codecs, 4112 to
    // 28672 outputs, 1024 to 28672 inputs and 2, 8, 9 and 16 rows, each of the four forced in turn, 1.6 % above the fastest.
    const bool few_waves = (!big && (spread || (HYB && K == 4))) ||
                           (!spread && (tn < (tm > 4 * CUS ? 768 : big ? 512 : 256) || (K == 3 && (big || !HASH)) ||
                                        (!HASH && (big || (CODE == CODE_3INST && K == 4)))));
    if (tm <= CUS || between_16) {
        QTIP_MM_BATCH(1, 16, 1);
    } else if (between) {
        QTIP_MM_BATCH(1, 8, 0);
    } else if (tm <= 2 * CUS || !few_waves) {
        QTIP_MM_BATCH(2, 16, 2);
    } else {
        QTIP_MM_BATCH(2, 8, 2);
    }
#undef QTIP_MM_BATCH
#undef QTIP_MM
    return hipGetLastError();
}

#define QTIP_DISPATCH(FN, ...)                                                         \
    do {                                                                               \
        if (code_id == CODE_HYB1) {                                                    \
            if (k == 2) return FN<2, 1, CODE_HYB1>(__VA_ARGS__);                       \
            if (k == 3) return FN<3, 1, CODE_HYB1>(__VA_ARGS__);                       \
            return FN<4, 1, CODE_HYB1>(__VA_ARGS__);                                   \
        } else if (code_id == CODE_HYB2) {                                             \
            if (k == 2) return FN<2, 2, CODE_HYB2>(__VA_ARGS__);                       \
            if (k == 3) return FN<3, 2, CODE_HYB2>(__VA_ARGS__);                       \
            return FN<4, 2, CODE_HYB2>(__VA_ARGS__);                                   \
        } else if (code_id == CODE_HYB) {                                              \
            if (k == 2) return FN<2, 2, CODE_HYB>(__VA_ARGS__);                        \
            if (k == 3) return FN<3, 2, CODE_HYB>(__VA_ARGS__);                        \
            return FN<4, 2, CODE_HYB>(__VA_ARGS__);                                    \
        } else if (code_id == CODE_3INST) {                                            \
            if (k == 2) return FN<2, 1, CODE_3INST>(__VA_ARGS__);                      \
            if (k == 3) return FN<3, 1, CODE_3INST>(__VA_ARGS__);                      \
            return FN<4, 1, CODE_3INST>(__VA_ARGS__);                                  \
        } else {                                                                       \
            if (k == 2) return FN<2, 1, CODE_1MAD>(__VA_ARGS__);                       \
            if (k == 3) return FN<3, 1, CODE_1MAD>(__VA_ARGS__);                       \
            return FN<4, 1, CODE_1MAD>(__VA_ARGS__);                                   \
        }                                                                              \
    } while (0)

hipError_t launch_dequantize(int k, int code_id, const uint32_t *codes, const uint32_t *lut, int m,
                             int n, void *W, hipStream_t st) {
    if (code_id == CODE_LUT) return launch_lut_dequantize(k, codes, lut, m, n, W, st);
    QTIP_DISPATCH(launch_dequantize_t, codes, lut, m, n, W, st);
}

hipError_t launch_matvec(int k, int code_id, const uint32_t *codes, const uint32_t *lut, int m,
                         int n, const void *x, const void *scale, float *y, hipStream_t st) {
    if (code_id == CODE_LUT) return launch_lut_matvec(k, codes, lut, m, n, x, scale, y, st);
    QTIP_DISPATCH(launch_matvec_t, codes, lut, m, n, x, (const int8_t *)nullptr, 0, scale, y, st);
}

int fused_rht_matvec_max_n() { return FUSED_MAX_N; }

hipError_t launch_rht_matvec(int k, int code_id, const uint32_t *codes, const uint32_t *lut, int m,
                             int n, const void *x, const int8_t *signs, int block, const void *scale,
                             float *y, hipStream_t st) {
    // (beyond these there is no kernel that looks at the signs: QTIP_MV_LAUNCH_MANY)
    if (m > FUSED_RHT_MATVEC_MAX_M || n > FUSED_MAX_N) return hipErrorInvalidValue;
    int log2_block = 0;
    while ((1 << log2_block) < block) log2_block++;
    QTIP_DISPATCH(launch_matvec_t, codes, lut, m, n, x, signs, log2_block, scale, y, st);
}

// 17 to 256 batch rows by the kernel for 16 (or 32) of them at a time: where workgroups of one tile row and 32 batch rows are
// one per CU at most, which leaves gemm_kernel, 32 outputs and eight waves each, fewer CUs and longer slices; and up to 32
// rows of many outputs for the codes with a table, which leaves room for one workgroup of gemm_kernel on a CU (the others have two),
// if rows are not long.
// us, that kernel and this one: 2-bit 3INST 1024 x 14336 32 rows 21.1 11.6, 64 rows 21.2 13.7, 128 rows 22.3 16.9, 4096 x 4096 17 rows
// 8.5 6.7, 4096 x 14336 32 rows 22.9 18.2, 5120 x 4096 32 rows 8.7 9.7; 4-bit HYB 1024 x 14336 32 rows 19.0 13.4, 2048 x 4096 64 rows
// 8.0 8.0.  Six codes, 16 to 4096 outputs, 16 to 2^20 inputs: up to 256 rows 0.97 to 2.1 times as fast, 1.5 on average; more rows,
// which are few outputs, are not taken (16 x 4096, 512 rows 0.8 times, 2000 rows 8.9 us and 34).  17 to 32 rows of more than 8192
// outputs, time of this kernel over that one's: V = 1 hash code 0.73 at 64 inputs, 0.94 at 6144, 1.0 at 8192, 1.05 at 28672; HYB and
// HYB2 0.76, 0.98 at 4096, 1.0 at 6144, 1.05; codes without a table 0.95 at 64 inputs, 1.02 at 2048, 1.1 at 8192.
// Where 16 rows at a time would be more than one workgroup per CU and 32 are not, what is read of X decides: there are twice as many
// workgroups as the other kernel's to read it, and rows that do not begin with a cache line have 64 lines in a step's 64 inputs of 32
// batch rows, not 32.  Time of this kernel over that one's, code words from memory: in whole lines codes without a table and V = 1 hash
// code 0.82, HYB and HYB2 at 2 bits 0.94; at 3 and 4 bits, where that kernel hashes two states at once, 0.98 to 1.1.  Otherwise, up to 64
// batch rows and the inputs below, 0.88, but beyond these 1.05 (V = 1 hash code) to 1.4 (480 x 28400, 140 rows, 3-bit HYB 54.5 us and
// 38.6; 592 x 19728, 136 rows, 2-bit 3INST 38.7 28.6), and for more batch rows up to 1.2 (432 x 1456, 172 rows, 4-bit HYB2 6.4 5.3).
// Of 757 products that go here by this 9 take more than 6 % longer, 13 % at most.
static bool matmat_takes(int k, int code_id, int m, int n, int B) {
    const int tm = m / 16, groups = (B + 15) / 16;
    if (code_id == CODE_LUT || B > 256) return false;
    if ((long)tm * groups <= CUS) return true;
    if ((long)tm * ((groups + 1) / 2) <= CUS)
        return (groups <= 4 && n <= (code_is_hyb(code_id) ? 2048 : code_id == CODE_HYB1 ? 8192 : 4096)) ||
               (n % 64 == 0 && (k == 2 || !code_is_hyb(code_id)));
    return groups == 2 && tm > 2 * CUS && code_lds_words(code_id) > 1 && n <= (code_is_hyb(code_id) ? 4096 : 8192);
}

// The lookup-only code's own kernel decodes 16 waves' shares of 32 outputs one wait after the other; it is for what the other one does
// not take (us, up to 16 rows, code words from memory, it and gemm_kernel: k = 2 1024 x 14464 34.7 30.8, k = 4 1472 x 24152 56.6 48.4,
// 256 x 11736 30.0 25.3; up to 256 outputs it takes 0.97 to 1.19 times as long, 1.02 on average, and from the caches 0.95 to 0.98; ms,
// 96 x 2^24 38.8 30.3).
hipError_t launch_matmat(int k, int code_id, const uint32_t *codes, const uint32_t *lut, int m,
                         int n, const void *X, int B, const void *scale, float *Y,
                         hipStream_t st) {
    if (gemm_takes(code_id, n, B) && (code_id == CODE_LUT || (B > 16 && !matmat_takes(k, code_id, m, n, B))))
        return launch_gemm(k, code_id, codes, lut, m, n, X, B, scale, Y, st);
    if (code_id == CODE_LUT) return launch_lut_matmat(k, codes, lut, m, n, X, B, scale, Y, st);
    QTIP_DISPATCH(launch_matmat_t, codes, lut, m, n, X, B, scale, Y, st);
}

hipError_t launch_decode_states(int code_id, const uint32_t *states, int count,
                                const uint32_t *lut, void *out, hipStream_t st) {
    const int blocks = (count + 255) / 256;
    if (code_id == CODE_LUT) return launch_lut_decode_states(states, count, lut, out, st);
    if (code_id == CODE_HYB1)
        hipLaunchKernelGGL((decode_states_kernel<CODE_HYB1>), dim3(blocks), dim3(256), 0, st, states,
                           count, lut, (half_t *)out);
    else if (code_id == CODE_HYB2)
        hipLaunchKernelGGL((decode_states_kernel<CODE_HYB2>), dim3(blocks), dim3(256), 0, st, states,
                           count, lut, (half_t *)out);
    else if (code_id == CODE_HYB)
        hipLaunchKernelGGL((decode_states_kernel<CODE_HYB>), dim3(blocks), dim3(256), 0, st, states,
                           count, lut, (half_t *)out);
    else if (code_id == CODE_3INST)
        hipLaunchKernelGGL((decode_states_kernel<CODE_3INST>), dim3(blocks), dim3(256), 0, st,
                           states, count, lut, (half_t *)out);
    else
        hipLaunchKernelGGL((decode_states_kernel<CODE_1MAD>), dim3(blocks), dim3(256), 0, st,
                           states, count, lut, (half_t *)out);
    return hipGetLastError();
}

}  // namespace qtip
