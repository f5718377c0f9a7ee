// Decode + batched product for prompts and large batches: Y = X W~^T with the weights decoded on the way
// into the matrix cores.
//
// v_mfma_f32_32x32x16_f16 with the activations as A (32 batch rows) and the decoded weights as B (32
// outputs), so that a result register holds 32 neighbouring outputs of one batch row and is stored as whole
// cache lines.  A step is 16 inputs, one tile J: lane l decodes eight neighbouring weights of output l % 32,
// inputs 8 (l / 32) .. + 7 of the tile, straight into the B operand.
//
// What bounds it.  Decoding eight weights costs a wave about 40 vector instructions, a matrix instruction
// keeps its unit busy for 32 cycles: a decoded operand has to meet eight batch groups (256 batch rows)
// before the matrix cores are the slower side.  So a wave owns RB groups of 32 outputs and all NBB groups of 32
// batch rows of its workgroup, and no weight is decoded twice in a workgroup.  Its loop interleaves the matrix
// instructions of a step with the decoding of the next step's weights, one piece after every matrix
// instruction, which leaves both units busy from one wave.
//
// The activations go from memory into LDS without passing through registers, KS tiles (KS * 32 bytes per batch row)
// at a time and one such stage ahead, and are shared by the WM waves that own different outputs; WK waves
// (or groups of WM) split the inputs instead where there are few outputs, and add up through LDS at the end.
// In LDS a row's 16-byte pieces are permuted by the row's number, so that the 16-byte reads of
// neighbouring rows fall on different banks; the copy into LDS fetches them in that order.
#include <type_traits>

#include "qtip_device.h"
#include "qtip_internal.h"

namespace qtip {
namespace {

typedef float float16_t __attribute__((ext_vector_type(16)));

// Where the eight weights of lane (i = output within its group of 32, h) of step J are: word index of the
// first and bit offset in it.  16 x 16 tiles: row i % 16 of the tile in tile row i / 16 of the group, second half
// of the row if h.  Lookup-only code: row i of block 2 J + h.
template <int K, int CODE>
__device__ __forceinline__ int first_bit(int i, int h) {
    return CODE == CODE_LUT ? 8 * K * i : 16 * K * (i & 15) + 8 * K * h;
}

// Sum of a 3INST word's halves into the low or the high half of a packed pair.  A register half-written by one
// of these may not be read by the very next instruction: the compiler puts a wait there, around such text too (unlike a read
// across lanes), which the callers make unnecessary with other instructions in between.
__device__ __forceinline__ void add_halves_low(uint32_t y, uint32_t &p) {
    asm("v_add_f16_sdwa %0, %1, %1 dst_sel:WORD_0 dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_1" : "=v"(p) : "v"(y));
}
__device__ __forceinline__ void add_halves_high(uint32_t y, uint32_t &p) {
    asm("v_add_f16_sdwa %0, %1, %1 dst_sel:WORD_1 dst_unused:UNUSED_PRESERVE src0_sel:WORD_0 src1_sel:WORD_1" : "+v"(p) : "v"(y));
}
__device__ __forceinline__ void add_halves_last(uint32_t y0, uint32_t y1, uint32_t &p) {
    asm("v_add_f16_sdwa %0, %1, %1 dst_sel:WORD_0 dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_1\n\t"
        "s_nop 0\n\t"
        "v_add_f16_sdwa %0, %2, %2 dst_sel:WORD_1 dst_unused:UNUSED_PRESERVE src0_sel:WORD_0 src1_sel:WORD_1\n\t"
        "s_nop 0"
        : "=&v"(p)
        : "v"(y0), "v"(y1));
}

// Eight weights from the 64 bits at their first one: what step<0> .. step<7>, called one after the other, leave in `raw` is made
// four packed pairs by packed(), a step later, so that nothing waits for a table read just made.
//   The hash codes hash two states at once in the halves of a register: states 4 K bits apart, which are two halves of
// one window at k = 4 and otherwise brought together by one v_perm_b32.  (One state at a time, values taken as soon as read and the
// table behind the first 64 KiB of LDS, where a read's address needs an instruction more: 64 rows of 8192 x 8192, k = 2 HYB 18.2 us
// and now 16.9, k = 3 HYB2 20.3 and 18.6, k = 4 HYB1 25.6 and 22.2; 40 rows of 4096 x 14336, HYB1, 29.3 and 25.0; with what is said
// at the copies of a stage.)
template <int K, int CODE> struct EightWeights {
    static constexpr int RAW = CODE == CODE_HYB2 ? 6 : CODE == CODE_HYB1 || CODE == CODE_LUT ? 8 : 4;
    uint64_t b64;
    uint32_t mm, lane4;
    const uint32_t *lut;  // LDS
    uint32_t w[2], t[2];
    __device__ __forceinline__ void init(const uint32_t *lds_lut) {
        lut = lds_lut;
        lane4 = (threadIdx.x & 31u) << 2;
        b64 = CODE == CODE_3INST ? INST_B : MAD_B;
        mm = INST_MM;
        asm volatile("" : "+v"(b64), "+v"(mm));
    }
    // w0, w1: two neighbouring words of the stream; selector: the bytes of (w0, w1) that start at the first bit
    __device__ __forceinline__ void start(uint32_t w0, uint32_t w1, uint32_t selector, uint32_t shift) {
        if constexpr (K == 4) {
            w[0] = w0;
            w[1] = w1;
        } else {
            w[0] = __builtin_amdgcn_perm(w0, w1, selector);
            w[1] = K == 2 ? 0u : w1 << shift;
        }
    }
    // the states at bits P (high half) and P + 4 K (low half)
    template <int P> __device__ __forceinline__ uint32_t state_pair() const {
        if constexpr (K == 4) return window32(w, P);
        else if constexpr (K == 2) return __builtin_amdgcn_perm(w[0] << P, w[0] << P, 0x03020201u);
        else return __builtin_amdgcn_perm(window32(w, P), window32(w, P + 12), 0x07060302u);
    }
    // low 16 bits of x x + x of both halves
    __device__ __forceinline__ static uint32_t hash_pair(uint32_t R) {
        uint32_t H;
        asm("v_pk_mad_u16 %0, %1, %1, %1" : "=v"(H) : "v"(R));
        return H;
    }
    template <int c> __device__ __forceinline__ void step(uint32_t (&raw)[RAW]) {
        if constexpr (CODE == CODE_3INST) {
            // (four vector instructions per call: a weight's sum of halves goes behind the next one's multiply-add,
            // which needs a wait state before its result is read)
            const uint32_t Z = lcg_mad64(window16(w, c * K), INST_A, b64);
            if constexpr (c % 2 == 1 && c < 7) add_halves_low(t[0], raw[c / 2]);
            if constexpr (c % 2 == 0 && c > 0) add_halves_high(t[1], raw[c / 2 - 1]);
            t[c & 1] = (Z & INST_MASK) ^ mm;
            if constexpr (c == 7) add_halves_last(t[0], t[1], raw[3]);
        } else if constexpr (CODE == CODE_1MAD) {
            const uint32_t X = lcg_mad64(window16(w, c * K), MAD_A, b64);
            const uint32_t s = __builtin_amdgcn_sad_u8(X, 0u, 0x4B000000u);  // float 2^23 + s
            t[c & 1] = __builtin_bit_cast(uint32_t, (__builtin_bit_cast(float, s) - 8389118.0f) * MAD_INV_SCALE);
            if constexpr (c & 1)
                raw[c / 2] = as_u32(half2_t{(half_t)__builtin_bit_cast(float, t[0]), (half_t)__builtin_bit_cast(float, t[1])});
        } else if constexpr (code_is_hyb(CODE)) {
            constexpr int j = c / 4;  // states j and j + 2
            if constexpr (c % 4 == 0) {
                const uint32_t R = state_pair<2 * K * j>();
                if constexpr (CODE == CODE_HYB2) raw[4 + j] = hyb2_sign_mask(R);
                t[0] = hash_pair(R);
                raw[j] = hyb_signed_lookup(lut, (t[0] >> 20) & 0xFFCu);
            } else if constexpr (c % 4 == 2) {
                raw[j + 2] = hyb_signed_lookup(lut, (t[0] >> 4) & 0xFFCu);
            }
        } else if constexpr (CODE == CODE_HYB1) {
            constexpr int j = c / 2;  // states j and j + 4
            if constexpr (c % 2 == 0) {
                t[0] = hash_pair(state_pair<K * j>());
                raw[j] = hyb_signed_lookup(lut, ((t[0] >> 18) & 0x3F80u) | lane4);
            } else {
                raw[j + 4] = hyb_signed_lookup(lut, ((t[0] >> 2) & 0x3F80u) | lane4);
            }
        } else {
            // 14 state bits to bits 14..1
            const uint32_t off = c * K < 17 ? (w[0] >> (17 - c * K)) & 0x7FFEu : window32(w, c * K - 17) & 0x7FFEu;
            raw[c] = *reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(lut) + off);
        }
    }
    __device__ __forceinline__ static half8_t packed(const uint32_t (&raw)[RAW]) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        u32x4 h;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            if constexpr (CODE == CODE_HYB1) h[c] = hyb1_pair(raw[2 * c], raw[2 * c + 1]);
            else if constexpr (CODE == CODE_LUT) h[c] = raw[2 * c] | (raw[2 * c + 1] << 16);
            else if constexpr (CODE == CODE_HYB2) h[c] = raw[c] ^ ((c < 2 ? raw[4 + c] >> 16 : raw[2 + c]) & 0x8000u);
            else h[c] = raw[c];
        }
        return __builtin_bit_cast(half8_t, h);
    }
};

// s_waitcnt that waits until at most n memory loads are outstanding, and for nothing else.
constexpr int vmcnt_only(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }

// A buffer of `bytes` bytes: what is read behind its end is 0.
__device__ __forceinline__ u32x4_t buffer_of(const void *p, size_t bytes) {
    const uint64_t at = reinterpret_cast<uintptr_t>(p);
    return u32x4_t{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at),
                   (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32)),
                   (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(bytes < 0xFFFFFFFFu ? bytes : 0xFFFFFFFFu)),
                   0x00020000u};
}
// 16 bytes per lane from byte `lane_offset` + `offset` of a buffer into LDS at `to`, lane by lane.  (Written
// out, because the compiler makes every later read of LDS wait for the copy, whatever it reads.  The kernel
// waits for its copies itself; the compiler's own waits only become longer by loads it does not count.)
__device__ __forceinline__ void copy_to_lds(u32x4_t buffer, uint32_t lane_offset, uint32_t offset, const char *to) {
    const uint32_t at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char *)to;
    asm volatile("s_mov_b32 m0, %3\n\t"
                 "s_nop 0\n\t"
                 "buffer_load_dwordx4 %0, %1, %2 offen lds"
                 :
                 : "v"(lane_offset), "s"(buffer), "s"(offset), "s"(at)
                 : "memory");
}

template <int N, class F, int I = 0>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, F, I + 1>(static_cast<F &&>(f));
    }
}

// Sizes of a workgroup's LDS.
template <int K, int CODE, int RB, int NBB, int WM, int WK, int KS> struct GemmLds {
    static constexpr bool LUT = CODE == CODE_LUT;
    static constexpr int SLICE = 32 * NBB * KS * 32;                       // activations of a stage
    static constexpr int STEP_BYTES = (LUT ? 8 : 4) * 8 * K;               // code words of a tile row and step
    static constexpr int CODE_ROW = KS * STEP_BYTES, CODE_ROWS = LUT ? RB : 2 * RB;  // of a wave and stage
    static constexpr int CODE_COPIES = (CODE_ROWS * CODE_ROW + 1023) / 1024, CODE_STAGE = CODE_COPIES * 1024;
    static constexpr int TABLE_WORDS = LUT ? 1 << 13 : code_lds_words(CODE) > 1 ? code_lds_words(CODE) : 0;
    // batch groups whose partial sums are in LDS at the same time, in the room of the activations
    static constexpr int SUM_BYTES = WM * WK * RB * 4096;
    static constexpr int SUMS = WK == 1 ? 0 : NBB * SUM_BYTES <= 2 * WK * SLICE ? NBB : (2 * WK * SLICE) / SUM_BYTES;
    static constexpr int BYTES = 2 * WK * SLICE + WM * WK * 2 * CODE_STAGE + (4 * TABLE_WORDS + 1023) / 1024 * 1024;
    static_assert(WK == 1 || (SUMS >= 1 && NBB % SUMS == 0), "whole rounds of partial sums");
    // (a kilobyte more, and one: us, 2-bit 3INST 4128 x 2048, 96 rows, 9.4 and 11.1, 10240 x 2048, 192 rows, 18.4 and 21.1)
    static_assert(TABLE_WORDS > 0 || RB * NBB > 1 || 2 * BYTES <= 160 * 1024, "32 x 32: two workgroups per CU");
};

template <int K, int CODE, int RB, int NBB, int WM, int WK, int KS>
__global__ __launch_bounds__(WM *WK * 64, RB *NBB > 4 ? 1 : 2) void gemm_kernel(
    const uint32_t *__restrict__ codes, const uint32_t *__restrict__ lut, int m, int n, const half_t *__restrict__ X,
    int B, const half_t *__restrict__ scale, float *__restrict__ Y) {
    constexpr bool LUT = CODE == CODE_LUT;
    constexpr int NWORDS = 8 * K, NT = WM * WK * 64;
    constexpr int BT = 32 * NBB, ROW = KS * 32;       // batch rows of a workgroup; bytes of a row per stage
    constexpr int UNITS = KS * 2, RPI = 64 / UNITS;   // 16-byte pieces of a row; rows per copy instruction
    using Lds = GemmLds<K, CODE, RB, NBB, WM, WK, KS>;
    constexpr int SLICE = Lds::SLICE, NCOPY = BT / RPI / WM;  // bytes of a stage; copy instructions per wave
    constexpr int SUMS_AT_ONCE = Lds::SUMS;
    // Stages that are summed in the matrix cores before the sums go to totals of their own: the rounding error of a long
    // chain grows with it (997 x 4096 x 14336, against binary64: 4.1e-7 in one chain of 256 matrix instructions,
    // 1.3e-7 in chains of 16).  The totals take as many registers as the running sums: at 256 batch rows a workgroup is
    // four waves with a SIMD's registers each (115 -> 149 us; up to 128 batch rows it costs 1 to 4 %).
    // With eight slices of the inputs a chain is a 128th of the inputs long, no longer than it was in the kernels that
    // had 17 to 64 rows before (1.6e-7 at 4096 inputs, 2.8e-7 at 14464; totals would halve that and cost HYB 3 to 5 %).
    // Only the lookup-only code had more, 16 slices up to 32 rows (1.3e-7 and 2.1e-7) and four with totals up to 64, so its
    // sums go to totals here too: 1.2e-7 and 1.3e-7; 24 rows, 4096 x 4096 12.6 -> 12.7 us, 2048 x 14464 35.7 -> 36.0, 8192 x
    // 8192 22.6 -> 23.1.
    constexpr int CHAIN = WK == 8 && !LUT ? 0 : 16 / KS;
    constexpr int AHEAD = 3, GROUPS = KS * NBB * RB;  // a group: one matrix instruction and what goes with it
    constexpr int STEP_BYTES = Lds::STEP_BYTES, CODE_ROW = Lds::CODE_ROW, CODE_ROWS = Lds::CODE_ROWS;
    constexpr int CODE_COPIES = Lds::CODE_COPIES, CODE_STAGE = Lds::CODE_STAGE;
    constexpr int COPIES = CODE_COPIES + NCOPY;
    // The group behind which a copy is made: the next stage's are spread over the first half of this one.  Code words come from
    // memory, not from the caches, and are waited for in the middle of a stage.  Where few batch rows make stages short, those
    // of the stage after the next are asked for as soon as this one's have all been read, at step KS - 2, a whole stage
    // ahead of that wait in place of half of one (8192 x 8192, 4-bit HYB, 32 rows 16.3 -> 14.8 us, 64 rows 21.4 -> 20.9, one
    // stage more ahead 22.1; but 200 rows of 12288 x 8192, 3-bit 3INST, 73.7 -> 75.0).
    constexpr bool EARLY = WM == 1;
    constexpr auto copy_group = [](int c) {
        if (!EARLY) return c * (GROUPS / 2) / COPIES;
        return c < CODE_COPIES ? (KS - 2) * NBB * RB + RB - 1 + c * (GROUPS / KS) / CODE_COPIES
                               : (c - CODE_COPIES) * (GROUPS / 2) / NCOPY;
    };
    // Copies made behind the code words of the next stage at the wait for them, and behind the next stage's last activations.
    constexpr int WAIT_GROUP = ((KS - 2) * NBB + NBB / 2) * RB;
    constexpr int BEHIND_CODES = [=] {
        int count = 0;
        for (int c = EARLY ? 0 : CODE_COPIES; c < COPIES; c++) count += copy_group(c) <= WAIT_GROUP;
        return count;
    }();
    constexpr int BEHIND_X = [=] {
        int count = 0;
        for (int c = 0; c < CODE_COPIES; c++) count += copy_group(c) > copy_group(COPIES - 1);
        return count;
    }();
    static_assert(KS >= 2 && 2 * CODE_COPIES + NCOPY <= 60, "a stage holds the step after the next; the count of a wait");
    static_assert(BT % (RPI * WM) == 0, "whole copies");
    // (in this order: the table's place in a read's 16 bits of offset)
    __shared__ struct {
        __attribute__((aligned(1024))) uint32_t lut[Lds::TABLE_WORDS];
        __attribute__((aligned(1024))) char x[2 * WK * SLICE];
        __attribute__((aligned(1024))) char codes[WM * WK * 2 * CODE_STAGE];
    } s_all;
    static_assert(sizeof(s_all) == Lds::BYTES, "as the launcher counts");
    uint32_t *const s_lut = s_all.lut;
    char *const s_x = s_all.x, *const s_codes = s_all.codes;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wm = wave % WM, wk = wave / WM;
    const int i = lane & 31, h = lane >> 5;
    const int o0 = (blockIdx.x * WM + wm) * (32 * RB);  // first output
    const int b0 = blockIdx.y * BT;
    // Places along the inputs are counted in pieces of eight, half a step each.  A slice's stages end where the slice ends, so
    // that a stage with less than KS steps is the first one, copied ahead of the loop: in the loop no copy looks where it
    // is (at 32 x 64, 4-bit HYB, 72 vector instructions a stage with that, 58 without).
    const int all = n / 8, per = (all + WK * UNITS - 1) / (WK * UNITS) * UNITS;  // of a slice
    const int P0 = wk * per, Pend = min(all, P0 + per);
    const int stages = per / UNITS, mine = P0 < Pend ? (Pend - P0 + UNITS - 1) / UNITS : 0;
    const int Pfirst = Pend - mine * UNITS;  // (may be less than P0, and less than 0)

    // The wave's code words of a stage: the KS tiles of a tile row lie one after the other, so whole 16
    // bytes are copied into LDS as they are.  (Any weights do ahead of a slice, their inputs are zeros.  The copies that the last
    // stage makes for one that does not come stay inside the buffer or bring zeros.)
    constexpr int r_first = LUT ? 32 : 16;
    const size_t line = (size_t)(LUT ? n / 8 : n / 16) * (4 * NWORDS);  // bytes of a tile row
    const int I_base = min(o0, m - 1) / r_first;
    const u32x4_t code_buffer =
        buffer_of(reinterpret_cast<const char *>(codes) + (size_t)I_base * line, ((size_t)(m / r_first) - I_base) * line);
    char *const my_codes = s_codes + wave * (2 * CODE_STAGE);
    uint32_t coff[CODE_COPIES];
    int ahead[CODE_COPIES];  // bytes from there to the first stage's
#pragma unroll
    for (int q = 0; q < CODE_COPIES; q++) {
        const int at = (64 * q + lane) * 16, r = min(at / CODE_ROW, CODE_ROWS - 1);
        const int I = min(o0 + r * r_first, m - 1) / r_first - I_base;  // (beyond m: any row)
        coff[q] = (uint32_t)I * (uint32_t)line + at % CODE_ROW;
        ahead[q] = max(at % CODE_ROW + Pfirst * (STEP_BYTES / 2), 0) - at % CODE_ROW;
    }
    const int bit = first_bit<K, CODE>(i, h);
    const int w0 = bit >> 5, w1 = (w0 + 1) % NWORDS;  // (wraps inside a tile: tail-biting)
    const uint32_t selector = 0x07060504u - (uint32_t)((bit & 31) >> 3) * 0x01010101u, shift = bit & 31;
    const char *const code_words = my_codes + (LUT ? h * 4 * NWORDS : (i >> 4) * CODE_ROW);
    auto copy_codes = [&](auto qc, uint32_t offset, uint32_t at, int buffer) {
        constexpr int q = decltype(qc)::value;
        copy_to_lds(code_buffer, offset, at, my_codes + buffer * CODE_STAGE + q * 1024);
    };
    // copies into LDS: lane = (row within the instruction, place of the piece)
    auto swizzle = [](int row) { return (row / (16 / UNITS)) & (UNITS - 1); };
    const int crow = lane / UNITS;
    char *const slice = s_x + wk * (2 * SLICE);
    const int rows = min(BT, B - b0);
    uint32_t xoff[NCOPY];
    const char *const xbase = reinterpret_cast<const char *>(X + (size_t)b0 * n);
    const u32x4_t x_buffer = buffer_of(xbase, (size_t)rows * 2 * n);
    auto copy_x = [&](auto qc, uint32_t offset, uint32_t at, int buffer) {
        constexpr int q = decltype(qc)::value;
        copy_to_lds(x_buffer, offset, at, slice + buffer * SLICE + (wm * NCOPY + q) * 1024);
    };
    // (the first stage's, on their way while the table is filled)
    static_for<CODE_COPIES>([&](auto qc) {
        if (mine > 0) copy_codes(qc, coff[decltype(qc)::value] + (uint32_t)ahead[decltype(qc)::value], 0, 0);
    });
    static_for<NCOPY>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        const int b = (wm * NCOPY + q) * RPI + crow;
        const int piece = (lane % UNITS) ^ swizzle(q * RPI + crow) ^ (NCOPY % 2 ? swizzle(wm * NCOPY * RPI) : 0);
        xoff[q] = (uint32_t)min(b, rows - 1) * (uint32_t)(2 * n) + 16 * piece;
        // what lies ahead of the slice is asked for beyond the buffer's end, so that zeros arrive
        if (mine > 0) copy_x(qc, Pfirst + piece >= P0 ? xoff[q] + (uint32_t)(16 * Pfirst) : 0xFFFFFF00u, 0, 0);
    });
    if constexpr (EARLY) {
        static_for<CODE_COPIES>([&](auto qc) {
            if (mine > 0) copy_codes(qc, coff[decltype(qc)::value], (uint32_t)min(Pfirst + UNITS, all - 1) * (STEP_BYTES / 2), 1);
        });
    }
    // a lane's place in a buffer: row i, piece 2 j + h
    const uint32_t xread = (uint32_t)i * ROW + (uint32_t)((h ^ swizzle(i)) << 4);

    if constexpr (LUT) {
        const uint4 *src = reinterpret_cast<const uint4 *>(lut);
        uint4 *dst = reinterpret_cast<uint4 *>(s_lut);
        for (int e = threadIdx.x; e < 2048; e += NT) dst[e] = src[e];
        __syncthreads();
    } else {
        stage_code_table<CODE>(lut, s_lut, NT);
    }
    EightWeights<K, CODE> dec[RB];
#pragma unroll
    for (int rb = 0; rb < RB; rb++) dec[rb].init(s_lut);
    float16_t acc[RB][NBB], total[RB][NBB];
#pragma unroll
    for (int rb = 0; rb < RB; rb++)
#pragma unroll
        for (int nb = 0; nb < NBB; nb++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[rb][nb][e] = 0.f, total[rb][nb][e] = 0.f;
    auto add_up = [&] {
#pragma unroll
        for (int rb = 0; rb < RB; rb++)
#pragma unroll
            for (int nb = 0; nb < NBB; nb++) total[rb][nb] += acc[rb][nb];
    };

    uint32_t wnext[RB][EightWeights<K, CODE>::RAW];  // the weights of the next step
    uint32_t cw[RB][2];  // the two words that the next eight weights start in
    auto read_codes = [&](int step, int buffer) {
#pragma unroll
        for (int rb = 0; rb < RB; rb++) {
            const char *p = code_words + buffer * CODE_STAGE + rb * (CODE_ROWS / RB) * CODE_ROW + step * STEP_BYTES;
            cw[rb][0] = *reinterpret_cast<const uint32_t *>(p + 4 * w0);
            cw[rb][1] = *reinterpret_cast<const uint32_t *>(p + 4 * w1);
        }
    };
    __builtin_amdgcn_s_waitcnt(vmcnt_only(0));  // the first stage is there
    __syncthreads();
    if (mine > 0) {
        read_codes(0, 0);
#pragma unroll
        for (int rb = 0; rb < RB; rb++) {
            dec[rb].start(cw[rb][0], cw[rb][1], selector, shift);
            static_for<8>([&](auto c) { dec[rb].template step<decltype(c)::value>(wnext[rb]); });
        }
        read_codes(1, 0);
    }
    // fresh: the running sums start again
    auto stage = [&](int s, auto fresh) {
        // first pieces of the next stage, and of the stage whose code words are copied in this one
        const uint32_t next = min(Pfirst + (s + 1) * UNITS, all - 1);
        const uint32_t codes_of = EARLY ? min(Pfirst + (s + 2) * UNITS, all - 1) : next;
        const char *const buf = slice + (s & 1) * SLICE;
        // the activations of a stage, KS * NBB operands, are read from LDS AHEAD operands before their use
        half8_t xv[AHEAD + 1];
        auto read_x = [&](auto rc) {
            constexpr int r = decltype(rc)::value;
            xv[r % (AHEAD + 1)] = *reinterpret_cast<const half8_t *>(buf + (xread ^ (r / NBB << 5)) + r % NBB * 32 * ROW);
        };
        static_for<AHEAD>([&](auto r) { read_x(r); });
        __builtin_amdgcn_sched_barrier(0);
        static_for<KS>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            half8_t wv[RB];
#pragma unroll
            for (int rb = 0; rb < RB; rb++) {
                wv[rb] = EightWeights<K, CODE>::packed(wnext[rb]);
                dec[rb].start(cw[rb][0], cw[rb][1], selector, shift);
            }
            static_for<NBB>([&](auto nbc) {
                constexpr int nb = decltype(nbc)::value, r = j * NBB + nb;
                if constexpr (r + AHEAD < KS * NBB) read_x(std::integral_constant<int, r + AHEAD>{});
                static_for<RB>([&](auto rbc) {
                    constexpr int rb = decltype(rbc)::value, group = r * RB + rb;
                    acc[rb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xv[r % (AHEAD + 1)], wv[rb],
                                                                         decltype(fresh)::value && j == 0 ? float16_t{} : acc[rb][nb], 0, 0, 0);
                    // the next stage's copies, spread over the first part of this one: a wave that issues several in a
                    // row waits for the memory pipeline, and the matrix cores with it
                    static_for<COPIES>([&](auto cc) {
                        constexpr int c = decltype(cc)::value;
                        if constexpr (copy_group(c) == group) {
                            if constexpr (EARLY && c == 0) {  // (the words read last, which the copy replaces, are in registers)
#pragma unroll
                                for (int rb = 0; rb < RB; rb++) asm volatile("" : "+v"(cw[rb][0]), "+v"(cw[rb][1]));
                            }
                            if constexpr (c < CODE_COPIES)
                                copy_codes(std::integral_constant<int, c>{}, coff[c], codes_of * (STEP_BYTES / 2),
                                           (s + !EARLY) & 1);
                            else
                                copy_x(std::integral_constant<int, c - CODE_COPIES>{}, xoff[c - CODE_COPIES], 16 * next, (s + 1) & 1);
                        }
                    });
                    static_for<8 / NBB>([&](auto pc) {
                        dec[rb].template step<nb * (8 / NBB) + decltype(pc)::value>(wnext[rb]);
                    });
                    // the words of the step after the next: of this stage, or, at its last steps, of the next
                    if constexpr (nb == NBB / 2 && rb == 0) {
                        if constexpr (j + 2 < KS) {
                            read_codes(j + 2, s & 1);
                        } else {
                            if constexpr (j + 2 == KS) __builtin_amdgcn_s_waitcnt(vmcnt_only(BEHIND_CODES));
                            read_codes(j + 2 - KS, (s + 1) & 1);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
        });
        // The copies of this stage have landed, everywhere.  Where waves own different inputs (WM = 1) each reads only what
        // it copied, and waits for nothing else: in step they all decoded and all used the matrix cores at the same time
        // (8192 x 8192, 4-bit HYB, 64 rows 24.8 -> 21.0 us, 32 rows 17.8 -> 16.9).
        __builtin_amdgcn_s_waitcnt(vmcnt_only(BEHIND_X));
        asm volatile("" ::: "memory");
        if constexpr (WM > 1) {
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
    };
    if constexpr (CHAIN == 0) {
        for (int s = 0; s < mine; s++) stage(s, std::false_type{});
    } else {
        for (int s = 0; s < mine;) {
            stage(s++, std::true_type{});
            for (int c = 1; c < CHAIN && s < mine; c++) stage(s++, std::false_type{});
            add_up();
        }
    }
    const auto &sum = [&]() -> auto & {
        if constexpr (CHAIN == 0) return acc;
        else return total;
    }();
    if constexpr (WM > 1)
        for (int s = mine; s < stages; s++) __builtin_amdgcn_s_barrier();  // (a slice with less or nothing to do)
    __builtin_amdgcn_s_waitcnt(vmcnt_only(0));  // (no copy is under way when the workgroup's LDS is another's)
    __syncthreads();

    // D element e of a lane: batch row 8 (e / 4) + 4 h + e % 4, output i
    if constexpr (WK == 1) {
#pragma unroll
        for (int rb = 0; rb < RB; rb++) {
            const int o = o0 + 32 * rb + i;
            if (o >= m) continue;
            const float sc = scale ? (float)scale[o] : 1.f;
#pragma unroll
            for (int nb = 0; nb < NBB; nb++)
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    const int b = b0 + 32 * nb + 8 * (e / 4) + 4 * h + e % 4;
                    if (b < B) Y[(size_t)b * m + o] = sum[rb][nb][e] * sc;
                }
        }
    } else {
        float *const sums = reinterpret_cast<float *>(s_x);  // [wk][wm][rb][nb of this round][e][lane]
        constexpr int BLOCKS = WM * RB * SUMS_AT_ONCE, PARTS = BLOCKS * 16;
#pragma unroll
        for (int nb0 = 0; nb0 < NBB; nb0 += SUMS_AT_ONCE) {
            if (nb0 > 0) __syncthreads();
#pragma unroll
            for (int rb = 0; rb < RB; rb++)
#pragma unroll
                for (int nb = 0; nb < SUMS_AT_ONCE; nb++)
#pragma unroll
                    for (int e = 0; e < 16; e++)
                        sums[(((wk * WM + wm) * RB + rb) * SUMS_AT_ONCE + nb) * 1024 + e * 64 + lane] = sum[rb][nb0 + nb][e];
            __syncthreads();
            for (int part = wave; part < PARTS; part += WM * WK) {
                const int e = part % 16, block = part / 16;
                const int nb = nb0 + block % SUMS_AT_ONCE, rb = block / SUMS_AT_ONCE % RB, mw = block / SUMS_AT_ONCE / RB;
                float v = 0.f;
#pragma unroll
                for (int kk = 0; kk < WK; kk++) v += sums[kk * (BLOCKS * 1024) + block * 1024 + e * 64 + lane];
                const int o = (blockIdx.x * WM + mw) * (32 * RB) + 32 * rb + i;
                const int b = b0 + 32 * nb + 8 * (e / 4) + 4 * h + e % 4;
                if (o < m && b < B) Y[(size_t)b * m + o] = scale ? v * (float)scale[o] : v;
            }
        }
    }
}

}  // namespace

// ------------------------------------------------------------------ launcher

// The ways a product is split: outputs and batch rows of a workgroup, and the time of a round of one workgroup per CU,
// `first` once and `round` for each (only their ratios matter here).  A large tile decodes a weight once for more batch
// rows; a small one leaves no CU idle where outputs or batch rows are few, and splits the inputs between its waves.  A
// round costs the lookup-only code more in the small ones, where every workgroup copies 32 KiB of table, and the V = 1
// hash code, a table read for every weight, more at 128 x 256, which has four waves.
// With each split forced in turn, six codes, k = 2 to 4, 18 shapes from 768 x 4096 and 28672 x 1024 to 5120 x 13824, 17 to
// 1024 rows: the one picked takes 0.15 % more than the fastest on average.  (With one column for all codes, 5.5 a round of 32 x
// 32 and 42 of 128 x 128, it was up to 39 % slower: 2-bit HYB 9216 x 4096, 96 rows, 30.8 us against 22.2, lookup-only 5120 x
// 5120, 256 rows, 65.7 against 48.9, 3-bit 3INST 28672 x 1024, 1024 rows, 118 against 101; with 45 for 128 x 128 lookup-only
// 20480 x 5120, 896 rows, 346 against 311.)  The worst that is left is HYB2 with a single round of 128 x 256 that 64 x 128
// beats: 4128 x 14464, 1024 rows, 280 us against 238.
struct GemmSplit {
    int outputs, rows;
    float first, round, round_lut, round_hyb1;
};
static constexpr GemmSplit GEMM_SPLITS[] = {
    {128, 256, 0.f, 74.f, 74.f, 80.f}, {128, 128, 0.f, 43.5f, 43.5f, 43.5f}, {64, 128, 2.f, 25.f, 25.f, 25.f},
    {64, 64, 5.f, 15.f, 15.5f, 15.f},  {32, 64, 2.f, 11.3f, 11.f, 11.3f}, {32, 32, 4.5f, 6.f, 7.7f, 6.f}};

// A workgroup addresses its batch rows and its wave's tile rows (16 bytes an input at most, less than 32 batch rows) with
// 32-bit byte offsets from uniform bases, kept within 2^31.
static bool offsets_fit(const GemmSplit &s, int n) { return (long)s.rows * 2 * n <= 1L << 31; }

// Kernels of the splits, in their order.  A stage is four tiles, 128 bytes of every batch row, which is what the memory
// pipeline likes (two tiles, 8192 x 8192, 4-bit HYB, 64 rows: 21 -> 27 us); two where four leave no room for the lookup-only
// code's table, at 32 x 64 (8192 x 8192, 48 rows, against 64 x 64, which leaves half of the CUs idle: 44 -> 26 us).
#define QTIP_GEMM_SPLITS(GO)                                             \
    GO(0, 1, 8, 4, 1, 4) GO(1, 1, 4, 4, 2, 4) GO(2, 1, 4, 2, 4, 4)       \
    GO(3, 1, 2, 2, 4, 4) GO(4, 1, 2, 1, 8, (CODE == CODE_LUT ? 2 : 4)) GO(5, 1, 1, 1, 8, 4)

template <int K, int CODE>
static hipError_t launch_gemm_t(const uint32_t *codes, const uint32_t *lut, int m, int n, const void *X, int B,
                                const void *scale, float *Y, hipStream_t st) {
    int best = -1;
    float least = 0.f;
#define QTIP_GEMM_FITS(I, RB, NBB, WM, WK, KS) GemmLds<K, CODE, RB, NBB, WM, WK, KS>::BYTES <= 160 * 1024,
    constexpr bool fits[] = {QTIP_GEMM_SPLITS(QTIP_GEMM_FITS)};
    for (int i = 0; i < 6; i++) {
        const GemmSplit &s = GEMM_SPLITS[i];
        const long gx = (m + s.outputs - 1) / s.outputs, gy = (B + s.rows - 1) / s.rows;
        if (!fits[i] || gy > 65535 || !offsets_fit(s, n)) continue;
        const float round = CODE == CODE_LUT ? s.round_lut : CODE == CODE_HYB1 ? s.round_hyb1 : s.round;
        const float t = s.first + round * (float)((gx * gy + CUS - 1) / CUS);
        if (best < 0 || t < least) best = i, least = t;
    }
    const dim3 grid((m + GEMM_SPLITS[best].outputs - 1) / GEMM_SPLITS[best].outputs,
                    (B + GEMM_SPLITS[best].rows - 1) / GEMM_SPLITS[best].rows);
#define QTIP_GEMM_GO(I, RB, NBB, WM, WK, KS)                                                                        \
    if constexpr (fits[I])                                                                                      \
        if (best == I) {                                                                                        \
            static_assert(32 * RB * WM == GEMM_SPLITS[I].outputs && 32 * NBB == GEMM_SPLITS[I].rows, "order"); \
            hipLaunchKernelGGL((gemm_kernel<K, CODE, RB, NBB, WM, WK, KS>), grid, dim3(WM * WK * 64), 0, st, codes, \
                               lut, m, n, (const half_t *)X, B, (const half_t *)scale, Y);                      \
        }
    QTIP_GEMM_SPLITS(QTIP_GEMM_GO)
#undef QTIP_GEMM_GO
#undef QTIP_GEMM_FITS
    return hipGetLastError();
}

// Rows of up to 2^22 inputs fit every split.  Longer rows are megabytes apart, which the copies into LDS bear badly (2^22
// inputs, 64 outputs and 64 rows, where nothing but the copies takes long: 9.5 ms; the 16-row kernel 3.1).  There the 16 x 16
// codes' own kernels are faster (4096 outputs, 2-bit HYB, 24 rows: 7.7 against 5.4 ms), the lookup-only code's are not (24 rows
// 9.3 against 11.8 ms, 200 rows 18 against 54), so its rows go on as long as the smallest split's offsets fit
// (and its grid takes the batch).
bool gemm_takes(int code_id, int n, int B) {
    return n <= 1 << 22 || (code_id == CODE_LUT && n <= 1 << 25 && B <= 32 * 65535);
}

hipError_t launch_gemm(int k, int code_id, const uint32_t *codes, const void *lut, int m, int n, const void *X, int B,
                       const void *scale, float *Y, hipStream_t st) {
    const uint32_t *tab = (const uint32_t *)lut;
#define QTIP_GEMM_CODE(CODE)                                                                    \
    case CODE:                                                                                  \
        if (k == 2) return launch_gemm_t<2, CODE>(codes, tab, m, n, X, B, scale, Y, st);        \
        if (k == 3) return launch_gemm_t<3, CODE>(codes, tab, m, n, X, B, scale, Y, st);        \
        return launch_gemm_t<4, CODE>(codes, tab, m, n, X, B, scale, Y, st);
    switch (code_id) {
        QTIP_GEMM_CODE(CODE_1MAD)
        QTIP_GEMM_CODE(CODE_3INST)
        QTIP_GEMM_CODE(CODE_HYB)
        QTIP_GEMM_CODE(CODE_HYB2)
        QTIP_GEMM_CODE(CODE_HYB1)
        default: break;
        QTIP_GEMM_CODE(CODE_LUT)
    }
#undef QTIP_GEMM_CODE
    return hipErrorInvalidValue;
}

}  // namespace qtip
