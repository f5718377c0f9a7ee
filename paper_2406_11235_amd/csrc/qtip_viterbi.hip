// GPU quantizer: the Viterbi algorithm on the (L, k, V) bitshift trellis (Section 2.3 of
// arXiv 2406.11235: value function and update rule; Section 3.1: edge rule), made
// tail-biting by Algorithm 4, one T_x x T_y block = one length-256 sequence (Section 4), for
// the computed codes of Algorithms 1-3 (L = 16, 16 x 16 blocks) and the lookup-only code of
// the appendix (L = 14, 32 x 8 blocks; the text below says 16 and 1024, read L and 2^L / 64).
//
// The recursion.  All 2^kV successors of a state share the state's low L - kV bits as their
// top bits, their "prefix" hi = y >> kV, so the value function of a step is
//     val_t[y] = best_t[y >> kV] + err_t[y],
//     best_{t+1}[hi] = min over p < 2^kV of val_t[p 2^(L-kV) + hi],      best_0 = 0,
// and only `best`, 2^(L-kV) binary32 numbers, passes from one step to the next.
//
// Forward kernel.  One workgroup of 1024 threads owns one sequence; `best` lives in LDS, twice
// (read one copy, write the other, one barrier per step; 2 x 64 KiB at kV = 2).  A thread owns
// 2^(6-kV) neighbouring prefixes and their 64 predecessor states, whose code values sit in its
// registers: it reads the few `best` entries those states hang on, forms the 64 values and
// takes the minima, per state one subtraction, one fused multiply-add and half a minimum.
// No arg-minimum is formed: a back-pointer costs more instructions per prefix (3 compares, 3
// adds-with-carry and a third minimum at kV = 2) than everything else the prefix needs.
// Instead `best` itself is written to HBM every J steps, and the walk back recomputes what it
// needs: of the states J steps before a known state only 2^(kV J) can lead to it, a tree that
// one wave evaluates from the stored `best` in a few hundred instructions.
//   What bounds it is the issue of those instructions: 2.8 cycles for the subtraction and 2.9 for the
// fused multiply-add, 4.35 for a minimum are 2020 cycles a step at kV = 2 and V = 1.  Measured (busy cycles of the
// counters over the steps of a pass): 2165 to 2190 in the 255 of the first pass and 2190 to 2210 in the 245 of the second, whether
// half of the CUs are at work or all of them; but the clock is 2.3 GHz with 128 sequences and 1.9 to 2.15 with thousands, so that a
// step takes 0.95 us there and 1.02 to 1.15 here.
// 2048 x 2048, 2-bit 3INST: 69.7 ms with back-pointers, 36.1 now (37.5 on another card).  (The subtractions on the matrix cores, one
// v_mfma_f32_16x16x1 for 16 registers, bit for bit the same: 34.7 ms, but BlockLDLQ's 128
// sequences 48.4 -> 48.8: its 32 cycles are not hidden behind other waves' vector instructions.)
//
// Walk back.  One wave per sequence and J steps at a time: it reads the 2^(kV J) stored minima
// below the current state (one contiguous run: `best` is stored with the state's low bits, which
// are fixed there, as the major index), and repeats the recursion level by level with the
// arguments kept; ties go to the lowest predecessor.  The same operations in the same order
// give the same bits as the forward kernel, so the walk is the one its minima imply.
// Where there are few sequences four waves share a tree, one p_1 (or a quarter of them) each, and
// compare their roots: BlockLDLQ of 2048 x 1024, 128 sequences at a time, 48.4 -> 46.0 ms; and with at most one
// sequence per CU, at kV = 3 three, one kernel does all of Algorithm 4 (viterbi_few_kernel; not at kV = 6 and 8, HYB with 3 and 4
// bits, and not for the lookup-only code, which it has no trees for: they take several launches whatever their number).
// The copies go through the caches as they come: written and read with the non-temporal hint the same
// case takes 46.4 ms, and thousands of sequences the same.
// Algorithm 4 is forward / walk to the middle / constrained forward / full walk; what the constraint already says about the
// ends of the second pass is not searched for (VitGeo::FORCED).
//
// Arithmetic (fixed, so that a CPU reference can repeat every decision): binary32,
//   e_j = C[y][j] - s[V t + j];
//   V = 1: value = fma(e_0, e_0, min)            (the first step: e_0 e_0)
//   V = 2: value = min + fma(e_1, e_1, e_0 e_0)
// with exactly these roundings (the file is compiled without contraction).
// Minima take the lowest predecessor on ties, the final state the lowest state.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "qtip_device.h"
#include "qtip_internal.h"

#pragma clang fp contract(off)

namespace qtip {
namespace {

constexpr int VT_T = 256;    // sequence length (one T_x x T_y block)
constexpr int VT_REGS = 64;  // states per thread

// LB = L, the number of state bits: 16 (NT = 1024 threads per sequence) for the codes of
// Algorithms 1-3, 14 (NT = 256) for the lookup-only code.
template <int KV, int V, int LB>
struct VitGeo {
    static constexpr int G = VT_T / V;              // steps
    static constexpr int NT = (1 << LB) / VT_REGS;  // threads per sequence
    static constexpr int OV = LB - KV;              // bits two consecutive states share
    static constexpr int NP = 1 << OV;              // prefixes = minima per step
    static constexpr int NC = 1 << KV;              // predecessors per prefix
    static constexpr bool WHOLE = NC <= VT_REGS;    // a prefix's predecessors fit one thread
    static constexpr int NB = WHOLE ? VT_REGS / NC : 1;  // prefixes per thread
    // Steps between two stored copies of `best`.  The tree of a walk has 2^(kV J) leaves, and
    // storing costs 4 NP / J bytes per step: 13 KiB at kV = 2 (J = 5, 16 leaves per lane), 3.4
    // TB/s over the chip, is as dense as pays; denser (J = 4) the stores bound the kernel.
    static constexpr int J = KV == 2 ? (LB == 16 ? 5 : 4) : KV == 3 ? 3 : KV == 4 ? 2 : 1;
    static constexpr int NLEAF = 1 << (KV * J);
    static constexpr int LOWB = LB - KV * (J + 1);  // low prefix bits, fixed within one tree
    static constexpr int NSEG = (G - 1 + J - 1) / J;  // trees of a walk from G - 1 to 0
    // Up to this many sequences a walk has four waves: a tree is a serial chain (leaves from memory,
    // about 1 us, then J levels), and four waves have a quarter of the leaves each.  Not at J < 3, where a
    // wave's share of the chain is no shorter than the exchange at the root (HYB k = 2, 256 tiles: 1009 us
    // with one wave, 1023 with four); and not where all SIMDs have walks enough to hide the chains
    // (3INST k = 2, us with one wave | four: 256 tiles 888 | 840, 1024 2555 | 2531, 2048 4634 | 4691;
    // lookup-only code, whose forward pass is a quarter as long: 256 456 | 431, 512 515 | 510, 1024 767 | 824).
    static constexpr int FEW = J < 3 ? 0 : LB == 16 ? 1024 : 512;
    static constexpr int MID = G / 2 - 1;           // the step the first walk goes down to
    static constexpr int NSEG_MID = (G - 1 - MID + J - 1) / J;
    static_assert(LOWB >= 0, "a tree's leaves are distinct states");
    // Algorithm 4's second pass knows the states around its ends: the first state's top bits are the overlap, so that one walk
    // leads to each of the 4096 states that the first T0 steps can reach, and `best` of step T0 is made at once; the last
    // state's low bits are the overlap too, so that the 2^kV states it may be are level 1 of a tree below a step G that only has
    // that prefix.  The pass takes steps T0 .. G - J - 1, and its walk trees down from G, the last one to step T0.  (Not at kV = 6
    // and 8, where that is one step, and not for the lookup-only code; and not for a sequence that is unbounded(), see there.)
    static constexpr bool FORCED = KV <= 4 && LB == 16;
    static constexpr int T0 = FORCED ? 12 / KV : 0, END = FORCED ? G : G - 1;
    static constexpr int NSEG2 = FORCED ? (G - T0 + J - 1) / J : NSEG;  // trees of a whole walk
    static constexpr int LAST = G - 1 - (NSEG - 1) * J;                 // levels of the last one
    static constexpr int COPIES = NSEG - 1;  // of a whole walk
    static_assert(!FORCED || (KV * T0 == 12 && NSEG2 == COPIES && END - T0 - (NSEG2 - 1) * J == LAST),
                  "forced or not, as many copies, and as many levels of the last tree");
    // LDS place of best[hi] (floats).  kV = 2 and 3: a thread's 16 or 8 minima are one row; written
    // as they stand, the 16-byte stores of neighbouring lanes would be a whole row apart and
    // land on two (four) of the eight 16-byte bank groups, so the row's pieces are rotated by an
    // amount that depends on the row, which spreads eight lanes over all eight groups here and
    // where the rows are read back.  kV = 6: the 64 entries that one wave reads are one row.
    __device__ static __forceinline__ int place(int hi) {
        if constexpr (KV == 2) return (hi & ~15) | ((((hi >> 2) + (hi >> 5)) & 3) << 2) | (hi & 3);
        else if constexpr (KV == 3) return (hi & ~7) | ((((hi >> 2) ^ (hi >> 5)) & 1) << 2) | (hi & 3);
        else if constexpr (KV == 6) return (hi & 15) * 68 + (hi >> 4);
        else if constexpr (KV == 8) return (hi >> 6) * 68 + (hi & 63);
        else return hi;
    }
    static constexpr int BEST_FLOATS = KV == 6 ? 16 * 68 : KV == 8 ? 4 * 68 : NP;
    // place of best[hi] in a stored copy
    __device__ static __forceinline__ uint32_t stored(uint32_t hi) {
        return ((hi & ((1u << LOWB) - 1u)) << (KV * J)) | (hi >> LOWB);
    }
    // the prefix at place i of a stored copy
    __device__ static __forceinline__ uint32_t prefix_at(uint32_t i) {
        return ((i & ((1u << (KV * J)) - 1u)) << LOWB) | (i >> (KV * J));
    }
};

// m = min(a, b) and min(a, b, c) as instructions: the builtins first "canonicalize" their
// operands, one extra instruction each, against signalling NaNs that cannot occur here.
__device__ __forceinline__ float min2(float a, float b) {
    float m;
    asm("v_min_f32 %0, %1, %2" : "=v"(m) : "v"(a), "v"(b));
    return m;
}
__device__ __forceinline__ float min3(float a, float b, float c) {
    float m;
    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(m) : "v"(a), "v"(b), "v"(c));
    return m;
}

// The code values of state y as a register: the binary32 value (V = 1), or the packed binary16
// pair with its signs applied (V = 2).
template <int CODE>
__device__ __forceinline__ uint32_t code_register(uint32_t y, const uint32_t *__restrict__ lut) {
    if constexpr (CODE == CODE_HYB) return as_u32(code_hyb(y, lut));
    else if constexpr (CODE == CODE_HYB2) return as_u32(code_hyb2(y, lut));
    else {
        half_t c;
        if constexpr (CODE == CODE_LUT) c = reinterpret_cast<const half_t *>(lut)[y];
        else if constexpr (CODE == CODE_HYB1) c = code_hyb1(y, reinterpret_cast<const uint16_t *>(lut));
        else c = CODE == CODE_3INST ? code_3inst(y) : code_1mad(y);
        return __builtin_bit_cast(uint32_t, (float)c);
    }
}
// val = value of a state with code register c on top of `best` b.  V = 2: the conversion to
// binary32 and the subtraction are one v_fma_mix_f32, (float)c * 1.0 - s: an exact product
// and one rounding.
template <int V>
__device__ __forceinline__ float state_value(uint32_t c, float s0, float s1, float b) {
    if constexpr (V == 2) {
        float e0, e1;
        asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(e0) : "v"(c), "v"(s0));
        asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(e1) : "v"(c), "v"(s1));
        return b + __builtin_fmaf(e1, e1, e0 * e0);
    } else {
        const float e = __builtin_bit_cast(float, c) - s0;
        return __builtin_fmaf(e, e, b);
    }
}

// Element u of the sequence of tile `tile`.  rotate = 1: rotated by T/2 (Algorithm 4's first call).
template <int CODE>
__device__ __forceinline__ float sequence_element(const float *__restrict__ W, int n, int tn, long tile, int u,
                                                  int rotate) {
    constexpr int LTY = code_log2_ty(CODE), TY = 1 << LTY, TX = VT_T >> LTY;  // the block is TX x TY
    const int I = (int)(tile / tn), J = (int)(tile % tn);
    const int s = rotate ? ((u + VT_T / 2) & (VT_T - 1)) : u;
    return W[(size_t)(TX * I + (s >> LTY)) * n + TY * J + (s & (TY - 1))];
}

// For prefixes whose predecessors a thread owns (kV <= 4): the entries of `best` (in LDS) that its states hang on, and the minima
// of a step from them.  Prefix i's predecessor p hangs on entry `under(i, p)`.
template <int KV> struct Hang {
    static constexpr int COUNT = KV == 2 ? 16 : 1 << KV;
    __host__ __device__ static constexpr int under(int i, int p) { return KV == 2 ? 4 * p + (i >> 2) : p; }
};
template <int KV, int V, int LB>
__device__ __forceinline__ void thread_reads(const float *__restrict__ in, int tid, float (&b)[Hang<KV>::COUNT]) {
    using Geo = VitGeo<KV, V, LB>;
    constexpr int BSTEP = Geo::OV - KV;
#pragma unroll
    for (int p = 0; p < Geo::NC; p++) {
        if constexpr (KV == 2) {
            const float4_t four = *reinterpret_cast<const float4_t *>(in + Geo::place((p << BSTEP) + 4 * tid));
#pragma unroll
            for (int a = 0; a < 4; a++) b[4 * p + a] = four[a];
        } else {
            b[p] = in[Geo::place((p << BSTEP) + (Geo::NB * tid >> KV))];
        }
    }
}
template <int KV, int V, int LB>
__device__ __forceinline__ void thread_minima(const float (&b)[Hang<KV>::COUNT], const uint32_t (&cr)[VT_REGS], float s0,
                                              float s1, float (&best)[VitGeo<KV, V, LB>::NB]) {
    constexpr int NC = VitGeo<KV, V, LB>::NC;
#pragma unroll
    for (int i = 0; i < VitGeo<KV, V, LB>::NB; i++) {
        auto value = [&](int p) { return state_value<V>(cr[i * NC + p], s0, s1, b[Hang<KV>::under(i, p)]); };
        if constexpr (KV == 2) {
            float v[NC];
#pragma unroll
            for (int p = 0; p < NC; p++) v[p] = value(p);
            best[i] = min3(min2(v[0], v[1]), v[2], v[3]);
        } else {
            float m = value(0);
#pragma unroll
            for (int p = 1; p + 1 < NC; p += 2) m = min3(m, value(p), value(p + 1));
            best[i] = min2(m, value(NC - 1));
        }
    }
}

// Whether a sequence's values might not all be finite: a sample beyond 2^59 or none at all, or a table entry that is not
// finite.  (Below that 256 squares of differences to code values, 65504 at most, stay below 2^127.)  Where all of
// them are finite, what the ends of the second pass are forced to is what a search finds: only walks from the forced first
// state have a finite value.  Where they are not, minima over infinite and undefined values decide, and the second pass
// searches over all states and steps.  `element` is the thread's of the sequence, if it has one; true for threads of the
// workgroup that see such a value.
template <int CODE> __device__ __forceinline__ bool unbounded(float element, int tid, const uint32_t *__restrict__ lut) {
    auto not_finite = [](uint32_t h) { return (h & 0x7C00u) == 0x7C00u; };
    bool is = tid < VT_T && !(__builtin_fabsf(element) <= 0x1p59f);
    if constexpr (CODE == CODE_HYB1) {
        if (tid < 1 << HYB1_Q) is |= not_finite(reinterpret_cast<const uint16_t *>(lut)[tid]);
    } else if constexpr (code_is_hyb(CODE)) {
        const uint32_t pair = tid < 1 << HYB_Q ? lut[tid] : 0u;
        is |= not_finite(pair) || not_finite(pair >> 16);
    }
    return is;
}
// Goes with a sequence's final state and overlap where its second pass has to be searched.
constexpr uint32_t SEARCHED = 0x80000000u;

// `best` of step T0 where the first state's top bits are O: entries ((O << 12) | 4 tid + i) mod NP, the others are infinite.  The
// one walk to each: minima over one finite value, in the order and with the roundings of the steps.
// (The second pass's 255 steps and the search for its last state are 245 steps at kV = 2, 242 or 243 in one launch: us, all steps and
// so, one card, 64 | 400 | 4096 sequences: 3INST k = 2 611 588 | 1256 1220 | 9235 9186, k = 3 638 620 | 1275 1243 | 8861 8707, k = 4
// 629 626 | 1313 1318 | 8245 8250, HYB k = 2 795 770 | 1512 1474 | 10634 10277, HYB1 k = 2 630 612 | 1380 1285 | 9784 9216.)
template <int KV, int V, int CODE, class Sample>
__device__ __forceinline__ float4_t forced_entries(uint32_t O, int tid, const uint32_t *__restrict__ lut, Sample sample) {
    using Geo = VitGeo<KV, V, 16>;
    constexpr int T0 = Geo::T0;
    auto state = [&](int j, uint32_t e) { return ((O << (KV * (j + 1))) | (e >> (KV * (T0 - 1 - j)))) & 0xFFFFu; };
    float v = 0.f;
#pragma unroll
    for (int j = 0; j < T0 - 1; j++)
        v = state_value<V>(code_register<CODE>(state(j, 4u * tid), lut), sample(j, 0), V == 2 ? sample(j, 1) : 0.f, v);
    float4_t best;
#pragma unroll
    for (int i = 0; i < 4; i++)
        best[i] = state_value<V>(code_register<CODE>(state(T0 - 1, 4u * tid + i), lut), sample(T0 - 1, 0),
                                 V == 2 ? sample(T0 - 1, 1) : 0.f, v);
    return best;
}
// Digit of step j < T0 of such a walk: the top kV bits of its state.
template <int KV> __device__ __forceinline__ uint32_t forced_digit(uint32_t O, int j) {
    return (O >> (16 - KV - KV * (j + 1))) & ((1u << KV) - 1u);
}

// Steps 0 (T0 where the ends are forced, see VitGeo) .. t_end - 1 of sequence tile0 + blockIdx.x, with `best` stored after every J steps
// counted from the last, G - 1 (copies c_lo .. c_hi - 1, copy c at step G - 1 - J (c + 1)), and, when
// t_end = G - 1, the best final state.  Where the ends are forced, copies are counted from G and the last one is of T0 (t_end is
// theirs: a pass that is searched all the same goes up to its own).  overlap != null: the first state's top L-kV bits and the
// last state's low L-kV bits are forced to overlap[slot] (Algorithm 4's second call).
// (four waves per SIMD, i.e. at most 128 registers, also where a workgroup is only four waves)
template <int KV, int V, int CODE>
__global__ __launch_bounds__((VitGeo<KV, V, code_state_bits(CODE)>::NT), 4) void viterbi_forward_kernel(
    const float *__restrict__ W, int n, int tn, long tile0, const uint32_t *__restrict__ lut, int rotate,
    const uint32_t *__restrict__ overlap, float *__restrict__ store, long slots, int c_lo, int c_hi, int t_end,
    uint32_t *__restrict__ final_state, float *__restrict__ final_value) {
    using Geo = VitGeo<KV, V, code_state_bits(CODE)>;
    constexpr int NP = Geo::NP, NC = Geo::NC, NB = Geo::NB, NT = Geo::NT, OV = Geo::OV, G = Geo::G, J = Geo::J;
    static_assert(code_is_hyb(CODE) == (V == 2), "V = 2 is the HYB code");
    static_assert(NT >= VT_T, "one thread per sequence element");
    __shared__ __attribute__((aligned(16))) float s_best[2][Geo::BEST_FLOATS];
    __shared__ __attribute__((aligned(16))) float s_seq[VT_T + 4];
    __shared__ float s_rv[NT / 64];
    __shared__ uint32_t s_ry[NT / 64], s_searched;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int slot = blockIdx.x;
    const float INF = __builtin_inff();
    const bool constrained = overlap != nullptr;
    const uint32_t given = constrained ? overlap[slot] : 0u, O = given & (uint32_t)(NP - 1);
    const bool forced = Geo::FORCED && constrained && !(given & SEARCHED);
    if (Geo::FORCED && constrained && !forced) t_end = c_lo == 0 ? G - 1 : G - 1 - J * (c_lo + 1);

    if constexpr (Geo::FORCED) {
        if (!constrained) {
            if (tid == 0) s_searched = 0u;
            __syncthreads();
        }
    }
    const float element = tid < VT_T ? sequence_element<CODE>(W, n, tn, tile0 + slot, tid, rotate) : 0.f;
    if (tid < VT_T) s_seq[tid] = element;
    if constexpr (Geo::FORCED) {
        if (!constrained && unbounded<CODE>(element, tid, lut)) s_searched = SEARCHED;
    }
    // (0 at step 0, but for a first state's top bits that are O; of step T0 all but the forced entries)
    for (int i = tid; i < NP; i += NT) s_best[0][Geo::place(i)] = constrained && (forced || (uint32_t)i != O) ? INF : 0.f;

    // register r of this thread is state (p, hi): WHOLE: p = r % NC, prefix NB tid + r / NC;
    // else (kV = 8) a quarter of a prefix's predecessors, p = 64 (lane / 16) + r
    const int my_hi = Geo::WHOLE ? NB * tid : 16 * wave + (lane & 15);
    auto state_of = [&](int r) -> uint32_t {
        if constexpr (Geo::WHOLE) return ((uint32_t)(r % NC) << OV) | (uint32_t)(my_hi + r / NC);
        else return ((uint32_t)(64 * (lane >> 4) + r) << OV) | (uint32_t)my_hi;
    };
    uint32_t cr[VT_REGS];
#pragma unroll
    for (int r = 0; r < VT_REGS; r++) {
        cr[r] = code_register<CODE>(state_of(r), lut);
        // (opaque to the compiler from here on, or it recomputes the codes inside the loop)
        asm volatile("" : "+v"(cr[r]));
    }
    __syncthreads();

    float *store_base = store + (size_t)slot * slots * NP;
    int until = (G - 1) % J;  // steps to the next one that is a multiple of J from the last
    if (until == 0) until = J;
    int c_now = (G - 1 - until) / J - 1;  // the copy that belongs to it
    int t = 0;
    if constexpr (Geo::FORCED) {
        if (forced) {
            int tid = threadIdx.x;
            asm volatile("" : "+v"(tid));  // (nothing that is made with it here is worth a register later)
            const float4_t first = forced_entries<KV, V, CODE>(O, tid, lut, [&](int u, int e) { return s_seq[V * u + e]; });
            *reinterpret_cast<float4_t *>(s_best[0] + Geo::place((int)(((O << 12) | (4u * tid)) & (uint32_t)(NP - 1)))) = first;
            __syncthreads();
            // (a loop of few registers, which the code values have, and of neighbouring stores: in the order of the prefixes
            // 256 workgroups of kV = 4 took 12 us for it)
            if (c_hi == Geo::NSEG2) {
                float *const dst = store_base + (size_t)(Geo::NSEG2 - 1 - c_lo) * NP;
#pragma unroll 1
                for (uint32_t i = tid; i < (uint32_t)NP; i += NT) dst[i] = s_best[0][Geo::place((int)Geo::prefix_at(i))];
            }
            t = Geo::T0;
            until = Geo::LAST;
            c_now = Geo::NSEG2 - 2;
        }
    }
    float s0 = s_seq[V * t], s1 = V == 2 ? s_seq[V * t + 1] : 0.f;

    auto step = [&](const float *__restrict__ in, float *__restrict__ out, int t) {
        // (the next step's samples are read ahead of the barrier)
        const float n0 = s_seq[V * (t + 1)], n1 = V == 2 ? s_seq[V * (t + 1) + 1] : 0.f;
        float best[NB];
        if constexpr (KV <= 4) {
            float b[Hang<KV>::COUNT];
            thread_reads<KV, V, code_state_bits(CODE)>(in, tid, b);
            thread_minima<KV, V, code_state_bits(CODE)>(b, cr, s0, s1, best);
        } else {
            // the 64 entries are one row of 68 floats, the same for the whole wave (kV = 6) or for
            // sixteen lanes (kV = 8)
            const float *row = in + 68 * (KV == 6 ? my_hi >> KV : lane >> 4);
            float m = INF;
#pragma unroll
            for (int p = 0; p < VT_REGS; p += 4) {
                const float4_t b = *reinterpret_cast<const float4_t *>(row + p);
                m = min3(m, state_value<V>(cr[p], s0, s1, b[0]), state_value<V>(cr[p + 1], s0, s1, b[1]));
                m = min3(m, state_value<V>(cr[p + 2], s0, s1, b[2]), state_value<V>(cr[p + 3], s0, s1, b[3]));
            }
            if constexpr (!Geo::WHOLE) {
                m = min2(m, __shfl_xor(m, 16, 64));
                m = min2(m, __shfl_xor(m, 32, 64));
            }
            best[0] = m;
        }
        if constexpr (NB >= 4) {
#pragma unroll
            for (int i = 0; i < NB; i += 4)
                *reinterpret_cast<float4_t *>(out + Geo::place(my_hi + i)) =
                    float4_t{best[i], best[i + 1], best[i + 2], best[i + 3]};
        } else if (Geo::WHOLE || lane < 16) {
            out[Geo::place(my_hi)] = best[0];
        }
        if (--until == 0) {  // `best` after this step is copy c_now
            until = J;
            if (c_now >= c_lo && c_now < c_hi && (Geo::WHOLE || lane < 16)) {
                float *dst = store_base + (size_t)(c_now - c_lo) * NP;
                // (where a thread's prefixes differ in the low bits alone, its places are a uniform distance apart: one
                // address and scalar additions; but the 3-bit V = 1 hash code's kernel, which is out of registers, would
                // spill 36 of them in place of 28: 4096 sequences 9.43 -> 9.57 ms)
                constexpr bool EVEN = NB <= 1 << Geo::LOWB && !(KV == 3 && CODE == CODE_HYB1);
#pragma unroll
                for (int i = 0; i < NB; i++) {
                    if constexpr (EVEN) (dst + (i << (KV * J)))[Geo::stored((uint32_t)my_hi)] = best[i];
                    else dst[Geo::stored((uint32_t)(my_hi + i))] = best[i];
                }
            }
            c_now--;
        }
        s0 = n0;
        s1 = n1;
        __syncthreads();
    };
    for (; t + 1 < t_end; t += 2) {
        step(s_best[0], s_best[1], t);
        step(s_best[1], s_best[0], t + 1);
    }
    if (t < t_end) step(s_best[0], s_best[1], t);
    if (t_end < G - 1) return;

    // the best allowed final state, lowest state on ties
    const float *in = s_best[(G - 1) & 1];
    float bv = INF;
    uint32_t by = 0xFFFFFFFFu;
    auto take_better = [&](bool ok, float v, uint32_t y) {
        const bool take = ok & ((v < bv) | ((v == bv) & (y < by)));
        bv = take ? v : bv;
        by = take ? y : by;
    };
#pragma unroll
    for (int r = 0; r < VT_REGS; r++) {
        const uint32_t y = state_of(r);
        take_better(!constrained | ((y & (uint32_t)(NP - 1)) == O),
                    state_value<V>(cr[r], s0, s1, in[Geo::place((int)(y >> KV))]), y);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) take_better(true, __shfl_xor(bv, off, 64), __shfl_xor(by, off, 64));
    if (lane == 0) {
        s_rv[wave] = bv;
        s_ry[wave] = by;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < NT / 64; w++) take_better(true, s_rv[w], s_ry[w]);
        final_state[slot] = Geo::FORCED && !constrained ? by | s_searched : by;
        final_value[slot] = bv;
    }
}

// ------------------------------------------------------------------- walk back

// x from the lane whose index differs in bit BIT alone, without LDS.
template <int BIT>
__device__ __forceinline__ uint32_t other_lane(uint32_t x) {
    if constexpr (BIT == 0) return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true);        // quad_perm [1, 0, 3, 2]
    else if constexpr (BIT == 1) return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true);   // quad_perm [2, 3, 0, 1]
    else if constexpr (BIT == 2)  // lane ^ 7 (row_half_mirror), then ^ 3 (quad_perm [3, 2, 1, 0])
        return __builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, true), 0x1B, 0xF, 0xF, true);
    else if constexpr (BIT == 3) return __builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, true);  // row_ror:8
    else if constexpr (BIT == 4) {  // rows 0 and 2 of the second result are rows 1 and 3 of x, and the other way round
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return threadIdx.x & 16 ? r[0] : r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return threadIdx.x & 32 ? r[0] : r[1];
    }
}

// What the waves of a sequence tell each other at the root of a tree: value and leaf of the best walk
// of each, twice, so that one barrier per tree is enough.
struct WalkRoot {
    float value[2][4];
    uint32_t leaf[2][4];
};

// One tree of JJ levels below state y at step t, whose leaves are the states of step t - JJ.
// Leaf l = (p_JJ ... p_1), digit p_j being the top kV bits of the state j steps back, is state
// (l << (L - kV JJ)) | (y >> kV JJ); the low WB bits of l are the wave, the next six the lane, the
// others a register.  Level j takes the minimum over p_j and moves one step forward; the wave's bits, of
// p_1, come last, at the root.  On return digit[j] = p_j of the best walk (the same in all lanes).
template <int KV, int V, int CODE, int JJ, int WB>
struct WalkTree {
    using Geo = VitGeo<KV, V, code_state_bits(CODE)>;
    static constexpr int LB = code_state_bits(CODE);
    static constexpr int LREG = WB + 6;  // the first bit of a leaf that is a register's
    static constexpr int regs(int bits) { return bits > LREG ? 1 << (bits - LREG) : 1; }
    static_assert(WB <= KV, "the wave is a part of the last digit");

    uint32_t y;
    int t, lane, wave;
    const uint32_t *lut;
    const float *seq;  // LDS
    WalkRoot *root;    // LDS
    float best;        // of the wave, at the root; of the tree when run() is through
    uint32_t args[JJ + 1];  // args[j]: kV bits per register of level j - 1

    __device__ __forceinline__ uint32_t node_state(int j, int m) const {  // level j, register m
        const uint32_t own = (uint32_t)(m << LREG) | (uint32_t)(lane << WB) | (uint32_t)wave;
        const uint32_t l = KV * j >= LREG ? own : own & ((1u << (KV * j)) - 1u);
        return ((l << (LB - KV * j)) | (y >> (KV * j))) & ((1u << LB) - 1u);
    }
    __device__ __forceinline__ float node_value(int j, int m, float b) const {
        const int u = V * (t - j);
        return state_value<V>(code_register<CODE>(node_state(j, m), lut), seq[u], V == 2 ? seq[u + 1] : 0.f, b);
    }

    template <int j>
    __device__ __forceinline__ void reduce(float (&v)[regs(KV * JJ)]) {
        constexpr int M = regs(KV * j), M1 = regs(KV * (j - 1)), A = M / M1;
        // digit j: its top bits tell registers apart, the next ones, if any, are lane bits, and the low
        // ones of digit 1 the wave
        constexpr int WAVE = j == 1 ? WB : 0;
        constexpr int LANE_LO = KV * (j - 1) + WAVE - WB, LANE_HI = (KV * j < LREG ? KV * j : LREG) - WB;
        constexpr int LBITS = LANE_HI > LANE_LO ? LANE_HI - LANE_LO : 0;
        const uint32_t mine = ((LBITS ? ((uint32_t)lane >> LANE_LO) & ((1u << LBITS) - 1u) : 0u) << WAVE) |
                              (WAVE ? (uint32_t)wave : 0u);
        uint32_t packed = 0;
#pragma unroll
        for (int m = 0; m < M1; m++) {
            float bv = v[m];
            uint32_t bp = mine;
#pragma unroll
            for (int a = 1; a < A; a++) {
                const bool lt = v[a * M1 + m] < bv;
                bv = lt ? v[a * M1 + m] : bv;
                bp = lt ? ((uint32_t)a << (LBITS + WAVE)) | mine : bp;
            }
            auto meet = [&](auto bit) {
                constexpr int BIT = decltype(bit)::value;
                if constexpr (BIT < LBITS) {
                    const float ov = __builtin_bit_cast(float, other_lane<LANE_LO + BIT>(__builtin_bit_cast(uint32_t, bv)));
                    const uint32_t op = other_lane<LANE_LO + BIT>(bp);
                    const bool take = ov < bv || (ov == bv && op < bp);
                    bv = take ? ov : bv;
                    bp = take ? op : bp;
                }
            };
            meet(std::integral_constant<int, 0>{});
            meet(std::integral_constant<int, 1>{});
            meet(std::integral_constant<int, 2>{});
            meet(std::integral_constant<int, 3>{});
            meet(std::integral_constant<int, 4>{});
            meet(std::integral_constant<int, 5>{});
            packed |= bp << (m * KV);
            if constexpr (j > 1) v[m] = node_value(j - 1, m, bv);
            else best = bv;
        }
        args[j] = packed;
        if constexpr (j > 1) reduce<j - 1>(v);
    }

    // stored: best at step t - JJ, or null for step 0 (0, or INF off the forced prefix)
    // turn: which of root's two places
    __device__ __forceinline__ void run(const float *__restrict__ stored, bool constrained, uint32_t O, int turn,
                                        uint32_t (&digit)[JJ + 1]) {
        constexpr int M = regs(KV * JJ);
        float v[M];
#pragma unroll
        for (int m = 0; m < M; m++) {
            const uint32_t hi = node_state(JJ, m) >> KV;
            v[m] = stored ? stored[Geo::stored(hi)]
                          : (constrained && hi != O) ? __builtin_inff() : 0.f;
        }
#pragma unroll
        for (int m = 0; m < M; m++) v[m] = node_value(JJ, m, v[m]);
        reduce<JJ>(v);
        uint32_t l = 0;  // (p_{j-1} ... p_1)
#pragma unroll
        for (int j = 1; j <= JJ; j++) {
            const uint32_t word = __builtin_amdgcn_readlane(args[j], (l >> WB) & 63u);
            const uint32_t m = KV * (j - 1) > LREG ? l >> LREG : 0u;
            digit[j] = (word >> (m * KV)) & ((1u << KV) - 1u);
            l |= digit[j] << (KV * (j - 1));
        }
        if constexpr (WB > 0) {
            if (lane == 0) {
                root->value[turn][wave] = best;
                root->leaf[turn][wave] = l;
            }
            __syncthreads();
            float bv = root->value[turn][0];
            l = root->leaf[turn][0];
#pragma unroll
            for (int w = 1; w < 1 << WB; w++) {
                const float ov = root->value[turn][w];
                const uint32_t ol = root->leaf[turn][w];
                const bool take = ov < bv || (ov == bv && (ol & ((1u << KV) - 1u)) < (l & ((1u << KV) - 1u)));
                bv = take ? ov : bv;
                l = take ? ol : l;
            }
            l = __builtin_amdgcn_readfirstlane(l);
            best = bv;
#pragma unroll
            for (int j = 1; j <= JJ; j++) digit[j] = (l >> (KV * (j - 1))) & ((1u << KV) - 1u);
        }
    }
};

// One wave per sequence, or four (WB = 2) where there are few.  pass 1: from the final state down to step G/2 - 1, whose low L-kV bits are
// the overlap of Algorithm 4.  pass 2: the whole walk; step t contributes the top kV bits of its
// state as stream bits t kV .. (t+1) kV - 1 (first bit = most significant bit of word 0).  The
// trees c_lo .. c_hi - 1 of the walk are done; where the workspace holds too few copies of `best`
// for the whole walk, the state it got to waits in final_state and the next launch adds its bits.
template <int KV, int V, int CODE, int WB>
__global__ __launch_bounds__(256) void viterbi_walk_kernel(
    const float *__restrict__ W, int n, int tn, long tile0, const uint32_t *__restrict__ lut, int pass,
    const float *__restrict__ store, long slots, int c_lo, int c_hi, uint32_t *__restrict__ final_state,
    const float *__restrict__ final_value, int count, uint32_t *__restrict__ overlap, uint32_t *__restrict__ codes,
    float *__restrict__ tile_err) {
    using Geo = VitGeo<KV, V, code_state_bits(CODE)>;
    constexpr int OV = Geo::OV, NP = Geo::NP, G = Geo::G, J = Geo::J, LB = code_state_bits(CODE);
    constexpr int NWORDS = KV * G / 32;
    __shared__ float s_seq[4][VT_T];
    __shared__ uint32_t s_sym[4][VT_T / 4];  // one byte per step
    __shared__ WalkRoot s_root;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int slot = WB ? blockIdx.x : blockIdx.x * 4 + wave;
    const bool first = WB == 0 || wave == 0;  // (all waves of a sequence know all of its walk)
    if (slot >= count) return;
    float *const seq = s_seq[wave];
    uint8_t *const sym = reinterpret_cast<uint8_t *>(s_sym[wave]);
#pragma unroll
    for (int i = 0; i < VT_T / 64; i++)
        seq[64 * i + lane] = sequence_element<CODE>(W, n, tn, tile0 + slot, 64 * i + lane, pass == 1);
    const bool constrained = pass == 2;
    const uint32_t given = constrained ? overlap[slot] : 0u, O = given & (uint32_t)(NP - 1);
    // (the wave's own LDS: its operations complete in order, the fences keep the compiler in line)
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    const bool forced = Geo::FORCED && constrained && !(given & SEARCHED);
    const int end = forced ? Geo::END : G - 1, nseg = forced ? Geo::NSEG2 : Geo::NSEG;
    // (the last tree of a walk that is not forced starts at step 0 and needs no copy)
    if (Geo::FORCED && constrained && !forced && c_hi == Geo::COPIES) c_hi = Geo::NSEG;
    // (a forced walk begins at a step G whose state has the overlap for a prefix)
    const uint32_t from = __builtin_amdgcn_readfirstlane(forced && c_lo == 0 ? O << KV : final_state[slot]);
    const uint32_t searched = constrained ? 0u : from & SEARCHED;
    uint32_t y = from & ((1u << LB) - 1u);
    s_sym[wave][lane] = 0;
    wave_sync();
    if (!forced && c_lo == 0 && lane == 0) sym[G - 1] = (uint8_t)(y >> OV);
    if (forced && c_hi == nseg && lane < Geo::T0) sym[lane] = (uint8_t)forced_digit<KV>(O, lane);
    const float *my_store = store + (size_t)slot * slots * NP;
    auto tree = [&](auto jj, int c) {
        constexpr int JJ = decltype(jj)::value;
        const int t = end - J * c;
        WalkTree<KV, V, CODE, JJ, WB> w;
        w.y = y;
        w.t = t;
        w.lane = lane;
        w.wave = WB ? wave : 0;
        w.root = &s_root;
        w.lut = lut;
        w.seq = seq;
        uint32_t digit[JJ + 1];
        w.run(t > JJ ? my_store + (size_t)(c - c_lo) * NP : nullptr, constrained, O, c & 1, digit);
        if (forced && first && c == 0 && tile_err && lane == 0) tile_err[tile0 + slot] = w.best;
#pragma unroll
        for (int j = 1; j <= JJ; j++) {
            y = (digit[j] << OV) | (y >> KV);
            if (lane == 0) sym[t - j] = (uint8_t)digit[j];
            if (first && pass == 1 && t - j == Geo::MID && lane == 0) overlap[slot] = (y & (uint32_t)(NP - 1)) | searched;
        }
    };
    for (int c = c_lo; c < c_hi; c++) {
        if (c == nseg - 1) tree(std::integral_constant<int, Geo::LAST>{}, c);  // (never the first pass's)
        else tree(std::integral_constant<int, J>{}, c);
    }
    if (!first || (pass == 1 && c_hi >= Geo::NSEG_MID)) return;
    wave_sync();
    if (c_hi < nseg && lane == 0) final_state[slot] = y | searched;
    if (pass == 1) return;
    if (lane < NWORDS) {
        uint32_t *const out = codes + (size_t)(tile0 + slot) * NWORDS + lane;
        uint32_t word = 0;
#pragma unroll
        for (int b = 0; b < 32; b++) {
            const int pos = 32 * lane + b;
            word = (word << 1) | ((sym[pos / KV] >> (KV - 1 - pos % KV)) & 1u);
        }
        *out = c_lo == 0 ? word : *out | word;
    }
    if (!forced && tile_err && lane == 0) tile_err[tile0 + slot] = final_value[slot];
}

// --------------------------------------------------- few sequences: all of Algorithm 4 in one workgroup

// With at most a few sequences per CU both the walks, serial chains of trees, and the parts of forward passes that are
// repeated where the workspace has no room for every copy are a large part of the time.  Here a workgroup keeps its code
// values in registers through both passes, and all of it walks back: each thread has its part of the next copy of `best` under
// way while a segment is walked; a copy is taken F steps forward by the same code as in the forward pass, and the last T steps
// of a segment are a tree of 4096 leaves, T levels: a thread per node of level T, then one wave.  F is what the number of
// copies asks for: `nseg` segments of T + F steps, lengths differing by one at most.
// The last forward step of a segment is only taken for the prefixes that the tree hangs on, a few of each thread; with F = 0
// level T takes entries and codes from the registers they arrive in.
//   What bounds it is still the issue of the forward steps: 255 and 242 of 2043 cycles (kV = 2, V = 1), 441 of 590 to 615 us.
// (Several launches and this one are compared where the launcher chooses; BlockLDLQ of 2048 x 256 11.44 | 10.01 ms, of 3-bit
// 1024 x 256 15.94 | 10.34.  With every copy through LDS and all of a tree's codes formed anew, 128 sequences, against 635,
// 641, 635 and 800 us on that card: 3INST k = 2 to 4 671, 693, 648, HYB 821.)
template <int KV, int V> struct FewGeo : VitGeo<KV, V, 16> {
    static constexpr int T = KV == 2 ? 6 : KV == 3 ? 4 : 3;    // levels of a tree
    static constexpr int NODES = 1 << (KV * (T - 1));          // of level T - 1
    static constexpr int FIXED = 4 - KV;                       // low bits that the prefixes of a tree's leaves share
    static constexpr int ARRAYS = KV == 3 ? 4 : 2;             // room for `best` of consecutive steps
    static constexpr int LONGEST = T + ARRAYS;                 // segment
    static constexpr int D1 = VitGeo<KV, V, 16>::G - 1 - VitGeo<KV, V, 16>::MID,
                         D2 = VitGeo<KV, V, 16>::G - VitGeo<KV, V, 16>::T0, D2_SEARCHED = VitGeo<KV, V, 16>::G - 1;  // steps walked
    static_assert(16 - KV * T == 4 && NODES <= 1024, "4096 leaves");
    static_assert(D1 > LONGEST, "two segments at least, so one copy");
    static constexpr bool fits(int d, int nseg) { return nseg > 0 && (d + nseg - 1) / nseg <= LONGEST; }
};

// f(integral_constant) of the one of 0 .. COUNT - 1 that the wave-uniform `which` is.
template <int COUNT, int FIRST = 0, class F>
__device__ __forceinline__ void one_of(uint32_t which, F f) {
    if constexpr (COUNT == 1) f(std::integral_constant<int, FIRST>{});
    else if (which & (uint32_t)(COUNT / 2)) one_of<COUNT / 2, FIRST + COUNT / 2>(which, f);
    else one_of<COUNT / 2, FIRST>(which, f);
}

template <int KV, int V, int CODE>
__global__ __launch_bounds__(1024, 4) void viterbi_few_kernel(const float *__restrict__ W, int n, int tn,
                                                              const uint32_t *__restrict__ lut, float *__restrict__ store,
                                                              long slots, int nseg1, int nseg2, uint32_t *__restrict__ codes,
                                                              float *__restrict__ tile_err) {
    using Geo = FewGeo<KV, V>;
    constexpr int NP = Geo::NP, NC = Geo::NC, NB = Geo::NB, OV = Geo::OV, G = Geo::G, T = Geo::T, NODES = Geo::NODES;
    constexpr int NWORDS = KV * G / 32, LB = 16, COUNT = Hang<KV>::COUNT, AHEAD = KV == 4 ? NB : COUNT;
    constexpr bool CODES_KEPT = KV < 4 || CODE == CODE_HYB1 || V == 2;  // level T takes its leaves' codes from registers
    static_assert(Geo::NT == 1024 && Geo::BEST_FLOATS == NP && NB % 4 == 0, "kV = 2 to 4");
    __shared__ __attribute__((aligned(16))) float s_best[Geo::ARRAYS][NP];
    __shared__ __attribute__((aligned(16))) float s_leaf[4096];  // `best` under a tree's leaves
    __shared__ __attribute__((aligned(16))) uint2 s_node[NODES];
    __shared__ uint2 s_four[KV == 2 ? 256 : 1];  // nodes of level 4
    __shared__ float s_seq[VT_T];
    __shared__ uint32_t s_sym[VT_T / 4];  // one byte per step
    __shared__ float s_rv[16];
    __shared__ uint32_t s_ry[16], s_state, s_searched;
    int tid = threadIdx.x, my_hi = NB * tid;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), slot = blockIdx.x;
    const float INF = __builtin_inff();
    uint8_t *const sym = reinterpret_cast<uint8_t *>(s_sym);
    float *const my_store = store + (size_t)slot * slots * NP;

    if (tid == 0) s_searched = 0u;
    __syncthreads();
    {
        const float element = tid < VT_T ? sequence_element<CODE>(W, n, tn, slot, tid, 0) : 0.f;
        if (tid < VT_T) s_seq[tid] = element;
        if (unbounded<CODE>(element, tid, lut)) s_searched = SEARCHED;
    }
    if (tid < VT_T / 4) s_sym[tid] = 0;
    uint32_t cr[VT_REGS];
#pragma unroll
    for (int r = 0; r < VT_REGS; r++) {
        cr[r] = code_register<CODE>(((uint32_t)(r % NC) << OV) | (uint32_t)(my_hi + r / NC), lut);
        asm volatile("" : "+v"(cr[r]));  // (as in the forward kernel)
    }

    uint32_t O = 0;
    for (int pass = 1; pass <= 2; pass++) {
        // (the second pass's ends are forced, see VitGeo: it begins at T0, and its walk at G, whose first segment's `best` is
        // where the forward pass stops and needs no copy)
        const bool constrained = pass == 2;
        const bool forced = constrained && !__builtin_amdgcn_readfirstlane(s_searched);
        const int rotate = constrained ? 0 : VT_T / 2, begin = forced ? Geo::T0 : 0, end = forced ? G : G - 1;
        const int nseg = !constrained ? nseg1 : forced ? nseg2 : min((int)slots + 1, Geo::D2_SEARCHED / T);
        const int D = !constrained ? Geo::D1 : forced ? Geo::D2 : Geo::D2_SEARCHED;
        const int uncopied = forced, last_copy = nseg - 1 - (constrained && !forced);  // (searched: the last segment starts at step 0)
        const int base = D / nseg, longer = D % nseg;
        auto sample = [&](int t, int e) { return s_seq[(V * t + e + rotate) & (VT_T - 1)]; };
        // the step that copy c, under segment c from the end, belongs to
        auto step_of = [&](int c) { return end - (c + 1) * base - min(c + 1, longer); };
        auto put = [&](float *to, const float *best) {
#pragma unroll
            for (int i = 0; i < NB; i += 4)
                *reinterpret_cast<float4_t *>(to + Geo::place(my_hi + i)) =
                    float4_t{best[i], best[i + 1], best[i + 2], best[i + 3]};
        };
        // (entry `hi` of step 0)
        auto first = [&](int hi) { return constrained && (uint32_t)hi != O ? INF : 0.f; };
        {
            float best[NB];
#pragma unroll
            for (int i = 0; i < NB; i++) best[i] = forced ? INF : first(my_hi + i);
            put(s_best[0], best);
        }
        __syncthreads();
        int c_now = last_copy, t_next = step_of(c_now);
        auto copy_at = [&](int c) { return my_store + (size_t)(c - uncopied) * NP; };
        auto next_copy = [&] {
            c_now--;
            t_next = c_now >= uncopied ? step_of(c_now) : -1;
        };
        auto store_copy = [&](const float *best) {
            float4_t *const to = reinterpret_cast<float4_t *>(copy_at(c_now));
#pragma unroll
            for (int i = 0; i < NB; i += 4)
                to[(uint32_t)(NB / 4 * tid + i / 4)] = float4_t{best[i], best[i + 1], best[i + 2], best[i + 3]};
            next_copy();
        };
        if (forced) {
            const float4_t first = forced_entries<KV, V, CODE>(O, tid, lut, sample);
            *reinterpret_cast<float4_t *>(s_best[0] + Geo::place((int)(((O << 12) | (4u * tid)) & (uint32_t)(NP - 1)))) = first;
            if (tid < Geo::T0) sym[tid] = (uint8_t)forced_digit<KV>(O, tid);
            __syncthreads();
            if constexpr (KV > 2) {
                float best[NB];
#pragma unroll
                for (int i = 0; i < NB; i++) best[i] = s_best[0][Geo::place(my_hi + i)];
                store_copy(best);
            }
        }
        float s0 = sample(begin, 0), s1 = V == 2 ? sample(begin, 1) : 0.f;
        auto step = [&](const float *in, float *out, int t) {
            // (the next step's samples are read ahead of the barrier)
            const float n0 = sample(t + 1, 0), n1 = V == 2 ? sample(t + 1, 1) : 0.f;
            float b[COUNT], best[NB];
            thread_reads<KV, V, LB>(in, tid, b);
            // A copy of step t_next is stored as it will be read, coalesced both times.
            if constexpr (KV == 2) {
                if (t == t_next) {
                    float4_t *const to = reinterpret_cast<float4_t *>(copy_at(c_now));
#pragma unroll
                    for (int p = 0; p < NC; p++)
                        (to + 1024 * p)[(uint32_t)tid] = float4_t{b[4 * p], b[4 * p + 1], b[4 * p + 2], b[4 * p + 3]};
                    next_copy();
                }
            }
            thread_minima<KV, V, LB>(b, cr, s0, s1, best);
            s0 = n0;
            s1 = n1;
            put(out, best);
            if constexpr (KV > 2) {
                if (t + 1 == t_next) store_copy(best);
            }
            __syncthreads();
        };
        const int stop = forced ? step_of(0) : G - 1;
        int t = begin;
        for (; t + 1 < stop; t += 2) {
            step(s_best[0], s_best[1], t);
            step(s_best[1], s_best[0], t + 1);
        }
        if (t < stop) step(s_best[0], s_best[1], t);
        static_assert((G - 1) % 2 == 1, "one step over");

        // the best allowed final state, lowest state on ties
        float bv = INF;
        uint32_t by = 0xFFFFFFFFu;
        auto take_better = [&](bool ok, float v, uint32_t y) {
            const bool take = ok & ((v < bv) | ((v == bv) & (y < by)));
            bv = take ? v : bv;
            by = take ? y : by;
        };
        if (!forced) {
            // (what is made with it here is not worth a register in the steps)
            int my_hi = NB * (int)threadIdx.x;
            asm volatile("" : "+v"(my_hi));
#pragma unroll
            for (int r = 0; r < VT_REGS; r++) {
                const uint32_t y = ((uint32_t)(r % NC) << OV) | (uint32_t)(my_hi + r / NC);
                take_better(!constrained | ((y & (uint32_t)(NP - 1)) == O),
                            state_value<V>(cr[r], s0, s1, s_best[1][Geo::place((int)(y >> KV))]), y);
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) take_better(true, __shfl_xor(bv, off, 64), __shfl_xor(by, off, 64));
            if (lane == 0) s_rv[wave] = bv, s_ry[wave] = by;
        }
        // (a segment's copy, on the way while the one before is walked)
        float pre[AHEAD];
        auto fetch = [&](int c) {  // (whether there is one or not: else the last one would have to be kept meanwhile)
            const float *const from = copy_at(min(c, last_copy));
            if constexpr (KV == 3) {
#pragma unroll
                for (int p = 0; p < NC; p++) pre[p] = (from + (p << (OV - KV)))[(uint32_t)tid];
            } else {
#pragma unroll
                for (int i = 0; i < AHEAD; i += 4) {
                    const float4_t four = (reinterpret_cast<const float4_t *>(from) + 256 * i)[(uint32_t)tid];
#pragma unroll
                    for (int e = 0; e < 4; e++) pre[i + e] = four[e];
                }
            }
        };
        uint32_t y;
        if (!forced) {
            fetch(0);
            __syncthreads();
            bv = INF;
            by = 0xFFFFFFFFu;
            for (int w = 0; w < 16; w++) take_better(true, s_rv[w], s_ry[w]);
            y = __builtin_amdgcn_readfirstlane(by) & 0xFFFFu;
            if (constrained && tid == 0) {
                sym[G - 1] = (uint8_t)(y >> OV);
                if (tile_err) tile_err[slot] = bv;
            }
        } else {  // what a copy of this step would bring, and a state of step G with the overlap for a prefix
            const float *const at = s_best[(stop - begin) & 1];
            if constexpr (KV == 4) {
#pragma unroll
                for (int i = 0; i < NB; i++) pre[i] = at[Geo::place(my_hi + i)];
            } else {
                thread_reads<KV, V, LB>(at, tid, pre);
            }
            __syncthreads();
            y = O << KV;
        }

        t = end;
        for (int c = 0; c < nseg; c++) {
            const int length = base + (c < longer), forward = length - T, u = t - length;
            // (nothing that depends on these is worth a register across segments: it would be one of the spilled ones)
            asm volatile("" : "+v"(tid), "+v"(my_hi));
            const int lane = tid & 63;
            // The entries of step u that the thread's states hang on.  (At kV = 4 four threads have the same sixteen, as many
            // loads from memory for a few bytes: there they go through LDS.)
            float through_lds[KV == 4 ? COUNT : 1];
            float(&b)[COUNT] = [&]() -> float(&)[COUNT] {
                if constexpr (KV == 4) return through_lds;
                else return pre;
            }();
            if constexpr (KV == 4) {
                if (c > last_copy) {
#pragma unroll
                    for (int i = 0; i < NB; i++) pre[i] = first(my_hi + i);
                }
                put(s_best[0], pre);
                __syncthreads();
            } else if (c > last_copy) {
#pragma unroll
                for (int p = 0; p < NC; p++) {
#pragma unroll
                    for (int a = 0; a < COUNT / NC; a++)
                        pre[COUNT / NC * p + a] = first((p << (OV - KV)) + COUNT / NC * tid + a);
                }
            }
            const uint32_t under = (y >> (KV * T)) & 15u;  // low bits of the leaves
            if (forward > 0) {
                if constexpr (KV == 4) {
                    thread_reads<KV, V, LB>(s_best[0], tid, b);
                } else {  // (LDS has step u for the way down)
#pragma unroll
                    for (int p = 0; p < NC; p++) {
                        if constexpr (KV == 2)
                            *reinterpret_cast<float4_t *>(s_best[0] + Geo::place((p << (OV - KV)) + 4 * tid)) =
                                float4_t{b[4 * p], b[4 * p + 1], b[4 * p + 2], b[4 * p + 3]};
                        else s_best[0][Geo::place((p << (OV - KV)) + tid)] = b[p];
                    }
                }
                for (int k = 0; k + 1 < forward; k++) {
                    float best[NB];
                    thread_minima<KV, V, LB>(b, cr, sample(u + k, 0), V == 2 ? sample(u + k, 1) : 0.f, best);
                    put(s_best[k + 1], best);
                    __syncthreads();
                    thread_reads<KV, V, LB>(s_best[k + 1], tid, b);
                }
                const float s0 = sample(u + forward - 1, 0), s1 = V == 2 ? sample(u + forward - 1, 1) : 0.f;
                // prefix my_hi + (a << FIXED) + (under >> KV) is leaf 4 tid + a's
                one_of<1 << Geo::FIXED>(under >> KV, [&](auto fc) {
                    float4_t best;
#pragma unroll
                    for (int a = 0; a < 4; a++) {
                        const int i = (a << Geo::FIXED) + decltype(fc)::value;
                        auto value = [&](int p) { return state_value<V>(cr[i * NC + p], s0, s1, b[Hang<KV>::under(i, p)]); };
                        float m = min2(value(0), value(1));
#pragma unroll
                        for (int p = 2; p < NC; p += 2) m = min3(m, value(p), value(p + 1));
                        best[a] = m;
                    }
                    *reinterpret_cast<float4_t *>(s_leaf + 4 * tid) = best;
                });
                __syncthreads();
            }

            // Leaf l = (p_T ... p_1), digit p_j being the top kV bits of the state j steps back; node (p_j ... p_1) of level j is
            // state (node << (16 - kV j)) | (y >> kV j).  A node carries its value and the digits of its best walk.
            auto node_state = [&](int j, uint32_t node) { return ((node << (LB - KV * j)) | (y >> (KV * j))) & 0xFFFFu; };
            // A node's code and samples, read and formed before what its value waits for.
            struct Node {
                uint32_t code;
                float s0, s1;
                __device__ __forceinline__ float value(float b) const { return state_value<V>(code, s0, s1, b); }
            };
            auto uniform = [](float v) {
                return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
            };
            auto node_of = [&](uint32_t state, int step) {
                return Node{code_register<CODE>(state, lut), uniform(sample(step, 0)), V == 2 ? uniform(sample(step, 1)) : 0.f};
            };
            // the minimum over the top digit of the nodes above `node`, and their walks with that digit behind
            auto best_below = [&](const uint2 *nodes, int count, uint32_t node, float &v, uint32_t &walk) {
                constexpr int AT_A_TIME = NC < 8 ? NC : 8;
#pragma unroll
                for (int p0 = 0; p0 < NC; p0 += AT_A_TIME) {
                    uint2 e[AT_A_TIME];
#pragma unroll
                    for (int p = 0; p < AT_A_TIME; p++) e[p] = nodes[(uint32_t)((p0 + p) * count) + node];
#pragma unroll
                    for (int p = 0; p < AT_A_TIME; p++) {
                        const float ev = __builtin_bit_cast(float, e[p].x);
                        const bool lt = p0 + p == 0 || ev < v;
                        v = lt ? ev : v;
                        walk = lt ? (e[p].y << KV) | (uint32_t)(p0 + p) : walk;
                    }
                    asm volatile("" : "+v"(v), "+v"(walk));
                }
            };
            // Level T's node is what the forward step calls a prefix, number `under` (its low bits) of the thread that has its
            // predecessors' codes, and where the copy is of this very step also their entries, in registers.  At kV = 4 that is
            // every fourth thread: computed codes are formed anew by 256 side by side, table codes would be as many reads.
            auto level_t = [&](int node, bool active, const uint32_t (&leaf)[NC], const float (&entry)[NC]) {
                const Node own = node_of(node_state(T - 1, (uint32_t)node), t - T + 1);
                const float s0 = sample(t - T, 0), s1 = V == 2 ? sample(t - T, 1) : 0.f;
                float m = INF;
                uint32_t digit = 0;
#pragma unroll
                for (int p = 0; p < NC; p++) {
                    const float v = state_value<V>(leaf[p], s0, s1, entry[p]);
                    const bool lt = p == 0 || v < m;
                    m = lt ? v : m;
                    digit = lt ? (uint32_t)p : digit;
                }
                if (active) s_node[node] = uint2{__builtin_bit_cast(uint32_t, own.value(m)), digit};
            };
            if constexpr (CODES_KEPT) {
                const int node = tid >> (KV - 2);
                uint32_t leaf[NC];
                float entry[NC];
                one_of<NB>(under & (uint32_t)(NB - 1), [&](auto ic) {
#pragma unroll
                    for (int p = 0; p < NC; p++) {
                        leaf[p] = cr[decltype(ic)::value * NC + p];
                        entry[p] = KV == 4 ? 0.f : b[Hang<KV>::under(decltype(ic)::value, p)];
                        // (else the cases become one with an index, and the arrays go to memory)
                        asm("; %2" : "+v"(leaf[p]), "+v"(entry[p]) : "i"(decltype(ic)::value));
                    }
                });
                if (KV == 4 || forward > 0) {
#pragma unroll
                    for (int p = 0; p < NC; p++) entry[p] = (forward > 0 ? s_leaf : s_best[0])[p * NODES + node];
                }
                level_t(node, (uint32_t)(tid & ((1 << (KV - 2)) - 1)) == under >> (6 - KV), leaf, entry);
            } else if (tid < NODES) {
                uint32_t leaf[NC];
                float entry[NC];
#pragma unroll
                for (int p = 0; p < NC; p++) {
                    entry[p] = (forward > 0 ? s_leaf : s_best[0])[p * NODES + tid];
                    leaf[p] = code_register<CODE>(node_state(T, (uint32_t)(p * NODES + tid)), lut);
                }
                level_t(tid, true, leaf, entry);
            }
            // (here, where few registers are in use: ahead of the steps above these would be spilled as they arrive)
            fetch(c + 1);
            // levels whose nodes are the lanes of wave 0
            constexpr int ROOTS = KV == 2 ? 3 : KV == 3 ? 2 : 1;
            const uint32_t me = (uint32_t)lane & ((1u << (KV * ROOTS)) - 1u);
            Node four{};
            if constexpr (KV == 2) {
                if (wave < 4) four = node_of(node_state(4, (uint32_t)tid), t - 4);
            }
            Node root[ROOTS + 1];
            if (wave == 0) {
#pragma unroll
                for (int j = 1; j <= ROOTS; j++) root[j] = node_of(node_state(j, me & ((1u << (KV * j)) - 1u)), t - j);
            }
            __syncthreads();
            if constexpr (KV == 2) {  // level 4: 256 nodes
                if (wave < 4) {
                    float m = INF;
                    uint32_t walk = 0;
                    best_below(s_node, 256, (uint32_t)tid, m, walk);
                    s_four[tid] = uint2{__builtin_bit_cast(uint32_t, four.value(m)), walk};
                }
                __syncthreads();
            }
            if (wave == 0) {
                float m = INF;
                uint32_t walk = 0;
                best_below(KV == 2 ? s_four : s_node, 1 << (KV * ROOTS), me, m, walk);
                // levels ROOTS to 1 across lanes: the lane's bits kV (j - 1) .. are digit j
                auto across = [&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    const uint32_t digit = (me >> (KV * (j - 1))) & (uint32_t)(NC - 1);
                    m = root[j].value(m);
                    walk = (walk << KV) | digit;
                    auto meet = [&](auto bit) {
                        constexpr int BIT = decltype(bit)::value;
                        if constexpr (BIT < KV) {
                            const float ov = __builtin_bit_cast(float, other_lane<KV * (j - 1) + BIT>(__builtin_bit_cast(uint32_t, m)));
                            const uint32_t ow = other_lane<KV * (j - 1) + BIT>(walk);
                            const bool take = ov < m || (ov == m && (ow & (uint32_t)(NC - 1)) < (walk & (uint32_t)(NC - 1)));
                            m = take ? ov : m;
                            walk = take ? ow : walk;
                        }
                    };
                    meet(std::integral_constant<int, 0>{});
                    meet(std::integral_constant<int, 1>{});
                    meet(std::integral_constant<int, 2>{});
                    meet(std::integral_constant<int, 3>{});
                };
                if constexpr (ROOTS >= 3) across(std::integral_constant<int, 3>{});
                if constexpr (ROOTS >= 2) across(std::integral_constant<int, 2>{});
                across(std::integral_constant<int, 1>{});
                walk = __builtin_amdgcn_readfirstlane(walk);
                if (forced && c == 0 && tile_err && lane == 0) tile_err[slot] = m;
                if (lane < T) sym[t - 1 - lane] = (uint8_t)((walk >> (KV * lane)) & (uint32_t)(NC - 1));
                uint32_t z = (walk << 4) | under;
                // and the steps that were taken forward
                for (int k = forward - 1; k >= 0; k--) {
                    const uint32_t p = (uint32_t)lane & (uint32_t)(NC - 1), state = (p << OV) | (z >> KV);
                    float v = node_of(state, u + k).value(s_best[k][Geo::place((int)(state >> KV))]);
                    uint32_t digit = p;
                    auto meet = [&](auto bit) {
                        constexpr int BIT = decltype(bit)::value;
                        if constexpr (BIT < KV) {
                            const float ov = __builtin_bit_cast(float, other_lane<BIT>(__builtin_bit_cast(uint32_t, v)));
                            const uint32_t od = other_lane<BIT>(digit);
                            const bool take = ov < v || (ov == v && od < digit);
                            v = take ? ov : v;
                            digit = take ? od : digit;
                        }
                    };
                    meet(std::integral_constant<int, 0>{});
                    meet(std::integral_constant<int, 1>{});
                    meet(std::integral_constant<int, 2>{});
                    meet(std::integral_constant<int, 3>{});
                    digit = __builtin_amdgcn_readfirstlane(digit);
                    if (lane == 0) sym[u + k] = (uint8_t)digit;
                    z = (digit << OV) | (z >> KV);
                }
                if (lane == 0) s_state = z;
            }
            __syncthreads();
            y = __builtin_amdgcn_readfirstlane(s_state);
            t = u;
        }
        O = y & (uint32_t)(NP - 1);  // (after the first pass: of step MID)
    }
    if (tid < NWORDS) {
        uint32_t word = 0;
#pragma unroll
        for (int b = 0; b < 32; b++) {
            const int pos = 32 * tid + b;
            word = (word << 1) | ((sym[pos / KV] >> (KV - 1 - pos % KV)) & 1u);
        }
        codes[(size_t)slot * NWORDS + tid] = word;
    }
}

// ------------------------------------------------------------------- launchers

// Words of a sequence in flight besides its copies of `best`: final state, overlap, final value.
constexpr int VT_HEAD_WORDS = 3;
constexpr size_t VT_HEAD_ALIGN = 256;

size_t head_bytes(long tiles) {
    const size_t b = (size_t)tiles * VT_HEAD_WORDS * sizeof(uint32_t);
    return (b + VT_HEAD_ALIGN - 1) / VT_HEAD_ALIGN * VT_HEAD_ALIGN;
}

// How a workspace is used: `tiles` sequences in flight, `slots` copies of `best` each.  With fewer
// slots than a walk needs the forward pass is repeated up to where the next copies lie.
struct Plan {
    long tiles;
    int slots;
    double cost;  // steps of one workgroup's passes, all batches together
};
// Trees of a pass's walk, and the step that its forward pass goes up to for copies from c on.
template <class Geo>
int segments_of(int pass) { return pass == 1 ? Geo::NSEG_MID : Geo::NSEG2; }
template <class Geo>
int last_step(int pass, int c) {
    if (pass == 2 && Geo::FORCED) return Geo::END - Geo::J * (c + 1) > Geo::T0 ? Geo::END - Geo::J * (c + 1) : Geo::T0;
    return c == 0 ? Geo::G - 1 : Geo::G - 1 - Geo::J * (c + 1);
}
template <class Geo>
double pass_steps(int slots, int pass) {
    double steps = 0;
    for (int c = 0; c < segments_of<Geo>(pass); c += slots) steps += last_step<Geo>(pass, c) - (pass == 2 ? Geo::T0 : 0);
    return steps;
}
template <class Geo>
Plan plan_for(long tiles, long ntiles, size_t ws_bytes) {
    constexpr long RESIDENT = 256L * (1024 / Geo::NT);  // workgroups the chip runs at a time
    Plan p{0, 0, 0};
    if (tiles > ntiles) tiles = ntiles;
    // whole rounds of workgroups, and batches of the same number of rounds
    if (tiles > RESIDENT && tiles < ntiles) {
        const long rounds = (ntiles + RESIDENT - 1) / RESIDENT, per = tiles / RESIDENT;
        const long batches = (rounds + per - 1) / per;
        tiles = (rounds + batches - 1) / batches * RESIDENT;
    }
    if (tiles <= 0 || head_bytes(tiles) >= ws_bytes) return p;
    const size_t copies = (ws_bytes - head_bytes(tiles)) / ((size_t)tiles * Geo::NP * sizeof(float));
    p.slots = (int)(copies < (size_t)Geo::COPIES ? copies : (size_t)Geo::COPIES);
    if (p.slots <= 0) return p;
    p.tiles = tiles;
    const double steps = pass_steps<Geo>(p.slots, 1) + pass_steps<Geo>(p.slots, 2);
    for (long t = 0; t < ntiles; t += tiles)
        p.cost += steps * (double)((((ntiles - t < tiles) ? ntiles - t : tiles) + RESIDENT - 1) / RESIDENT);
    return p;
}
// The cheaper of two ways: as many sequences at a time as find room for every copy a walk needs, or
// as many as the caller sized the workspace for.
template <class Geo>
Plan make_plan(long ntiles, size_t ws_bytes, size_t sized_for) {
    auto room_for = [&](size_t per_tile) {
        long t = (long)(ws_bytes / per_tile);
        while (t > 0 && head_bytes(t) + (size_t)t * per_tile > ws_bytes) t--;
        return t;
    };
    const Plan a = plan_for<Geo>(room_for((size_t)Geo::COPIES * Geo::NP * sizeof(float)), ntiles, ws_bytes);
    const Plan b = plan_for<Geo>(room_for(sized_for), ntiles, ws_bytes);
    if (b.tiles == 0) return a;
    return a.tiles && a.cost <= b.cost ? a : b;
}

template <int KV, int V, int CODE>
hipError_t quantize_gpu_t(const float *W, int m, int n, int ld, const uint32_t *lut, uint32_t *codes,
                          float *tile_err, void *ws, size_t ws_bytes, hipStream_t st) {
    using Geo = VitGeo<KV, V, code_state_bits(CODE)>;
    constexpr int TY = 1 << code_log2_ty(CODE), TX = VT_T / TY;
    const int tn = n / TY;
    const long ntiles = (long)(m / TX) * tn;
    // One launch for at most one sequence per CU; three at kV = 3, where walks and forward passes repeat the most steps.  (us, with
    // the workspace callers are told to bring, 128 | 256 | 512 sequences, several launches and one: 3INST k = 2 698 619 | 724
    // 663 | 1272 1307, k = 3 982 644 | 984 650 | 1992 1292, k = 4 761 636 | 762 642 | 1331 1284, HYB k = 2 920 796 | 916 801 |
    // 1534 1600; k = 3 of 768 2023 1933, of 1024 2695 2579.  With room for every copy k = 2 618 588 | 640 686, k = 3 659 562 |
    // 675 596 | 1187 1186, of 520 1650 1745 and of 768 1702 1768, k = 4 649 594 | 666 601 | 1153 1192, HYB 756 743 | 767 746 | 1425
    // 1492: the launches stay apart there, all of them storing every copy, at kV = 2 if more than half of the CUs have a
    // sequence, at kV = 3 if some have three.)
    if constexpr (KV <= 4 && code_state_bits(CODE) == 16) {
        using Few = FewGeo<KV, V>;
        if (ntiles <= (KV == 3 ? 3 * CUS : CUS)) {
            const size_t copy_bytes = (size_t)ntiles * Geo::NP * sizeof(float);
            const size_t room = ws_bytes > head_bytes(ntiles) ? (ws_bytes - head_bytes(ntiles)) / copy_bytes : 0;
            const long slots = (long)(room < (size_t)VT_T ? room : (size_t)VT_T);
            const bool pays = ntiles <= (KV == 2 ? CUS / 2 : KV == 3 ? 2 * CUS : CUS) || slots < Geo::COPIES;
            const int nseg1 = (int)(slots < Few::D1 / Few::T ? slots : Few::D1 / Few::T);
            const int nseg2 = (int)(slots + 1 < Few::D2 / Few::T ? slots + 1 : Few::D2 / Few::T);
            // (copies for segments of a walk over all steps: at some sizes one fewer would do)
            const bool room_for_walk = Few::fits(Geo::G - 1, (int)slots + 1);
            if (pays && room_for_walk && Few::fits(Few::D1, nseg1) && Few::fits(Few::D2, nseg2)) {
                hipLaunchKernelGGL((viterbi_few_kernel<KV, V, CODE>), dim3((unsigned)ntiles), dim3(1024), 0, st, W, ld, tn,
                                   lut, (float *)((char *)ws + head_bytes(ntiles)), slots, nseg1, nseg2, codes, tile_err);
                return hipGetLastError();
            }
        }
    }
    const size_t sized_for = quantize_gpu_workspace(KV / V, V, 1) - head_bytes(1);
    const Plan plan = make_plan<Geo>(ntiles, ws_bytes, sized_for);
    const long cap = plan.tiles;
    if (cap <= 0) return hipErrorInvalidValue;
    uint32_t *final_state = (uint32_t *)ws;
    uint32_t *overlap = final_state + cap;
    float *final_value = (float *)(overlap + cap);
    float *store = (float *)((char *)ws + head_bytes(cap));
    for (long tile0 = 0; tile0 < ntiles; tile0 += cap) {
        const int cnt = (int)(ntiles - tile0 < cap ? ntiles - tile0 : cap);
        const bool few = cnt <= Geo::FEW;
        for (int pass = 1; pass <= 2; pass++) {
            const int nseg = segments_of<Geo>(pass);
            for (int c_lo = 0; c_lo < nseg; c_lo += plan.slots) {
                // (the last tree of a whole walk that is not forced starts at step 0 and needs no copy)
                int c_hi = c_lo + plan.slots < nseg ? c_lo + plan.slots : nseg;
                if (!Geo::FORCED && c_hi == Geo::NSEG - 1) c_hi = Geo::NSEG;
                const int t_end = last_step<Geo>(pass, c_lo);
                if (t_end > 0)
                    hipLaunchKernelGGL((viterbi_forward_kernel<KV, V, CODE>), dim3(cnt), dim3(Geo::NT), 0, st, W, ld,
                                       tn, tile0, lut, pass == 1, pass == 1 ? (const uint32_t *)nullptr : overlap,
                                       store, (long)plan.slots, c_lo, c_hi, t_end, final_state, final_value);
                hipLaunchKernelGGL((few ? viterbi_walk_kernel<KV, V, CODE, Geo::FEW ? 2 : 0> : viterbi_walk_kernel<KV, V, CODE, 0>),
                                   dim3(few ? cnt : (cnt + 3) / 4), dim3(256), 0, st, W, ld, tn, tile0, lut, pass,
                                   (const float *)store, (long)plan.slots, c_lo, c_hi, final_state,
                                   (const float *)final_value, cnt, overlap, codes, tile_err);
                if (c_hi == nseg) break;
            }
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

// Bytes per sequence in flight that callers are told to bring (at kV = 2 half, at kV = 3 and 4 less,
// of what a whole walk's copies take: with thousands in flight fewer at a time do as well, with few one launch
// takes longer segments, and in between the forward pass is repeated in part, see Plan).
size_t quantize_gpu_workspace(int k, int V, long tiles) {
    size_t per_step;  // words
    switch (k * V) {
        case 2: per_step = 2048; break;
        case 8: per_step = 256; break;
        default: per_step = 1024; break;
    }
    return head_bytes(tiles) + (size_t)tiles * (VT_T / V) * per_step * sizeof(uint32_t);
}

hipError_t launch_quantize_gpu(int k, int code_id, const float *W, int m, int n, int ld, const uint32_t *lut,
                               uint32_t *codes, float *tile_err, void *ws, size_t ws_bytes,
                               hipStream_t st) {
    if (code_id == CODE_HYB1) {
        if (k == 2) return quantize_gpu_t<2, 1, CODE_HYB1>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
        if (k == 3) return quantize_gpu_t<3, 1, CODE_HYB1>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
        return quantize_gpu_t<4, 1, CODE_HYB1>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
    } else if (code_id == CODE_LUT) {
        if (k == 2) return quantize_gpu_t<2, 1, CODE_LUT>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
        if (k == 3) return quantize_gpu_t<3, 1, CODE_LUT>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
        return quantize_gpu_t<4, 1, CODE_LUT>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
    } else if (code_id == CODE_HYB2) {
        if (k == 2) return quantize_gpu_t<4, 2, CODE_HYB2>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
        if (k == 3) return quantize_gpu_t<6, 2, CODE_HYB2>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
        return quantize_gpu_t<8, 2, CODE_HYB2>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
    } else if (code_id == CODE_HYB) {
        if (k == 2) return quantize_gpu_t<4, 2, CODE_HYB>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
        if (k == 3) return quantize_gpu_t<6, 2, CODE_HYB>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
        return quantize_gpu_t<8, 2, CODE_HYB>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
    } else if (code_id == CODE_3INST) {
        if (k == 2) return quantize_gpu_t<2, 1, CODE_3INST>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
        if (k == 3) return quantize_gpu_t<3, 1, CODE_3INST>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
        return quantize_gpu_t<4, 1, CODE_3INST>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
    } else {
        if (k == 2) return quantize_gpu_t<2, 1, CODE_1MAD>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
        if (k == 3) return quantize_gpu_t<3, 1, CODE_1MAD>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
        return quantize_gpu_t<4, 1, CODE_1MAD>(W, m, n, ld, lut, codes, tile_err, ws, ws_bytes, st);
    }
}

}  // namespace qtip
