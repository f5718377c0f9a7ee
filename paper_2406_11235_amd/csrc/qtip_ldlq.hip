// BlockLDLQ with the trellis quantizer as its rounder (Algorithm 5 of arXiv 2406.11235;
// T_x = T_y = 16 for the codes of Algorithms 1-3, T_x = 32 and T_y = 8 for the lookup-only
// code, whose smaller group size is the reason the paper gives for that shape; the comments
// below say 16 for T_y = G): the block LDL decomposition of the proxy Hessian and the loop over
// column blocks, last to first, that quantizes x = W_j + (W - What)_{>j} A_{>j,j} tile by
// tile with the GPU Viterbi quantizer and feeds the error of every finished block forward.
//
// Block LDL (H = L D L^T, L unit block lower triangular, D block diagonal, A = L - I) runs
// in binary64 on the device, right-looking, in panels of 8 block columns with two launches each.
// It is a one-off of n^3/3 multiply-adds per layer.
//
// The feedback sum is written so that a CPU reference can repeat it bit for bit, because
// what it feeds is a quantizer, whose decisions are not continuous: binary32, one fused
// multiply-add per term E[r][i] A[i][c], the terms taken block by block from the last
// column block down, ascending inside a block (the order in which a running sum that is
// updated after every finished block receives them).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qtip_device.h"
#include "qtip_internal.h"

namespace qtip {
namespace {

// G = T_y = block size of the decomposition = width of a sequence's block of the matrix

// ------------------------------------------------------------------ block LDL
//
// In 16 x 16 blocks, on the binary64 matrix cores.  Everything is kept transposed and by blocks: T_ji = S_ij^T (S
// the trailing matrix, j <= i) and M_ji = L_ij^T = D_j^-1 T_ji, each as the result layout of
// v_mfma_f64_16x16x4_f64: lane l, register t holds row 4 t + l / 16, column l % 16.  In that layout a block is at
// the same time a B operand, and, transposed, an A operand of a product that contracts over its rows, and these are the
// only products there are:
//     M_ji = D_j^-1 T_ji,        T_ki -= T_jk^T M_ji   (S_ik -= L_ij S_kj^T)   for j < k <= i.
// The workspace holds T and M by blocks of 2 KiB, which a wave reads and writes as they are.
//
// Panels of 8 block columns, two launches each.  ldl_panel_kernel: a workgroup has a wave for each of the panel's own 8
// block rows but the first, one to four for block rows below, and one for the pivots; a row's wave holds its 8 blocks in registers.
// The pivots' wave inverts D_j, the waves meet once per block column, and while the others take the two products above it
// takes those that its next pivot needs itself.  It has its SIMD to itself: a binary64 matrix instruction of another wave holds
// that up for 64 cycles at a time (a wave's priority does not help: 388 us -> 397), which was 1200 cycles of each of the
// panel's first four block columns.  Every workgroup factors the panel's own rows again, which costs little (the inversions
// are a serial chain) and saves a launch per panel.  ldl_update_panel_kernel: the panel's products with the next
// panel's block columns.  Those with everything further right are taken beside the next panel, in its launch.
// What bounds it is the chain of block columns, 4330 cycles each: rows of the pivot 280, inversion 2280, its way to LDS 530, the
// meeting 160, two dependent products 900, the loop 190; the first three of a panel wait 2500 more for the products of the other
// rows, which have three SIMDs; and the launch between two panels, 4 us.  n = 2048, g = 16: 1744 us with two launches
// per block column, the inversion with five barriers per pivot and the products on the vector units, 388 us with the pivots
// inverted by the waves of their rows, 343 with a wave for the pivots, 318 us now; g = 8: 475 us -> 383 -> 368 (144 bytes a lane
// of its pivots' wave lie in private memory).  Meeting twice, or handing the next pivot's products' operands over through a flag half-way through the
// inversion, so that they run before the meeting, is no faster (350 to 371 us): the other rows are what is late then.

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef double double2_t __attribute__((ext_vector_type(2)));
constexpr int LDL_PANEL = 8;

__device__ __forceinline__ double *ldl_block(double *base, int nb, int k, int i) {
    return base + ((size_t)k * nb + i) * 256;
}
// (a lane's four numbers are neighbours: two 16-byte accesses, in LDS as in memory; as four of 8 bytes n = 1040 took 154.0 us in
// place of 150.5, 2048 331 in place of 318, 4096 1123 in place of 1077)
__device__ __forceinline__ double4_t ldl_load(const double *block, int lane) {
    const double2_t lo = *reinterpret_cast<const double2_t *>(block + 4 * lane);
    const double2_t hi = *reinterpret_cast<const double2_t *>(block + 4 * lane + 2);
    return double4_t{lo[0], lo[1], hi[0], hi[1]};
}
__device__ __forceinline__ void ldl_store(double *block, int lane, double4_t v) {
    *reinterpret_cast<double2_t *>(block + 4 * lane) = double2_t{v[0], v[1]};
    *reinterpret_cast<double2_t *>(block + 4 * lane + 2) = double2_t{v[2], v[3]};
}
// c + X^T Y, the contraction over the rows of X and Y
__device__ __forceinline__ double4_t ldl_product(double4_t x, double4_t y, double4_t c) {
#pragma unroll
    for (int t = 0; t < 4; t++) c = __builtin_amdgcn_mfma_f64_16x16x4f64(x[t], y[t], c, 0, 0, 0);
    return c;
}

// T from the lower triangle of H, a diagonal block's upper half from its lower one (what H holds above its diagonal is
// nobody's to read, the blocks between the two 8 x 8 blocks of a g = 8 pivot included), and zeros where A has no block of
// its own: block row i, four block columns from j0 on, by one wave.
__device__ __forceinline__ void ldl_init(const double *__restrict__ H, double *__restrict__ T, float *__restrict__ A, int n,
                                         int i, int j0, int lane) {
    const int nb = n >> 4, r = lane >> 2, m = lane & 3;  // row r, columns 4 m .. 4 m + 3 of the block
    const double *h = H + (size_t)(16 * i + r) * n + 4 * m;
    float *a = A + (size_t)(16 * i + r) * n + 4 * m;
    double v[4][4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const int j = j0 + e;
        if (j >= nb || j > i) continue;
#pragma unroll
        for (int c = 0; c < 4; c++)
            v[e][c] = j < i || 4 * m + c <= r ? h[16 * j + c] : H[(size_t)(16 * i + 4 * m + c) * n + 16 * i + r];
    }
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const int j = j0 + e;
        if (j < nb && j >= i) {
#pragma unroll
            for (int c = 0; c < 4; c++) a[16 * j + c] = 0.f;
        }
        if (j >= nb || j > i) continue;
        double *t = ldl_block(T, nb, j, i) + lane;
#pragma unroll
        for (int c = 0; c < 4; c++) t[64 * c] = v[e][c];
    }
}
// Block columns below `columns`, four per wave.
__global__ __launch_bounds__(256) void ldl_init_kernel(const double *__restrict__ H, double *__restrict__ T,
                                                       float *__restrict__ A, int n, int columns) {
    const int w = blockIdx.x * 4 + (threadIdx.x >> 6), of = (columns + 3) / 4;
    if (w < of * (n >> 4)) ldl_init(H, T, A, n, w / of, 4 * (w % of), threadIdx.x & 63);
}

// The value that lane p of this row of 16 lanes has.  (What reads across lanes may not follow the vector instruction that
// wrote its register within two wait states, which is left to whoever writes it as text: it begins with them.)
template <int p>
__device__ __forceinline__ double row_value(double a) {
    double v;
    asm volatile("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "=&v"(v) : "v"(a), "n"(p));
    return v;
}

// Rows of a symmetric block in the result layout: a[c] = entry (l % 16, c) in lane l.  The lane has column l % 16, four of
// its entries; through a piece of LDS that is the wave's own, rows 18 apart.  (Six exchanges of lane rows per register in its
// place: 476 cycles, this 300.)
constexpr int LDL_ROW = 18;
__device__ __forceinline__ void ldl_rows(double4_t d, double *s_rows, int lane, double (&a)[16]) {
    double *const mine = s_rows + (lane & 15) * LDL_ROW;
#pragma unroll
    for (int t = 0; t < 4; t++) mine[4 * t + (lane >> 4)] = d[t];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int c = 0; c < 16; c += 2) {
        const double2_t two = *reinterpret_cast<const double2_t *>(mine + c);
        a[c] = two[0];
        a[c + 1] = two[1];
    }
}
// The other way: entries 4 t + g, g = l / 16, of the lane's row: an A operand with the rows as they are.
__device__ __forceinline__ double4_t ldl_operand(const double (&a)[16], int g) {
    double4_t v;
#pragma unroll
    for (int t = 0; t < 4; t++) {
        const double e = g & 1 ? a[4 * t + 1] : a[4 * t], o = g & 1 ? a[4 * t + 3] : a[4 * t + 2];
        v[t] = g & 2 ? o : e;
    }
    return v;
}

// 1 / d to the last bit or two: the hardware's reciprocal (2^-26) and two Newton steps.
__device__ __forceinline__ double reciprocal(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
    return __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
}

// The other columns of pivot p: a[c] += f * a_p[c], c != p, a_p the row that lane p of this row of 16 lanes holds; returns
// the reciprocal of the next pivot (reciprocal() of lane p + 1's a[p + 1]), whose chain runs between the columns.  One
// piece of text, so that the waits are in it and nothing can come in between: two wait states before the first read
// across lanes, two columns between the next pivot's column and its broadcast, one behind the hardware's reciprocal.
// (Column by column, with the waits left to what stood between, the compiler put an exchange of lane rows one instruction
// before the read of its result.)
template <int p>
__device__ __forceinline__ double ldl_eliminate(double (&a)[16], double f) {
    double d, r, e;
#define COLUMN(C) "v_fmac_f64_dpp %" #C ", %" #C ", %[f] row_newbcast:%[p] row_mask:0xf bank_mask:0xf\n\t"
    asm volatile("s_nop 1\n\t" COLUMN(0) COLUMN(1) COLUMN(2)
                 "v_mov_b64_dpp %[d], %0 row_newbcast:%[next] row_mask:0xf bank_mask:0xf\n\t" COLUMN(3)
                 "v_rcp_f64_e32 %[r], %[d]\n\t" COLUMN(4) COLUMN(5) COLUMN(6)
                 "v_fma_f64 %[e], -%[d], %[r], 1.0\n\t" COLUMN(7) COLUMN(8)
                 "v_fma_f64 %[r], %[e], %[r], %[r]\n\t" COLUMN(9) COLUMN(10)
                 "v_fma_f64 %[e], -%[d], %[r], 1.0\n\t" COLUMN(11) COLUMN(12)
                 "v_fma_f64 %[r], %[e], %[r], %[r]\n\t" COLUMN(13) COLUMN(14)
                 : "+v"(a[(p + 1) & 15]), "+v"(a[(p + 2) & 15]), "+v"(a[(p + 3) & 15]), "+v"(a[(p + 4) & 15]),
                   "+v"(a[(p + 5) & 15]), "+v"(a[(p + 6) & 15]), "+v"(a[(p + 7) & 15]), "+v"(a[(p + 8) & 15]),
                   "+v"(a[(p + 9) & 15]), "+v"(a[(p + 10) & 15]), "+v"(a[(p + 11) & 15]), "+v"(a[(p + 12) & 15]),
                   "+v"(a[(p + 13) & 15]), "+v"(a[(p + 14) & 15]), "+v"(a[(p + 15) & 15]), [d] "=&v"(d), [r] "=&v"(r),
                   [e] "=&v"(e)
                 : [f] "v"(f), [p] "n"(p), [next] "n"((p + 1) & 15));
#undef COLUMN
    return r;
}

// Gauss-Jordan elimination of [D | I] in place, without pivoting (D is positive definite): lane l of a row of 16 holds
// row l.  Rows are not scaled on the way: `scale` is 1 / pivot of the lane's row, and the inverse is scale * a in
// the end.  After pivots 0 .. P - 1 the first P columns hold the identity's part, and `inv` is 1 / pivot P.
template <int p, int END>
__device__ __forceinline__ void ldl_invert(double (&a)[16], double &inv, double &scale, int row) {
    if constexpr (p < END) {
        const double f = row == p ? 0.0 : -a[p] * inv;
        scale = row == p ? inv : scale;
        inv = ldl_eliminate<p>(a, f);
        a[p] = row == p ? 1.0 : f;
        ldl_invert<p + 1, END>(a, inv, scale, row);
    }
}

// L_ij in binary32 from E = L_ij^T.
__device__ __forceinline__ void ldl_emit(float *__restrict__ A, int n, int i, int j, int lane, double4_t e) {
    float *a = A + (size_t)(16 * i + (lane & 15)) * n + 16 * j + (lane >> 4);
#pragma unroll
    for (int t = 0; t < 4; t++) a[4 * t] = (float)e[t];
}

// T_ki -= sum over the block columns j of the panel at J0 of T_jk^T M_ji, for the TB x TB blocks from (k0, i0) on that
// have k <= i, by one wave.
template <int TB>
__device__ __forceinline__ void ldl_update(double *T, const double *Ms, int nb, int J0, int k0, int i0, int lane) {
    int k[TB], i[TB];
#pragma unroll
    for (int e = 0; e < TB; e++) {
        k[e] = min(k0 + e, nb - 1);
        i[e] = min(i0 + e, nb - 1);
    }
    double4_t acc[TB][TB], old[TB][TB];
    // the operands of three block columns ahead: another XCD's workgroup has just written them, so they come from
    // behind the L2
    constexpr int AHEAD = 3;
    double4_t x[AHEAD + 1][TB], y[AHEAD + 1][TB];
    auto load = [&](int j, int to) {
#pragma unroll
        for (int e = 0; e < TB; e++) {
            x[to][e] = ldl_load(ldl_block(T, nb, J0 + j, k[e]), lane);
            y[to][e] = ldl_load(ldl_block(const_cast<double *>(Ms), nb, J0 + j, i[e]), lane);
        }
    };
#pragma unroll
    for (int j = 0; j < AHEAD; j++) load(j, j);
#pragma unroll
    for (int a = 0; a < TB; a++)
#pragma unroll
        for (int b = 0; b < TB; b++) {
            acc[a][b] = double4_t{0.0, 0.0, 0.0, 0.0};
            old[a][b] = ldl_load(ldl_block(T, nb, min(k[a], i[b]), max(k[a], i[b])), lane);
        }
#pragma unroll
    for (int j = 0; j < LDL_PANEL; j++) {
        if (j + AHEAD < LDL_PANEL) load(j + AHEAD, (j + AHEAD) % (AHEAD + 1));
#pragma unroll
        for (int a = 0; a < TB; a++)
#pragma unroll
            for (int b = 0; b < TB; b++)
                acc[a][b] = ldl_product(x[j % (AHEAD + 1)][a], y[j % (AHEAD + 1)][b], acc[a][b]);
    }
#pragma unroll
    for (int a = 0; a < TB; a++)
#pragma unroll
        for (int b = 0; b < TB; b++) {
            if (i0 + b >= nb || k0 + a > i0 + b) continue;
            ldl_store(ldl_block(T, nb, k[a], i[b]), lane, old[a][b] - acc[a][b]);
        }
}
// The same for the w-th pair of block groups, kp <= ip, of the triangle from block b0 on.
template <int TB>
__device__ __forceinline__ void ldl_update_triangle(double *T, const double *Ms, int nb, int J0, int b0, int w, int lane) {
    int ip = (int)((__builtin_sqrtf(8.f * (float)w + 1.f) - 1.f) * 0.5f);  // w = ip (ip + 1) / 2 + kp
    while ((ip + 1) * (ip + 2) / 2 <= w) ip++;
    while (ip * (ip + 1) / 2 > w) ip--;
    ldl_update<TB>(T, Ms, nb, J0, b0 + TB * (w - ip * (ip + 1) / 2), b0 + TB * ip, lane);
}
// The block columns of the panel behind the one at J0: a block per workgroup, two of the panel's block columns per wave, all
// operands asked for at once.  (A block per wave was 32 matrix instructions one behind the other: with this and with T made beside
// the first panel n = 512 takes 71.8 us in place of 75.3, 1040 154.7 in place of 163.9, 2048 332 in place of 342.)
__global__ __launch_bounds__(256) void ldl_update_panel_kernel(double *__restrict__ T, const double *__restrict__ Ms,
                                                               int nb, int J0) {
    static_assert(LDL_PANEL == 8, "four waves of two block columns");
    __shared__ __attribute__((aligned(16))) double s_sum[3][256];
    const int w = blockIdx.x, k = J0 + LDL_PANEL + w % LDL_PANEL, i = J0 + LDL_PANEL + w / LDL_PANEL;
    if (i >= nb || k > i) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, j = J0 + 2 * wave;
    double *const block = ldl_block(T, nb, k, i);
    double4_t x[2], y[2], old = {0.0, 0.0, 0.0, 0.0}, sum = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int e = 0; e < 2; e++) {
        x[e] = ldl_load(ldl_block(T, nb, j + e, k), lane);
        y[e] = ldl_load(ldl_block(const_cast<double *>(Ms), nb, j + e, i), lane);
    }
    if (wave == 0) old = ldl_load(block, lane);
#pragma unroll
    for (int e = 0; e < 2; e++) sum = ldl_product(x[e], y[e], sum);
    if (wave > 0) ldl_store(s_sum[wave - 1], lane, sum);
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int e = 0; e < 3; e++) sum += ldl_load(s_sum[e], lane);
    ldl_store(block, lane, old - sum);
}

// The waves of a panel's workgroup: wave 0 inverts pivots, the others whose number is not a multiple of 4 have a block row
// each, so that the inversions have their SIMD to themselves (a binary64 matrix instruction holds it for 64 cycles).
constexpr int ldl_waves(int rows) { return LDL_PANEL + rows + (LDL_PANEL + rows - 2) / 3; }
// Block row, counted from the panel's first, of the p-th of those waves: the long ones first, so that the three SIMDs have as much.
__device__ __forceinline__ int ldl_row_of(int p) {
    return p == 0 ? LDL_PANEL : p < 3 || (p >= 6 && p < 8) ? LDL_PANEL - p : p < 6 ? p : p + 1;
}
// (the waves meet for what is in LDS; results on their way to memory are nobody's business here)
__device__ __forceinline__ void ldl_meet() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The first `groups` workgroups: block columns J0 .. J0 + np - 1, and `rows` block rows below them per workgroup.  The others:
// what the panel before has to subtract behind this one, TB x TB blocks per wave, on the CUs that the chain leaves idle; beside
// the first panel the blocks of T behind it, where H is given.
template <int G, int TB, int rows>
__global__ __launch_bounds__(ldl_waves(rows) * 64) void ldl_panel_kernel(double *__restrict__ T, double *__restrict__ Ms,
                                                                         float *__restrict__ A, int n, int J0, int groups,
                                                                         int pairs, double *__restrict__ Dout,
                                                                         const double *__restrict__ H) {
    static_assert(LDL_PANEL == 8, "ldl_row_of");
    // D_j^-1 as an A operand, and what L_ij^T is made with (for G = 8 see below)
    __shared__ __attribute__((aligned(16))) double s_inv[2][256];
    __shared__ __attribute__((aligned(16))) double s_out[2][G == 8 ? 256 : 1];
    __shared__ __attribute__((aligned(16))) double s_t[2][LDL_PANEL][256];  // T_ij of the panel's own rows
    __shared__ __attribute__((aligned(16))) double s_d[2][256];             // the next pivot, column j not yet taken off
    __shared__ __attribute__((aligned(16))) double s_rows[16 * LDL_ROW];
    const int nb = n >> 4, np = min(LDL_PANEL, nb - J0);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if ((int)blockIdx.x >= groups) {
        const int w0 = (blockIdx.x - groups) * ldl_waves(rows) + wave, waves = (gridDim.x - groups) * ldl_waves(rows);
        for (int w = w0; w < pairs; w += waves) ldl_update_triangle<TB>(T, Ms, nb, J0 - LDL_PANEL, J0 + LDL_PANEL, w, lane);
        if (H) {
            const int of = (nb - LDL_PANEL + 3) / 4;
            for (int w = w0; w < of * nb; w += waves) ldl_init(H, T, A, n, w / of, LDL_PANEL + 4 * (w % of), lane);
        }
        return;
    }
    const double4_t zero = {0.0, 0.0, 0.0, 0.0};
    if (wave == 0) {
        const int row = lane & 15, g = lane >> 4;
        double4_t d = ldl_load(ldl_block(T, nb, J0, J0), lane);
        for (int j = 0; j < np; j++) {
            const int buf = j & 1;
            double a[16];
            ldl_rows(d, s_rows, lane, a);
            double scale = 1.0;
            double inv = reciprocal(row_value<0>(a[0]));
            if constexpr (G == 16) {
                ldl_invert<0, 16>(a, inv, scale, row);
            } else {
                // Half-way the first 8 rows hold the inverse of D's first 8 x 8 block, the last 8 the second
                // block of D in 8 x 8 blocks and, negative, the entry of L between the two.
                ldl_invert<0, 8>(a, inv, scale, row);
                if (blockIdx.x == 0 && g == 0 && row >= 8) {
#pragma unroll
                    for (int c = 0; c < 8; c++) {
                        A[(size_t)(16 * (J0 + j) + row) * n + 16 * (J0 + j) + c] = (float)-a[c];
                        if (Dout) Dout[(size_t)(J0 + j) * 128 + 64 + (row - 8) * 8 + c] = a[8 + c];
                    }
                }
                double f[16];
#pragma unroll
                for (int c = 0; c < 16; c++) f[c] = c < 8 ? a[c] * scale : 0.0;
                ldl_invert<8, 16>(a, inv, scale, row);
#pragma unroll
                for (int c = 0; c < 16; c++) f[c] = row < 8 ? f[c] : a[c] * scale;
                ldl_store(s_out[buf], lane, ldl_operand(f, g));
            }
            const double4_t op = ldl_operand(a, g) * scale;
            ldl_store(s_inv[buf], lane, op);
            ldl_meet();
            if (blockIdx.x == 0 && Dout) {
                if constexpr (G == 16) {
#pragma unroll
                    for (int q = 0; q < 4; q++) Dout[(size_t)(J0 + j) * 256 + 64 * q + lane] = d[q];
                } else if (row < 8) {
#pragma unroll
                    for (int q = 0; q < 2; q++) Dout[(size_t)(J0 + j) * 128 + (4 * q + g) * 8 + row] = d[q];
                }
            }
            if (j + 1 < np) {
                const double4_t t = ldl_load(s_t[buf][j + 1], lane), before = ldl_load(s_d[buf], lane);
                d = ldl_product(t, -ldl_product(op, t, zero), before);
            }
        }
        return;
    }
    const int rel = wave & 3 ? ldl_row_of(wave - 1 - (wave >> 2)) : -1;
    const bool own = rel < LDL_PANEL;  // of the panel's own block rows
    const int i = rel < 0 ? nb : own ? J0 + rel : J0 + rel + (int)blockIdx.x * rows;
    const bool some = i < nb;
    const bool speaks = own ? blockIdx.x == 0 : true;  // writes results
    double4_t t[LDL_PANEL];
#pragma unroll
    for (int j = 0; j < LDL_PANEL; j++) {
        t[j] = zero;
        if (some && j < np && j <= rel) t[j] = ldl_load(ldl_block(T, nb, J0 + j, i), lane);
    }
#pragma unroll
    for (int j = 0; j < LDL_PANEL; j++) {
        if (j >= np) break;
        const int buf = j & 1;
        if (some && own && rel > j) ldl_store(s_t[buf][rel], lane, t[j]);
        if (j + 1 < LDL_PANEL && some && rel == j + 1) ldl_store(s_d[buf], lane, t[j + 1 < LDL_PANEL ? j + 1 : 0]);
        ldl_meet();
        if (some && rel > j) {
            const double4_t m = ldl_product(ldl_load(s_inv[buf], lane), t[j], zero);
            const double4_t neg = -m;
            auto take_off = [&](int k) {  // (the next pivot's own is its wave's)
                if (k < np && k <= rel && rel != j + 1) t[k] = ldl_product(ldl_load(s_t[buf][k], lane), neg, t[k]);
            };
            if (j + 1 < LDL_PANEL) take_off(j + 1);
            // (results leave while products of the three waves of the SIMD run: after the last one 347 us in place of 338)
            if (speaks) {
                if (!own) {
                    ldl_store(ldl_block(T, nb, J0 + j, i), lane, t[j]);
                    ldl_store(ldl_block(Ms, nb, J0 + j, i), lane, m);
                }
                if constexpr (G == 8) ldl_emit(A, n, i, J0 + j, lane, ldl_product(ldl_load(s_out[buf], lane), t[j], zero));
                else ldl_emit(A, n, i, J0 + j, lane, m);
            }
#pragma unroll
            for (int k = j + 2; k < LDL_PANEL; k++) take_off(k);
        }
    }
}

// ------------------------------------------------------------------ Algorithm 5

// The feedback of Algorithm 5 as a running sum: X starts as W; when column block j is done,
// its error E_j = (W - What)[:, 16j:16j+16] is fed to every column before it,
//     X[r][c] += sum_{i in block j, ascending} E_j[r][i] A[16 j + i][c],   c < 16 j,
// one fused multiply-add per term.  When block j's turn comes, X[:, 16j:16j+16] is its x.
// Per element the terms arrive by blocks from the last one down and ascending inside a
// block: that order is the definition both sides use.  A thread owns one column and 8 rows:
// 16 values of A in registers, the rows' errors are wave-uniform.
constexpr int UPD_ROWS = 8;
template <int G>
__global__ __launch_bounds__(256) void ldlq_update_kernel(const float *__restrict__ Eslab,
                                                          const float *__restrict__ A, int m, int n, int j,
                                                          float *__restrict__ X) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    const int r0 = blockIdx.y * UPD_ROWS;
    if (c >= j * G) return;
    float a[G];
#pragma unroll
    for (int i = 0; i < G; i++) a[i] = A[(size_t)(j * G + i) * n + c];
#pragma unroll
    for (int rr = 0; rr < UPD_ROWS; rr++) {
        const int r = r0 + rr;
        if (r >= m) break;
        float acc = X[(size_t)r * n + c];
#pragma unroll
        for (int i = 0; i < G; i++) acc = __builtin_fmaf(Eslab[(size_t)r * G + i], a[i], acc);
        X[(size_t)r * n + c] = acc;
    }
}

__global__ void ldlq_copy_kernel(const float *__restrict__ src, float *__restrict__ dst, size_t count) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

// After block j is quantized: its error slab E_j and What from the decoded slab, and the
// slab's codes and errors to their places in the matrix's tile order.
// (TX x G is the block that is one sequence, so the slab holds m / TX of them.)
template <int G, int TX>
__global__ __launch_bounds__(256) void ldlq_finish_kernel(const float *__restrict__ W,
                                                          const half_t *__restrict__ slab,
                                                          const uint32_t *__restrict__ slab_codes,
                                                          const float *__restrict__ slab_err, int m, int n,
                                                          int j, int nwords, float *__restrict__ Eslab,
                                                          float *__restrict__ What,
                                                          uint32_t *__restrict__ codes,
                                                          float *__restrict__ tile_err) {
    const int idx = blockIdx.x * 256 + threadIdx.x;
    const int r = idx / G, c = idx % G;
    if (r >= m) return;
    const float w = (float)slab[(size_t)r * G + c];
    const size_t at = (size_t)r * n + j * G + c;
    Eslab[(size_t)r * G + c] = W[at] - w;
    if (What) What[at] = w;
    const int tn = n / G;
    if (idx < (m / TX) * nwords) {
        const int I = idx / nwords, wd = idx % nwords;
        codes[((size_t)I * tn + j) * nwords + wd] = slab_codes[idx];
    }
    if (tile_err && idx < m / TX) tile_err[(size_t)idx * tn + j] = slab_err[idx];
}

size_t align256(size_t b) { return (b + 255) / 256 * 256; }

}  // namespace

size_t block_ldl_workspace(int n) { return 2 * align256((size_t)n * n * sizeof(double)); }

template <int G>
static hipError_t block_ldl_t(const double *H, int n, float *A, double *Dout, void *ws, hipStream_t st) {
    double *T = (double *)ws;
    double *Ms = (double *)((char *)ws + align256((size_t)n * n * sizeof(double)));
    const int nb = n / 16;
    // T behind the first panel beside that panel's chain, if a quarter of the CUs is idle there.
    const bool late = nb > LDL_PANEL && nb - LDL_PANEL <= CUS * 3 / 4;
    const int columns = late ? LDL_PANEL : nb;
    hipLaunchKernelGGL(ldl_init_kernel, dim3(((columns + 3) / 4 * nb + 3) / 4), dim3(256), 0, st, H, T, A, n, columns);
    for (int J0 = 0; J0 < nb; J0 += LDL_PANEL) {
        const int below = nb - J0 - LDL_PANEL;  // block rows below the panel
        // as few rows per workgroup as keep it at one workgroup per CU: they take the matrix cores from the chain
        const int rows = below <= 256 ? 1 : below <= 512 ? 2 : 4;
        const int groups = below > 0 ? (below + rows - 1) / rows : 1, waves = ldl_waves(rows);
        // 2 x 2 blocks per wave while that is half a wave per SIMD; single blocks, a shorter chain, otherwise
        const int p2 = J0 > 0 && below > 0 ? (below + 1) / 2 : 0, pairs2 = p2 * (p2 + 1) / 2;
        const int pairs = rows > 1 || pairs2 >= 512 ? pairs2 : p2 > 0 ? below * (below + 1) / 2 : 0;
        // Workgroups beside the chain: no more than there are CUs for, if that is at least half of them.
        const int idle = CUS - groups;
        int beside = J0 == 0 && late ? idle : (pairs + waves - 1) / waves;
        if (idle > 0 && beside > idle && beside <= 2 * idle) beside = idle;
        const dim3 grid(groups + beside), block(waves * 64);
        const double *const behind = J0 == 0 && late ? H : nullptr;
#define QTIP_LDL_PANEL(TB, ROWS) \
    hipLaunchKernelGGL((ldl_panel_kernel<G, TB, ROWS>), grid, block, 0, st, T, Ms, A, n, J0, groups, pairs, Dout, behind)
        if (rows == 4) QTIP_LDL_PANEL(2, 4);
        else if (rows == 2) QTIP_LDL_PANEL(2, 2);
        else if (pairs2 >= 512) QTIP_LDL_PANEL(2, 1);
        else QTIP_LDL_PANEL(1, 1);
#undef QTIP_LDL_PANEL
        if (below > 0)
            hipLaunchKernelGGL(ldl_update_panel_kernel, dim3(below * LDL_PANEL), dim3(256), 0, st, T, (const double *)Ms, nb, J0);
    }
    return hipGetLastError();
}

hipError_t launch_block_ldl(const double *H, int n, int g, float *A, double *Dout, void *ws, hipStream_t st) {
    return g == 8 ? block_ldl_t<8>(H, n, A, Dout, ws, st) : block_ldl_t<16>(H, n, A, Dout, ws, st);
}

// Workspace of the loop: the running sum X (m x n), the error slab (m x G), the decoded
// slab (fp16 m x G), the slab's codes and errors, then the Viterbi quantizer's own workspace.
static size_t ldlq_fixed_bytes(int m, int n, int k, int G, int TX) {
    return align256((size_t)m * n * 4) + align256((size_t)m * G * 4) + align256((size_t)m * G * 2) +
           align256((size_t)(m / TX) * 8 * k * 4) + align256((size_t)(m / TX) * 4);
}

// (sized for 16 x 16 blocks, which is also enough for 32 x 8)
size_t quantize_ldlq_workspace(int m, int n, int k, int V, long tiles) {
    if (tiles > m / 16) tiles = m / 16;
    return ldlq_fixed_bytes(m, n, k, 16, 16) + quantize_gpu_workspace(k, V, tiles);
}

template <int G, int TX>
static hipError_t quantize_ldlq_t(int k, int code_id, const float *W, const float *A, int m, int n,
                                  const uint32_t *lut, uint32_t *codes, float *What, float *tile_err,
                                  void *ws, size_t ws_bytes, hipStream_t st) {
    char *p = (char *)ws;
    float *X = (float *)p;
    p += align256((size_t)m * n * 4);
    float *Eslab = (float *)p;
    p += align256((size_t)m * G * 4);
    half_t *slab = (half_t *)p;
    p += align256((size_t)m * G * 2);
    uint32_t *slab_codes = (uint32_t *)p;
    p += align256((size_t)(m / TX) * 8 * k * 4);
    float *slab_err = (float *)p;
    p += align256((size_t)(m / TX) * 4);
    const size_t fixed = ldlq_fixed_bytes(m, n, k, G, TX);
    if (ws_bytes <= fixed) return hipErrorInvalidValue;
    const size_t qbytes = ws_bytes - fixed;
    const int nwords = 8 * k;
    const dim3 egrid((m * G + 255) / 256);
    hipLaunchKernelGGL(ldlq_copy_kernel, dim3(1024), dim3(256), 0, st, W, X, (size_t)m * n);
    for (int j = n / G - 1; j >= 0; j--) {
        // column block j of X is complete: quantize it in place (row stride n)
        hipError_t e = launch_quantize_gpu(k, code_id, X + (size_t)j * G, m, G, n, lut, slab_codes, slab_err, p,
                                           qbytes, st);
        if (e != hipSuccess) return e;
        e = launch_dequantize(k, code_id, slab_codes, lut, m, G, slab, st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((ldlq_finish_kernel<G, TX>), egrid, dim3(256), 0, st, W, (const half_t *)slab,
                           (const uint32_t *)slab_codes, (const float *)slab_err, m, n, j, nwords, Eslab, What,
                           codes, tile_err);
        if (j > 0)
            hipLaunchKernelGGL(ldlq_update_kernel<G>, dim3((j * G + 255) / 256, (m + UPD_ROWS - 1) / UPD_ROWS),
                               dim3(256), 0, st, (const float *)Eslab, A, m, n, j, X);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_quantize_ldlq(int k, int V, int code_id, const float *W, const float *A, int m, int n,
                                const uint32_t *lut, uint32_t *codes, float *What, float *tile_err,
                                void *ws, size_t ws_bytes, hipStream_t st) {
    (void)V;
    if (code_id == CODE_LUT)
        return quantize_ldlq_t<8, 32>(k, code_id, W, A, m, n, lut, codes, What, tile_err, ws, ws_bytes, st);
    return quantize_ldlq_t<16, 16>(k, code_id, W, A, m, n, lut, codes, What, tile_err, ws, ws_bytes, st);
}

}  // namespace qtip
