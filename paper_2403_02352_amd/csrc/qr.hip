// r×r pieces of the CholeskyQR orthonormalisation (fp32, batched over sequences).
// The orthonormal factor they lead to is the U of Eq.5 (UᵀU = I, text after Eq.8).
//
//  (r below is padded to a multiple of 4 by the caller, see prepare_kernel)
//  1. gram_prepare: sum the split-K partial Gram matrices, Jacobi-scale them to unit diagonal
//     (S' = D·S·D, D = diag(S)^-1/2), add the shift, and initialise the work matrices.
//  2. factor_inverse: blocked right-looking Cholesky of S' = L·Lᵀ carried out on the augmented
//     matrix [S'; I], which yields [L; L^-T] at once: the triangular inverse needs no second
//     sweep.  One launch per 64-wide block column j: the tiles of block column j first apply the
//     rank-64 update of panel j-1 and are then eliminated against the diagonal tile (recomputed
//     redundantly by each of them, so a launch has no internal dependencies).  The trailing tiles
//     are updated lazily: on odd j only block column j+1 (the next panel) is brought up to date, on
//     even j every trailing tile applies the two panels it lacks (j-2 and j-1) in one visit, which
//     halves the passes over the trailing matrix.  The inverse comes out as Binv[n][k] = (L^-1)[n][k]·D[k], the
//     B operand of the product Z·R^-1 that the GEMM kernel then applies to the tall matrix.
//  3. factor_inverse_dataflow: the same factorisation as ONE launch of co-resident workgroups that keep
//     their tiles in registers and hand finished panel tiles to each other through global memory (second
//     half of this file); the form used whenever the whole batch fits one launch.
//  4. factor_inverse_single: 1 and the factorisation of a single block column (r <= 64), one workgroup per item and no hand-over.
#include "common.h"

#include <algorithm>
#include <utility>

namespace atp {
namespace {

constexpr int NB = 64;  // block size of the factorisation

// development aid: with ATP_DF_TRACE defined (never in the library build) item 0 records time stamps
#ifdef ATP_DF_TRACE
__device__ long long g_df_trace[1024];
#define DF_STAMP(idx) do { if (blockIdx.y == 0 && threadIdx.x == 0) g_df_trace[idx] = wall_clock64(); } while (0)
#else
#define DF_STAMP(idx) do { } while (0)
#endif

// ---------------------------------------------------------------------------
// Set-up of one factorisation, one workgroup per 64×64 tile (ti, tj); r is a multiple of 4 (the caller pads to it), of which the
// first r_true rows and columns belong to the matrix:
//   dinv[j] = 1/sqrt(sum_p Spart[p][j][j])   (1 if the diagonal entry is not positive and finite)
//   S'[i][j] = (sum_p Spart[p][i][j])·dinv[i]·dinv[j] (+ shift on the diagonal)   for tj <= ti
//              (the Gram kernel fills the lower 256×256 tiles of the partial sums only); padding is a unit diagonal, which leaves
//              the factorisation of the rest as it is and never raises `info`;
//   Y = I on the tiles with tj >= ti (null: the single-launch factorisation needs no start value);
//   Binv = 0 where the factorisation never writes but the product Z·R^-1 reads: tj > ti, and, unless
//   zero_all is set, only inside the 256-wide diagonal block (the MFMA product stops its K loop at
//   the end of the diagonal block of a triangular operand).
// NaN entries become the one that arithmetic makes.
// Also clears the item's hand-over flags of the single-launch factorisation (flags may be null) and arms its exchange slots (wx: wx_words words
// per item are set to the "not written yet" pattern).
// HBM-bound (nparts reads of the lower triangle).  Every tile forms the 128 scale factors it needs itself: the 128·nparts diagonal
// loads travel with the tile's own and come from L2, where a launch of its own for dinv cost 5 µs per factorisation.
// NP = number of partial sums, a constant so that all loads of a thread are in flight together.
template <int NP>
__global__ void __launch_bounds__(256) prepare_kernel(const float* __restrict__ Sp, int64_t pstride, float* __restrict__ S,
                                                      float* __restrict__ dinv, float* __restrict__ Y, float* __restrict__ Binv,
                                                      bf16_t* __restrict__ Bh, bf16_t* __restrict__ Bl, int r, int r_true, float shift,
                                                      int zero_all, unsigned* __restrict__ flags, int flag_words, uint4* __restrict__ wx,
                                                      int wx_words) {
    __shared__ float sc[2][NB];
    const int b = blockIdx.z, ti = blockIdx.y, tj = blockIdx.x, tid = threadIdx.x;
    const int64_t base = (int64_t)b * r * r;
    if (flags) {
        const int first = (ti * gridDim.x + tj) * 256 + tid, step = gridDim.x * gridDim.y * 256;
        for (int e = first; e < flag_words; e += step) flags[(int64_t)b * flag_words + e] = 0u;
        const uint4 unset = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
        for (int e = first; e < wx_words / 4; e += step) wx[(int64_t)b * (wx_words / 4) + e] = unset;
    }
    const int j = tj * NB + (tid & 15) * 4;
    if (tj <= ti) {
        f32x4 s[4], part[NP][4];
        float dg = 0.f, dpart[NP];
        const int k = (tid < NB ? ti : tj) * NB + (tid & 63);   // diagonal entry of the first 128 threads
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const float* src = Sp + (int64_t)p * pstride + base;
            dpart[p] = (tid < 2 * NB && k < r) ? src[(int64_t)k * r + k] : 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = ti * NB + (tid >> 4) + 16 * q;
                part[p][q] = (i < r && j < r) ? *reinterpret_cast<const f32x4*>(src + (int64_t)i * r + j) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) s[q] = part[0][q];
        dg = dpart[0];
#pragma unroll
        for (int p = 1; p < NP; ++p) {
            dg += dpart[p];
#pragma unroll
            for (int q = 0; q < 4; ++q) s[q] += part[p][q];
        }
        if (tid < 2 * NB) {
            const float di = (dg > 0.f && dg < 3.0e38f) ? 1.0f / sqrtf(dg) : 1.0f;
            sc[tid >> 6][tid & 63] = di;
            if (ti == tj && tid < NB && k < r) dinv[(int64_t)b * r + k] = di;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int li = (tid >> 4) + 16 * q, i = ti * NB + li;
            if (i >= r || j >= r) continue;
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float t = s[q][e] * sc[0][li], dj = sc[1][(tid & 15) * 4 + e];
                v[e] = t * dj;
                if (i == j + e) v[e] = i < r_true ? fmaf(t, dj, shift) : 1.f + shift;   // the diagonal rounds once
                if (v[e] != v[e]) v[e] = __uint_as_float(0x7fc00000u);                  // (the exchange slots reserve another NaN)
            }
            *reinterpret_cast<f32x4*>(S + base + (int64_t)i * r + j) = v;
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int i = ti * NB + (tid >> 4) + 16 * q;
        if (i >= r || j >= r) continue;
        const int64_t o = base + (int64_t)i * r + j;
        if (Y && tj >= ti) {
            f32x4 e;
#pragma unroll
            for (int v = 0; v < 4; ++v) e[v] = (i == j + v) ? 1.f : 0.f;
            *reinterpret_cast<f32x4*>(Y + o) = e;
        }
        if (tj > ti && (zero_all || (i >> 8) == (j >> 8))) {
            if (Binv) *reinterpret_cast<f32x4*>(Binv + o) = f32x4{0.f, 0.f, 0.f, 0.f};
            if (Bh) {
                *reinterpret_cast<uint2*>(Bh + o) = make_uint2(0u, 0u);
                *reinterpret_cast<uint2*>(Bl + o) = make_uint2(0u, 0u);
            }
        }
    }
}

// Joint right-looking elimination of the two 64×64 tiles, four columns per step (the block index
// is a compile-time constant so that the half tile row each thread keeps in registers is indexed
// statically).   reg[t] = T_sel[a][2t + half].
//   exchange 1: the raw values of the 4 block columns of every row (both tiles);
//   every thread then factors the 4×4 pivot block redundantly and reduces its own row:
//     x_k = current value of T[a][4B+k] after columns 4B .. 4B+k-1 are eliminated, f_k = x_k / piv_k;
//   exchange 2: the x_k of the diagonal tile's rows;
//   trailing columns cc > 4B+3:  T[a][cc] -= sum_k f_k(a) · x_k(cc).
// Columns stay unscaled until they are final (L[a][c] = x_c(a) / sqrt(piv_c)).
// A pivot at or below PIVOT_DROP (the scaled Gram matrix has unit diagonal; rounding noise of its entries is
// ~1e-5) means the column has no energy left beyond noise: the column is dropped (its multipliers and its
// column of L / row of L^-1 are zero) instead of being divided by, so nothing can grow without bound and
// every output stays finite.  Such a pivot is always below the level that sets `info`.
constexpr float PIVOT_DROP = 1e-6f;
__device__ __forceinline__ float drop_rcp(float piv) { return piv > PIVOT_DROP ? __builtin_amdgcn_rcpf(piv) : 0.f; }
__device__ __forceinline__ float drop_rsq(float piv) { return piv > PIVOT_DROP ? __builtin_amdgcn_rsqf(piv) : 0.f; }

struct ElimLds {
    float4 raw[2][2][NB];  // [buffer][tile][row]
    float4 xs[2][NB];      // [buffer][row of the diagonal tile]
};

template <int B>
__device__ __forceinline__ void elim_block(float (&reg)[32], ElimLds& L, int sel, int half, int a, float flag_below,
                                           int& bad_col) {
    constexpr int buf = B & 1;
    {
        float* w = reinterpret_cast<float*>(&L.raw[buf][sel][a]);
        w[half] = reg[2 * B];
        w[half + 2] = reg[2 * B + 1];
    }
    __syncthreads();
    const float4 p0 = L.raw[buf][0][4 * B + 0], p1 = L.raw[buf][0][4 * B + 1];
    const float4 p2 = L.raw[buf][0][4 * B + 2], p3 = L.raw[buf][0][4 * B + 3];
    const float4 R = L.raw[buf][sel][a];
    // pivot block: xp[i][k] = x_k of pivot row i (lower triangle), piv_k = xp[k][k]
    const float piv0r = p0.x;
    const float i0 = drop_rcp(piv0r);
    const float x10 = p1.x, x20 = p2.x, x30 = p3.x;
    const float piv1r = fmaf(-x10 * i0, x10, p1.y);
    const float i1 = drop_rcp(piv1r);
    const float x21 = fmaf(-x20 * i0, x10, p2.y);
    const float x31 = fmaf(-x30 * i0, x10, p3.y);
    const float piv2r = fmaf(-x21 * i1, x21, fmaf(-x20 * i0, x20, p2.z));
    const float i2 = drop_rcp(piv2r);
    const float x32 = fmaf(-x31 * i1, x21, fmaf(-x30 * i0, x20, p3.z));
    const float piv3r = fmaf(-x32 * i2, x32, fmaf(-x31 * i1, x31, fmaf(-x30 * i0, x30, p3.w)));
    const float i3 = drop_rcp(piv3r);
    if (bad_col < 0) {
        if (!(piv0r >= flag_below)) bad_col = 4 * B;
        else if (!(piv1r >= flag_below)) bad_col = 4 * B + 1;
        else if (!(piv2r >= flag_below)) bad_col = 4 * B + 2;
        else if (!(piv3r >= flag_below)) bad_col = 4 * B + 3;
    }
    // own row
    const float x0 = R.x, f0 = x0 * i0;
    const float x1 = fmaf(-f0, x10, R.y), f1 = x1 * i1;
    const float x2 = fmaf(-f1, x21, fmaf(-f0, x20, R.z)), f2 = x2 * i2;
    const float x3 = fmaf(-f2, x32, fmaf(-f1, x31, fmaf(-f0, x30, R.w))), f3 = x3 * i3;
    if (sel == 0 && half == 0) L.xs[buf][a] = make_float4(x0, x1, x2, x3);
    // final (scaled) values of the block columns owned by this thread
    reg[2 * B] = (half ? x1 * drop_rsq(piv1r) : x0 * drop_rsq(piv0r));
    reg[2 * B + 1] = (half ? x3 * drop_rsq(piv3r) : x2 * drop_rsq(piv2r));
    __syncthreads();
#pragma unroll
    for (int t = 2 * B + 2; t < 32; ++t) {
        const float4 d = L.xs[buf][2 * t + half];
        reg[t] = fmaf(-f3, d.w, fmaf(-f2, d.z, fmaf(-f1, d.y, fmaf(-f0, d.x, reg[t]))));
    }
    __builtin_amdgcn_sched_barrier(0);  // keep the steps apart: no hoarding of values in registers
}


// ---------------------------------------------------------------------------
// W = L^-T of one 64×64 symmetric positive definite tile T = L·Lᵀ, for the single-launch
// factorisation (L itself is not needed there).  The elimination of [T; I] above, 16 columns per stage, arranged for latency:
//  * row a of T is dead once its 16-column block has been eliminated, and row a of the identity part is born in that stage, so
//    64 rows are live throughout;
//  * wave 0 eliminates the 16 columns of a stage by itself, a live row per lane.  The 16 pivot rows are held by each of its
//    four rows of 16 lanes as well: x_k(c) reaches the lanes as the broadcast operand of the multiply-add (DPP), so a pivot
//    costs no LDS exchange and no barrier;
//  * the columns to the right take the 16 multipliers at once, T -= f·xᵀ on the matrix cores, a 16-row group per wave, the next
//    stage's columns first.  The fp32 matrix instruction adds its products one by one in the order of the pivots, so every entry is the same
//    chain of multiply-adds as column by column;
//  * the other columns, the scaling of the final ones and their stores run in waves 1 to 3 while wave 0 is in the next stage;
//  * the stages are one loop: the code runs cold in every workgroup, and four copies of it took 2.4 µs to fetch.
// A chain of 64 pivots: 3050 cycles per stage, 1700 of them the panel of 16 columns in one wave, bound by instruction issue (about 21 per pivot
// at 4.5 cycles), the rest the update of the next stage's columns on the matrix cores, two barriers and two round trips through LDS.
// ---------------------------------------------------------------------------
constexpr int EP = 20;   // row pitch of a 64×16 column block in LDS (16-byte aligned rows; reads and writes of 16 rows fall into different banks)
struct alignas(16) Elim2Lds {
    float raw[NB][EP];      // the 16 columns of the next stage
    float unit[16][EP];     // rows of the identity, as they are born
    float xs[2][NB][EP];    // [stage % 2][row]: x_k of the live rows
    float piv[4][16];       // [stage]: the pivots
    float ninv[4][16];      // -1/pivot, 0 where it is dropped
    int stored;             // waves whose part of the published tile has arrived
};

__device__ __forceinline__ void df_st16(float* p, f32x4 v);
__device__ __forceinline__ void df_stores_done();

// lane C of each row of 16 lanes, to all lanes of that row
template <int C>
__device__ __forceinline__ float row_bcast(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + C, 0xf, 0xf, true));
}
// d += m·(lane C of the row of s).  A DPP operand must not have been written by the two instructions before; the compiler does not look into
// these statements, so the order that keeps the distance is written out below (they are volatile and stay in it).
template <int C>
__device__ __forceinline__ void fma_bcast(float& d, float s, float m) {
    asm volatile("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(d) : "v"(s), "v"(m), "n"(C));
}

// columns C .. 15 take the multipliers of pivot K
template <int K, int C>
__device__ __forceinline__ void elim2_row(float (&D)[16], float (&P)[16], float nd, float np) {
    if constexpr (C < 16) {
        fma_bcast<C>(D[C], D[K], nd);
        fma_bcast<C>(P[C], D[K], np);
        elim2_row<K, C + 1>(D, P, nd, np);
    }
}

// Pivot K of a stage: D the pivot rows, P the live row of the lane, ninv = -1/pivot (0: dropped); next and piv: those of pivot K+1.  Column K+1 of the pivot rows
// comes first, and the reciprocal of the next pivot is on its way while the other columns follow.  The distances that the hardware does not
// keep by itself: two instructions from the write of a register to its DPP read and from a compare to the select, one after a reciprocal.
#define ATP_FMA_BCAST(d, s, m, c) "v_fmac_f32_dpp " d ", " s ", " m " row_newbcast:" c " row_mask:0xf bank_mask:0xf\n\t"
#define ATP_DPP(op, d, s, c) op " " d ", " s " row_newbcast:" c " row_mask:0xf bank_mask:0xf\n\t"
template <int K>
__device__ __forceinline__ void elim2_pivot(float (&D)[16], float (&P)[16], float ninv, float& next, float& piv) {
    float nd, np, rcp;
    if constexpr (K <= 12) {
        asm volatile("v_mul_f32 %[nd], %[dk], %[n]\n\tv_mul_f32 %[np], %[pk], %[n]\n\t"
                     ATP_FMA_BCAST("%[d1]", "%[dk]", "%[nd]", "%[c1]") ATP_FMA_BCAST("%[p1]", "%[dk]", "%[np]", "%[c1]")
                     ATP_FMA_BCAST("%[d2]", "%[dk]", "%[nd]", "%[c2]")
                     ATP_DPP("v_rcp_f32_dpp", "%[rcp]", "%[d1]", "%[c1]") ATP_DPP("v_mov_b32_dpp", "%[piv]", "%[d1]", "%[c1]")
                     ATP_FMA_BCAST("%[p2]", "%[dk]", "%[np]", "%[c2]")
                     "v_cmp_lt_f32 vcc, %[drop], %[piv]\n\t"
                     ATP_FMA_BCAST("%[d3]", "%[dk]", "%[nd]", "%[c3]") ATP_FMA_BCAST("%[p3]", "%[dk]", "%[np]", "%[c3]")
                     "v_cndmask_b32 %[next], 0, -%[rcp], vcc"
                     : [nd] "=&v"(nd), [np] "=&v"(np), [d1] "+v"(D[K + 1]), [p1] "+v"(P[K + 1]), [d2] "+v"(D[K + 2]), [p2] "+v"(P[K + 2]),
                       [d3] "+v"(D[K + 3]), [p3] "+v"(P[K + 3]), [rcp] "=&v"(rcp), [piv] "=&v"(piv), [next] "=&v"(next)
                     : [dk] "v"(D[K]), [pk] "v"(P[K]), [n] "v"(ninv), [drop] "s"(PIVOT_DROP), [c1] "n"(K + 1), [c2] "n"(K + 2), [c3] "n"(K + 3)
                     : "vcc");
        elim2_row<K, K + 4>(D, P, nd, np);
    } else if constexpr (K == 13) {
        asm volatile("v_mul_f32 %[nd], %[dk], %[n]\n\tv_mul_f32 %[np], %[pk], %[n]\n\t"
                     ATP_FMA_BCAST("%[d1]", "%[dk]", "%[nd]", "14") ATP_FMA_BCAST("%[p1]", "%[dk]", "%[np]", "14")
                     ATP_FMA_BCAST("%[d2]", "%[dk]", "%[nd]", "15")
                     ATP_DPP("v_rcp_f32_dpp", "%[rcp]", "%[d1]", "14") ATP_DPP("v_mov_b32_dpp", "%[piv]", "%[d1]", "14")
                     ATP_FMA_BCAST("%[p2]", "%[dk]", "%[np]", "15")
                     "v_cmp_lt_f32 vcc, %[drop], %[piv]\n\ts_nop 1\n\t"
                     "v_cndmask_b32 %[next], 0, -%[rcp], vcc"
                     : [nd] "=&v"(nd), [np] "=&v"(np), [d1] "+v"(D[14]), [p1] "+v"(P[14]), [d2] "+v"(D[15]), [p2] "+v"(P[15]), [rcp] "=&v"(rcp),
                       [piv] "=&v"(piv), [next] "=&v"(next)
                     : [dk] "v"(D[13]), [pk] "v"(P[13]), [n] "v"(ninv), [drop] "s"(PIVOT_DROP)
                     : "vcc");
    } else {
        asm volatile("v_mul_f32 %[nd], %[dk], %[n]\n\tv_mul_f32 %[np], %[pk], %[n]\n\t"
                     ATP_FMA_BCAST("%[d1]", "%[dk]", "%[nd]", "15") ATP_FMA_BCAST("%[p1]", "%[dk]", "%[np]", "15")
                     "s_nop 0\n\t"
                     ATP_DPP("v_rcp_f32_dpp", "%[rcp]", "%[d1]", "15") ATP_DPP("v_mov_b32_dpp", "%[piv]", "%[d1]", "15")
                     "v_cmp_lt_f32 vcc, %[drop], %[piv]\n\ts_nop 1\n\t"
                     "v_cndmask_b32 %[next], 0, -%[rcp], vcc\n\ts_nop 1"   // (the last wait is for what follows)
                     : [nd] "=&v"(nd), [np] "=&v"(np), [d1] "+v"(D[15]), [p1] "+v"(P[15]), [rcp] "=&v"(rcp), [piv] "=&v"(piv), [next] "=&v"(next)
                     : [dk] "v"(D[14]), [pk] "v"(P[14]), [n] "v"(ninv), [drop] "s"(PIVOT_DROP)
                     : "vcc");
    }
}
#undef ATP_FMA_BCAST
#undef ATP_DPP

template <int... Ks>
__device__ __forceinline__ void elim2_panel(std::integer_sequence<int, Ks...>, float (&D)[16], float (&P)[16], float (&ninv)[16], float (&piv)[16]) {
    piv[0] = row_bcast<0>(D[0]);
    ninv[0] = -drop_rcp(piv[0]);
    (elim2_pivot<Ks>(D, P, ninv[Ks], ninv[Ks + 1], piv[Ks + 1]), ...);
}

// the 16-row group of the diagonal tile that a wave works on: wave 0 has the one with the least to do besides the next stage's columns
__device__ __forceinline__ int elim2_group(int wave) { return wave < 2 ? 1 - wave : wave; }

// All 256 threads.  `acc[j]`: rows 16g .. 16g+15 of T (g = elim2_group(wave)), columns 16j .. 16j+15, in the C layout of the 16×16 product
// (column lane % 16, rows 4·(lane / 16) .. +3); only the lower 16×16 tiles are used.  Columns from `cols` on are those of the identity.
// W leaves in `Wt` (upper triangular, zeros below) and in `slot` (may be null), the exchange slot: four groups of 16 columns, group q at slot + 1024·q, as
// operands of the 16×16×4 product: [row / 16][(row / 4) % 4][column][row % 4].  Each is sent when its stage is over, so the workgroup that
// consumes W works through it behind this elimination.
// `store` is called by waves 1 to 3 in the first stage; `publish` (may be null) is the hand-over flag of what it stores, raised in the
// second, by when the stores have completed.
// Returns the first column whose pivot is below `flag_below`, else -1.  Ends with a block barrier.
template <class F>
__device__ __forceinline__ int diag_inverse_factor(const f32x4 (&acc)[4], float (*Wt)[NB + 1], Elim2Lds& L, int tid, int cols, float flag_below,
                                                   float* slot, unsigned* publish, F store) {
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), g = elim2_group(w), l16 = lane & 15, kq = lane >> 4;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 right[3] = {acc[1], acc[2], acc[3]};       // the column groups after the stage's
    float A[4];
    const int stages = cols > 48 ? 4 : (cols + 15) / 16;
    const auto write_columns = [&](const f32x4& c) {
#pragma unroll
        for (int v = 0; v < 4; ++v) L.raw[16 * g + 4 * kq + v][l16] = c[v];
    };
    // operands of T -= f·xᵀ: lane (l16, kq) holds k = 4s + kq of row l16 of a 16-row group
    const auto update = [&](f32x4& c, int B, int group) {
        const float* x = &L.xs[B & 1][16 * group + l16][kq];
#pragma unroll
        for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f32_16x16x4f32(A[s], x[4 * s], c, 0, 0, 0);
    };
    const auto next_columns = [&](int B) {
        const float *f = &L.xs[B & 1][16 * g + l16][kq], *n = &L.ninv[B][kq];
#pragma unroll
        for (int s = 0; s < 4; ++s) A[s] = f[4 * s] * n[4 * s];
        update(right[0], B, B + 1);
        write_columns(right[0]);
        right[0] = right[1];
        right[1] = right[2];
        __syncthreads();   // the next stage's columns are in raw
    };
    const auto send = [&](int B, int rg) {   // columns 16B .. 16B+15 of row group rg, 0 where the rows are still those of T
        const float scale = drop_rsq(L.piv[B][l16]);
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = rg <= B ? L.xs[B & 1][16 * rg + 4 * kq + e][l16] * scale : 0.f;
        if (slot) df_st16(slot + 1024 * B + 256 * rg + 4 * lane, v);
#pragma unroll
        for (int e = 0; e < 4; ++e) Wt[16 * rg + 4 * kq + e][16 * B + l16] = v[e];
    };
    const auto raise = [&]() {   // the last of three waves
        df_stores_done();
        if (lane == 0 && atomicAdd(&L.stored, 1) == 2) __hip_atomic_store(publish, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    write_columns(acc[0]);
    L.unit[tid >> 4][tid & 15] = (tid >> 4) == (tid & 15) ? 1.f : 0.f;
    if (tid == 0) L.stored = 0;
    if (tid < NB) L.piv[tid >> 4][tid & 15] = 1.f;   // stages that are left out
    __syncthreads();
    if (w == 0) {
#pragma unroll 1
        for (int B = 0;; ++B) {
            float D[16], P[16], ninv[16], piv[16];
            // the lane's live row; group B, whose rows are born, from the identity
            const float* dp = L.raw[16 * B + l16];
            const float* pp = kq == B ? L.unit[l16] : L.raw[lane];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 d4 = *reinterpret_cast<const float4*>(dp + 4 * q), p4 = *reinterpret_cast<const float4*>(pp + 4 * q);
                D[4 * q] = d4.x; D[4 * q + 1] = d4.y; D[4 * q + 2] = d4.z; D[4 * q + 3] = d4.w;
                P[4 * q] = p4.x; P[4 * q + 1] = p4.y; P[4 * q + 2] = p4.z; P[4 * q + 3] = p4.w;
            }
            if (B == 1) right[0] = right[1] = zero;   // this wave's rows are born
            if (B == 2) update(right[0], 1, 3);       // and their columns 48 .. 63 were left
            elim2_panel(std::make_integer_sequence<int, 15>{}, D, P, ninv, piv);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                *reinterpret_cast<f32x4*>(&L.xs[B & 1][lane][4 * q]) = f32x4{P[4 * q], P[4 * q + 1], P[4 * q + 2], P[4 * q + 3]};
                *reinterpret_cast<f32x4*>(&L.ninv[B][4 * q]) = f32x4{ninv[4 * q], ninv[4 * q + 1], ninv[4 * q + 2], ninv[4 * q + 3]};
                *reinterpret_cast<f32x4*>(&L.piv[B][4 * q]) = f32x4{piv[4 * q], piv[4 * q + 1], piv[4 * q + 2], piv[4 * q + 3]};
            }
            __syncthreads();
            if (B + 1 == stages) break;
            next_columns(B);
        }
    } else {
#pragma unroll 1
        for (int B = 0;; ++B) {
            if (B == 1 && publish) raise();
            if (B > 0) {
                if (B < 3) update(right[0], B - 1, B + 1);
                if (B == 1) update(right[1], 0, 3);
                send(B - 1, w);
                if (w == 1) send(B - 1, 0);
            } else {
                store();
            }
            if (B == g) right[0] = right[1] = right[2] = zero;   // rows that are born in this stage start from zero
            __syncthreads();
            if (B + 1 == stages) break;
            next_columns(B);
        }
    }
    send(stages - 1, w);
    for (int q = stages; q < 4; ++q) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) Wt[16 * w + 4 * kq + e][16 * q + l16] = v[e] = w == q && 4 * kq + e == l16 ? 1.f : 0.f;
        if (slot) df_st16(slot + 1024 * q + 256 * w + 4 * lane, v);
    }
    const uint64_t bad = __builtin_amdgcn_ballot_w64(!(L.piv[kq][l16] >= flag_below));
    if (stages == 1 && w > 0 && publish) raise();
    __syncthreads();
    return bad ? (int)__builtin_ctzll(bad) : -1;
}

template <int... Bs>
__device__ __forceinline__ void elim_all(std::integer_sequence<int, Bs...>, float (&reg)[32], ElimLds& L, int sel,
                                         int half, int a, float flag_below, int& bad_col) {
    (elim_block<Bs>(reg, L, sel, half, a, flag_below, bad_col), ...);
}

// ---------------------------------------------------------------------------
// One block column of the augmented factorisation (see the header of this file).
// Tile kinds handled by a workgroup (tile = 64×64, k = its block column):
//   S-kind (i, k), i >= k >= j : tile of S'; panel operand A = L(i, j-1)
//   Y-kind (c, k), c <= k, k >= j : tile of Y (= L^-T when final); panel operand A = Y(c, j-1)
// update (j >= 1, not for the fresh identity tile Y(j, j)):  T -= A · L(k, j-1)ᵀ
// k > j : store T back.   k == j : eliminate the 64 columns of T together with the diagonal
// tile Tjj = S'(j, j) - L(j, j-1)·L(j, j-1)ᵀ and store the result as L(i, j) / Y(c, j) + Binv.
// ---------------------------------------------------------------------------
constexpr int LP = NB + 4;  // padded row length of the MFMA operand tiles (16-byte aligned rows)

// 64×64 tile -> LDS (row-major, padded), optionally negated; rows/cols past r read as zero
__device__ __forceinline__ void tile_to_lds(float (*dst)[LP], const float* __restrict__ src, int r, int row0, int col0,
                                            float sign, bool enable, int tid) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int row = (tid >> 4) + 16 * q, c4 = (tid & 15) * 4;
        const int gr = row0 + row, gc = col0 + c4;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (enable && gr < r && gc < r) v = *reinterpret_cast<const float4*>(src + (int64_t)gr * r + gc);
        *reinterpret_cast<float4*>(&dst[row][c4]) = make_float4(sign * v.x, sign * v.y, sign * v.z, sign * v.w);
    }
}

__global__ void __launch_bounds__(256, 2) factor_step_kernel(float* S, float* Lf, float* Y, const float* __restrict__ dinv,
                                                             float* Binv, bf16_t* Bh, bf16_t* Bl, int r, int nblk, int j,
                                                             int32_t* info, float flag_below) {
    // MFMA operands (-A and L(k, j-1), row-major) during the update; the tiles T and Tjj afterwards
    __shared__ __align__(16) float lds_a[NB * LP];
    __shared__ __align__(16) float lds_b[NB * LP];
    __shared__ __align__(16) ElimLds elds;
    float (*Am)[LP] = reinterpret_cast<float (*)[LP]>(lds_a);
    float (*Bm)[LP] = reinterpret_cast<float (*)[LP]>(lds_b);
    float (*As)[NB + 1] = reinterpret_cast<float (*)[NB + 1]>(lds_a);
    float (*Bs)[NB + 1] = reinterpret_cast<float (*)[NB + 1]>(lds_b);

    const int b = blockIdx.y;
    const int m = nblk - j;
    int id = blockIdx.x;
    // ---- decode the tile ----------------------------------------------------------------------
    bool ykind, panel;
    int rb, kb;  // row block (i or c) and column block k
    if (id < m) { ykind = false; panel = true; rb = j + id; kb = j; }
    else if (id < m + j + 1) { ykind = true; panel = true; rb = id - m; kb = j; }
    else if (j & 1) {
        // odd block column: only the tiles of the next block column are brought up to date
        id -= m + j + 1;
        panel = false;
        kb = j + 1;
        if (id < m - 1) { ykind = false; rb = j + 1 + id; }
        else { ykind = true; rb = id - (m - 1); }   // c in 0..j-1
    } else {
        id -= m + j + 1;
        panel = false;
        const int nt1 = m * (m - 1) / 2;  // S-kind trailing tiles (i, k), j < k <= i
        if (id < nt1) {
            ykind = false;
            // row-wise enumeration of the triangle: rows ii = 0..m-2 (i = j+1+ii) hold ii+1 tiles
            int ii = (int)((sqrtf(8.f * id + 1.f) - 1.f) * 0.5f);
            while ((ii + 1) * (ii + 2) / 2 <= id) ++ii;
            while (ii * (ii + 1) / 2 > id) --ii;
            rb = j + 1 + ii;
            kb = j + 1 + (id - ii * (ii + 1) / 2);
        } else {
            id -= nt1;
            ykind = true;
            rb = id / (m - 1);            // c in 0..j-1
            kb = j + 1 + id % (m - 1);
        }
    }
    const int64_t boff = (int64_t)b * r * r;
    float* Sb = S + boff;
    float* Lb = Lf + boff;
    float* Yb = Y + boff;
    float* own = ykind ? Yb : Sb;
    const int r0 = rb * NB, c0 = kb * NB;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    const int wr = wave >> 1, wc = wave & 1;   // 32×32 quadrant of the tile owned by this wave

    // Tiles of block column j (and j+1 on odd j) lack panel j-1 only; the other trailing tiles are
    // visited on even j only and lack panels j-2 and j-1.
    const int npanels = (j == 0) ? 0 : ((panel || (j & 1)) ? 1 : 2);
    auto stage_panel = [&](int q) {
        const int pb = j - npanels + q;            // panel block column
        const bool update = !(ykind && rb > pb);   // row rb of Y is still the identity row before block column rb
        tile_to_lds(Am, ykind ? Yb : Lb, r, r0, pb * NB, -1.f, update, tid);
        tile_to_lds(Bm, Lb, r, c0, pb * NB, 1.f, true, tid);
    };
    // the operands of the first pending update are requested first: they are needed first
    if (npanels) stage_panel(0);
    // ---- accumulators start from the own tile (and the diagonal tile) in MFMA C layout ---------------
    // C layout: element v of lane -> row 8*(v/4) + 4*lh + v%4, column l32 (within the quadrant);
    // out-of-range entries pad with the identity
    f32x16 acc, accj;
    {
        const int gc = c0 + 32 * wc + l32;
        const int rq = 32 * wr + 4 * lh;   // first row of this lane within the tile
        if (r0 + NB <= r && c0 + NB <= r) {
            // tile completely inside the matrix (the diagonal tile then is too): plain strided loads
            const float* po = own + (int64_t)(r0 + rq) * r + gc;
            const float* pj = Sb + (int64_t)(c0 + rq) * r + gc;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t o = (int64_t)(8 * (v >> 2) + (v & 3)) * r;
                acc[v] = po[o];
                accj[v] = panel ? pj[o] : 0.f;
            }
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = rq + 8 * (v >> 2) + (v & 3);
                const int gr = r0 + row, gj = c0 + row;
                acc[v] = (gr < r && gc < r) ? own[(int64_t)gr * r + gc] : ((gr == gc) ? 1.f : 0.f);
                accj[v] = 0.f;
                if (panel) accj[v] = (gj < r && gc < r) ? Sb[(int64_t)gj * r + gc] : ((gj == gc) ? 1.f : 0.f);
            }
        }
    }
    // ---- pending rank-64 updates on the matrix cores (fp32 MFMA): T -= A(·, p) · L(k, p)ᵀ ------------
    for (int q = 0; q < npanels; ++q) {
        if (q > 0) {
            __syncthreads();
            stage_panel(q);
        }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < NB / 8; ++g) {
            // lanes of half lh take k = 8g + 4*lh .. +3: one 16-byte read per operand feeds 4 MFMAs
            const float4 a4 = *reinterpret_cast<const float4*>(&Am[32 * wr + l32][8 * g + 4 * lh]);
            const float4 b4 = *reinterpret_cast<const float4*>(&Bm[32 * wc + l32][8 * g + 4 * lh]);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.x, b4.x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.y, b4.y, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.z, b4.z, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.w, b4.w, acc, 0, 0, 0);
            if (panel) {
                const float4 c4 = *reinterpret_cast<const float4*>(&Bm[32 * wr + l32][8 * g + 4 * lh]);
                accj = __builtin_amdgcn_mfma_f32_32x32x2f32(-c4.x, b4.x, accj, 0, 0, 0);
                accj = __builtin_amdgcn_mfma_f32_32x32x2f32(-c4.y, b4.y, accj, 0, 0, 0);
                accj = __builtin_amdgcn_mfma_f32_32x32x2f32(-c4.z, b4.z, accj, 0, 0, 0);
                accj = __builtin_amdgcn_mfma_f32_32x32x2f32(-c4.w, b4.w, accj, 0, 0, 0);
            }
        }
    }
    if (npanels) __syncthreads();
    if (!panel) {
        const int gc = c0 + 32 * wc + l32;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int gr = r0 + 32 * wr + 8 * (v >> 2) + 4 * lh + (v & 3);
            if (gr < r && gc < r) own[(int64_t)gr * r + gc] = acc[v];
        }
        return;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int row = 32 * wr + 8 * (v >> 2) + 4 * lh + (v & 3), col = 32 * wc + l32;
        As[row][col] = acc[v];
        Bs[row][col] = accj[v];
    }
    __syncthreads();

    // ---- joint elimination of the 64 columns; every thread keeps half a tile row in registers --
    const int sel = tid >> 7;         // 0: diagonal tile, 1: own tile
    const int a = tid & 63;           // row
    const int half = (tid >> 6) & 1;  // column parity owned (uniform per wave)
    float reg[32];
#pragma unroll
    for (int t = 0; t < 32; ++t) reg[t] = sel ? As[a][2 * t + half] : Bs[a][2 * t + half];
    int bad_col = -1;                          // first column whose pivot is below the flag level
    elim_all(std::make_integer_sequence<int, NB / 4>{}, reg, elds, sel, half, a, flag_below, bad_col);
    if (!ykind && rb == j && tid == 0 && info && bad_col >= 0 && (c0 + bad_col) < r && info[b] == 0)
        info[b] = c0 + bad_col + 1;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 32; ++t) {
        if (sel) As[a][2 * t + half] = reg[t];
        else Bs[a][2 * t + half] = reg[t];
    }
    __syncthreads();
    // ---- store ---------------------------------------------------------------------------------------
    if (!ykind) {
        const bool diag = (rb == j);
        // 16-byte row pieces
        for (int e = tid; e < NB * NB / 4; e += 256) {
            const int row = e >> 4, col = (e & 15) * 4;
            const int gr = r0 + row, gc = c0 + col;
            if (gr < r && gc < r) {
                f32x4 v;
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = diag ? ((row >= col + q) ? Bs[row][col + q] : 0.f) : As[row][col + q];
                *reinterpret_cast<f32x4*>(Lb + (int64_t)gr * r + gc) = v;
            }
        }
    } else {
        const float* db = dinv + (int64_t)b * r;
        for (int e = tid; e < NB * NB / 4; e += 256) {
            const int row = e >> 4, col = (e & 15) * 4;
            const int gr = r0 + row, gc = c0 + col;
            if (gr < r && gc < r) {
                f32x4 v;
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = As[row][col + q];
                *reinterpret_cast<f32x4*>(Yb + (int64_t)gr * r + gc) = v;
            }
        }
        if (Bh && !Binv && (r & 7) == 0) {
            // hi/lo planes of R^-1 (transposed tile): 8 consecutive rows of one column are 8 consecutive
            // bf16 of a Binv row: one 16-byte store per plane
            for (int e = tid; e < NB * NB / 8; e += 256) {
                const int col = e >> 3, row8 = (e & 7) * 8;
                const int gr = r0 + row8, gc = c0 + col;
                if (gr < r && gc < r) {   // r is a multiple of 8: the 8 rows are in range together
                    float v[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) v[q] = As[row8 + q][col] * db[gr + q];
                    uint4 h, l;
                    uint32_t* hp = reinterpret_cast<uint32_t*>(&h);
                    uint32_t* lp = reinterpret_cast<uint32_t*>(&l);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t hh = pack_bf2(v[2 * q], v[2 * q + 1]);
                        hp[q] = hh;
                        lp[q] = pack_bf2(v[2 * q] - bf2f((bf16_t)(hh & 0xffffu)), v[2 * q + 1] - bf2f((bf16_t)(hh >> 16)));
                    }
                    const int64_t o = boff + (int64_t)gc * r + gr;
                    *reinterpret_cast<uint4*>(Bh + o) = h;
                    *reinterpret_cast<uint4*>(Bl + o) = l;
                }
            }
        } else {
            for (int e = tid; e < NB * NB; e += 256) {
                const int col = e >> 6, row = e & 63;   // row fastest: consecutive addresses in Binv
                const int gr = r0 + row, gc = c0 + col;
                if (gr < r && gc < r) {
                    const float v = As[row][col] * db[gr];
                    const int64_t o = boff + (int64_t)gc * r + gr;
                    if (Binv) Binv[o] = v;
                    if (Bh) {
                        const bf16_t h = f2bf(v);
                        Bh[o] = h;
                        Bl[o] = f2bf(v - bf2f(h));
                    }
                }
            }
        }
    }
}


// ---------------------------------------------------------------------------
// Single-launch factorisation: the same augmented block factorisation as above, carried out by one
// grid of co-resident workgroups that hand tiles to each other through global memory and per-tile
// flags instead of kernel boundaries.  Every 64×64 tile lives in the accumulator registers of the
// workgroup that owns it for the whole factorisation; only finished panel tiles travel.
//
// Stacked tile rows: S-rows i (tiles S'(i,k), k <= i) and Y-rows c (tiles Y(c,k), k >= c, Y = L^-T).
//   T(rho,k) = init - sum_{p<k} P(rho,p)·L(k,p)ᵀ ,   P(rho,k) = T(rho,k)·W_k ,   W_k = L_kk^-T
// (init = S'(i,k) for S-rows, 0 for Y-rows; the sum starts at p = c for Y-row c with P(c,c) = W_c).
// Roles inside one item's group of workgroups:
//   spine workgroup i (one per block row) owns S'(i,i-2), S'(i,i-1) and S'(i,i): applies the panels p <= i-3 as
//     they appear, forms L(i,i-2) once W_{i-2} is published, brings T(i,i-1) and T(i,i) up to panel i-2, and then, once W_{i-1} is
//     published, forms L(i,i-1) and the Schur complement of the diagonal tile, factorises it together with an identity tile
//     (which yields W_i) and publishes W_i.
//     From W_{i-1} to W_i takes 9 µs at r = 1024: 6 of elimination, 0.7 for the last columns to cross, 0.8 for the quarter of L(i,i-1) and
//     of the diagonal update that depends on them, and 1.5 by which a workgroup is late for them.  With S'(i,i-2) in a bulk
//     workgroup, flags for every tile and the elimination in four-column steps it took 12.3 (r = 1024, batch 4: 204 -> 147 µs; 256: 55 -> 42);
//   bulk workgroups own the remaining tiles, dealt round-robin in order of block column so that a
//     workgroup's slots are sorted by urgency.  Step q: finalise the slots of block column q (product
//     with W_q), publish them, then apply panel q to every later slot.
// Every workgroup walks the steps in the same global order (step, block column), so the oldest
// unfinished task is always at the head of its owner's queue: no cycle of waits, provided the whole
// grid is resident (the host bounds the grid by the number of compute units).  Waits are bounded: a
// workgroup that spins too long raises the item's abort word, sets info = -1 and exits; every other
// wait of that item then ends as well.
// ---------------------------------------------------------------------------
constexpr int DF_SPIN_LIMIT = 1 << 22;   // polls of a flag, each a round trip through memory: seconds, well beyond any healthy wait
constexpr int DF_MAX_NBLK = 32;
constexpr int DF_FLAG_WORDS = 2 * DF_MAX_NBLK * DF_MAX_NBLK + 64;   // per item; the last 64 words hold the abort word
// Exchange slots: what the critical path of the factorisation waits for travels without a flag.  A slot (a dense 64×64 tile) is armed with a
// bit pattern that no number has (all ones: a NaN, and not the one that arithmetic makes; gram_prepare lets no other NaN in) before the
// launch; a consumer loads its part until no word shows the pattern any more, so a tile that is torn or partly there only looks unfinished.
// Against a flag (stores, wait for them, flag; poll, load) that saves two round trips through memory, 2 µs per hand-over.
// W_i travels in four pieces: columns of W = L^-T become final from left to right as the elimination proceeds, the producer stores a group of
// 16 columns as soon as it is final, and the next spine workgroup forms the matching 16 columns of L(i+1,i) = T(i+1,i)·W_i and their share of the
// update of its diagonal tile at once.  When the last group arrives only a quarter of that work is left.
constexpr unsigned DF_UNSET = 0xFFFFFFFFu;
// tiles of the bulk workgroups: all of S' below the third diagonal and all of Y above its diagonal
__host__ __device__ constexpr int df_bulk_tiles(int nb) { return (nb > 3 ? (nb - 2) * (nb - 3) / 2 : 0) + nb * (nb - 1) / 2; }
constexpr int DF_SLOT_WORDS = NB * NB;
enum DfSlot { DF_SLOT_W, DF_SLOT_L1, DF_SLOT_L2, DF_SLOT_L3, DF_SLOT_T, DF_SLOTS };   // of a block row i: W_i, L(i,i-1), L(i,i-2), L(i,i-3), T(i,i-1)
__host__ __device__ constexpr int df_wx_words(int nblk) { return nblk * DF_SLOTS * DF_SLOT_WORDS; }   // per item

struct DfArgs {
    float* S; float* Lf; float* Y; const float* dinv;
    float* Binv; bf16_t* Bh; bf16_t* Bl;
    unsigned* flags;
    float* wx;              // exchange slots, df_wx_words(nblk) per item
    int32_t* info;
    int r, nblk, nbulk;
    int spin_limit;         // polls before a wait gives up
    int last_by_32;         // see df_last_by_32
    float flag_below;
};


// Panel tiles travel between workgroups of one running kernel, possibly on different XCDs (each has
// an L2 of its own).  They are written and read with agent-scope ("sc1") accesses, which are coherent
// across the device by themselves: no cache-wide write-back or invalidate is needed, and ordering is
// plain completion order (s_waitcnt before the flag is raised; the flag is polled with relaxed loads).
// The loads are issued through inline assembly, both tiles of an update in flight before one wait.
// eight 16-byte loads in flight, then one wait, in ONE statement: the compiler never sees a register
// whose load is still outstanding
__device__ __forceinline__ void df_ld16x8(const float* const (&p)[8], f32x4 (&v)[8]) {
    asm volatile(
        "global_load_dwordx4 %0, %8, off sc1\n\t"
        "global_load_dwordx4 %1, %9, off sc1\n\t"
        "global_load_dwordx4 %2, %10, off sc1\n\t"
        "global_load_dwordx4 %3, %11, off sc1\n\t"
        "global_load_dwordx4 %4, %12, off sc1\n\t"
        "global_load_dwordx4 %5, %13, off sc1\n\t"
        "global_load_dwordx4 %6, %14, off sc1\n\t"
        "global_load_dwordx4 %7, %15, off sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
        : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "v"(p[4]), "v"(p[5]), "v"(p[6]), "v"(p[7])
        : "memory");
}
// A store of more than 8 bytes reads its data registers for two more cycles after it has issued; the
// compiler pads its own stores but cannot see into this statement, so the padding is part of it (without it
// the next instruction may overwrite the data registers: seen as an LDS address stored in place of a value).
__device__ __forceinline__ void df_st16(float* p, f32x4 v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void df_stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ bool df_written(const f32x4& v) {
    return __float_as_uint(v[0]) != DF_UNSET && __float_as_uint(v[1]) != DF_UNSET && __float_as_uint(v[2]) != DF_UNSET &&
           __float_as_uint(v[3]) != DF_UNSET;
}

// Column groups of W on their way from an exchange slot into the registers of a wave, in the operand order that the slot holds them in: no LDS,
// no barrier.  Group Q takes Q+1 pieces (W is upper triangular).
struct DfW { f32x4 g0[1], g1[2], g2[3], g3[4]; };
template <int Q>
__device__ __forceinline__ auto& df_group(DfW& w) {
    if constexpr (Q == 0) return w.g0;
    else if constexpr (Q == 1) return w.g1;
    else if constexpr (Q == 2) return w.g2;
    else return w.g3;
}
template <int Q>
__device__ __forceinline__ void df_load_group(DfW& w, const float* slot, int lane) {
    const float* p = slot + 1024 * Q + 4 * lane;
    auto& v = df_group<Q>(w);
    if constexpr (Q == 0)
        asm volatile("global_load_dwordx4 %0, %1, off sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(v[0]) : "v"(p) : "memory");
    else if constexpr (Q == 1)
        asm volatile("global_load_dwordx4 %0, %2, off sc1\n\tglobal_load_dwordx4 %1, %2, off offset:1024 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]) : "v"(p) : "memory");
    else if constexpr (Q == 2)
        asm volatile("global_load_dwordx4 %0, %3, off sc1\n\tglobal_load_dwordx4 %1, %3, off offset:1024 sc1\n\t"
                     "global_load_dwordx4 %2, %3, off offset:2048 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]) : "v"(p) : "memory");
    else
        asm volatile("global_load_dwordx4 %0, %4, off sc1\n\tglobal_load_dwordx4 %1, %4, off offset:1024 sc1\n\t"
                     "global_load_dwordx4 %2, %4, off offset:2048 sc1\n\tglobal_load_dwordx4 %3, %4, off offset:3072 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]) : "v"(p) : "memory");
}
// all four groups in flight together
__device__ __forceinline__ void df_load_groups(DfW& w, const float* slot, int lane) {
    const float *p0 = slot + 4 * lane, *p1 = p0 + 1024, *p2 = p0 + 2048, *p3 = p0 + 3072;
    asm volatile(
        "global_load_dwordx4 %0, %10, off sc1\n\t"
        "global_load_dwordx4 %1, %11, off sc1\n\tglobal_load_dwordx4 %2, %11, off offset:1024 sc1\n\t"
        "global_load_dwordx4 %3, %12, off sc1\n\tglobal_load_dwordx4 %4, %12, off offset:1024 sc1\n\t"
        "global_load_dwordx4 %5, %12, off offset:2048 sc1\n\t"
        "global_load_dwordx4 %6, %13, off sc1\n\tglobal_load_dwordx4 %7, %13, off offset:1024 sc1\n\t"
        "global_load_dwordx4 %8, %13, off offset:2048 sc1\n\tglobal_load_dwordx4 %9, %13, off offset:3072 sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(w.g0[0]), "=&v"(w.g1[0]), "=&v"(w.g1[1]), "=&v"(w.g2[0]), "=&v"(w.g2[1]), "=&v"(w.g2[2]), "=&v"(w.g3[0]), "=&v"(w.g3[1]),
          "=&v"(w.g3[2]), "=&v"(w.g3[3])
        : "v"(p0), "v"(p1), "v"(p2), "v"(p3)
        : "memory");
}
template <int Q>
__device__ __forceinline__ bool df_complete(DfW& w) {
    const auto& v = df_group<Q>(w);
    bool ok = true;
#pragma unroll
    for (int g = 0; g <= Q; ++g) ok = ok && df_written(v[g]);
    return __all(ok);
}

template <class F>
__device__ __forceinline__ void for_groups(F f) {
    f(std::integral_constant<int, 0>{}); f(std::integral_constant<int, 1>{}); f(std::integral_constant<int, 2>{}); f(std::integral_constant<int, 3>{});
}

// a wave's wait on an exchange slot ends without what it waits for: an eighth of the spin limit of a flag (a poll of data reads 1 to 22
// pieces of 16 bytes per lane, 1 µs and more), or the item's abort word
__device__ __forceinline__ bool df_gives_up(int spins, unsigned* abort_w, int spin_limit) {
    return spins > spin_limit / 8 || ((spins & 63) == 63 && __hip_atomic_load(abort_w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// One wave: until group Q has arrived.  What the last look at all of the slot (df_load_groups) found is used, so a consumer that comes late
// takes everything in one round trip (1 µs); one that comes early polls no more than the group it waits for.
// false = gave up (spin limit or the item's abort word).
template <int Q>
__device__ __forceinline__ bool df_wait_group(DfW& w, const float* slot, unsigned* abort_w, int spin_limit, int lane) {
    if (df_complete<Q>(w)) return true;
    df_load_groups(w, slot, lane);
    for (int spins = 0; !df_complete<Q>(w); ++spins) {
        df_load_group<Q>(w, slot, lane);
        if (df_gives_up(spins, abort_w, spin_limit)) return false;
    }
    return true;
}

// Column group Q of L = T·W for the wave's 16 rows (wave w: rows 16w..16w+15), 16×16×4 fp32 MFMA.
// T row-major [row][k] (pitch LP).  W is upper triangular: k < 16(Q+1).
// Lane (l16, kq): the MFMA step (g, e) contracts k = 16g + 4kq + e in lane group kq.
// The result goes to Lm[row][16Q + col] (pitch LP).
template <int Q>
__device__ __forceinline__ void df_l_group(float (*Lm)[LP], const float (*Tm)[LP], DfW& wv, int w, int l16, int kq) {
    const auto& v = df_group<Q>(wv);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g <= Q; ++g) {
        const float4 a4 = *reinterpret_cast<const float4*>(&Tm[16 * w + l16][16 * g + 4 * kq]);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a4.x, v[g][0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a4.y, v[g][1], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a4.z, v[g][2], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a4.w, v[g][3], acc, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) Lm[16 * w + 4 * kq + e][16 * Q + l16] = acc[e];
}

// acc[j] += L[16w.., group q]·L[16j.., group q]ᵀ for the 16×16 tiles j <= w of tile row w (the lower
// triangle is all the elimination of the diagonal tile reads)
__device__ __forceinline__ void df_syrk_group(f32x4 (&acc)[4], const float (*Lm)[LP], int q, int w, int l16, int kq) {
    const float4 a4 = *reinterpret_cast<const float4*>(&Lm[16 * w + l16][16 * q + 4 * kq]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (j > w) continue;
        const float4 b4 = *reinterpret_cast<const float4*>(&Lm[16 * j + l16][16 * q + 4 * kq]);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4.x, b4.x, acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4.y, b4.y, acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4.z, b4.z, acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4.w, b4.w, acc[j], 0, 0, 0);
    }
}

// Three 64×64 tiles, 16 bytes of each of 4 rows per thread and tile, and what has arrived of a W, all in flight together: one round trip.
// The first lies in a matrix with rows of length r, of which `rows` rows exist from it on (those behind are read as its first and count as zero),
// the others in one with rows of length ld (NB: exchange slots).
__device__ __forceinline__ void df_load_tiles(f32x4 (&v)[12], DfW& w, const float* t0, int rows, const float* t1, const float* t2, int ld,
                                              const float* slot, int r, int tid) {
    const int row = tid >> 4, c4 = (tid & 15) * 4;
    unsigned o[4], o0[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        o[q] = (unsigned)((row + 16 * q) * ld + c4) * 4u;
        o0[q] = (unsigned)((row + 16 * q < rows ? row + 16 * q : 0) * r + c4) * 4u;
    }
    const unsigned w0 = (tid & 63) * 16, w1 = w0 + 4096, w2 = w0 + 8192, w3 = w0 + 12288;
#define ATP_LD(n, off, base) "global_load_dwordx4 %" #n ", %" #off ", %" #base " sc1\n\t"
#define ATP_LDW(n, off, imm) "global_load_dwordx4 %" #n ", %" #off ", %33 offset:" #imm " sc1\n\t"
    asm volatile(
        ATP_LD(0, 22, 34) ATP_LD(1, 23, 34) ATP_LD(2, 24, 34) ATP_LD(3, 25, 34)
        ATP_LD(4, 26, 35) ATP_LD(5, 27, 35) ATP_LD(6, 28, 35) ATP_LD(7, 29, 35)
        ATP_LD(8, 26, 36) ATP_LD(9, 27, 36) ATP_LD(10, 28, 36) ATP_LD(11, 29, 36)
        ATP_LDW(12, 30, 0) ATP_LDW(13, 31, 0) ATP_LDW(14, 31, 1024) ATP_LDW(15, 32, 0) ATP_LDW(16, 32, 1024) ATP_LDW(17, 32, 2048)
        ATP_LDW(18, 37, 0) ATP_LDW(19, 37, 1024) ATP_LDW(20, 37, 2048) ATP_LDW(21, 37, 3072)
        "s_waitcnt vmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7]), "=&v"(v[8]), "=&v"(v[9]),
          "=&v"(v[10]), "=&v"(v[11]), "=&v"(w.g0[0]), "=&v"(w.g1[0]), "=&v"(w.g1[1]), "=&v"(w.g2[0]), "=&v"(w.g2[1]), "=&v"(w.g2[2]),
          "=&v"(w.g3[0]), "=&v"(w.g3[1]), "=&v"(w.g3[2]), "=&v"(w.g3[3])
        : "v"(o0[0]), "v"(o0[1]), "v"(o0[2]), "v"(o0[3]), "v"(o[0]), "v"(o[1]), "v"(o[2]), "v"(o[3]), "v"(w0), "v"(w1), "v"(w2), "s"(slot),
          "s"(t0), "s"(t1), "s"(t2), "v"(w3)
        : "memory");
#undef ATP_LD
#undef ATP_LDW
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (row + 16 * q >= rows) v[q] = f32x4{0.f, 0.f, 0.f, 0.f};
}
__device__ __forceinline__ void df_tile_to_lds(float (*dst)[LP], const f32x4 (&v)[12], int first, float sign, int tid) {
#pragma unroll
    for (int q = 0; q < 4; ++q) *reinterpret_cast<f32x4*>(&dst[(tid >> 4) + 16 * q][(tid & 15) * 4]) = v[first + q] * sign;
}

// a tile of LDS into an exchange slot (row-major)
template <int THREADS>
__device__ __forceinline__ void df_store_slot(float* slot, const float (*src)[LP], int tid) {
    constexpr int N = (NB * NB / 4 + THREADS - 1) / THREADS;
    f32x4 v[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int e = (tid + j * THREADS) & (NB * NB / 4 - 1);
        v[j] = *reinterpret_cast<const f32x4*>(&src[e >> 4][(e & 15) * 4]);
    }
#pragma unroll
    for (int j = 0; j < N; ++j)
        if (tid + j * THREADS < NB * NB / 4) df_st16(slot + 4 * (tid + j * THREADS), v[j]);
}

// One wave's part of a tile in an exchange slot, until every word of it has been written.  false = gave up.
__device__ __forceinline__ bool df_wait_tile(f32x4& v0, f32x4& v1, f32x4& v2, f32x4& v3, const float* slot, unsigned* abort_w, int spin_limit, int tid) {
    const float *p0 = slot + 4 * tid, *p1 = p0 + 1024, *p2 = p0 + 2048, *p3 = p0 + 3072;
    for (int spins = 0;; ++spins) {
        asm volatile("global_load_dwordx4 %0, %4, off sc1\n\tglobal_load_dwordx4 %1, %5, off sc1\n\t"
                     "global_load_dwordx4 %2, %6, off sc1\n\tglobal_load_dwordx4 %3, %7, off sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(v0), "=&v"(v1), "=&v"(v2), "=&v"(v3) : "v"(p0), "v"(p1), "v"(p2), "v"(p3) : "memory");
        if (__all(df_written(v0) && df_written(v1) && df_written(v2) && df_written(v3))) return true;
        if (df_gives_up(spins, abort_w, spin_limit)) return false;
    }
}

// Two 64×64 tiles (rows ra0.., columns ca0.. of Ma and rows rb0.., columns cb0.. of Mb) -> LDS, row-major
// with pitch LP; the first is multiplied by sa.  Entries outside the r×r matrix read as zero.
__device__ __forceinline__ void df_tiles_to_lds(float (*da)[LP], const float* Ma, int ra0, int ca0, float sa, float (*dbm)[LP],
                                                const float* Mb, int rb0, int cb0, bool two, int r, int tid) {
    f32x4 v[8];
    const float* ptr[8];
    bool ok[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const bool second = q >= 4;
        const int row = (tid >> 4) + 16 * (q & 3), c4 = (tid & 15) * 4;
        const int gr = (second ? rb0 : ra0) + row, gc = (second ? cb0 : ca0) + c4;
        ok[q] = (gr < r) && (gc < r) && (two || !second);
        ptr[q] = (second ? Mb : Ma) + (ok[q] ? (int64_t)gr * r + gc : 0);   // out of range: a valid address, value dropped
    }
    df_ld16x8(ptr, v);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const bool second = q >= 4;
        if (second && !two) continue;
        const int row = (tid >> 4) + 16 * (q & 3), c4 = (tid & 15) * 4;
        const float sg = second ? 1.f : sa;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
        if (ok[q]) o = v[q] * sg;
        *reinterpret_cast<f32x4*>(second ? &dbm[row][c4] : &da[row][c4]) = o;
    }
}

// one thread: wait until all three flags are up (they may be the same); the loads of a poll are in flight together
__device__ __forceinline__ bool df_poll(unsigned* f1, unsigned* f2, unsigned* f3, unsigned* abort_w, int spin_limit) {
    for (int spins = 0;; ++spins) {
        const unsigned v1 = __hip_atomic_load(f1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned v2 = __hip_atomic_load(f2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned v3 = __hip_atomic_load(f3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (v1 && v2 && v3) return true;
        if (spins > spin_limit) return false;
        if ((spins & 255) == 255 && __hip_atomic_load(abort_w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return false;
        __builtin_amdgcn_s_sleep(1);
    }
}

// acc += Am[32wr + ·][:] · (bsign · Bm[32wc + ·][:])ᵀ   (64-deep, operands row-major [row][k] in LDS)
__device__ __forceinline__ void df_mma(f32x16& acc, const float (*Am)[LP], const float (*Bm)[LP], int wr, int wc, int l32,
                                       int lh, float bsign) {
#pragma unroll
    for (int g = 0; g < NB / 8; ++g) {
        const float4 a4 = *reinterpret_cast<const float4*>(&Am[32 * wr + l32][8 * g + 4 * lh]);
        const float4 b4 = *reinterpret_cast<const float4*>(&Bm[32 * wc + l32][8 * g + 4 * lh]);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.x, bsign * b4.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.y, bsign * b4.y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.z, bsign * b4.z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.w, bsign * b4.w, acc, 0, 0, 0);
    }
}

// W as it lies in the registers of every wave -> LDS, row-major [k][n]; wave w writes column group w
__device__ __forceinline__ void df_w_to_lds(float (*Wm)[LP], DfW& wv, int w, int l16, int kq) {
    for_groups([&](auto Q) {
        constexpr int q = decltype(Q)::value;
        if (w != q) return;
        const auto& v = df_group<q>(wv);
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) Wm[16 * g + 4 * kq + e][16 * q + l16] = g <= q ? v[g <= q ? g : 0][e] : 0.f;
    });
}

// returns Am · W with W row-major [k][n] in LDS, 32×32×2 fp32 MFMA
__device__ __forceinline__ f32x16 df_times_w(const float (*Am)[LP], const float (*Wm)[LP], int wr, int wc, int l32, int lh) {
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
    for (int g = 0; g < NB / 8; ++g) {
        const float4 a4 = *reinterpret_cast<const float4*>(&Am[32 * wr + l32][8 * g + 4 * lh]);
        const int k0 = 8 * g + 4 * lh, n = 32 * wc + l32;
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.x, Wm[k0 + 0][n], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.y, Wm[k0 + 1][n], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.z, Wm[k0 + 2][n], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.w, Wm[k0 + 3][n], acc, 0, 0, 0);
    }
    return acc;
}

// accumulator (MFMA C layout: element v of a lane -> row 8*(v/4) + 4*lh + v%4, column l32 of the wave's
// 32×32 quadrant) -> LDS tile, row-major with pitch P
template <int P>
__device__ __forceinline__ void df_acc_to_lds(float (*dst)[P], const f32x16& acc, int wr, int wc, int l32, int lh) {
#pragma unroll
    for (int v = 0; v < 16; ++v) dst[32 * wr + 8 * (v >> 2) + 4 * lh + (v & 3)][32 * wc + l32] = acc[v];
}

// 64×64 tile of a global r×r matrix -> accumulator; out-of-range entries read as `diag_pad` on the
// global diagonal and 0 elsewhere
__device__ __forceinline__ f32x16 df_load_acc(const float* __restrict__ M, int r, int r0, int c0, int wr, int wc, int l32,
                                              int lh, float diag_pad) {
    f32x16 acc;
    const int gc = c0 + 32 * wc + l32;
    const int rq = 32 * wr + 4 * lh;
    if (r0 + NB <= r && c0 + NB <= r) {
        const float* po = M + (int64_t)(r0 + rq) * r + gc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = po[(int64_t)(8 * (v >> 2) + (v & 3)) * r];
    } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int gr = r0 + rq + 8 * (v >> 2) + (v & 3);
            acc[v] = (gr < r && gc < r) ? M[(int64_t)gr * r + gc] : ((gr == gc) ? diag_pad : 0.f);
        }
    }
    return acc;
}

// LDS tile (row-major, pitch P) -> global r×r matrix with agent-scope stores (a panel tile other workgroups
// will read), 16-byte row pieces where the shape allows
template <int P, int THREADS = 256>
__device__ __forceinline__ void df_store_tile(float* __restrict__ M, const float (*src)[P], int r, int r0, int c0, int tid) {
    constexpr int N = (NB * NB / 4 + THREADS - 1) / THREADS;
    f32x4 v[N];   // (out of LDS before the first store: the compiler moves no read over one)
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int e = tid + j * THREADS, row = (e >> 4) & (NB - 1), col = (e & 15) * 4;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[j][q] = src[row][col + q];
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int e = tid + j * THREADS, gr = r0 + (e >> 4), gc = c0 + (e & 15) * 4;
        if (e < NB * NB / 4 && gr < r && gc < r) df_st16(M + (int64_t)gr * r + gc, v[j]);
    }
}

// Finished Y tile (rows r0.., columns c0.. of Y = L^-T, row-major with pitch P in LDS) -> its transposed
// place in Binv[n][k] = Y[k][n]·dinv[k], as fp32 and/or as hi/lo bf16 planes
template <int P>
__device__ __forceinline__ void df_store_binv(const float (*src)[P], const float* __restrict__ db, float* Binv, bf16_t* Bh,
                                              bf16_t* Bl, int64_t boff, int r, int r0, int c0, int tid) {
    if (Bh && !Binv && (r & 7) == 0) {
        for (int e = tid; e < NB * NB / 8; e += 256) {
            const int col = e >> 3, row8 = (e & 7) * 8;
            const int gr = r0 + row8, gc = c0 + col;
            if (gr < r && gc < r) {
                float v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = src[row8 + q][col] * db[gr + q];
                uint4 h, l;
                uint32_t* hp = reinterpret_cast<uint32_t*>(&h);
                uint32_t* lp = reinterpret_cast<uint32_t*>(&l);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t hh = pack_bf2(v[2 * q], v[2 * q + 1]);
                    hp[q] = hh;
                    lp[q] = pack_bf2(v[2 * q] - bf2f((bf16_t)(hh & 0xffffu)), v[2 * q + 1] - bf2f((bf16_t)(hh >> 16)));
                }
                const int64_t o = boff + (int64_t)gc * r + gr;
                *reinterpret_cast<uint4*>(Bh + o) = h;
                *reinterpret_cast<uint4*>(Bl + o) = l;
            }
        }
    } else {
        for (int e = tid; e < NB * NB; e += 256) {
            const int col = e >> 6, row = e & 63;
            const int gr = r0 + row, gc = c0 + col;
            if (gr < r && gc < r) {
                const float v = src[row][col] * db[gr];
                const int64_t o = boff + (int64_t)gc * r + gr;
                if (Binv) Binv[o] = v;
                if (Bh) {
                    const bf16_t h = f2bf(v);
                    Bh[o] = h;
                    Bl[o] = f2bf(v - bf2f(h));
                }
            }
        }
    }
}

template <int NT>
__global__ void __launch_bounds__(256, 1) factor_dataflow_kernel(DfArgs a) {
    __shared__ __align__(16) float lds_a[NB * LP];
    __shared__ __align__(16) float lds_b[NB * LP];
    __shared__ __align__(16) Elim2Lds elds;
    __shared__ __align__(16) float lds_l[NB * LP];     // the product with W as it is formed, group by group
    __shared__ __align__(16) float lds_m[NB * LP], lds_t[NB * LP];
    __shared__ int s_ok, s_gave_up;
    float (*Am)[LP] = reinterpret_cast<float (*)[LP]>(lds_a);
    float (*Bm)[LP] = reinterpret_cast<float (*)[LP]>(lds_b);
    float (*As)[NB + 1] = reinterpret_cast<float (*)[NB + 1]>(lds_a);
    float (*Bs)[NB + 1] = reinterpret_cast<float (*)[NB + 1]>(lds_b);
    float (*Am2)[LP] = reinterpret_cast<float (*)[LP]>(lds_l);
    float (*Lm2)[LP] = reinterpret_cast<float (*)[LP]>(lds_m);
    float (*Tm)[LP] = reinterpret_cast<float (*)[LP]>(lds_t);

    const int b = blockIdx.y;
    const int r = a.r, nb = a.nblk;
    const int64_t boff = (int64_t)b * r * r;
    float* Sb = a.S + boff;
    float* Lb = a.Lf + boff;
    float* Yb = a.Y + boff;
    const float* db = a.dinv + (int64_t)b * r;
    unsigned* fl = a.flags + (int64_t)b * DF_FLAG_WORDS;
    unsigned* abort_w = fl + 2 * DF_MAX_NBLK * DF_MAX_NBLK;
    float* wxb = a.wx + (int64_t)b * df_wx_words(nb);
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    const int wr = wave >> 1, wc = wave & 1;
    const int l16 = lane & 15, kq = lane >> 4;
    const int grp = elim2_group(__builtin_amdgcn_readfirstlane(wave));

    auto slot_of = [&](int row, DfSlot kind) { return wxb + (int64_t)(row * DF_SLOTS + kind) * DF_SLOT_WORDS; };
    // flag of the finished panel tile in stacked row `row` (S-rows 0..nb-1, Y-rows nb..2nb-1), block column p
    auto flag_of = [&](int row, int p) { return fl + row * nb + p; };
    // whole workgroup waits for up to three flags; false = give up (abort raised)
    auto wg_wait = [&](unsigned* f1, unsigned* f2, unsigned* f3) -> bool {
        if (tid == 0) {
            const bool ok = df_poll(f1, f2, f3, abort_w, a.spin_limit);
            if (!ok) {
                __hip_atomic_store(abort_w, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (a.info) a.info[b] = -1;
            }
            s_ok = ok ? 1 : 0;
        }
        __syncthreads();
        const int ok = s_ok;
        __syncthreads();      // s_ok may be rewritten from here on
        return ok != 0;
    };
    // publish: every wave's stores of the tile have completed, then one thread raises the flag
    auto wg_publish = [&](unsigned* f) {
        df_stores_done();
        __syncthreads();
        if (tid == 0) __hip_atomic_store(f, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };

    // a wait of some wave on an exchange slot gave up (looked at after a barrier): raise the item's abort word and flag the result
    if (tid == 0) s_gave_up = 0;
    __syncthreads();
    auto gave_up = [&]() -> bool {
        const int any = s_gave_up;
        __syncthreads();      // no wave is in its next wait before all have looked
        if (!any) return false;
        if (tid == 0) {
            __hip_atomic_store(abort_w, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (a.info) a.info[b] = -1;
        }
        return true;
    };
    // column group Q of W_k; what is there of W_k before (df_load_groups, df_load_tiles) is used
    DfW wv;
    auto wait_group = [&](auto Q, int k) {
        constexpr int q = decltype(Q)::value;
        const float* slot = slot_of(k, DF_SLOT_W);
        if (!df_wait_group<q>(wv, slot, abort_w, a.spin_limit, lane)) s_gave_up = 1;
    };

    const int g = blockIdx.x;
    if (g < nb) {
        // ------------------------------------------------------------------ spine of block row i
        const int i = g;
        const int r0 = i * NB;
        DF_STAMP(i * 8 + 0);
        f32x16 acc_d = df_load_acc(Sb, r, r0, r0, wr, wc, l32, lh, 1.f);
        f32x16 acc_s, acc_q;
        if (i > 0) acc_s = df_load_acc(Sb, r, r0, r0 - NB, wr, wc, l32, lh, 0.f);
        if (i > 1) {
            acc_q = df_load_acc(Sb, r, r0, r0 - 2 * NB, wr, wc, l32, lh, 0.f);
            f32x4 v[12];
            for (int p = 0; p + 4 <= i; ++p) {
                if (!wg_wait(flag_of(i, p), flag_of(i - 1, p), flag_of(i - 2, p))) return;
                df_load_tiles(v, wv, Lb + (int64_t)r0 * r + p * NB, r - r0, Lb + (int64_t)(r0 - NB) * r + p * NB, Lb + (int64_t)(r0 - 2 * NB) * r + p * NB, r,
                              slot_of(i - 2, DF_SLOT_W), r, tid);
                df_tile_to_lds(Am, v, 0, -1.f, tid);    // -L(i,p), L(i-1,p), L(i-2,p)
                df_tile_to_lds(Bm, v, 4, 1.f, tid);
                df_tile_to_lds(Am2, v, 8, 1.f, tid);
                __syncthreads();
                df_mma(acc_q, Am, Am2, wr, wc, l32, lh, 1.f);
                df_mma(acc_s, Am, Bm, wr, wc, l32, lh, 1.f);
                df_mma(acc_d, Am, Am, wr, wc, l32, lh, -1.f);
                __syncthreads();
            }
            // Panels i-3 and i-2 are what the next diagonal tile waits for, and in them L(i,i-2) and T(i,i-1), which workgroup i+1 waits for.
            // Tiles of the spine come through exchange slots, those of panel i-3 in one round trip with what has arrived of W_{i-2}.
            DF_STAMP(256 + i * 8 + 0);
            if (i > 2) {
                const float *l3 = slot_of(i, DF_SLOT_L3), *l2 = slot_of(i - 1, DF_SLOT_L2), *l1 = slot_of(i - 2, DF_SLOT_L1);
                for (int spins = 0;; ++spins) {
                    df_load_tiles(v, wv, l3, NB, l2, l1, NB, slot_of(i - 2, DF_SLOT_W), NB, tid);
                    bool ok = true;
#pragma unroll
                    for (int q = 0; q < 12; ++q) ok = ok && df_written(v[q]);
                    if (__all(ok)) break;
                    if (df_gives_up(spins, abort_w, a.spin_limit)) { s_gave_up = 1; break; }
                }
                DF_STAMP(256 + i * 8 + 1);
                df_tile_to_lds(Am, v, 0, -1.f, tid);
                df_tile_to_lds(Bm, v, 4, 1.f, tid);
                df_tile_to_lds(Am2, v, 8, 1.f, tid);
                __syncthreads();
                if (gave_up()) return;
                df_mma(acc_q, Am, Am2, wr, wc, l32, lh, 1.f);
                df_mma(acc_s, Am, Bm, wr, wc, l32, lh, 1.f);
                __syncthreads();
            } else {
                df_load_groups(wv, slot_of(i - 2, DF_SLOT_W), lane);
            }
            df_acc_to_lds<LP>(Lm2, acc_q, wr, wc, l32, lh);
            // L(i-1,i-2) is formed here for a second time, next to L(i,i-2), from the T(i-1,i-2) that workgroup i-1 sends: waiting for its
            // L(i-1,i-2) instead puts the formation and a hand-over between W_{i-2} and W_{i-1} (12.7 µs per block row).
            if (!df_wait_tile(v[0], v[1], v[2], v[3], slot_of(i - 1, DF_SLOT_T), abort_w, a.spin_limit, tid)) s_gave_up = 1;
            df_tile_to_lds(Bm, v, 0, 1.f, tid);
            __syncthreads();
            DF_STAMP(256 + i * 8 + 2);
            for_groups([&](auto Q) {
                wait_group(Q, i - 2);
                df_l_group<decltype(Q)::value>(Am2, Lm2, wv, wave, l16, kq);
                df_l_group<decltype(Q)::value>(Tm, Bm, wv, wave, l16, kq);
            });
            __syncthreads();
            if (gave_up()) return;
            DF_STAMP(256 + i * 8 + 3);
            if (i + 1 < nb) df_store_slot<256>(slot_of(i, DF_SLOT_L2), Am2, tid);
            df_store_tile<LP>(Lb, Am2, r, r0, r0 - 2 * NB, tid);
            df_mma(acc_s, Am2, Tm, wr, wc, l32, lh, -1.f);
            df_acc_to_lds<LP>(Lm2, acc_s, wr, wc, l32, lh);   // T(i,i-1)
            wg_publish(flag_of(i, i - 2));
            DF_STAMP(256 + i * 8 + 4);
            if (i + 1 < nb) df_store_slot<256>(slot_of(i, DF_SLOT_T), Lm2, tid);
            if (i > 2) df_mma(acc_d, Am, Am, wr, wc, l32, lh, -1.f);
            df_mma(acc_d, Am2, Am2, wr, wc, l32, lh, -1.f);
        }
        DF_STAMP(i * 8 + 1);
        float (*Lm)[LP] = Am2;
        unsigned* pending = nullptr;   // flag of L(i,i-1), raised from inside the elimination
        // T_ii with the panels p <= i-2 applied (T in Bs); the panel i-1 follows below, group by group
        df_acc_to_lds<NB + 1>(Bs, acc_d, wr, wc, l32, lh);
        f32x4 accp[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) accp[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (i > 0) {
            if (i == 1) {   // T(1,0) is the tile of S' as it is
                df_acc_to_lds<LP>(Lm2, acc_s, wr, wc, l32, lh);
                __syncthreads();
                if (nb > 2) df_store_slot<256>(slot_of(1, DF_SLOT_T), Lm2, tid);
            }
            df_load_groups(wv, slot_of(i - 1, DF_SLOT_W), lane);
            __syncthreads();
            for_groups([&](auto Q) {
                constexpr int q = decltype(Q)::value;
                wait_group(Q, i - 1);                              // 16 columns of W_{i-1}
                if (q == 3) DF_STAMP(i * 8 + 2);
                df_l_group<q>(Lm, Lm2, wv, wave, l16, kq);         // 16 columns of L(i,i-1)
                __syncthreads();
                df_syrk_group(accp, Lm, q, grp, l16, kq);
            });
            if (gave_up()) return;
            pending = flag_of(i, i - 1);
            DF_STAMP(i * 8 + 3);
        } else {
            __syncthreads();
        }
        // T_ii -= L(i,i-1)·L(i,i-1)ᵀ on the lower 16×16 tiles, into the registers that the elimination works on
        f32x4 td[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) td[j][v] = Bs[16 * grp + 4 * kq + v][16 * j + l16] - accp[j][v];
        DF_STAMP(i * 8 + 4);
        // W_i = L_ii^-T of the Schur complement T_ii (W in As)
        {
            const int bad_col = diag_inverse_factor(td, As, elds, tid, r - r0, a.flag_below, slot_of(i, DF_SLOT_W), pending,
                                                    [&]() {
                                                        if (i > 0 && i + 2 < nb) df_store_slot<192>(slot_of(i, DF_SLOT_L1), Lm, tid - 64);
                                                        if (i > 0) df_store_tile<LP, 192>(Lb, Lm, r, r0, r0 - NB, tid - 64);
                                                    });
            if (tid == 0 && a.info && bad_col >= 0 && (r0 + bad_col) < r) atomicCAS(a.info + b, 0, r0 + bad_col + 1);
        }
        DF_STAMP(i * 8 + 5);
        if (i + 1 < nb) {   // (nobody takes the last one)
            df_store_tile<NB + 1>(Yb, As, r, r0, r0, tid);
            wg_publish(flag_of(nb + i, i));
        }
        DF_STAMP(i * 8 + 6);
        df_store_binv<NB + 1>(As, db, a.Binv, a.Bh, a.Bl, boff, r, r0, r0, tid);
        DF_STAMP(i * 8 + 7);
        return;
    }

    // ---------------------------------------------------------------------- bulk workgroup w
    const int w = g - nb;
    const int ntiles = df_bulk_tiles(nb);
    const int per = nb - 3;
    f32x16 acc[NT];
    int kcol[NT], rrow[NT];   // block column; stacked row (S-row i, or nb + c for Y-row c); kcol < 0: empty slot
#pragma unroll
    for (int s = 0; s < NT; ++s) {
        const int t = s * a.nbulk + w;
        kcol[s] = -1; rrow[s] = 0;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[s][v] = 0.f;
        if (t < ntiles) {
            int k, idx;
            // block column k holds the S-rows k+3 .. nb-1 and the Y-rows 0 .. k-1: nb-3 tiles up to k = nb-3, then nb-2 and nb-1
            if (per > 0 && t < (nb - 2) * per) { k = t / per; idx = t - k * per; }
            else {
                idx = t - (nb > 3 ? (nb - 2) * per : 0);
                k = nb - 2;
                if (idx >= nb - 2) { idx -= nb - 2; k = nb - 1; }
            }
            const int nS = max(nb - k - 3, 0);
            kcol[s] = k;
            if (idx < nS) {
                rrow[s] = k + 3 + idx;
                acc[s] = df_load_acc(Sb, r, rrow[s] * NB, k * NB, wr, wc, l32, lh, 0.f);
            } else {
                rrow[s] = nb + (idx - nS);
            }
        }
    }
    for (int q = 0; q < nb; ++q) {
        if (w == 0) DF_STAMP(512 + q * 4 + 0);
        // finalise the slots of block column q:  P = T·W_q, group by group behind the elimination that produces W_q
#pragma unroll
        for (int s = 0; s < NT; ++s) {
            if (kcol[s] != q) continue;
            const bool ykind = rrow[s] >= nb;
            const int r0 = (ykind ? rrow[s] - nb : rrow[s]) * NB;
            df_acc_to_lds<LP>(Am, acc[s], wr, wc, l32, lh);
            df_load_groups(wv, slot_of(q, DF_SLOT_W), lane);
            __syncthreads();
            // (the tile of df_last_by_32 is the last one dealt, so it is in the last register tile of its workgroup)
            const bool by_32 = s == NT - 1 && a.last_by_32 && q == nb - 1 && rrow[s] == 2 * nb - 2;
            for_groups([&](auto Q) {
                wait_group(Q, q);
                if (!by_32) df_l_group<decltype(Q)::value>(Am2, Am, wv, wave, l16, kq);
            });
            if (by_32) {
                df_w_to_lds(Bm, wv, wave, l16, kq);
                __syncthreads();
                const f32x16 pr = df_times_w(Am, Bm, wr, wc, l32, lh);
                df_acc_to_lds<LP>(Am2, pr, wr, wc, l32, lh);
            }
            __syncthreads();
            if (gave_up()) return;
            if (!ykind && rrow[s] == q + 3) df_store_slot<256>(slot_of(rrow[s], DF_SLOT_L3), Am2, tid);
            df_store_tile<LP>(ykind ? Yb : Lb, Am2, r, r0, q * NB, tid);
            wg_publish(flag_of(rrow[s], q));
            if (ykind) df_store_binv<LP>(Am2, db, a.Binv, a.Bh, a.Bl, boff, r, r0, q * NB, tid);
            __syncthreads();
        }
        if (w == 0) DF_STAMP(512 + q * 4 + 1);
        // apply panel q to the later slots
#pragma unroll
        for (int s = 0; s < NT; ++s) {
            if (kcol[s] <= q) continue;                    // empty, finished, or just finalised
            const bool ykind = rrow[s] >= nb;
            if (ykind && rrow[s] - nb > q) continue;       // Y-row c starts at panel c
            if (!wg_wait(flag_of(rrow[s], q), flag_of(kcol[s], q), flag_of(kcol[s], q))) return;
            const int r0 = (ykind ? rrow[s] - nb : rrow[s]) * NB;
            df_tiles_to_lds(Am, ykind ? Yb : Lb, r0, q * NB, -1.f, Bm, Lb, kcol[s] * NB, q * NB, true, r, tid);
            __syncthreads();
            df_mma(acc[s], Am, Bm, wr, wc, l32, lh, 1.f);
            __syncthreads();
        }
        if (w == 0) DF_STAMP(512 + q * 4 + 2);
    }
}

// One block row (r <= 64): sum of the partial Gram matrices, scaling, shift and factorisation of an item in one workgroup, the arithmetic of
// prepare_kernel and of the spine's elimination.  What bounds such a factorisation is launches and latency: block of 128×64 with r = 32,
// eleven of them, 305 -> 245 µs without the launch for the set-up, the arming of slots and the flags.
__global__ void __launch_bounds__(256, 1) factor_single_kernel(const float* __restrict__ Sp, int nparts, int64_t pstride, float* __restrict__ dinv,
                                                               float* Binv, bf16_t* Bh, bf16_t* Bl, int r, int r_true, float shift, int32_t* info,
                                                               float flag_below) {
    __shared__ __align__(16) float lds_a[NB * LP];
    __shared__ __align__(16) float lds_b[NB * LP];
    __shared__ __align__(16) Elim2Lds elds;
    __shared__ float sc[NB];
    float (*As)[NB + 1] = reinterpret_cast<float (*)[NB + 1]>(lds_a);
    float (*Bs)[LP] = reinterpret_cast<float (*)[LP]>(lds_b);
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
    const int grp = elim2_group(__builtin_amdgcn_readfirstlane(tid >> 6)), j = (tid & 15) * 4;
    const float* src = Sp + (int64_t)b * r * r;
    f32x4 s[4];
    float dg = 0.f;
    for (int p = 0; p < nparts; ++p, src += pstride) {
        const float d = tid < r ? src[(int64_t)tid * r + tid] : 0.f;
        dg = p ? dg + d : d;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = (tid >> 4) + 16 * q;
            const f32x4 v = i < r && j < r ? *reinterpret_cast<const f32x4*>(src + (int64_t)i * r + j) : f32x4{0.f, 0.f, 0.f, 0.f};
            s[q] = p ? s[q] + v : v;
        }
    }
    if (tid < NB) {
        const float di = (dg > 0.f && dg < 3.0e38f) ? 1.0f / sqrtf(dg) : 1.0f;
        sc[tid] = di;
        if (tid < r) dinv[(int64_t)b * r + tid] = di;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int i = (tid >> 4) + 16 * q;
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float t = s[q][e] * sc[i], dj = sc[j + e];
            v[e] = t * dj;
            if (i == j + e) v[e] = i < r_true ? fmaf(t, dj, shift) : i < r ? 1.f + shift : 1.f;
        }
        *reinterpret_cast<f32x4*>(&Bs[i][j]) = v;
    }
    __syncthreads();
    f32x4 td[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) td[c][v] = Bs[16 * grp + 4 * kq + v][16 * c + l16];
    const int bad_col = diag_inverse_factor(td, As, elds, tid, r, flag_below, nullptr, nullptr, []() {});
    if (tid == 0 && info && bad_col >= 0 && bad_col < r && info[b] == 0) info[b] = bad_col + 1;
    df_store_binv<NB + 1>(As, sc, Binv, Bh, Bl, (int64_t)b * r * r, r, 0, 0, tid);
}

}  // namespace


namespace {
int g_df_spin_limit = DF_SPIN_LIMIT;
constexpr int DF_MAX_CU = 256;   // an MI355X; a partition of one has fewer
// compute units of the current device (the single-launch factorisation runs one workgroup on each and needs them
// all resident at once), asked once so that a partitioned or smaller device is sized correctly
int compute_units() {
    static int n = 0;
    if (n == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            n = std::min(v, DF_MAX_CU);
        else
            n = DF_MAX_CU;
        (void)hipGetLastError();
    }
    return n;
}
// The last tile of the inverse that is a product with the last W, row nblk-2 of Y, is formed by the 32×32×2 matrix instruction where the
// launch was once dealt so that a workgroup had two tiles of the last block column (three or four block rows, five from 29 items on 256
// compute units), by the 16×16×4 one elsewhere.  The two add in another order, with the same precision: results keep their bits.
// The detour through LDS comes once, at the end of the chain: 362.5 -> 363.6 µs for a basis (bf16, L = 576, d = 512, r = 256, one
// iteration), 506 µs with and without it at batch 42.
int df_last_by_32(int nblk, int items) {
    return nblk >= 3 && nblk <= 5 && nblk - 1 > std::min(compute_units() / items - nblk, ((nblk - 1) * (nblk - 1) + 4) / 5);
}
// Workgroups per item of the single-launch factorisation, 0 = shape not covered.  Five tiles per bulk workgroup: with three, 48 workgroups that
// poll instead of 43 beside a spine of 16, four items of r = 1024 take 1425 µs against 1394 (bf16, L = 2112, d = 2048, one iteration), one of
// r = 2048 2547 against 2539; short chains would like three (2 × r = 256 355 against 373, 1 × r = 1024 1123 against 1130).
// Six tiles are what the registers hold, and a batch that needs them is taken: the launch per block column, which has no such limit, is slower
// at every one of these shapes, 25 × r = 384 1104 against 794 µs, 16 × 512 1334 against 887, 8 × 768 1885 against 1193, 6 × 896 2175
// against 1352, 4 × 1152 2717 against 1734, 2 × 1664 3768 against 2305 (bf16; fp32, where the products take most, 1.16 to 1.20 times), with
// U against float64 the same to 1e-3 of its error.
int dataflow_group(int nblk, int items, int cus, int& nt) {
    if (nblk < 2 || nblk > DF_MAX_NBLK || items < 1) return 0;
    const int ntiles = df_bulk_tiles(nblk), room = cus / items - nblk;   // (one workgroup per compute unit)
    const int nbulk = std::min(room, (ntiles + 4) / 5);
    if (nbulk < 1) return 0;
    nt = (ntiles + nbulk - 1) / nbulk;
    return nt > 6 ? 0 : nblk + nbulk;
}
}  // namespace

bool factor_dataflow_ok(int r, int batch, bool whole_batch) {
    const int nblk = (r + NB - 1) / NB;
    int nt;
    if (batch < 1) return false;
    if (nblk == 1) return true;   // factor_inverse_single: workgroups that wait for nobody
    // the whole batch in one launch, or at least one item per launch
    return dataflow_group(nblk, whole_batch ? batch : 1, compute_units(), nt) != 0;
}

void factor_dataflow_set_spin_limit(int polls) { g_df_spin_limit = polls >= 1 ? polls : DF_SPIN_LIMIT; }

namespace {
// items of a launch: as many as keep every workgroup of it resident at once
int dataflow_items(int nblk, int batch, int cus) {
    if (nblk < 2 || nblk > DF_MAX_NBLK) return 0;
    int nt, n = std::min(batch, cus / (nblk + 1));   // (a spine and one workgroup beside it)
    while (n > 0 && dataflow_group(nblk, n, cus, nt) == 0) --n;
    return n;
}
}  // namespace

// For the items of one launch, which the next launch takes over: the flag words, then the exchange slots.  The size is that of a whole device,
// which no part of one exceeds: a question about sizes does not touch the GPU.
size_t factor_dataflow_flag_bytes(int r, int batch) {
    const int nblk = (r + NB - 1) / NB;
    return (size_t)dataflow_items(nblk, batch, DF_MAX_CU) * (DF_FLAG_WORDS + df_wx_words(nblk)) * sizeof(unsigned);
}

hipError_t factor_inverse_dataflow(hipStream_t st, const float* Spart, int nparts, int64_t pstride, float* S, float* dinv, float* Lf, float* Y,
                                   float* Binv, bf16_t* Bh, bf16_t* Bl, unsigned* flags, int r, int r_true, float shift, int zero_all,
                                   int32_t* info, float flag_below, int batch) {
    const int nblk = (r + NB - 1) / NB, cus = compute_units(), per_launch = dataflow_items(nblk, batch, cus);
    int nt = 0;
    if (per_launch < 1) return hipErrorInvalidValue;
    const int G = dataflow_group(nblk, per_launch, cus, nt);
    for (int item0 = 0; item0 < batch; item0 += per_launch) {
        const int n = std::min(batch - item0, per_launch);
        const int64_t o = (int64_t)item0 * r * r;
        DfArgs a;
        a.S = S + o; a.Lf = Lf + o; a.Y = Y + o; a.dinv = dinv + (int64_t)item0 * r;
        a.Binv = Binv ? Binv + o : nullptr; a.Bh = Bh ? Bh + o : nullptr; a.Bl = Bl ? Bl + o : nullptr;
        a.flags = flags; a.info = info ? info + item0 : nullptr;
        a.wx = reinterpret_cast<float*>(flags + (size_t)n * DF_FLAG_WORDS);
        a.spin_limit = g_df_spin_limit;
        a.last_by_32 = df_last_by_32(nblk, per_launch);
        a.r = r; a.nblk = nblk; a.nbulk = G - nblk; a.flag_below = flag_below;
        const hipError_t e = gram_prepare(st, Spart + o, nparts, pstride, a.S, dinv + (int64_t)item0 * r, a.Y, a.Binv, a.Bh, a.Bl, r, r_true, shift,
                                          zero_all, n, flags);
        if (e != hipSuccess) return e;
        const dim3 grid(G, n), block(256);
        switch (nt) {   // (2 does not occur: two block rows have one tile, more have at least three to a workgroup)
            case 1: hipLaunchKernelGGL(factor_dataflow_kernel<1>, grid, block, 0, st, a); break;
            case 3: hipLaunchKernelGGL(factor_dataflow_kernel<3>, grid, block, 0, st, a); break;
            case 4: hipLaunchKernelGGL(factor_dataflow_kernel<4>, grid, block, 0, st, a); break;
            case 5: hipLaunchKernelGGL(factor_dataflow_kernel<5>, grid, block, 0, st, a); break;
            default: hipLaunchKernelGGL(factor_dataflow_kernel<6>, grid, block, 0, st, a); break;
        }
    }
    return hipGetLastError();
}

hipError_t factor_inverse_single(hipStream_t st, const float* Spart, int nparts, int64_t pstride, float* dinv, float* Binv, bf16_t* Bh, bf16_t* Bl,
                                 int r, int r_true, float shift, int32_t* info, float flag_below, int batch) {
    if (r < 1 || r > NB || (r & 3) || nparts < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(factor_single_kernel, dim3(batch), dim3(256), 0, st, Spart, nparts, pstride, dinv, Binv, Bh, Bl, r, r_true, shift, info,
                       flag_below);
    return hipGetLastError();
}

hipError_t gram_prepare(hipStream_t st, const float* Spart, int nparts, int64_t pstride, float* S, float* dinv,
                        float* Y, float* Binv, bf16_t* Bh, bf16_t* Bl, int r, int r_true, float shift, int zero_all, int batch,
                        unsigned* flags) {
    if (r & 3) return hipErrorInvalidValue;
    const int nblk = (r + NB - 1) / NB;
    const auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(nblk, nblk, batch), dim3(256), 0, st, Spart, pstride, S, dinv, flags ? nullptr : Y, Binv, Bh, Bl, r,
                           r_true, shift, zero_all, flags, DF_FLAG_WORDS,
                           flags ? reinterpret_cast<uint4*>(flags + (size_t)batch * DF_FLAG_WORDS) : nullptr,
                           nblk <= DF_MAX_NBLK ? df_wx_words(nblk) : 0);
    };
    switch (nparts) {
        case 1: launch(prepare_kernel<1>); break;
        case 2: launch(prepare_kernel<2>); break;
        case 3: launch(prepare_kernel<3>); break;
        case 4: launch(prepare_kernel<4>); break;
        case 5: launch(prepare_kernel<5>); break;
        case 6: launch(prepare_kernel<6>); break;
        case 7: launch(prepare_kernel<7>); break;
        case 8: launch(prepare_kernel<8>); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t factor_inverse(hipStream_t st, float* S, float* Lf, float* Y, const float* dinv, float* Binv, bf16_t* Bh,
                          bf16_t* Bl, int r, int32_t* info, float flag_below, int batch,
                          hipError_t (*after)(void* ctx, int j), void* ctx) {
    const int nblk = (r + NB - 1) / NB;
    for (int j = 0; j < nblk; ++j) {
        const int m = nblk - j;
        int tiles = m + j + 1;                                   // block column j of S and of Y
        if (j & 1) tiles += (m - 1) + ((m > 1) ? j : 0);        // odd j: the tiles of block column j+1
        else if (j >= 2) tiles += m * (m - 1) / 2 + j * (m - 1);  // even j: every trailing tile
        hipLaunchKernelGGL(factor_step_kernel, dim3(tiles, batch), dim3(256), 0, st, S, Lf, Y, dinv, Binv, Bh, Bl, r, nblk,
                           j, info, flag_below);
        if (after) {
            const hipError_t e = after(ctx, j);
            if (e != hipSuccess) return e;
        }
    }
    return hipGetLastError();
}

}  // namespace atp
