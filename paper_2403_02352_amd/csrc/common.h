// Shared declarations of the ATP HIP library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace atp {

typedef uint16_t bf16_t;  // raw bfloat16 bits in memory

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// two floats -> packed pair of bfloat16 (lo in bits 0..15), round to nearest even: one
// v_cvt_pk_bf16_f32 on gfx950
__device__ __forceinline__ uint32_t pack_bf2(float a, float b) {
    const f32x2 v = {a, b};
    union { bf16x2 h; uint32_t u; } c;
    c.h = __builtin_convertvector(v, bf16x2);
    return c.u;
}
__device__ __forceinline__ bf16_t f2bf(float f) { return (bf16_t)(pack_bf2(f, 0.f) & 0xffffu); }
__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) const void glb_void;

// 16-byte-per-lane asynchronous copy global -> LDS written as inline assembly: the compiler neither
// tracks it nor adds waits of its own for it (with the builtin it inserts a full vmcnt(0) drain at
// the head of a loop whose body reads a stage that was filled one trip earlier).  The global address
// is a wave-uniform base (SGPR pair) plus a 32-bit byte offset per lane, the LDS address `lds` a
// wave-uniform byte address (lane q lands at lds + 16·q): three instructions per copy and no vector
// address arithmetic in the loop.
// M0 is written by the copy and is named in the clobber list so that the compiler never assumes a value
// of its own survives the statement (the compiler warns about any reserved register there; silenced).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void copy16_untracked(const void* base, unsigned off_bytes, unsigned lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off_bytes), "s"(base), "s"(lds) : "memory", "m0");
}
#pragma clang diagnostic pop

// Fragments of an operand that lies in LDS as it lies in memory, rows of k by columns, come from the transposing LDS read: each
// of 16 lanes names four consecutive 16-bit elements of a row (lanes 4i .. 4i+3 the 16 columns of row i) and lane c receives
// column c of the four rows.  Position p of a row of W elements holds 16-byte chunk p ^ column_swz<W>(row), which puts the four
// rows that 32 lanes take at once in different 64-byte spans of the banks.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <int W>
__device__ __forceinline__ int column_swz(int row) {
    static_assert(W == 64 || W % 128 == 0, "row width");
    return W == 64 ? ((row >> 1) & 1) << 2 : (row & 3) << 2;
}

// byte offset, from the first of 16 rows, of what this lane names for the 32 columns from `col` (a multiple of 32) on
template <int W>
__device__ __forceinline__ int column_frag_offset(int lane, int col) {
    const int row = 8 * (lane >> 5) + ((lane & 15) >> 2);
    return row * W * 2 + (((col >> 3) ^ column_swz<W>(row)) + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) * 16 + (lane & 1) * 8;
}

// 8 consecutive rows of one column: the A or B operand of a 32x32x16 product (column lane % 32, rows 8·(lane / 32) .. +7)
template <int W>
__device__ __forceinline__ bf16x8 read_column_frag(const uint4* base, int ofs) {
    const unsigned at = (unsigned)(uintptr_t)(lds_void*)base + (unsigned)ofs;
    union { s16x4 h[2]; bf16x8 b; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)at);
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(at + 4 * W * 2));
    return u.b;
}

// ---------------------------------------------------------------------------
// C = A · Bᵀ  with both operands K-contiguous ("NT" product), batched.
//   A[M,K] (lda), B[N,K] (ldb); fp32 accumulate.  With a_cols (b_cols) the operand is stored as A[K,M] (B[K,N]) instead.
// MFMA path: operands are bf16.  A value that needs more than bf16 precision is held as a
// hi + lo pair of bf16 planes (hi = bf16(x), lo = bf16(x - hi), ≈16 mantissa bits); when both
// operands carry a lo plane the product is formed from three MFMA products (hi·hi, hi·lo,
// lo·hi, ≈2^-17 relative error), with lo_lo from four (all of the held values).
// Any subset of the outputs may be requested (null = skip):
//   C32 / C16 (+C16lo) : C[M,N] row-major (ldc);  CT32 / CT16 : Cᵀ[N,M] (ldct).
// SWIGLU epilogue: B has 2·Nh rows (gate rows then up rows); the output has Nh
// columns: SiLU(A·gateᵀ) ⊙ (A·upᵀ).  N below is Nh in that case.
// ---------------------------------------------------------------------------
struct GemmArgs {
    const void* A = nullptr;
    const void* A_lo = nullptr;
    const void* B = nullptr;
    const void* B_lo = nullptr;
    int64_t lda = 0, ldb = 0, sA = 0, sB = 0;  // leading dims, batch strides (elements)
    int M = 0, N = 0, K = 0, batch = 1;
    int a_cols = 0, b_cols = 0;
    int lo_lo = 0;
    float* C32 = nullptr;
    bf16_t* C16 = nullptr;
    bf16_t* C16lo = nullptr;
    int64_t ldc = 0, sC = 0;
    float* CT32 = nullptr;
    bf16_t* CT16 = nullptr;
    int64_t ldct = 0, sCT = 0;
    int swiglu = 0;
    // K range limit per output tile for triangular B (B[n][k] = 0 for k > n): 1 = on.  When B is a
    // row block of the triangular matrix, n_origin is the index of its first row.
    int b_lower = 0;
    int n_origin = 0;
    // symmetric output (A == B): only tiles with tileN <= tileM are computed and written; the
    // strictly upper tiles of the output are left untouched
    int symmetric = 0;
    // split-K: slice z of the K range writes a partial product to C32 + z*sKsplit (C32 only)
    int ksplit = 0;
    int64_t sKsplit = 0;
};

enum OperandType { OP_BF16 = 0, OP_F32 = 1 };

// MFMA path (bf16 operands, optional lo planes).  Requirements: K % 64 == 0 (K % 32 == 0 with lo
// planes), lda/ldb/sA/sB % 8 == 0, pointers 16-byte aligned; a_cols only with b_cols (and with lo planes both or none),
// with M % 8 == 0 (a_cols) and N, rounded up to a multiple of 8, within a row (b_cols); b_lower only for B[N,K].
hipError_t gemm_nt_mfma(hipStream_t st, const GemmArgs& g);
bool gemm_nt_mfma_ok(const GemmArgs& g);
bool gemm_nt_mfma_big(const GemmArgs& g);  // true when the 256×256 tile configuration is chosen

// Strided path (any layout, any size; the "simt" of the names is its first, scalar form: it runs on the matrix cores).  ta/tb give the
// element type of A/B; bf16 operands may carry a lo plane (same strides) that is added on load.
struct SimtArgs {
    const void* A = nullptr;
    const void* A_lo = nullptr;
    const void* B = nullptr;
    const void* B_lo = nullptr;
    int64_t a_rs = 0, a_cs = 0, b_rs = 0, b_cs = 0;  // A(m,k) = A[m*a_rs + k*a_cs]; B(n,k) = B[n*b_rs + k*b_cs]
    int64_t sA = 0, sB = 0;
    int M = 0, N = 0, K = 0, batch = 1;
    float* C32 = nullptr;
    bf16_t* C16 = nullptr;
    bf16_t* C16lo = nullptr;
    int64_t ldc = 0, sC = 0;
    float* CT32 = nullptr;
    bf16_t* CT16 = nullptr;
    int64_t ldct = 0, sCT = 0;
    int swiglu = 0;
};
hipError_t gemm_simt(hipStream_t st, OperandType ta, OperandType tb, const SimtArgs& g);

// ---------------------------------------------------------------------------
// streaming passes
// ---------------------------------------------------------------------------
// out[b][c][r] = in[b][r][c]   (rows×cols -> cols×rows), elem_bytes 2 or 4; out row length ld_out
hipError_t transpose_batched(hipStream_t st, const void* in, void* out, int rows, int cols,
                             int64_t ld_out, int64_t s_in, int64_t s_out, int batch, int elem_bytes);
// Omega generator: out[d*r] fp32 N(0,1), counter-based
hipError_t fill_gaussian(hipStream_t st, float* out, int64_t n, uint64_t seed);
hipError_t fill_zero_i32(hipStream_t st, int32_t* p, int64_t n);
// the fp32 matrix in[rows][cols] with zeros outside it, as bf16 out[rows_out][cols_out] (elem_bytes 2) or transposed as fp32
// out[cols_out][rows_out] (elem_bytes 4); also clears zero[0 .. n_zero)
hipError_t start_block(hipStream_t st, const float* in, void* out, int rows, int cols, int rows_out, int cols_out, int elem_bytes,
                       int32_t* zero, int n_zero);
// out[b][0 .. rows_out)[0 .. ld_out) = in[b][0 .. rows)[0 .. cols) with zeros outside it
hipError_t pad_matrix(hipStream_t st, const void* in, void* out, int rows, int cols, int64_t rows_out, int ld_out, int batch, int elem_bytes);
// elements from .. ld-1 of `rows` rows of 2-byte or 4-byte elements set to zero, for up to eight matrices (null: skipped)
struct ZeroTail { void* m; int64_t rows, from, ld; int elem_bytes; };
hipError_t zero_tails(hipStream_t st, const ZeroTail (&z)[8]);
// out = sum of `parts` fp32 arrays of n elements (n a multiple of 8, 16-byte aligned), rounded to bf16
hipError_t sum_parts(hipStream_t st, const float* in, int parts, bf16_t* out, int64_t n);
// rotary position encoding of the rows of in [batch][L][dq] (heads of width dh, half-split pairs); in == out allowed
hipError_t rope_rows(hipStream_t st, const void* in, void* out, int batch, int L, int dq, int dh, float base, int pos0,
                     int elem_bytes);

// a contiguous rows×cols block of every batch item, copied into another matrix (leading dimension and batch strides in elements)
struct ConcatBlock { const void* in; void* out; int64_t rows, cols, ld_out, s_in, s_out; };
hipError_t concat_blocks(hipStream_t st, const ConcatBlock (&b)[4], int batch, int elem_bytes);
// row-wise normalisation of a factored matrix H = P·C: coefficient side (Cc = C - row mean, null: no centring, Cc = C; Cn = Cc·diag(gain))
// and basis side (Pn[i] = P[i] / sqrt(p_i·M·p_iᵀ/d + eps), with PM = P·M, M = Cc·Ccᵀ, given in fp32)
hipError_t norm_coeff(hipStream_t st, const void* C, const float* gain, void* Cc, void* Cn, int64_t rows, int d,
                      int elem_bytes);
hipError_t norm_basis(hipStream_t st, const void* P, const float* PM, void* Pn, int64_t rows, int m, int d, float eps,
                      int elem_bytes);

// ---------------------------------------------------------------------------
// r×r pieces of the CholeskyQR (fp32, batched)
// ---------------------------------------------------------------------------
// (in all of these r is a multiple of 4; the caller pads the matrix)
// Sum `nparts` partial Gram matrices (stride `pstride` elements; only their lower 64×64-tile
// triangle is read), scale to unit diagonal (dinv_j = 1/sqrt(S_jj), 1 if S_jj is not positive and
// finite), add `shift` to the diagonal; rows and columns r_true .. r-1 become those of the identity.  Also sets Y = I
// on its upper tile triangle (not for the single-launch factorisation, which is named by passing its flags) and zeroes the
// part of Binv that factor_inverse leaves unwritten (all of its strict upper tile triangle when
// zero_all is set, else only inside the 256-wide diagonal blocks).
hipError_t gram_prepare(hipStream_t st, const float* Spart, int nparts, int64_t pstride, float* S, float* dinv,
                        float* Y, float* Binv, bf16_t* Bh, bf16_t* Bl, int r, int r_true, float shift, int zero_all, int batch,
                        unsigned* flags = nullptr);
// Cholesky S = L·Lᵀ (S is overwritten with intermediate trailing blocks, L goes to Lf) and Binv[n][k] = (L^-1)[n][k]·dinv[k] (lower triangular).
// info[b] receives the first column (1-based) whose pivot is below `flag_below` (kept if already
// non-zero); pivots that are not positive are replaced by a tiny positive value: no NaN appears.
// Binv is written as fp32 (Binv) and/or as a hi/lo pair of bf16 planes (Bh, Bl); null = skip.
// `after` (may be null) is called on the host after the launch of every 64-wide block column j
// (0-based): rows 0 .. 64(j+1)-1 of Binv are final once that launch has run.
hipError_t factor_inverse(hipStream_t st, float* S, float* Lf, float* Y, const float* dinv, float* Binv, bf16_t* Bh,
                          bf16_t* Bl, int r, int32_t* info, float flag_below, int batch,
                          hipError_t (*after)(void* ctx, int j) = nullptr, void* ctx = nullptr);

// gram_prepare and the same factorisation as ONE launch per group of items: co-resident workgroups keep their tiles in
// registers and hand finished panel tiles to each other through global memory, with a flag per tile or, on the critical
// path, through exchange slots whose content says whether it has arrived (`flags`: factor_dataflow_flag_bytes(r, batch)
// bytes; gram_prepare clears the flags and arms the slots, for every launch anew).
// Covers 64 < r <= 2048 when a group of workgroups fits the chip (factor_dataflow_ok); needs every
// workgroup of a launch resident at the same time, so it must not share the GPU with another such
// launch.  Lf and Y receive the panel tiles (scratch).  info = -1 if a wait inside the kernel gave up.
// factor_dataflow_ok: the shape is covered; with whole_batch, also that all items fit ONE launch (items
// beyond that run as further launches one after the other; from four launches on that costs more than the
// launch-per-block-column factorisation, whose launches take all items at once: r = 1024, 14 factorisations of 16 items
// 9.2 against 8.7 ms, of 8 items 4.6 against 5.9).
bool factor_dataflow_ok(int r, int batch, bool whole_batch);
size_t factor_dataflow_flag_bytes(int r, int batch);
// polls after which a wait inside the kernel gives up (< 1: the default, far beyond any healthy wait)
void factor_dataflow_set_spin_limit(int polls);
hipError_t factor_inverse_dataflow(hipStream_t st, const float* Spart, int nparts, int64_t pstride, float* S, float* dinv, float* Lf, float* Y,
                                   float* Binv, bf16_t* Bh, bf16_t* Bl, unsigned* flags, int r, int r_true, float shift, int zero_all,
                                   int32_t* info, float flag_below, int batch);

// gram_prepare and the factorisation in one launch of a workgroup per item, for r <= 64 (a single block row; nobody waits for anybody)
hipError_t factor_inverse_single(hipStream_t st, const float* Spart, int nparts, int64_t pstride, float* dinv, float* Binv, bf16_t* Bh, bf16_t* Bl,
                                 int r, int r_true, float shift, int32_t* info, float flag_below, int batch);

// ---------------------------------------------------------------------------
// attention over n_k keys (n_k = r principal keys, or L for the dense comparator)
// ---------------------------------------------------------------------------
struct AttnArgs {
    const void* Q = nullptr;   // [batch, L, dq]
    const void* K = nullptr;   // [batch, nk, dq]
    const void* V = nullptr;   // [batch, nk, dq]
    void* O = nullptr;         // [batch, L, dq]
    int batch = 1, L = 0, nk = 0, nk_pad = 0, dq = 0, heads = 1;
    float scale = 0.f;
    // first-order (linearised) variant, Eq.8: weights 1·U + scale·q·K'ᵀ instead of exp(·)
    int linearised = 0;
    const float* colsum = nullptr;  // [batch, nk_pad] column sums of U (1·U), zero padded
    int norm_rowsum = 0;            // 0: divide by n_tokens + scale·(q·K'ᵀ)·(1·U)ᵀ; 1: by the row sum of the map
    float n_tokens = 0.f;           // rows of U
};
hipError_t attention_bf16(hipStream_t st, const AttnArgs& a);  // d_h in {64,128}
hipError_t attention_f32(hipStream_t st, const AttnArgs& a);   // d_h <= 256
// out[b][j] = sum_i U[b][i][j] (fp32), j < r; out rows have length ld_out >= r, the rest is zeroed
hipError_t column_sums(hipStream_t st, const void* U, float* out, int L, int r, int64_t ld_out, int batch, int elem_bytes);

// ---------------------------------------------------------------------------
// alternating rank-1 extraction (Alg.1): d <= 4096, d % 4 == 0
// ---------------------------------------------------------------------------
size_t alternating_workspace(int batch, int L, int d);
hipError_t alternating_bases(hipStream_t st, const void* X, int batch, int L, int d, int r, int sweeps, const float* V0,
                             void* U, void* B, int32_t* info, void* workspace, int elem_bytes);

// ---------------------------------------------------------------------------
// Rayleigh–Ritz canonicalisation (cyclic Jacobi on T = B·Bᵀ) and diagnostics
// ---------------------------------------------------------------------------
// T [batch][r][r] is diagonalised in place, R receives the eigenvectors as rows; W: scratch for the products of rotations,
// batch·ceil(r/64)·4096 floats (none for r <= 64)
hipError_t ritz_jacobi(hipStream_t st, float* T, float* R, float* W, int r, int batch, int sweeps);
hipError_t ritz_order(hipStream_t st, const float* T, const float* R, const float* colsum, int64_t ld_cs, int* rank,
                      float* RsT, float* sigma, int* zero_sum, int r, int batch, float zero_tol);
hipError_t ritz_fallback_sign(hipStream_t st, void* U, void* B, const int* zero_sum, int L, int d, int r, int batch,
                              int elem_bytes);
// part: scratch, 2·batch·r floats
hipError_t ritz_diagnostics(hipStream_t st, const float* T, const float* sigma, int r, int batch, float* part, float* diag);

}  // namespace atp
