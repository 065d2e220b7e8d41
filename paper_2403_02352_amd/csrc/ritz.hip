// Rayleigh–Ritz canonicalisation of a basis pair (U_r, B_r) (Eq.9: the rows of X' are σ_i·v_iᵀ in
// descending order): eigen-decomposition T = B_r·B_rᵀ = R·Λ·Rᵀ by the cyclic two-sided Jacobi method
// (fp32), then U_r ← U_r·R, B_r ← Rᵀ·B_r with the columns ordered by descending eigenvalue and signed
// so that 1ᵀ·u_i ≥ 0.  Also the diagnostics the paper uses to choose r: captured energy (Fig.5) and
// the SVD-entropy low-rankness ⌈2^μ⌉ (Eq.4) of the estimated singular values.
//
// Jacobi in blocks of 32 indices.  A round pairs the blocks (round-robin) and runs two launches: jacobi_pair_kernel
// takes the 64×64 diagonal sub-matrix of every block pair into LDS and annihilates each of its cross entries once, 32
// steps of 32 disjoint rotations, keeping their product W; jacobi_apply_kernel carries the W of all pairs to T (W_P·T_PQ·W_Qᵀ) and
// to the eigenvector rows (W_P·R_P) with fp32 MFMA.  Every
// second round (for r <= 128 each of the three) also annihilates the entries inside the blocks, and a rotation leaves the larger of its
// two diagonal entries at the smaller index.  Without either, each entry once a sweep, a sweep got less far than one that goes index by
// index: after ten, spectra 0.9^i and groups of eight at r = 300 were left with off-diagonal entries of 4e-6 to 1e-5 of the largest
// eigenvalue (index by index 7e-8 to 4e-7, now 1e-7 or less).  It costs a quarter: r = 512, ten sweeps, 6.44 -> 8.33 ms.
// r <= 64 is one launch, whose sweeps are r-1 steps of a round-robin over the indices themselves: with the 63 steps of two blocks of 32, ten sweeps took 440 µs whatever r was, at r = 1 six times what a launch per step took.
//
// What bounds it: the chain of dependent steps (48 in a round on average), each at best an LDS round trip plus the rotation formula
// (about 0.5 µs).
// A launch per step instead, with every step a pass over T and R, cost 7.4 µs per step: at r = 512, ten sweeps, 37.8 ms for the whole
// call against 8.3 ms.
#include "common.h"

namespace atp {
namespace {

constexpr int JB = 32;            // block size
constexpr int JW = 2 * JB;        // indices of a block pair
constexpr int JP = 96;            // LDS row pitch: rows of opposite parity start in opposite halves of the 64 banks

// blocks of pair i in round k of the round-robin schedule over nb (even) blocks; first < second
__device__ __forceinline__ void block_pair(int i, int k, int nb, int& first, int& second) {
    const int m = nb - 1;
    const int x = i == 0 ? m : (k + i) % m, y = i == 0 ? k : (k - i + m) % m;
    first = min(x, y); second = max(x, y);
}
// matrix index of local index l (0 .. 63) of a block pair
__device__ __forceinline__ int pair_index(int l, int first, int second) { return (l < JB ? first : second - 1) * JB + l; }

// rotation that annihilates the entry pq of [[pp, pq], [pq, qq]]: J = [[c, s], [-s, c]] as s and u = s/(1 + c); identity when the
// entry is zero (as it is for padding indices, whose rows and columns are zero).  The entry is divided by through its mantissa and
// exponent, so every size that fp32 holds is rotated, denormal ones included: a plain hardware reciprocal ends below 2^-126 and above 2^126.
// Hardware reciprocals and roots (1 unit in the last place): an angle that is off by 1e-7 leaves 1e-7 of the entry, and what keeps the
// rotation orthogonal is u against s, where the same error counts s²/2 at most.  Every wave derives all 32 rotations of a step, so
// these instructions count: a launch of 34 steps took 32.7 µs against 37.6 with correctly rounded divisions.
__device__ __forceinline__ void jacobi_su(float app, float aqq, float apq, float& s, float& u) {
    const float tau = __builtin_ldexpf(0.5f * (aqq - app), -__builtin_amdgcn_frexp_expf(apq)) * __builtin_amdgcn_rcpf(__builtin_amdgcn_frexp_mantf(apq));
    const float t = __builtin_copysignf(__builtin_amdgcn_rcpf(fabsf(tau) + __builtin_amdgcn_sqrtf(fmaf(tau, tau, 1.f))), tau);
    const float c = __builtin_amdgcn_rsqf(fmaf(t, t, 1.f));
    s = t * c;
    u = s * __builtin_amdgcn_rcpf(1.f + c);
    if (apq == 0.f) { s = 0.f; u = 0.f; }
}
// (x, y) <- (c·x - s·y, s·x + c·y) with c = 1 - s·u never rounded to fp32: near convergence a rounded c is too large by up to
// half a unit on average, which scaled the whole spectrum up by 6e-5 in ten sweeps at r = 512 (3e-6 this way)
__device__ __forceinline__ void rotate(float s, float u, float x, float y, float& xr, float& yr) {
    xr = fmaf(-s, fmaf(u, x, y), x);
    yr = fmaf(s, fmaf(-u, y, x), y);
}

// indices (p < q) of rotation i (0 .. 31) in step k: the 32 cross pairs of two blocks (32 steps), 16 pairs inside each
// block (31 steps of a round-robin over 32), or m/2 pairs of the first m indices (m even, m-1 steps) and the padding in neighbours
enum StepKind { STEP_CROSS, STEP_WITHIN, STEP_ROBIN };
template <StepKind KIND>
__device__ __forceinline__ void step_pair(int i, int k, int m, int& p, int& q) {
    if constexpr (KIND == STEP_CROSS) { p = i; q = JB + ((i + k) & (JB - 1)); }
    else if constexpr (KIND == STEP_ROBIN) {
        int a = 2 * i, b = 2 * i + 1;
        if (2 * i < m) {
            a = m - 1; b = k;
            if (i) {
                a = k + i; if (a >= m - 1) a -= m - 1;
                b = k - i; if (b < 0) b += m - 1;
            }
        }
        p = min(a, b); q = max(a, b);
    } else {
        int e = i & 15, a = JB - 1, b = k;
        if (e) {
            a = k + e; if (a >= JB - 1) a -= JB - 1;
            b = k - e; if (b < 0) b += JB - 1;
        }
        p = min(a, b) + (i >> 4) * JB; q = max(a, b) + (i >> 4) * JB;
    }
}

// One step: A0 -> A1 = J·A0·Jᵀ (every thread two 2×2 blocks of the 32×32 grid of rotation pairs), W <- J·W in place.  Between blocks, J with
// its rows exchanged where that puts the larger diagonal entry first: what is written changes places, no arithmetic.  (A round-robin
// over the indices themselves converges worse with exchanges.)
// Lane l of every wave derives rotation l % 32, so the step needs a single barrier.
template <StepKind KIND>
__device__ __forceinline__ void jacobi_step(const float* A0, float* A1, float* W, int k, int m, int wave, int lane) {
    const int j = lane & 31;
    int pj, qj;
    step_pair<KIND>(j, k, m, pj, qj);
    float sj, uj;
    const float app = A0[pj * JP + pj], aqq = A0[qj * JP + qj], apq = A0[pj * JP + qj];
    jacobi_su(app, aqq, apq, sj, uj);
    // (padding, whose entries are zero, stays last)
    const uint64_t swaps = KIND == STEP_ROBIN ? 0 : __builtin_amdgcn_ballot_w64(apq != 0.f && aqq > app);
    const bool swap_j = (swaps >> j) & 1;
    const int tpj = swap_j ? qj : pj, tqj = swap_j ? pj : qj;
    const auto lane_of = [](float x, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l)); };
#pragma unroll
    for (int h = 0; h < 32; h += 16) {
        int pi, qi;
        step_pair<KIND>(2 * wave + (lane >> 5) + h, k, m, pi, qi);
        const float b00 = A0[pi * JP + pj], b01 = A0[pi * JP + qj], b10 = A0[qi * JP + pj], b11 = A0[qi * JP + qj];
        const float w00 = W[pi * JP + j], w01 = W[pi * JP + j + 32], w10 = W[qi * JP + j], w11 = W[qi * JP + j + 32];
        const float s0 = lane_of(sj, 2 * wave + h), s1 = lane_of(sj, 2 * wave + h + 1);
        const float u0 = lane_of(uj, 2 * wave + h), u1 = lane_of(uj, 2 * wave + h + 1);
        const float si = lane < 32 ? s0 : s1, ui = lane < 32 ? u0 : u1;
        const bool swap_i = (swaps >> (2 * wave + (lane >> 5) + h)) & 1;
        const int tpi = swap_i ? qi : pi, tqi = swap_i ? pi : qi;
        float r00, r01, r10, r11, x, y;
        rotate(si, ui, b00, b10, r00, r10);
        rotate(si, ui, b01, b11, r01, r11);
        rotate(sj, uj, r00, r01, x, y);
        A1[tpi * JP + tpj] = x;
        A1[tpi * JP + tqj] = y;
        rotate(sj, uj, r10, r11, x, y);
        A1[tqi * JP + tpj] = x;
        A1[tqi * JP + tqj] = y;
        rotate(si, ui, w00, w10, x, y);
        W[tpi * JP + j] = x;
        W[tqi * JP + j] = y;
        rotate(si, ui, w01, w11, x, y);
        W[tpi * JP + j + 32] = x;
        W[tqi * JP + j + 32] = y;
    }
    __syncthreads();
}

// One workgroup per (block pair of round k, item): the rotations of the pair's 64×64 sub-matrix of T.  Their product goes to
// Wout[item][pair][64][64].  With a single pair (nb == 2) all `sweeps` sweeps run here, over the r indices; T and the product (then all of
// R) are the results.
__global__ void __launch_bounds__(512) jacobi_pair_kernel(float* __restrict__ T, float* __restrict__ Wout, int64_t w_stride, int w_rows,
                                                           int r, int nb, int k, int sweeps) {
    __shared__ float A[2][JW * JP];
    __shared__ float W[JW * JP];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int fb, sb;
    block_pair(blockIdx.x, k, nb, fb, sb);
    float* Tb = T + (int64_t)blockIdx.y * r * r;
    for (int e = tid; e < JW * JW; e += 512) {
        const int i = e >> 6, j = e & 63, gi = pair_index(i, fb, sb), gj = pair_index(j, fb, sb);
        A[0][i * JP + j] = (gi < r && gj < r) ? Tb[(int64_t)gi * r + gj] : 0.f;
        W[i * JP + j] = i == j ? 1.f : 0.f;
    }
    __syncthreads();
    int buf = 0;
    if (nb == 2) {
        const int m = r + (r & 1);
        for (int sw = 0; sw < sweeps; ++sw)
            for (int t = 0; t < m - 1; ++t, buf ^= 1) jacobi_step<STEP_ROBIN>(A[buf], A[buf ^ 1], W, t, m, wave, lane);
    } else {
        if (k % 2 == 0 || nb == 4)
            for (int t = 0; t < JB - 1; ++t, buf ^= 1) jacobi_step<STEP_WITHIN>(A[buf], A[buf ^ 1], W, t, 0, wave, lane);
        for (int t = 0; t < JB; ++t, buf ^= 1) jacobi_step<STEP_CROSS>(A[buf], A[buf ^ 1], W, t, 0, wave, lane);
    }
    float* Wb = Wout + (int64_t)blockIdx.y * w_stride + (int64_t)blockIdx.x * JW * JW;
    for (int e = tid; e < JW * JW; e += 512) {
        const int i = e >> 6, j = e & 63;
        if (i < w_rows && j < w_rows) Wb[i * w_rows + j] = W[i * JP + j];
        if (nb == 2 && i < r && j < r) Tb[(int64_t)i * r + j] = A[buf][i * JP + j];
    }
}

// acc (the wave's 16×16 piece, rows 16·(wave/4), columns 16·(wave%4)) = A·B of two 64×64 LDS matrices (pitch LP); B is read as
// B[k][n], or as B[n][k] when NT
constexpr int LP = JW + 4;
template <bool NT>
__device__ __forceinline__ f32x4 tile_product(const float* A, const float* B, int wave, int lane) {
    const int row = 16 * (wave >> 2) + (lane & 15), col = 16 * (wave & 3) + (lane & 15), kq = lane >> 4;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < JW; k += 4) {
        const float b = NT ? B[col * LP + k + kq] : B[(k + kq) * LP + col];
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(A[row * LP + k + kq], b, acc, 0, 0, 0);
    }
    return acc;
}

// One workgroup per 64×64 tile: tiles (P, Q <= P) of the symmetric T (the mirror tile is written from the same values), then
// tiles of 64 columns of the eigenvector rows of pair P.  Every tile is read and written by its own workgroup only, so both
// updates are in place.  Two 64³ products per tile are 2 µs of matrix-core time; 36 + 64 workgroups at r = 512.
__global__ void __launch_bounds__(1024) jacobi_apply_kernel(float* __restrict__ T, float* __restrict__ R, const float* __restrict__ Wall,
                                                            int r, int nb, int k) {
    __shared__ float WP[JW * LP], WQ[JW * LP], X[JW * LP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int np = nb / 2, ntri = np * (np + 1) / 2;
    const bool on_T = (int)blockIdx.x < ntri;
    int P, Q;
    if (on_T) {
        const int t = blockIdx.x;
        P = (int)((sqrtf(8.f * t + 1.f) - 1.f) * 0.5f);
        while ((P + 1) * (P + 2) / 2 <= t) ++P;
        while (P * (P + 1) / 2 > t) --P;
        Q = t - P * (P + 1) / 2;
    } else {
        P = (blockIdx.x - ntri) % np;
        Q = (blockIdx.x - ntri) / np;   // 64-column tile
    }
    int fp, sp, fq = 0, sq = 0;
    block_pair(P, k, nb, fp, sp);
    if (on_T) block_pair(Q, k, nb, fq, sq);
    float* M = (on_T ? T : R) + (int64_t)blockIdx.y * r * r;
    const float* Wb = Wall + (int64_t)blockIdx.y * np * JW * JW;
    for (int e = tid; e < JW * JW; e += 1024) {
        const int i = e >> 6, j = e & 63, gi = pair_index(i, fp, sp), gj = on_T ? pair_index(j, fq, sq) : Q * JW + j;
        WP[i * LP + j] = Wb[(int64_t)P * JW * JW + e];
        if (on_T) WQ[i * LP + j] = Wb[(int64_t)Q * JW * JW + e];
        X[i * LP + j] = (gi < r && gj < r) ? M[(int64_t)gi * r + gj] : 0.f;
    }
    __syncthreads();
    f32x4 acc = tile_product<false>(WP, X, wave, lane);
    const int row = 16 * (wave >> 2) + 4 * (lane >> 4), col = 16 * (wave & 3) + (lane & 15);
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) X[(row + v) * LP + col] = acc[v];
    __syncthreads();
    if (on_T) {
        acc = tile_product<true>(X, WQ, wave, lane);
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 4; ++v) X[(row + v) * LP + col] = acc[v];
        __syncthreads();
    }
    for (int e = tid; e < JW * JW; e += 1024) {
        const int i = e >> 6, j = e & 63;
        const int gi = pair_index(i, fp, sp), gj = on_T ? pair_index(j, fq, sq) : Q * JW + j;
        // the lower triangle of a diagonal tile stands for both halves: T stays exactly symmetric
        if (gi < r && gj < r) M[(int64_t)gi * r + gj] = (on_T && P == Q && j > i) ? X[j * LP + i] : X[i * LP + j];
        if (on_T && P != Q) {
            const int hi = pair_index(j, fp, sp), hj = pair_index(i, fq, sq);   // (lane varies the row of X: the mirror row is contiguous)
            if (hi < r && hj < r) M[(int64_t)hj * r + hi] = X[j * LP + i];
        }
    }
}

__global__ void __launch_bounds__(256) ritz_identity_kernel(float* __restrict__ R, int r) {
    const int b = blockIdx.z, i = blockIdx.y, j = blockIdx.x * 256 + threadIdx.x;
    if (j < r) R[((int64_t)b * r + i) * r + j] = (i == j) ? 1.f : 0.f;
}

// rank of eigenvalue i in descending order (ties: lower index first); lam = diag(T), gathered into LDS first (r <= 4096)
__global__ void __launch_bounds__(256) ritz_rank_kernel(const float* __restrict__ T, int r, int* __restrict__ rank) {
    __shared__ float lam[4096];
    const int b = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
    const float* Tb = T + (int64_t)b * r * r;
    for (int j = threadIdx.x; j < r; j += 256) lam[j] = Tb[(int64_t)j * r + j];
    __syncthreads();
    if (i >= r) return;
    const float li = lam[i];
    int cnt = 0;
#pragma unroll 8
    for (int j = 0; j < r; ++j) {
        const float lj = lam[j];
        cnt += (lj > li || (lj == li && j < i)) ? 1 : 0;
    }
    rank[(int64_t)b * r + i] = cnt;
}

// One workgroup (64 threads) per eigenvector i: sign from 1ᵀ·u_i = (1ᵀU)·R[:, i]; writes row rank_i of
// RsT (= signed eigenvector), sigma[rank_i] and the "sum is numerically zero" flag.
__global__ void __launch_bounds__(64) ritz_order_kernel(const float* __restrict__ T, const float* __restrict__ R,
                                                        const float* __restrict__ colsum, int64_t ld_cs,
                                                        const int* __restrict__ rank, float* __restrict__ RsT,
                                                        float* __restrict__ sigma, int* __restrict__ zero_sum, int r,
                                                        float zero_tol) {
    const int b = blockIdx.y, i = blockIdx.x, lane = threadIdx.x;
    const float* row = R + ((int64_t)b * r + i) * r;
    float t = 0.f;
    for (int k = lane; k < r; k += 64) t = fmaf(colsum[(int64_t)b * ld_cs + k], row[k], t);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off);
    const int dst = rank[(int64_t)b * r + i];
    const bool small = fabsf(t) < zero_tol;
    const float sg = (!small && t < 0.f) ? -1.f : 1.f;
    float* out = RsT + ((int64_t)b * r + dst) * r;
    for (int k = lane; k < r; k += 64) out[k] = sg * row[k];
    if (lane == 0) {
        const float lam = T[((int64_t)b * r + i) * r + i];
        sigma[(int64_t)b * r + dst] = sqrtf(fmaxf(lam, 0.f));
        zero_sum[(int64_t)b * r + dst] = small ? 1 : 0;
    }
}

// Fallback sign rule for components whose 1ᵀ·u_i is numerically zero: make the largest-magnitude
// entry of b_i positive.  One workgroup per flagged component.
template <typename T>
__global__ void __launch_bounds__(256) ritz_fallback_sign_kernel(T* __restrict__ U, T* __restrict__ B,
                                                                 const int* __restrict__ zero_sum, int L, int d, int r) {
    __shared__ float smax[256];
    __shared__ int sidx[256];
    const int b = blockIdx.y, i = blockIdx.x, tid = threadIdx.x;
    if (!zero_sum[(int64_t)b * r + i]) return;
    T* brow = B + ((int64_t)b * r + i) * d;
    float best = -1.f; int bi = 0;
    for (int c = tid; c < d; c += 256) {
        float v;
        if constexpr (sizeof(T) == 2) v = bf2f(brow[c]); else v = brow[c];
        if (fabsf(v) > best) { best = fabsf(v); bi = c; }
    }
    smax[tid] = best; sidx[tid] = bi;
    __syncthreads();
    for (int s = 128; s >= 1; s >>= 1) {
        if (tid < s) {
            if (smax[tid + s] > smax[tid] || (smax[tid + s] == smax[tid] && sidx[tid + s] < sidx[tid])) {
                smax[tid] = smax[tid + s]; sidx[tid] = sidx[tid + s];
            }
        }
        __syncthreads();
    }
    float lead;
    if constexpr (sizeof(T) == 2) lead = bf2f(brow[sidx[0]]); else lead = brow[sidx[0]];
    if (!(lead < 0.f)) return;
    __syncthreads();
    for (int c = tid; c < d; c += 256) {
        if constexpr (sizeof(T) == 2) brow[c] = brow[c] ^ 0x8000u; else brow[c] = -brow[c];
    }
    T* ucol = U + (int64_t)b * L * r + i;
    for (int l = tid; l < L; l += 256) {
        if constexpr (sizeof(T) == 2) ucol[(int64_t)l * r] = ucol[(int64_t)l * r] ^ 0x8000u; else ucol[(int64_t)l * r] = -ucol[(int64_t)l * r];
    }
}

// part[b][i] = { max_{j≠i} |T_ij|, |T_ii| }: one wave per row
__global__ void __launch_bounds__(256) ritz_rowmax_kernel(const float* __restrict__ T, int r, float2* __restrict__ part) {
    const int b = blockIdx.y, lane = threadIdx.x & 63, i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= r) return;
    const float* row = T + ((int64_t)b * r + i) * r;
    float off = 0.f, lam = 0.f;
    for (int j = lane; j < r; j += 64) {
        const float v = fabsf(row[j]);
        if (i == j) lam = v; else off = fmaxf(off, v);
    }
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) { off = fmaxf(off, __shfl_xor(off, s)); lam = fmaxf(lam, __shfl_xor(lam, s)); }
    if (lane == 0) part[(int64_t)b * r + i] = make_float2(off, lam);
}

// diag[b] = { Σ λ (= ‖B_r‖²_F), max_{i≠j} |T_ij| / max_i λ_i, μ = -log2 Σ (σ_i/Σσ)², ⌈2^μ⌉ }
__global__ void __launch_bounds__(256) ritz_diag_kernel(const float2* __restrict__ part, const float* __restrict__ sigma, int r,
                                                        float* __restrict__ diag) {
    __shared__ float sh[4][256];
    const int b = blockIdx.x, tid = threadIdx.x;
    float off = 0.f, lmax = 0.f, s1 = 0.f, s2 = 0.f;
    for (int i = tid; i < r; i += 256) {
        const float2 m = part[(int64_t)b * r + i];
        off = fmaxf(off, m.x); lmax = fmaxf(lmax, m.y);
        const float s = sigma[(int64_t)b * r + i];
        s1 += s; s2 += s * s;
    }
    sh[0][tid] = off; sh[1][tid] = lmax; sh[2][tid] = s1; sh[3][tid] = s2;
    __syncthreads();
    for (int s = 128; s >= 1; s >>= 1) {
        if (tid < s) {
            sh[0][tid] = fmaxf(sh[0][tid], sh[0][tid + s]);
            sh[1][tid] = fmaxf(sh[1][tid], sh[1][tid + s]);
            sh[2][tid] += sh[2][tid + s];
            sh[3][tid] += sh[3][tid + s];
        }
        __syncthreads();
    }
    if (tid == 0) {
        const float sum1 = sh[2][0], sum2 = sh[3][0];
        const float mu = (sum1 > 0.f && sum2 > 0.f) ? -log2f(sum2 / (sum1 * sum1)) : 0.f;
        diag[b * 4 + 0] = sum2;
        diag[b * 4 + 1] = (sh[1][0] > 0.f) ? sh[0][0] / sh[1][0] : 0.f;
        diag[b * 4 + 2] = mu;
        diag[b * 4 + 3] = ceilf(exp2f(mu) - 1e-4f);
    }
}

}  // namespace

hipError_t ritz_jacobi(hipStream_t st, float* T, float* R, float* W, int r, int batch, int sweeps) {
    const int nb = 2 * ((r + JW - 1) / JW), np = nb / 2;
    if (nb == 2) {
        hipLaunchKernelGGL(jacobi_pair_kernel, dim3(1, batch), dim3(512), 0, st, T, R, (int64_t)r * r, r, r, nb, 0, sweeps);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(ritz_identity_kernel, dim3((r + 255) / 256, r, batch), dim3(256), 0, st, R, r);
    for (int sw = 0; sw < sweeps; ++sw)
        for (int k = 0; k < nb - 1; ++k) {
            hipLaunchKernelGGL(jacobi_pair_kernel, dim3(np, batch), dim3(512), 0, st, T, W, (int64_t)np * JW * JW, JW, r, nb, k, 1);
            hipLaunchKernelGGL(jacobi_apply_kernel, dim3(np * (np + 1) / 2 + np * ((r + JW - 1) / JW), batch), dim3(1024), 0, st, T, R, W, r, nb, k);
        }
    return hipGetLastError();
}

hipError_t ritz_order(hipStream_t st, const float* T, const float* R, const float* colsum, int64_t ld_cs, int* rank,
                      float* RsT, float* sigma, int* zero_sum, int r, int batch, float zero_tol) {
    hipLaunchKernelGGL(ritz_rank_kernel, dim3((r + 255) / 256, batch), dim3(256), 0, st, T, r, rank);
    hipLaunchKernelGGL(ritz_order_kernel, dim3(r, batch), dim3(64), 0, st, T, R, colsum, ld_cs, rank, RsT, sigma, zero_sum, r,
                       zero_tol);
    return hipGetLastError();
}

hipError_t ritz_fallback_sign(hipStream_t st, void* U, void* B, const int* zero_sum, int L, int d, int r, int batch,
                              int elem_bytes) {
    if (elem_bytes == 2)
        hipLaunchKernelGGL(ritz_fallback_sign_kernel<bf16_t>, dim3(r, batch), dim3(256), 0, st, (bf16_t*)U, (bf16_t*)B, zero_sum,
                           L, d, r);
    else
        hipLaunchKernelGGL(ritz_fallback_sign_kernel<float>, dim3(r, batch), dim3(256), 0, st, (float*)U, (float*)B, zero_sum, L,
                           d, r);
    return hipGetLastError();
}

hipError_t ritz_diagnostics(hipStream_t st, const float* T, const float* sigma, int r, int batch, float* part, float* diag) {
    hipLaunchKernelGGL(ritz_rowmax_kernel, dim3((r + 3) / 4, batch), dim3(256), 0, st, T, r, (float2*)part);
    hipLaunchKernelGGL(ritz_diag_kernel, dim3(batch), dim3(256), 0, st, (const float2*)part, sigma, r, diag);
    return hipGetLastError();
}

}  // namespace atp
