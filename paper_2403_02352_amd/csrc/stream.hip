// HBM-bound streaming passes: batched transposes (the fp32 path's Xᵀ, bf16 operands whose rows start at no multiple of 16 bytes),
// padding, fills, the start block and its counter-based Gaussian generator, concatenation and Norm of factored pairs, rotary encoding.
#include "common.h"

#include <algorithm>
#include <type_traits>

namespace atp {
namespace {

constexpr int TT = 64;  // transpose tile

// out[b][c][r] = in[b][r][c]; out rows have length ld_out (>= rows), what lies past `rows` keeps its value.
template <typename T>
__global__ void __launch_bounds__(256) transpose_kernel(const T* __restrict__ in, T* __restrict__ out, int rows,
                                                        int cols, int64_t ld_out, int64_t s_in, int64_t s_out) {
    __shared__ T tile[TT][TT + 2];
    const int b = blockIdx.z;
    const T* src = in + (int64_t)b * s_in;
    T* dst = out + (int64_t)b * s_out;
    const int r0 = blockIdx.y * TT, c0 = blockIdx.x * TT;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;  // 64 × 4
    for (int i = ty; i < TT; i += 4) {
        const int r = r0 + i, c = c0 + tx;
        tile[i][tx] = (r < rows && c < cols) ? src[(int64_t)r * cols + c] : (T)0;
    }
    __syncthreads();
    for (int i = ty; i < TT; i += 4) {
        const int c = c0 + i, r = r0 + tx;
        if (c < cols && r < rows) dst[(int64_t)c * ld_out + r] = tile[tx][i];
    }
}

// Same operation for 2-byte elements when every extent is a multiple of 8: global traffic moves as
// 16-byte pieces (8 elements) on both sides, the 64×64 tile turns in LDS.
__global__ void __launch_bounds__(256) transpose_u16x8_kernel(const uint16_t* __restrict__ in, uint16_t* __restrict__ out,
                                                              int rows, int cols, int64_t ld_out, int64_t s_in,
                                                              int64_t s_out) {
    __shared__ __align__(16) uint16_t tile[TT][TT + 2];
    const int b = blockIdx.z;
    const uint16_t* src = in + (int64_t)b * s_in;
    uint16_t* dst = out + (int64_t)b * s_out;
    const int r0 = blockIdx.y * TT, c0 = blockIdx.x * TT;
    for (int v = threadIdx.x; v < TT * 8; v += 256) {
        const int i = v >> 3, q = v & 7;
        const int r = r0 + i, c = c0 + 8 * q;
        uint4 x = make_uint4(0u, 0u, 0u, 0u);
        if (r < rows && c < cols) x = *reinterpret_cast<const uint4*>(src + (int64_t)r * cols + c);
        uint32_t* d = reinterpret_cast<uint32_t*>(&tile[i][8 * q]);
        d[0] = x.x; d[1] = x.y; d[2] = x.z; d[3] = x.w;
    }
    __syncthreads();
    for (int v = threadIdx.x; v < TT * 8; v += 256) {
        const int i = v >> 3, q = v & 7;
        const int c = c0 + i, r = r0 + 8 * q;
        if (c < cols && r < rows) {
            uint4 x;
            x.x = (uint32_t)tile[8 * q + 0][i] | ((uint32_t)tile[8 * q + 1][i] << 16);
            x.y = (uint32_t)tile[8 * q + 2][i] | ((uint32_t)tile[8 * q + 3][i] << 16);
            x.z = (uint32_t)tile[8 * q + 4][i] | ((uint32_t)tile[8 * q + 5][i] << 16);
            x.w = (uint32_t)tile[8 * q + 6][i] | ((uint32_t)tile[8 * q + 7][i] << 16);
            *reinterpret_cast<uint4*>(dst + (int64_t)c * ld_out + r) = x;
        }
    }
}

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// Element i is a function of (seed, i) only: 64 hashed bits -> two uniforms -> Box–Muller.
__global__ void gaussian_kernel(float* out, int64_t n, uint64_t seed) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t h = mix64(mix64(seed) + 0x9e3779b97f4a7c15ull * (uint64_t)(i + 1));
    const float u1 = ((float)(uint32_t)(h >> 40) + 0.5f) * (1.0f / 16777216.0f);        // 24 bits, (0,1)
    const float u2 = ((float)(uint32_t)((h >> 16) & 0xffffffu) + 0.5f) * (1.0f / 16777216.0f);
    out[i] = sqrtf(-2.0f * logf(u1)) * cosf(6.28318530717958647692f * u2);
}

__global__ void zero_i32_kernel(int32_t* p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// Start block in the form its product reads it, padded with zeros: rounded to bf16 as it lies, or turned (fp32 path), and `zero`
// cleared in the same pass.
__global__ void __launch_bounds__(256) start_block_bf16_kernel(const float* __restrict__ in, bf16_t* __restrict__ out, int rows, int cols,
                                                               int cols_out, int64_t n_out, int32_t* __restrict__ zero, int n_zero) {
    const int64_t first = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
    for (int64_t e = first; e < n_zero; e += step) zero[e] = 0;
    for (int64_t e = first; e < n_out; e += step) {
        const int64_t r = e / cols_out, c = e % cols_out;
        out[e] = (r < rows && c < cols) ? f2bf(in[r * cols + c]) : (bf16_t)0;
    }
}
__global__ void __launch_bounds__(256) start_block_f32_kernel(const float* __restrict__ in, float* __restrict__ out, int rows, int cols,
                                                              int rows_out, int cols_out, int32_t* __restrict__ zero, int n_zero) {
    __shared__ float tile[TT][TT + 1];
    const int r0 = blockIdx.y * TT, c0 = blockIdx.x * TT, tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    if (blockIdx.y == 0)
        for (int e = blockIdx.x * 256 + threadIdx.x; e < n_zero; e += gridDim.x * 256) zero[e] = 0;
    for (int i = ty; i < TT; i += 4) tile[i][tx] = (r0 + i < rows && c0 + tx < cols) ? in[(int64_t)(r0 + i) * cols + c0 + tx] : 0.f;
    __syncthreads();
    for (int i = ty; i < TT; i += 4) {
        const int c = c0 + i, r = r0 + tx;
        if (c < cols_out && r < rows_out) out[(int64_t)c * rows_out + r] = tile[tx][i];
    }
}

template <typename T>
__global__ void __launch_bounds__(256) pad_matrix_kernel(const T* __restrict__ in, T* __restrict__ out, int rows, int cols, int64_t rows_out,
                                                         int ld_out) {
    const int64_t b = blockIdx.x / rows_out, i = blockIdx.x % rows_out;
    const T* src = in + (b * rows + i) * cols;
    T* dst = out + (int64_t)blockIdx.x * ld_out;
    for (int j = threadIdx.x; j < ld_out; j += 256) dst[j] = (i < rows && j < cols) ? src[j] : (T)0;
}

struct ZeroTails { ZeroTail t[8]; };
__global__ void __launch_bounds__(256) zero_tails_kernel(ZeroTails a) {
    const ZeroTail& z = a.t[blockIdx.y];
    const int64_t nc = z.ld - z.from;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < z.rows * nc; i += (int64_t)gridDim.x * 256) {
        const int64_t e = i / nc * z.ld + z.from + i % nc;
        if (z.elem_bytes == 2) reinterpret_cast<uint16_t*>(z.m)[e] = 0;
        else reinterpret_cast<uint32_t*>(z.m)[e] = 0u;
    }
}

// Four blocks copied into wider (or taller) matrices in one launch, blockIdx.y = block, in pieces of sizeof(T) bytes.  2^tpr threads
// share a row, so that short rows fill a workgroup.  HBM-bound: pairs of width 1024 joined at L = d = 4096 (67 MB) took 35 µs as four
// launches that moved single elements.
struct ConcatArgs { ConcatBlock b[4]; int tpr[4]; };
template <typename T>
__global__ void __launch_bounds__(256) concat_kernel(ConcatArgs a) {
    const ConcatBlock& k = a.b[blockIdx.y];
    const T* src = reinterpret_cast<const T*>(k.in) + (int64_t)blockIdx.z * k.s_in;
    T* dst = reinterpret_cast<T*>(k.out) + (int64_t)blockIdx.z * k.s_out;
    const int tpr = a.tpr[blockIdx.y], sub = threadIdx.x >> tpr, lane = threadIdx.x & ((1 << tpr) - 1), rpb = 256 >> tpr;
    for (int64_t i = (int64_t)blockIdx.x * rpb + sub; i < k.rows; i += (int64_t)gridDim.x * rpb)
        for (int64_t j = lane; j < k.cols; j += 1 << tpr) dst[i * k.ld_out + j] = src[i * k.cols + j];
}

// N consecutive elements as floats, and back (N = 8: 16 bytes of bf16, 32 of fp32; N = 4: 8 and 16; rows start at multiples of that)
template <int N, typename T>
__device__ __forceinline__ void load_row(const T* p, float (&x)[N]) {
    if constexpr (N == 1) {
        if constexpr (sizeof(T) == 2) x[0] = bf2f(*p); else x[0] = *p;
    } else if constexpr (N == 4) {
        if constexpr (sizeof(T) == 2) {
            const uint2 u = *reinterpret_cast<const uint2*>(p);
            x[0] = __uint_as_float(u.x << 16); x[1] = __uint_as_float(u.x & 0xffff0000u);
            x[2] = __uint_as_float(u.y << 16); x[3] = __uint_as_float(u.y & 0xffff0000u);
        } else {
            const f32x4 a = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = a[e];
        }
    } else if constexpr (sizeof(T) == 2) {
        const uint4 u = *reinterpret_cast<const uint4*>(p);
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) { x[2 * e] = __uint_as_float(w[e] << 16); x[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u); }
    } else {
        const f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) { x[e] = a[e]; x[4 + e] = b[e]; }
    }
}
template <int N, typename T>
__device__ __forceinline__ void store_row(T* p, const float (&x)[N]) {
    if constexpr (N == 1) {
        if constexpr (sizeof(T) == 2) *p = f2bf(x[0]); else *p = x[0];
    } else if constexpr (N == 4) {
        if constexpr (sizeof(T) == 2) *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf2(x[0], x[1]), pack_bf2(x[2], x[3]));
        else *reinterpret_cast<f32x4*>(p) = f32x4{x[0], x[1], x[2], x[3]};
    } else if constexpr (sizeof(T) == 2) {
        *reinterpret_cast<uint4*>(p) = make_uint4(pack_bf2(x[0], x[1]), pack_bf2(x[2], x[3]), pack_bf2(x[4], x[5]), pack_bf2(x[6], x[7]));
    } else {
        *reinterpret_cast<f32x4*>(p) = f32x4{x[0], x[1], x[2], x[3]};
        *reinterpret_cast<f32x4*>(p + 4) = f32x4{x[4], x[5], x[6], x[7]};
    }
}

// Rotary position encoding, half-split pairing: within a head of width 2·half, coordinate j < half of row i is paired with
// j + half and the pair is rotated by (pos0 + i)·base^(-2j/dh).  A workgroup takes `rows` rows, up to ROPE_J values of j and one of
// `groups` groups of heads: it forms their sines and cosines once, in LDS, for all of its heads (formed per pair they took longer than
// the memory traffic), then moves N elements per access.  2 × 2048 × 4096 bf16 (67 MB), 32 heads: the call took 12 µs less.
// in == out allowed.
constexpr int ROPE_J = 256;
template <int N, typename T>
__global__ void __launch_bounds__(256) rope_kernel(const T* in, T* out, int L, int dq, int half, int j_step, int rows, int groups, float log2_base,
                                                   int pos0) {
    __shared__ float sn[ROPE_J], cs[ROPE_J];   // rows·J values, J·rows <= ROPE_J
    const int nj = (half + j_step - 1) / j_step, bx = (int)(blockIdx.x / groups), group = (int)(blockIdx.x % groups);
    const int row0 = bx / nj * rows, j0 = bx % nj * j_step;
    const int J = min(half - j0, j_step), dh = 2 * half, n_rows = min(rows, L - row0);
    for (int e = threadIdx.x; e < n_rows * J; e += 256) {
        const float freq = exp2f(-2.0f * (float)(j0 + e % J) / (float)dh * log2_base);
        sincosf((float)(pos0 + row0 + e / J) * freq, &sn[e], &cs[e]);
    }
    __syncthreads();
    const unsigned per = J / N;
    const int all = dq / dh, h0 = (int)((int64_t)group * all / groups), heads = (int)((int64_t)(group + 1) * all / groups) - h0;
    const unsigned n = (unsigned)n_rows * heads * per;   // (the host keeps it below 2^31)
    for (unsigned e = threadIdx.x; e < n; e += 256) {
        const int rest = (int)(e / per), jc = (int)(e - (unsigned)rest * per) * N, r = rest / heads, h = h0 + rest - r * heads;
        const int64_t o = ((int64_t)blockIdx.y * L + row0 + r) * dq + (int64_t)h * dh + j0 + jc;
        float x[N], y[N];
        load_row<N>(in + o, x);
        load_row<N>(in + o + half, y);
#pragma unroll
        for (int t = 0; t < N; ++t) {
            const float c = cs[r * J + jc + t], s = sn[r * J + jc + t], a = x[t];
            x[t] = a * c - y[t] * s;
            y[t] = a * s + y[t] * c;
        }
        store_row<N>(out + o, x);
        store_row<N>(out + o + half, y);
    }
}

// sum of the partial products of a product split along k
__global__ void __launch_bounds__(256) sum_parts_kernel(const float* __restrict__ in, int parts, bf16_t* __restrict__ out, int64_t n) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
    if (i >= n) return;
    float s[8], x[8];
    load_row<8>(in + i, s);
    for (int p = 1; p < parts; ++p) {
        load_row<8>(in + p * n + i, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] += x[e];
    }
    store_row<8>(out + i, s);
}

// Row-wise normalisation carried through a factored matrix H = P·C (one workgroup per row; HBM-bound, so 8 elements per access
// where the row length is a multiple of 8).
// Coefficient side: Cc[j][:] = C[j][:] - mean_j, Cn = Cc · diag(gain); without centring (Cc null) Cc is C itself.
template <int N, typename T>
__global__ void __launch_bounds__(256) norm_coeff_kernel(const T* __restrict__ C, const float* __restrict__ gain,
                                                         T* __restrict__ Cc, T* __restrict__ Cn, int d) {
    __shared__ float red[4];
    const int64_t row = blockIdx.x;
    const T* src = C + row * d;
    float mean = 0.f, x[N], g[N];
    if (Cc) {
        float s = 0.f;
        for (int j = threadIdx.x * N; j < d; j += 256 * N) {
            load_row<N>(src + j, x);
#pragma unroll
            for (int e = 0; e < N; ++e) s += x[e];
        }
        for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
        __syncthreads();
        mean = (red[0] + red[1] + red[2] + red[3]) / (float)d;
    }
    for (int j = threadIdx.x * N; j < d; j += 256 * N) {
        load_row<N>(src + j, x);
#pragma unroll
        for (int e = 0; e < N; ++e) { g[e] = gain[j + e]; x[e] -= mean; }
        if (Cc) store_row<N>(Cc + row * d + j, x);
#pragma unroll
        for (int e = 0; e < N; ++e) x[e] *= g[e];
        store_row<N>(Cn + row * d + j, x);
    }
}

// Basis side: var_i = (1/d)·p_i·M·p_iᵀ with T = P·M given; Pn[i][:] = P[i][:] / sqrt(var_i + eps).
template <int N, typename T>
__global__ void __launch_bounds__(256) norm_basis_kernel(const T* __restrict__ P, const float* __restrict__ PM,
                                                         T* __restrict__ Pn, int m, float inv_d, float eps) {
    __shared__ float red[4];
    const int64_t row = blockIdx.x;
    const T* p = P + row * m;
    const float* t = PM + row * m;
    float s = 0.f, x[N], y[N];
    for (int j = threadIdx.x * N; j < m; j += 256 * N) {
        load_row<N>(p + j, x);
        load_row<N>(t + j, y);
#pragma unroll
        for (int e = 0; e < N; ++e) s += x[e] * y[e];
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    const float var = fmaxf((red[0] + red[1] + red[2] + red[3]) * inv_d, 0.f);
    const float sc = 1.0f / sqrtf(var + eps);
    for (int j = threadIdx.x * N; j < m; j += 256 * N) {
        load_row<N>(p + j, x);
#pragma unroll
        for (int e = 0; e < N; ++e) x[e] *= sc;
        store_row<N>(Pn + row * m + j, x);
    }
}

}  // namespace

hipError_t start_block(hipStream_t st, const float* in, void* out, int rows, int cols, int rows_out, int cols_out, int elem_bytes,
                       int32_t* zero, int n_zero) {
    if (elem_bytes == 2) {
        const int64_t n = (int64_t)rows_out * cols_out, blocks = (n + 1023) / 1024;
        hipLaunchKernelGGL(start_block_bf16_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, st, in, (bf16_t*)out, rows, cols,
                           cols_out, n, zero, n_zero);
        return hipGetLastError();
    }
    const dim3 grid((cols_out + TT - 1) / TT, (rows_out + TT - 1) / TT);
    if (grid.y > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(start_block_f32_kernel, grid, dim3(256), 0, st, in, (float*)out, rows, cols, rows_out, cols_out, zero, n_zero);
    return hipGetLastError();
}

hipError_t pad_matrix(hipStream_t st, const void* in, void* out, int rows, int cols, int64_t rows_out, int ld_out, int batch, int elem_bytes) {
    if (batch * rows_out > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(batch * rows_out));
    if (elem_bytes == 2)
        hipLaunchKernelGGL(pad_matrix_kernel<uint16_t>, grid, dim3(256), 0, st, (const uint16_t*)in, (uint16_t*)out, rows, cols, rows_out, ld_out);
    else
        hipLaunchKernelGGL(pad_matrix_kernel<uint32_t>, grid, dim3(256), 0, st, (const uint32_t*)in, (uint32_t*)out, rows, cols, rows_out, ld_out);
    return hipGetLastError();
}

hipError_t zero_tails(hipStream_t st, const ZeroTail (&z)[8]) {
    ZeroTails a;
    int64_t most = 0;
    int n = 0;
    for (const ZeroTail& t : z)
        if (t.m && t.rows > 0 && t.from < t.ld) {
            a.t[n++] = t;
            most = t.rows * (t.ld - t.from) > most ? t.rows * (t.ld - t.from) : most;
        }
    if (n == 0) return hipSuccess;
    const int64_t blocks = (most + 255) / 256;
    hipLaunchKernelGGL(zero_tails_kernel, dim3((unsigned)(blocks < 1024 ? blocks : 1024), n), dim3(256), 0, st, a);
    return hipGetLastError();
}

namespace {
template <typename T>
hipError_t launch_concat(hipStream_t st, ConcatArgs a, int batch, int per) {   // per: elements in a T
    int64_t blocks = 1;
    for (int i = 0; i < 4; ++i) {
        ConcatBlock& k = a.b[i];
        k.cols /= per; k.ld_out /= per; k.s_in /= per; k.s_out /= per;
        a.tpr[i] = 0;
        while (a.tpr[i] < 8 && (1ll << a.tpr[i]) < k.cols) ++a.tpr[i];
        const int64_t n = (k.rows + (256 >> a.tpr[i]) - 1) / (256 >> a.tpr[i]);
        blocks = n > blocks ? n : blocks;
    }
    hipLaunchKernelGGL(concat_kernel<T>, dim3((unsigned)(blocks < 4096 ? blocks : 4096), 4, batch), dim3(256), 0, st, a);
    return hipGetLastError();
}
}  // namespace

hipError_t concat_blocks(hipStream_t st, const ConcatBlock (&b)[4], int batch, int elem_bytes) {
    ConcatArgs a;
    const int per = 16 / elem_bytes;
    bool whole = true;   // every row of every block is made of aligned 16-byte pieces
    for (int i = 0; i < 4; ++i) {
        a.b[i] = b[i];
        whole = whole && b[i].cols % per == 0 && b[i].ld_out % per == 0 && b[i].s_in % per == 0 && b[i].s_out % per == 0 &&
                (((uintptr_t)b[i].in | (uintptr_t)b[i].out) & 15) == 0;
    }
    if (whole) return launch_concat<uint4>(st, a, batch, per);
    return elem_bytes == 2 ? launch_concat<uint16_t>(st, a, batch, 1) : launch_concat<uint32_t>(st, a, batch, 1);
}

hipError_t norm_coeff(hipStream_t st, const void* C, const float* gain, void* Cc, void* Cn, int64_t rows, int d, int elem_bytes) {
    if (rows <= 0) return hipSuccess;
    if (rows > 0x7fffffff) return hipErrorInvalidValue;
    const auto go = [&](auto kern, auto* t) {
        using T = std::remove_reference_t<decltype(*t)>;
        hipLaunchKernelGGL(kern, dim3((unsigned)rows), dim3(256), 0, st, (const T*)C, gain, (T*)Cc, (T*)Cn, d);
    };
    if (elem_bytes == 2) go(d % 8 ? norm_coeff_kernel<1, bf16_t> : norm_coeff_kernel<8, bf16_t>, (bf16_t*)nullptr);
    else go(d % 8 ? norm_coeff_kernel<1, float> : norm_coeff_kernel<8, float>, (float*)nullptr);
    return hipGetLastError();
}

hipError_t norm_basis(hipStream_t st, const void* P, const float* PM, void* Pn, int64_t rows, int m, int d, float eps,
                      int elem_bytes) {
    if (rows <= 0) return hipSuccess;
    if (rows > 0x7fffffff) return hipErrorInvalidValue;
    const auto go = [&](auto kern, auto* t) {
        using T = std::remove_reference_t<decltype(*t)>;
        hipLaunchKernelGGL(kern, dim3((unsigned)rows), dim3(256), 0, st, (const T*)P, PM, (T*)Pn, m, 1.0f / (float)d, eps);
    };
    if (elem_bytes == 2) go(m % 8 ? norm_basis_kernel<1, bf16_t> : norm_basis_kernel<8, bf16_t>, (bf16_t*)nullptr);
    else go(m % 8 ? norm_basis_kernel<1, float> : norm_basis_kernel<8, float>, (float*)nullptr);
    return hipGetLastError();
}

hipError_t sum_parts(hipStream_t st, const float* in, int parts, bf16_t* out, int64_t n) {
    const int64_t blocks = (n / 8 + 255) / 256;
    if (n % 8 || blocks > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(sum_parts_kernel, dim3((unsigned)blocks), dim3(256), 0, st, in, parts, out, n);
    return hipGetLastError();
}

hipError_t rope_rows(hipStream_t st, const void* in, void* out, int batch, int L, int dq, int dh, float base, int pos0,
                     int elem_bytes) {
    const int half = dh / 2, nj = (half + ROPE_J - 1) / ROPE_J, heads = dq / dh;
    const int J = nj == 1 ? half : ((half + nj - 1) / nj + 7) & ~7;   // even shares of wide heads, whole accesses
    // Two workgroups per compute unit (512) as far as the sizes go: more rows to a workgroup only while that many remain, and where rows
    // are too few for them the heads are dealt out as well.  With as many rows as ROPE_J sines
    // allow, 4 × 4096 rows of 128 heads of 8 in bf16 took 60 µs against 15 (single elements in both halves then, four at a time now),
    // 2048 of them 42 against 9.
    const int64_t target = 512, row_share = (int64_t)L * batch / target;
    const int rows = (int)std::max<int64_t>(1, std::min<int64_t>(row_share, ROPE_J / J));
    const int64_t nb = (int64_t)((L + rows - 1) / rows) * ((half + J - 1) / J);
    const int groups = (int)std::max<int64_t>(1 + ((int64_t)rows * J * heads >> 30), std::min<int64_t>(target / (nb * batch), heads));
    const int64_t nx = nb * groups;
    if (nx > 0x7fffffff || batch > 65535) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nx, batch);
    const float lb = log2f(base);
    const auto go = [&](auto kern, auto* t) {
        using T = std::remove_reference_t<decltype(*t)>;
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, (const T*)in, (T*)out, L, dq, half, J, rows, groups, lb, pos0);
    };
    if (elem_bytes == 2) go(half % 4 ? rope_kernel<1, bf16_t> : half % 8 ? rope_kernel<4, bf16_t> : rope_kernel<8, bf16_t>, (bf16_t*)nullptr);
    else go(half % 4 ? rope_kernel<1, float> : half % 8 ? rope_kernel<4, float> : rope_kernel<8, float>, (float*)nullptr);
    return hipGetLastError();
}

hipError_t transpose_batched(hipStream_t st, const void* in, void* out, int rows, int cols, int64_t ld_out,
                             int64_t s_in, int64_t s_out, int batch, int elem_bytes) {
    if (rows <= 0 || cols <= 0 || batch <= 0) return hipSuccess;
    dim3 grid((cols + TT - 1) / TT, (rows + TT - 1) / TT, batch);
    if (grid.y > 65535 || grid.z > 65535) return hipErrorInvalidValue;
    const bool vec8 = elem_bytes == 2 && rows % 8 == 0 && cols % 8 == 0 && ld_out % 8 == 0 && s_in % 8 == 0 &&
                      s_out % 8 == 0 && ((((uintptr_t)in) | ((uintptr_t)out)) & 15) == 0;
    if (vec8)
        hipLaunchKernelGGL(transpose_u16x8_kernel, grid, dim3(256), 0, st, (const uint16_t*)in, (uint16_t*)out, rows, cols,
                           ld_out, s_in, s_out);
    else if (elem_bytes == 2)
        hipLaunchKernelGGL(transpose_kernel<uint16_t>, grid, dim3(256), 0, st, (const uint16_t*)in, (uint16_t*)out,
                           rows, cols, ld_out, s_in, s_out);
    else
        hipLaunchKernelGGL(transpose_kernel<uint32_t>, grid, dim3(256), 0, st, (const uint32_t*)in, (uint32_t*)out,
                           rows, cols, ld_out, s_in, s_out);
    return hipGetLastError();
}

hipError_t fill_gaussian(hipStream_t st, float* out, int64_t n, uint64_t seed) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(gaussian_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, out, n, seed);
    return hipGetLastError();
}

hipError_t fill_zero_i32(hipStream_t st, int32_t* p, int64_t n) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_i32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

}  // namespace atp
