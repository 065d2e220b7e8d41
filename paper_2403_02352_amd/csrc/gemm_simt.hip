// GEMM with element strides on the matrix cores:  C(m,n) = sum_k A(m,k) · B(n,k).
// Serves the ATP_F32 storage path (v_mfma_f32_32x32x2f32: fp32 products, fp32 accumulation) and, on the
// bf16 path, every shape or alignment the asynchronous kernel of gemm_mfma.hip does not cover.
//
// A tile goes global -> registers -> LDS, because only this way can an operand be turned, widened, added to its lo
// plane, masked at a ragged edge and read at any alignment.  Tile kt is multiplied out of one of two LDS buffers
// while tile kt+1 waits in registers and tile kt+2 is on its way: what bounds these products at the sizes they
// meet is the latency of a few k-tiles, not the arithmetic.  An operand may be contiguous along k or along its rows (a
// transposed operand needs no pass of its own); LDS always holds rows of k, padded by 16 bytes, so a fragment read is
// one conflict-free 16-byte access.
//
// Order of the sums.  The fp32 matrix instructions add their products one by one, k ascending, each with a single rounding (compared bit
// by bit with a chain of fmaf, denormal results included).  On the fp32 path every output is therefore one chain over k = 0 .. K-1,
// whatever the tile: the same bits as scalar fused multiply-adds in that order give.  The trailing columns of U_r
// magnify the last bits of these products a few hundred times where the spectrum of X falls below its noise, up to two thousand: an
// order that changes with the tile shows there as 1e-4.
//
// Tile choice.  The fp32 matrix cores do 256 flop per clock and compute unit, so what counts is that the 256 compute
// units have work: 128×128 tiles when at least 192 of them exist, else 64×64, else 32×32.  The four waves of a 32×32 tile take a
// 16×16 quarter each (fp32), or share the tile and split k, their sums meeting in LDS at the end (bf16).
// Measured on one MI355X against a scalar-FMA kernel with 64×64 tiles: four products (512×768)·(768×128) 151 -> 12 µs, the block at
// that shape 5.07 -> 0.89 ms, 2096×968 with k = 8 (tiles that are all epilogue) 15.1 -> 14 µs.
#include "common.h"

#include <type_traits>

namespace atp {
namespace {

__device__ __forceinline__ float silu_f(float x) { return x / (1.0f + expf(-x)); }

__device__ __forceinline__ bf16x8 u4_bf16x8(const uint4& u) {
    union { uint4 u; bf16x8 b; } c;
    c.u = u;
    return c.b;
}

// One operand: element (row, k) at p[row·rs + k·cs], optional lo plane added to it.
// mode 0: contiguous along k (cs == 1), 1: contiguous along the rows (rs == 1), 2: neither.
struct Operand {
    const void* p;
    const void* lo;
    int64_t rs, cs;
    int rows, K;
    int mode;
    int vec;   // elements a load may take at once along the contiguous direction: 8 / 4 (whole pieces), 2, 1
};

template <typename T> __device__ __forceinline__ float widen(T x);
template <> __device__ __forceinline__ float widen<float>(float x) { return x; }
template <> __device__ __forceinline__ float widen<bf16_t>(bf16_t x) { return bf2f(x); }

typedef f32x4 f32x4_4 __attribute__((aligned(4)));   // four floats at a multiple of four bytes: all that a 16-byte load needs

// Pieces of a tile run along the contiguous direction of the operand (along k where there is none).  A thread's pieces lie at even
// distances, so it keeps the address and the coordinates of its first one in tile 0; everything else is the same for all threads.
// Registers: with addresses per piece and form of the operand, hoisted out of the k loop, and element loads under conditions of their
// own, the kernels took 260 to 446, one workgroup on a compute unit that has LDS for two to four.  Now 115 to 255: four products
// (512×768)·(768×768) 63 -> 41 µs, 2096×968 with k = 8 22.6 -> 14.
template <typename T>
struct First {
    const T *p, *lo;
    int row, k;
};
template <typename T>
__device__ __forceinline__ First<T> first_piece(const Operand& o, int row, int k) {
    const int64_t off = (int64_t)row * o.rs + (int64_t)k * o.cs;
    const T* lo = reinterpret_cast<const T*>(o.lo);
    return {reinterpret_cast<const T*>(o.p) + off, lo ? lo + off : nullptr, row, k};
}

// ---- fp32 tiles: ROWS × BK floats in LDS, pitch BK + 4; a piece is four elements --
// PERM: each group of eight k lies in LDS as 0 2 4 6 1 3 5 7, so that the four k of a lane half, every second one, are one 16-byte read
template <typename T, int ROWS, int BK, int NT, bool PERM>
struct LoadF32 {
    static constexpr int P = BK + 4, N = ROWS * BK / 4 / NT, WORDS = ROWS * P;
    static constexpr int CK = BK / 4, CR = ROWS / 4;   // pieces of a row of k, of a column of rows
    static_assert(ROWS * BK % (4 * NT) == 0 && NT % CK == 0 && NT % CR == 0, "tile / threads mismatch");
    f32x4 v[N];
    static __device__ __forceinline__ First<T> first(const Operand& o, int row0, int tid) {
        return o.mode == 1 ? first_piece<T>(o, row0 + 4 * (tid % CR), tid / CR) : first_piece<T>(o, row0 + tid / CK, 4 * (tid % CK));
    }
    static __device__ __forceinline__ f32x4 piece(const T* q) {
        if constexpr (sizeof(T) == 4) return *reinterpret_cast<const f32x4_4*>(q);
        else {
            const uint2 u = *reinterpret_cast<const uint2*>(q);
            return f32x4{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                         __uint_as_float(u.y & 0xffff0000u)};
        }
    }
    __device__ __forceinline__ void load(const Operand& o, const First<T>& f, int row0, int kt) {
        const bool by_row = o.mode == 1, wide = sizeof(T) == 4 ? o.mode != 2 : o.vec >= 4;
        const int64_t tile = (int64_t)kt * BK * o.cs, step = by_row ? (NT / CR) * o.cs : (NT / CK) * o.rs, along = by_row ? o.rs : o.cs;
        const int room = by_row ? o.rows - f.row : o.K - kt * BK - f.k;   // elements from here to the end along the piece
        if (wide && row0 + ROWS <= o.rows && (kt + 1) * BK <= o.K) {   // a tile inside the matrix
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] = piece(f.p + (tile + i * step));
            if (f.lo)
#pragma unroll
                for (int i = 0; i < N; ++i) v[i] += piece(f.lo + (tile + i * step));
            return;
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (room <= 0 || (by_row ? f.k + kt * BK + i * (NT / CR) >= o.K : f.row + i * (NT / CK) >= o.rows)) continue;
            const T* q = f.p + (tile + i * step);
            const T* l = f.lo + (tile + i * step);
            if (wide && room >= 4) {
                v[i] = piece(q);
                if (f.lo) v[i] += piece(l);
            } else {   // element by element, those past the end from the last one's place and then zero
                f32x4 x;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = widen<T>(q[min(e, room - 1) * along]);
                if (f.lo)
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] += widen<T>(l[min(e, room - 1) * along]);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i][e] = e < room ? x[e] : 0.f;
            }
        }
    }
    __device__ __forceinline__ void store(float* lds, int mode, int tid) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int c = i * NT + tid;
            if (mode == 1) {
                const int k = c / (ROWS / 4), rq = c % (ROWS / 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) lds[(4 * rq + e) * P + (PERM ? (k & ~7) + 4 * (k & 1) + ((k & 7) >> 1) : k)] = v[i][e];
            } else if constexpr (PERM) {
                const int q = c % (BK / 4);
                float* d = lds + (c / (BK / 4)) * P + 8 * (q >> 1) + 2 * (q & 1);
                *reinterpret_cast<f32x2*>(d) = f32x2{v[i][0], v[i][2]};
                *reinterpret_cast<f32x2*>(d + 4) = f32x2{v[i][1], v[i][3]};
            } else {
                *reinterpret_cast<f32x4*>(lds + (c / (BK / 4)) * P + 4 * (c % (BK / 4))) = v[i];
            }
        }
    }
};

// ---- bf16 tiles: ROWS × BK bf16 in LDS, pitch BK + 8; a piece is 8 elements along k, or 2 (k) × 8 (rows) ---------
template <int ROWS, int BK, int NT>
struct LoadBF16 {
    static constexpr int P = BK + 8, N = ROWS * BK / 8 / NT, WORDS = ROWS * P / 2;
    static constexpr int CK = BK / 8, CR = ROWS / 8;
    static_assert(ROWS * BK % (16 * NT) == 0 && NT % CK == 0 && NT % CR == 0, "tile / threads mismatch");
    uint4 v[N];
    static __device__ __forceinline__ First<bf16_t> first(const Operand& o, int row0, int tid) {
        return o.mode == 1 ? first_piece<bf16_t>(o, row0 + 8 * (tid % CR), 2 * (tid / CR)) : first_piece<bf16_t>(o, row0 + tid / CK, 8 * (tid % CK));
    }
    __device__ __forceinline__ void load(const Operand& o, const First<bf16_t>& f, int row0, int kt) {
        const bool by_row = o.mode == 1;
        const int64_t tile = (int64_t)kt * BK * o.cs, step = by_row ? 2 * (NT / CR) * o.cs : (NT / CK) * o.rs, along = by_row ? o.rs : o.cs;
        const int room = by_row ? o.rows - f.row : o.K - kt * BK - f.k;
        // pieces 2j and 2j + 1 of a by_row operand are two consecutive k
        const auto at = [&](int i) { return f.p + (tile + (by_row ? (i / 2) * step + (i & 1) * o.cs : i * step)); };
        if (o.vec >= 8 && row0 + ROWS <= o.rows && (kt + 1) * BK <= o.K) {   // a tile inside the matrix
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] = *reinterpret_cast<const uint4*>(at(i));
            return;
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            v[i] = make_uint4(0u, 0u, 0u, 0u);
            if (room <= 0 || (by_row ? f.k + kt * BK + 2 * (i / 2) * (NT / CR) + (i & 1) >= o.K : f.row + i * (NT / CK) >= o.rows)) continue;
            const bf16_t* q = at(i);
            if (o.vec >= 8) v[i] = *reinterpret_cast<const uint4*>(q);
            else {   // two or one at a time, those past the end from the last one's place and then zero
                uint32_t w[4];
                if (o.vec >= 2) {   // 4-byte loads; K is even, so a pair is inside or outside as a whole
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[e] = *reinterpret_cast<const uint32_t*>(q + min(2 * e, room - 2));
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[e] = 2 * e < room ? w[e] : 0u;
                } else {
                    uint32_t x[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[e] = q[min(e, room - 1) * along];
#pragma unroll
                    for (int e = 0; e < 8; e += 2) w[e / 2] = (e < room ? x[e] : 0u) | (e + 1 < room ? x[e + 1] << 16 : 0u);
                }
                v[i] = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
    }
    __device__ __forceinline__ void store(float* lds_f, int mode, int tid) const {
        bf16_t* lds = reinterpret_cast<bf16_t*>(lds_f);
        if (mode == 1) {
#pragma unroll
            for (int i = 0; i < N / 2; ++i) {
                const int c = i * NT + tid, k = 2 * (c / (ROWS / 8)), rq = c % (ROWS / 8);
                const uint32_t* a = reinterpret_cast<const uint32_t*>(&v[2 * i]);
                const uint32_t* b = reinterpret_cast<const uint32_t*>(&v[2 * i + 1]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    *reinterpret_cast<uint32_t*>(lds + (8 * rq + 2 * e) * P + k) = (a[e] & 0xffffu) | (b[e] << 16);
                    *reinterpret_cast<uint32_t*>(lds + (8 * rq + 2 * e + 1) * P + k) = (a[e] >> 16) | (b[e] & 0xffff0000u);
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int c = i * NT + tid;
                *reinterpret_cast<uint4*>(lds + (c / (BK / 8)) * P + 8 * (c % (BK / 8))) = v[i];
            }
        }
    }
};

// BM×BN block tile, waves of (UT·TM)×(UT·TN), UT = 32 or 16 the matrix instruction's tile; KW waves share a wave tile and take every
// KW-th k-step (bf16 only: on the fp32 path the order of a sum is fixed).
// BF: operands stay bf16 (v_mfma_f32_32x32x16_bf16: exact products, fp32 accumulation), else everything is fp32.
template <typename TA, typename TB, bool BF, int BM, int BN, int UT, int TM, int TN, int KW, int BK, bool SWIGLU>
__global__ void __launch_bounds__((BM / (UT * TM)) * (BN / (UT * TN)) * KW * 64, 2)
gemm_strided_kernel(SimtArgs p, Operand oa, Operand ob, int tilesM, int tilesN) {
    static_assert((BF && UT == 32) || (!BF && KW == 1), "one chain over k on the fp32 path");
    constexpr int NWN = BN / (UT * TN), NWT = (BM / (UT * TM)) * NWN, NT = NWT * KW * 64;
    using LA = std::conditional_t<BF, LoadBF16<BM, BK, NT>, LoadF32<TA, BM, BK, NT, UT == 32>>;
    using LB = std::conditional_t<BF, LoadBF16<BN, BK, NT>, LoadF32<TB, BN, BK, NT, UT == 32>>;
    using Acc = std::conditional_t<UT == 32, f32x16, f32x4>;
    constexpr int NV = UT == 32 ? 16 : 4;   // accumulator registers
    constexpr int NB2 = SWIGLU ? 2 : 1;
    constexpr int STAGE = LA::WORDS + NB2 * LB::WORDS;
    static_assert(KW == 1 || (KW - 1) * NWT * TM * TN * NB2 * 1024 <= 2 * STAGE, "the partial sums meet in the stages");
    __shared__ __align__(16) float lds[2 * STAGE];
    // consecutive workgroup ids go to the 8 XCDs in turn: each XCD gets a contiguous run of the tile list (tile column
    // fastest), so the tiles that share rows of A share an L2
    int id = blockIdx.x;
    if ((gridDim.x & 7) == 0) id = (id & 7) * (gridDim.x >> 3) + (id >> 3);
    const int bz = id / (tilesM * tilesN), m0 = id / tilesN % tilesM * BM, n0 = id % tilesN * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kw = wave / NWT, wt = wave % NWT, wm = wt / NWN, wn = wt % NWN;
    const int l32 = lane & (UT - 1), lh = lane / UT;   // column of the accumulators, and which of their rows
    oa.p = reinterpret_cast<const TA*>(oa.p) + (int64_t)bz * p.sA;
    if (oa.lo) oa.lo = reinterpret_cast<const TA*>(oa.lo) + (int64_t)bz * p.sA;
    ob.p = reinterpret_cast<const TB*>(ob.p) + (int64_t)bz * p.sB;
    if (ob.lo) ob.lo = reinterpret_cast<const TB*>(ob.lo) + (int64_t)bz * p.sB;
    Operand ob2 = ob;   // SWIGLU: the up rows, N rows further on
    if constexpr (SWIGLU) ob2.p = reinterpret_cast<const TB*>(ob.p) + (int64_t)p.N * ob.rs;

    Acc acc[NB2][TM][TN];
#pragma unroll
    for (int h = 0; h < NB2; ++h)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < NV; ++v) acc[h][i][j][v] = 0.f;

    struct Regs { LA a; LB b, b2; };
    const auto fa = LA::first(oa, m0, tid);
    const auto fb = LB::first(ob, n0, tid);
    const auto fb2 = LB::first(ob2, n0, tid);
    auto load = [&](Regs& r, int kt) {
        r.a.load(oa, fa, m0, kt);
        r.b.load(ob, fb, n0, kt);
        if constexpr (SWIGLU) r.b2.load(ob2, fb2, n0, kt);
    };
    auto store = [&](const Regs& r, int buf) {
        r.a.store(lds + buf * STAGE, oa.mode, tid);
        r.b.store(lds + buf * STAGE + LA::WORDS, ob.mode, tid);
        if constexpr (SWIGLU) r.b2.store(lds + buf * STAGE + LA::WORDS + LB::WORDS, ob.mode, tid);
    };
    auto compute = [&](int buf, int kt) {
        const float* sa = lds + buf * STAGE;
        const float* sb = sa + LA::WORDS;
        if constexpr (BF) {
            const bf16_t* ha = reinterpret_cast<const bf16_t*>(sa);
#pragma unroll
            for (int s = 0; s < BK / 16 / KW; ++s) {
                const int k = 16 * (s * KW + kw) + 8 * lh;
                bf16x8 a[TM];
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    a[i] = u4_bf16x8(*reinterpret_cast<const uint4*>(ha + (32 * (wm * TM + i) + l32) * LA::P + k));
#pragma unroll
                for (int h = 0; h < NB2; ++h)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const bf16_t* hb = reinterpret_cast<const bf16_t*>(sb + h * LB::WORDS);
                        const bf16x8 b = u4_bf16x8(*reinterpret_cast<const uint4*>(hb + (32 * (wn * TN + j) + l32) * LB::P + k));
#pragma unroll
                        for (int i = 0; i < TM; ++i) acc[h][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b, acc[h][i][j], 0, 0, 0);
                    }
            }
        } else if constexpr (UT == 16) {
            const int left = min(BK, p.K - kt * BK);   // (zeros from there on; block of 128×64 with r = 32: 367 µs with all of them, 354 without)
#pragma unroll 1
            for (int k0 = 0; k0 < left; k0 += 32)
#pragma unroll
                for (int k = k0; k < k0 + 32; k += 4) {   // lanes of quarter lh take k + lh; rows of 132 floats: the 64 lanes meet 64 banks
                    float a[TM];
#pragma unroll
                    for (int i = 0; i < TM; ++i) a[i] = sa[(16 * (wm * TM + i) + l32) * LA::P + k + lh];
#pragma unroll
                    for (int h = 0; h < NB2; ++h)
#pragma unroll
                        for (int j = 0; j < TN; ++j) {
                            const float b = sb[h * LB::WORDS + (16 * (wn * TN + j) + l32) * LB::P + k + lh];
#pragma unroll
                            for (int i = 0; i < TM; ++i) acc[h][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b, acc[h][i][j], 0, 0, 0);
                        }
                }
        } else {
#pragma unroll
            for (int s = 0; s < BK / 8; ++s) {
                // lanes of half lh take k = lh, 2 + lh, 4 + lh, 6 + lh: one 16-byte read per operand feeds four MFMAs
                const int k = 8 * s + 4 * lh;
                f32x4 a[TM];
#pragma unroll
                for (int i = 0; i < TM; ++i) a[i] = *reinterpret_cast<const f32x4*>(sa + (32 * (wm * TM + i) + l32) * LA::P + k);
#pragma unroll
                for (int h = 0; h < NB2; ++h)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const f32x4 b = *reinterpret_cast<const f32x4*>(sb + h * LB::WORDS + (32 * (wn * TN + j) + l32) * LB::P + k);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
#pragma unroll
                            for (int i = 0; i < TM; ++i) acc[h][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[e], acc[h][i][j], 0, 0, 0);
                    }
            }
        }
    };

    const int nkt = (p.K + BK - 1) / BK;
    // tile kt is in LDS, tile kt+1 in registers, tile kt+2 on its way
    Regs r0, r1;
    load(r0, 0);
    if (nkt > 1) load(r1, 1);
    store(r0, 0);
    for (int kt = 0; kt < nkt; kt += 2) {
        if (kt + 2 < nkt) load(r0, kt + 2);
        __syncthreads();   // tile kt is in its buffer, and nobody reads the other one any more
        compute(0, kt);
        if (kt + 1 >= nkt) break;
        store(r1, 1);
        if (kt + 3 < nkt) load(r1, kt + 3);
        __syncthreads();
        compute(1, kt + 1);
        if (kt + 2 < nkt) store(r0, 0);
    }
    if constexpr (KW > 1) {   // the waves' shares meet in LDS, added in a fixed order
        __syncthreads();
        constexpr int PER = NB2 * TM * TN * 1024;
        if (kw > 0) {
            float* d = lds + ((kw - 1) * NWT + wt) * PER + lane;
#pragma unroll
            for (int h = 0; h < NB2; ++h)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int v = 0; v < 16; ++v) d[(((h * TM + i) * TN + j) * 16 + v) * 64] = acc[h][i][j][v];
        }
        __syncthreads();
        if (kw > 0) return;
#pragma unroll
        for (int q = 0; q < KW - 1; ++q) {
            const float* d = lds + (q * NWT + wt) * PER + lane;
#pragma unroll
            for (int h = 0; h < NB2; ++h)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[h][i][j][v] += d[(((h * TM + i) * TN + j) * 16 + v) * 64];
        }
    }

    if constexpr (SWIGLU) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < NV; ++v) acc[0][i][j][v] = silu_f(acc[0][i][j][v]) * acc[NB2 - 1][i][j][v];
    }
    // one output after the other, each with a pointer of its own that walks down the rows
    const auto each = [&](int64_t row_step, int64_t col_step, auto put) {   // put(offset in the output, value)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int row0 = m0 + UT * (wm * TM + i) + 4 * lh, col = n0 + UT * (wn * TN + j) + l32;
                if (col >= p.N) continue;
                int64_t at = (int64_t)row0 * row_step + (int64_t)col * col_step;
#pragma unroll
                for (int g = 0; g < NV / 4; ++g, at += 4 * row_step)
#pragma unroll
                    for (int e = 0; e < 4; ++e, at += row_step)
                        if (row0 + 8 * g + e < p.M) put(at, acc[0][i][j][4 * g + e]);
            }
    };
    if (p.C32) each(p.ldc, 1, [&, d = p.C32 + (int64_t)bz * p.sC](int64_t at, float x) { d[at] = x; });
    if (p.C16) each(p.ldc, 1, [&, d = p.C16 + (int64_t)bz * p.sC](int64_t at, float x) { d[at] = f2bf(x); });
    if (p.C16lo) each(p.ldc, 1, [&, d = p.C16lo + (int64_t)bz * p.sC](int64_t at, float x) { d[at] = f2bf(x - bf2f(f2bf(x))); });
    if (p.CT16) each(1, p.ldct, [&, d = p.CT16 + (int64_t)bz * p.sCT](int64_t at, float x) { d[at] = f2bf(x); });
    if (p.CT32) {
        float* d = p.CT32 + (int64_t)bz * p.sCT;
        // four consecutive rows of an accumulator are one 16-byte piece of a row of Cᵀ; single elements would touch a line each
        if (p.M % 4 == 0 && p.ldct % 4 == 0 && p.sCT % 4 == 0 && ((uintptr_t)p.CT32 & 15) == 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int row0 = m0 + UT * (wm * TM + i) + 4 * lh, col = n0 + UT * (wn * TN + j) + l32;
                    if (col >= p.N) continue;
                    float* q = d + (int64_t)col * p.ldct + row0;
                    const Acc& c = acc[0][i][j];
#pragma unroll
                    for (int g = 0; g < NV / 4; ++g)
                        if (row0 + 8 * g < p.M) *reinterpret_cast<f32x4*>(q + 8 * g) = f32x4{c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]};
                }
        } else each(1, p.ldct, [&](int64_t at, float x) { d[at] = x; });
    }
}

// how the loads of an operand may be widened: `piece` elements at once need 16-byte (8-byte when bf16 is widened to
// fp32) pieces at aligned addresses that are inside or outside the matrix as a whole
Operand operand(const void* ptr, const void* lo, int64_t rs, int64_t cs, int64_t sbatch, int rows, int K, int es, int piece) {
    Operand o;
    o.p = ptr; o.lo = lo; o.rs = rs; o.cs = cs; o.rows = rows; o.K = K;
    o.mode = cs == 1 ? 0 : (rs == 1 ? 1 : 2);
    const int64_t ld = o.mode == 0 ? rs : cs;
    const auto fits = [&](int n) {
        return o.mode != 2 && ld % n == 0 && sbatch % n == 0 && (((uintptr_t)ptr | (uintptr_t)lo) % (size_t)(n * es)) == 0 &&
               ((o.mode == 0 ? K : rows) % n == 0);
    };
    o.vec = fits(piece) ? piece : (es == 2 && o.mode == 0 && K % 2 == 0 && fits(2) ? 2 : 1);
    return o;
}

template <typename TA, typename TB, bool BF, int BM, int BN, int UT, int TM, int TN, int KW, int BK, bool SWIGLU>
hipError_t launch_tile(hipStream_t st, const SimtArgs& g, const Operand& oa, const Operand& ob) {
    const int tm = (g.M + BM - 1) / BM, tn = (g.N + BN - 1) / BN;
    const int64_t tiles = (int64_t)tm * tn * g.batch;
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    constexpr int NT = (BM / (UT * TM)) * (BN / (UT * TN)) * KW * 64;
    hipLaunchKernelGGL((gemm_strided_kernel<TA, TB, BF, BM, BN, UT, TM, TN, KW, BK, SWIGLU>), dim3((unsigned)tiles), dim3(NT), 0, st, g, oa, ob, tm, tn);
    return hipGetLastError();
}

template <typename TA, typename TB, bool BF, bool SWIGLU>
hipError_t launch_strided(hipStream_t st, const SimtArgs& g) {
    constexpr int piece = BF ? 8 : 4;
    const Operand oa = operand(g.A, g.A_lo, g.a_rs, g.a_cs, g.sA, g.M, g.K, sizeof(TA), piece);
    const Operand ob = operand(g.B, g.B_lo, g.b_rs, g.b_cs, g.sB, g.N, g.K, sizeof(TB), piece);
    const auto tiles = [&](int t) { return (int64_t)((g.M + t - 1) / t) * ((g.N + t - 1) / t) * g.batch; };
    constexpr int BK = BF ? 64 : 32;
    if (tiles(128) >= 192) return launch_tile<TA, TB, BF, 128, SWIGLU ? 64 : 128, 32, 2, SWIGLU ? 1 : 2, 1, BK, SWIGLU>(st, g, oa, ob);
    if (tiles(64) >= 192) return launch_tile<TA, TB, BF, 64, 64, 32, 1, 1, 1, BK, SWIGLU>(st, g, oa, ob);
    return launch_tile<TA, TB, BF, 32, 32, BF ? 32 : 16, 1, 1, BF ? 4 : 1, 128, SWIGLU>(st, g, oa, ob);
}

}  // namespace

hipError_t gemm_simt(hipStream_t st, OperandType ta, OperandType tb, const SimtArgs& g) {
    if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return hipSuccess;
    if (ta == OP_F32 && tb == OP_F32)
        return g.swiglu ? launch_strided<float, float, false, true>(st, g) : launch_strided<float, float, false, false>(st, g);
    if (ta == OP_BF16 && tb == OP_BF16) {
        // operands with a lo plane carry more than bf16: they are widened and multiplied in fp32
        if (g.A_lo || g.B_lo) return g.swiglu ? hipErrorInvalidValue : launch_strided<bf16_t, bf16_t, false, false>(st, g);
        return g.swiglu ? launch_strided<bf16_t, bf16_t, true, true>(st, g) : launch_strided<bf16_t, bf16_t, true, false>(st, g);
    }
    if (g.swiglu) return hipErrorInvalidValue;
    if (ta == OP_BF16) return launch_strided<bf16_t, float, false, false>(st, g);
    return launch_strided<float, bf16_t, false, false>(st, g);
}

}  // namespace atp
