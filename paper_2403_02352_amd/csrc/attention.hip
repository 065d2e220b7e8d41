// Softmax attention of all L queries over n_k keys/values (Fig.2b, Tab.1 row
// "Attention"; Eq.1 with K', V' in place of K, V).  n_k = r on the ATP path,
// n_k = L for the dense comparator.  The L×n_k score matrix lives only in
// registers: scores of a 64-key tile come out of the MFMA unit, the online
// softmax (running row max and row sum) is applied in registers, and the
// probabilities feed the value MFMA directly.
//
// bf16 kernel layout trick: the score tile is computed transposed,
// Sᵀ = K'·Qᵀ, so that every lane owns ONE query column (all 16 accumulator
// registers of a 32×32 MFMA tile belong to the same query).  Row max / row sum
// are then in-lane reductions plus one exchange between the two lane halves,
// and the probabilities are already laid out as the B operand of
// Oᵀ += V'ᵀ·Pᵀ.  Rows of the K' tile are fetched in a permuted order (bits 2 and
// 3 of the row index swapped) so that the 8 consecutive accumulator registers a
// lane feeds to the second MFMA correspond to 8 consecutive keys.  The value tile
// is staged as it lies in memory, keys by features, and two transposing LDS reads
// give a lane 8 keys of one feature.
// (A pass that turned V' first cost a launch: attention of 384 queries over 96
// keys, 12 heads of 64, 11.9 -> 9.1 µs without it.)
#include "common.h"

namespace atp {
namespace {

__device__ __forceinline__ bf16x8 u4_as_bf16x8(const uint4& u) {
    union { uint4 u; bf16x8 b; } c;
    c.u = u;
    return c.b;
}

constexpr int QT = 128;  // queries per workgroup (4 waves × 32)


// Tiles sit in LDS as plain rows of W 16-byte chunks (W = 16, 8 or 4); position p of row r holds chunk
// p ^ tile_swz<W>(r).  A 16-byte-per-lane LDS read is served 16 lanes at a time (16 × 16 B = all 64
// banks), and the 16 lanes of such a group read the same chunk of 16 consecutive rows (in some
// order): 16/W rows share one 256-byte bank span, so the swizzle counts those spans.
template <int W>
__device__ __forceinline__ int tile_swz(int r) {
    static_assert(W == 16 || W == 8 || W == 4, "row width");
    return W == 16 ? (r & 15) : W == 8 ? ((r >> 1) & 7) : ((r >> 2) & 3);
}

// The key/value tiles travel global -> LDS with asynchronous 16-byte copies (no registers), two
// stages: the copies of tile t+1 fly while tile t is multiplied.  Consecutive lanes of a copy
// fetch consecutive chunks of one row.
// LIN selects the first-order variant (Eq.8): the weight of key j is (1·U)_j + scale·<q, k_j>, no
// exponential and no running maximum; the normaliser is accumulated beside the numerator.
// KT = keys per tile (64, or 32: half the LDS and fewer live registers, so more workgroups per CU).
template <int DH, bool LIN, int KT>
__global__ void __launch_bounds__(256, KT == 32 ? 3 : 2) attn_bf16_kernel(AttnArgs a, float c_log2e) {
    constexpr int CK = DH / 8;            // 16-byte chunks per K-tile row
    constexpr int NKS = DH / 16;          // k-steps of the score MFMA
    constexpr int NCT = DH / 32;          // 32-row tiles of Oᵀ
    constexpr int NT = KT / 32;           // 32-key score tiles per key tile
    constexpr int KRPI = 64 / CK;         // K rows per copy instruction
    constexpr int NKI = KT / KRPI / 4;    // K copy instructions per wave and tile
    static_assert(NKI >= 1, "tile too small for four waves");
    __shared__ __align__(16) uint4 sK0[KT * CK];
    __shared__ __align__(16) uint4 sK1[KT * CK];
    __shared__ __align__(16) uint4 sV0[KT * CK];
    __shared__ __align__(16) uint4 sV1[KT * CK];

    // 1-D grid over (batch item, head, query block).  Consecutive workgroup ids go to the 8 XCDs in
    // turn: all query blocks of one (item, head) are given to one XCD, whose L2 then serves the
    // re-reads of that head's keys and values.
    const int nqb = (a.L + QT - 1) / QT, nbh = a.batch * a.heads;
    int bh, qb;
    if ((nbh & 7) == 0) {
        const int slot = blockIdx.x >> 3;
        bh = (blockIdx.x & 7) + 8 * (slot / nqb);
        qb = slot % nqb;
    } else {
        bh = blockIdx.x / nqb;
        qb = blockIdx.x % nqb;
    }
    const int b = bh / a.heads, h = bh % a.heads;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    const int q = qb * QT + wave * 32 + l32;
    const bf16_t* Qp = reinterpret_cast<const bf16_t*>(a.Q) + ((int64_t)b * a.L) * a.dq + h * DH;
    const bf16_t* Kp = reinterpret_cast<const bf16_t*>(a.K) + ((int64_t)b * a.nk) * a.dq + h * DH;
    const bf16_t* Vp = reinterpret_cast<const bf16_t*>(a.V) + ((int64_t)b * a.nk) * a.dq + h * DH;
    const float* csum = LIN ? a.colsum + (int64_t)b * a.nk_pad : nullptr;

    // per-lane pieces of the copy addresses
    int k_row[NKI];
    unsigned k_chunk[NKI], v_chunk[NKI];   // byte offsets
#pragma unroll
    for (int i = 0; i < NKI; ++i) {
        const int row = (i * 4 + wave) * KRPI + lane / CK;
        k_row[i] = row;
        k_chunk[i] = (unsigned)(((lane % CK) ^ tile_swz<CK>(row)) * 16);
        v_chunk[i] = (unsigned)(((lane % CK) ^ column_swz<DH>(row)) * 16);
    }
    // LDS byte address of this wave's first copy slot in each stage array (scalar registers); every
    // copy is a scalar base plus a 32-bit lane offset, untracked by the compiler: all waits for them
    // are explicit
    const unsigned wave_s = (unsigned)__builtin_amdgcn_readfirstlane(wave) * 1024u;
    const unsigned lK0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_void*)sK0) + wave_s;
    const unsigned lK1 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_void*)sK1) + wave_s;
    const unsigned lV0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_void*)sV0) + wave_s;
    const unsigned lV1 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_void*)sV1) + wave_s;
    const unsigned row_bytes = (unsigned)a.dq * 2u;
    auto issue = [&](int kt0, const uint4* sK, const uint4*) {
        const unsigned lk = (sK == sK0) ? lK0 : lK1, lv = (sK == sK0) ? lV0 : lV1;
#pragma unroll
        for (int i = 0; i < NKI; ++i) {
            const int key = min(kt0 + k_row[i], a.nk - 1);  // rows past the end: any valid row, masked below
            copy16_untracked(Kp, (unsigned)key * row_bytes + k_chunk[i], lk + (unsigned)i * 4096u);
            copy16_untracked(Vp, (unsigned)key * row_bytes + v_chunk[i], lv + (unsigned)i * 4096u);
        }
    };

    // query fragments (B operand of the score MFMA): 8 consecutive features per lane and k-step
    bf16x8 qf[NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
        uint4 v = make_uint4(0, 0, 0, 0);
        if (q < a.L) v = *reinterpret_cast<const uint4*>(Qp + (int64_t)q * a.dq + ks * 16 + lh * 8);
        qf[ks] = u4_as_bf16x8(v);
    }

    f32x16 o[NCT];
#pragma unroll
    for (int i = 0; i < NCT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[i][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    // S-tile row i holds key perm(i): bits 2 and 3 swapped
    const int prow = (l32 & ~0xC) | ((l32 & 4) << 1) | ((l32 & 8) >> 1);
    const int pswz = tile_swz<CK>(prow);
    int v_col[NCT];
#pragma unroll
    for (int i = 0; i < NCT; ++i) v_col[i] = column_frag_offset<DH>(lane, 32 * i);
    // Rows past the last key hold copies of it; their weight is zero, but zero times infinity is not: they become zeros.
    auto clear_tail = [&](int kt0, uint4* sV) {
        if (kt0 + KT <= a.nk) return;   // the same for every wave
        for (int c = (a.nk - kt0) * CK + tid; c < KT * CK; c += 256) sV[c] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
    };

    auto compute = [&](int kt0, const uint4* sK, const uint4* sV) {
        // ---- scores: Sᵀ[key, query] ------------------------------------------------
        f32x16 s[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int v = 0; v < 16; ++v) s[t][v] = 0.f;
            const int row = 32 * t + prow;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                const bf16x8 kf = u4_as_bf16x8(sK[row * CK + ((2 * ks + lh) ^ pswz)]);
                s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], s[t], 0, 0, 0);
            }
        }
        if constexpr (LIN) {
            // weights (1·U)_key + scale·s; keys past the end weigh nothing.  The 8 consecutive
            // accumulator registers of a lane are 8 consecutive keys.
            float acc_den = 0.f;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const int key0 = kt0 + 32 * t + 16 * g + 8 * lh;
                    const f32x4 c0 = *reinterpret_cast<const f32x4*>(csum + key0);
                    const f32x4 c1 = *reinterpret_cast<const f32x4*>(csum + key0 + 4);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float cj = e < 4 ? c0[e] : c1[e - 4];
                        const float sv = s[t][8 * g + e] * c_log2e;   // c_log2e carries the plain scale here
                        const bool live = (key0 + e) < a.nk;
                        const float pv = live ? cj + sv : 0.f;
                        acc_den += a.norm_rowsum ? pv : (live ? sv * cj : 0.f);
                        s[t][8 * g + e] = pv;
                    }
                }
            l_run += acc_den;
        } else {
            if (kt0 + KT > a.nk) {  // only the last tile can be ragged
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int key = kt0 + 32 * t + 16 * (v >> 3) + 8 * lh + (v & 7);
                        if (key >= a.nk) s[t][v] = -INFINITY;
                    }
            }
            float mloc = -INFINITY;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) mloc = fmaxf(mloc, s[t][v]);
            mloc = fmaxf(mloc, __shfl_xor(mloc, 32));
            const float m_new = fmaxf(m_run, mloc);
            // the running maximum settles after a few tiles: rescale only when some query of this wave
            // raised it (the factor is exactly 1 otherwise)
            if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {
                const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c_log2e);
                l_run *= alpha;
#pragma unroll
                for (int i = 0; i < NCT; ++i)
#pragma unroll
                    for (int v = 0; v < 16; ++v) o[i][v] *= alpha;
                m_run = m_new;
            }
            const float mc = m_run * c_log2e;
            float psum = 0.f;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float pv = __builtin_amdgcn_exp2f(fmaf(s[t][v], c_log2e, -mc));
                    s[t][v] = pv;
                    psum += pv;
                }
            l_run += psum;
        }

        // ---- Oᵀ += V'ᵀ · Pᵀ ---------------------------------------------------------
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                uint4 pu;
                pu.x = pack_bf2(s[t][8 * tt + 0], s[t][8 * tt + 1]);
                pu.y = pack_bf2(s[t][8 * tt + 2], s[t][8 * tt + 3]);
                pu.z = pack_bf2(s[t][8 * tt + 4], s[t][8 * tt + 5]);
                pu.w = pack_bf2(s[t][8 * tt + 6], s[t][8 * tt + 7]);
                const bf16x8 pf = u4_as_bf16x8(pu);
#pragma unroll
                for (int i = 0; i < NCT; ++i) {
                    const bf16x8 vf = read_column_frag<DH>(sV, v_col[i] + (32 * t + 16 * tt) * DH * 2);
                    o[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf, o[i], 0, 0, 0);
                }
            }
    };

    const int ntiles = (a.nk + KT - 1) / KT;
    issue(0, sK0, sV0);
    for (int kt = 0; kt < ntiles; kt += 2) {
        // the explicit vmcnt(0) makes this wave's copies of tile kt land before the barrier (the
        // compiler does not count asynchronous LDS copies as something a barrier has to wait for)
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();  // everybody's copies have landed; stage 1 is free
        if (kt + 1 < ntiles) issue((kt + 1) * KT, sK1, sV1);
        clear_tail(kt * KT, sV0);
        compute(kt * KT, sK0, sV0);
        if (kt + 1 < ntiles) {
            __builtin_amdgcn_s_waitcnt(0x0F70);
            __syncthreads();
            if (kt + 2 < ntiles) issue((kt + 2) * KT, sK0, sV0);
            clear_tail((kt + 1) * KT, sV1);
            compute((kt + 1) * KT, sK1, sV1);
        }
    }
    __syncthreads();

    // ---- normalise; the output tile turns in a wave-private LDS tile [32 queries][DH + 8] so that
    //      each query row leaves as 16-byte pieces -------------------------------------------------
    float l_tot = l_run + __shfl_xor(l_run, 32);
    if (LIN && !a.norm_rowsum) l_tot += a.n_tokens;
    const float inv = 1.0f / l_tot;
    // (row pitch DH elements; 16-byte piece p of query row q sits at piece p ^ (q & (DH/8 - 1)))
    static_assert(32 * DH * 2 <= KT * CK * 16 && 4 * 32 * DH * 2 <= 4 * KT * CK * 16, "output staging: one stage array per wave");
    bf16_t* ob = reinterpret_cast<bf16_t*>(wave == 0 ? sK0 : wave == 1 ? sK1 : wave == 2 ? sV0 : sV1);
#pragma unroll
    for (int i = 0; i < NCT; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            uint2 w;
            w.x = pack_bf2(o[i][4 * g + 0] * inv, o[i][4 * g + 1] * inv);
            w.y = pack_bf2(o[i][4 * g + 2] * inv, o[i][4 * g + 3] * inv);
            const int piece = (4 * i + g) ^ (l32 & (DH / 8 - 1));   // features 32i + 8g + 4lh .. +3 live in piece 4i + g
            *reinterpret_cast<uint2*>(ob + l32 * DH + piece * 8 + 4 * lh) = w;
        }
    constexpr int CPQ = DH / 8;  // 16-byte pieces per query row
#pragma unroll
    for (int it = 0; it < 32 * CPQ / 64; ++it) {
        const int c = it * 64 + lane, qq = c / CPQ, part = c % CPQ;
        const int qg = qb * QT + wave * 32 + qq;
        const uint4 v = *reinterpret_cast<const uint4*>(ob + qq * DH + (part ^ (qq & (CPQ - 1))) * 8);
        if (qg < a.L)
            *reinterpret_cast<uint4*>(reinterpret_cast<bf16_t*>(a.O) + ((int64_t)b * a.L + qg) * a.dq + h * DH + part * 8) = v;
    }
}

// ---------------------------------------------------------------------------
// fp32 storage path: same scheme on v_mfma_f32_32x32x2f32 (fp32 products and sums, expf).  A wave owns 32 queries and sees the
// scores transposed, one query per lane.  Accumulator register v of lane half lh belongs to key 8·(v/4) + 4·lh + v%4, so register v
// is at once the B operand of a k-step of Oᵀ += V'ᵀ·Pᵀ over the two keys of its halves: probabilities go from one product to the
// next without moving, and V' is read in its natural layout.
// KS = waves that share a query block, each with every KS-th tile of 32 keys (their sums meet in LDS): 1 when there are enough
// query blocks for the chip, else 4.  DP = head width padded to 64, 128 or 256 (zeros).
// Bound by the fp32 matrix cores (256 flop per clock and compute unit).  With one wave per query and scalar products this
// kernel took 358 µs of the 1.47 ms of a block of 4 × 512 × 768 with r = 128 (12 heads of 64); the block now takes 1.15 ms.
// ---------------------------------------------------------------------------
template <int DP, int KS, bool LIN>
__global__ void __launch_bounds__(256, 1) attn_f32_kernel(AttnArgs a, int dh, int vec) {
    constexpr int PK = DP + 4, PV = DP + 8;   // LDS row pitches: conflict-free 16-byte rows of K', 4 rows of V' half a bank span apart
    constexpr int TK = 32 * KS;               // keys per stage
    constexpr int NCT = DP / 32, NL = TK * DP / 4 / 256;
    constexpr int NQ = 4 / KS;
    __shared__ __align__(16) float sK[TK * PK];
    __shared__ __align__(16) float sV[TK * PV];
    const int b = blockIdx.z, h = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, lh = lane >> 5;
    const int kw = wave / NQ;
    const int q = (blockIdx.x * NQ + wave % NQ) * 32 + l32;
    const float* Qp = reinterpret_cast<const float*>(a.Q) + ((int64_t)b * a.L + min(q, a.L - 1)) * a.dq + h * dh;
    const float* Kp = reinterpret_cast<const float*>(a.K) + ((int64_t)b * a.nk) * a.dq + h * dh;
    const float* Vp = reinterpret_cast<const float*>(a.V) + ((int64_t)b * a.nk) * a.dq + h * dh;
    const float* csum = LIN ? a.colsum + (int64_t)b * a.nk_pad : nullptr;
    // four features of a row; zeros past the end of the head
    const auto quad = [&](const float* row, int c) {
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (vec) { if (c < dh) v = *reinterpret_cast<const f32x4*>(row + c); }
        else {
#pragma unroll
            for (int e = 0; e < 4; ++e) if (c + e < dh) v[e] = row[c + e];
        }
        return v;
    };
    f32x4 qf[DP / 8];   // features 8s + 4·lh .. +3, scaled
#pragma unroll
    for (int s = 0; s < DP / 8; ++s) qf[s] = quad(Qp, 8 * s + 4 * lh) * a.scale;
    f32x4 kr[NL], vr[NL];
    const auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int c = i * 256 + tid, key = k0 + c / (DP / 4), f = 4 * (c % (DP / 4));
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            kr[i] = key < a.nk ? quad(Kp + (int64_t)key * a.dq, f) : zero;
            vr[i] = key < a.nk ? quad(Vp + (int64_t)key * a.dq, f) : zero;
        }
    };
    f32x16 o[NCT];
#pragma unroll
    for (int i = 0; i < NCT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[i][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    load(0);
    for (int k0 = 0; k0 < a.nk; k0 += TK) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int c = i * 256 + tid, row = c / (DP / 4), f = 4 * (c % (DP / 4));
            *reinterpret_cast<f32x4*>(sK + row * PK + f) = kr[i];
            *reinterpret_cast<f32x4*>(sV + row * PV + f) = vr[i];
        }
        __syncthreads();
        if (k0 + TK < a.nk) load(k0 + TK);
        const int kb = k0 + 32 * kw;
        if (kb >= a.nk) continue;
        f32x16 s;
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = 0.f;
        // The matrix instruction adds one product after the other: a score of one chain over 256 features carried 2.6 times the error of
        // the tree sums of a wave per query.  Sums of 16 features, added up, carry less than those; 256 features take sums of 8, added
        // up over 64.
        constexpr int NU = DP == 256 ? 1 : 2, NM = DP == 256 ? 8 : DP / 8;   // k-groups of 8 in a sum, in an intermediate one
#pragma unroll
        for (int t = 0; t < DP / 8; t += NM) {
            f32x16 mid;
#pragma unroll
            for (int u = t; u < t + NM; u += NU) {
                f32x16 part;
#pragma unroll
                for (int v = 0; v < 16; ++v) part[v] = 0.f;
#pragma unroll
                for (int w = u; w < u + NU; ++w) {
                    const f32x4 kf = *reinterpret_cast<const f32x4*>(sK + (32 * kw + l32) * PK + 8 * w + 4 * lh);
#pragma unroll
                    for (int e = 0; e < 4; ++e) part = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[e], qf[w][e], part, 0, 0, 0);
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) mid[v] = u == t ? part[v] : mid[v] + part[v];
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] += mid[v];
        }
        if constexpr (LIN) {
            // first-order variant (Eq.8): weight (1·U)_j + <q, k_j>·scale; keys past the end weigh nothing
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int key = kb + 8 * (v >> 2) + 4 * lh + (v & 3);
                const bool live = key < a.nk;
                const float cj = csum[key];   // padded with zeros to a multiple of 64 keys
                const float pv = live ? cj + s[v] : 0.f;
                l_run += a.norm_rowsum ? pv : (live ? s[v] * cj : 0.f);
                s[v] = pv;
            }
        } else {
            float mloc = -INFINITY;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                if (kb + 8 * (v >> 2) + 4 * lh + (v & 3) >= a.nk) s[v] = -INFINITY;
                mloc = fmaxf(mloc, s[v]);
            }
            mloc = fmaxf(mloc, __shfl_xor(mloc, 32));
            const float m_new = fmaxf(m_run, mloc);
            if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {   // the factor is exactly 1 otherwise
                const float alpha = m_new > m_run ? expf(m_run - m_new) : 1.f;
                l_run *= alpha;
#pragma unroll
                for (int i = 0; i < NCT; ++i)
#pragma unroll
                    for (int v = 0; v < 16; ++v) o[i][v] *= alpha;
                m_run = m_new;
            }
            // no finite score so far (this wave's keys may all be at -inf while another's are not): weights of zero, not -inf - -inf
            const float m_ref = m_run == -INFINITY ? 0.f : m_run;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                s[v] = expf(s[v] - m_ref);
                l_run += s[v];
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float* vrow = sV + (32 * kw + 8 * (v >> 2) + 4 * lh + (v & 3)) * PV + l32;
#pragma unroll
            for (int i = 0; i < NCT; ++i) o[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(vrow[32 * i], s[v], o[i], 0, 0, 0);
        }
    }
    if constexpr (KS > 1) {   // wave 0 adds the other waves' shares, in order, at the common maximum
        constexpr int PER = (NCT * 16 + 2) * 64;
        static_assert((KS - 1) * PER <= TK * (PK + PV) && PER <= TK * PK, "shares fit the stages");
        __syncthreads();
        float* share = wave == 1 ? sK : wave == 2 ? sV : sV + PER;
        if (wave) {
#pragma unroll
            for (int i = 0; i < NCT; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) share[(16 * i + v) * 64 + lane] = o[i][v];
            share[NCT * 16 * 64 + lane] = m_run;
            share[(NCT * 16 + 1) * 64 + lane] = l_run;
        }
        __syncthreads();
        if (wave) return;
        float f[KS];
        if constexpr (LIN) {
#pragma unroll
            for (int w = 0; w < KS; ++w) f[w] = 1.f;
        } else {
            float m_all = m_run;
#pragma unroll
            for (int w = 1; w < KS; ++w) {
                f[w] = (w == 1 ? sK : w == 2 ? sV : sV + PER)[NCT * 16 * 64 + lane];
                m_all = fmaxf(m_all, f[w]);
            }
            f[0] = expf(m_run - m_all);
#pragma unroll
            for (int w = 1; w < KS; ++w) f[w] = expf(f[w] - m_all);
        }
        l_run *= f[0];
#pragma unroll
        for (int i = 0; i < NCT; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[i][v] *= f[0];
#pragma unroll
        for (int w = 1; w < KS; ++w) {
            const float* p = w == 1 ? sK : w == 2 ? sV : sV + PER;
#pragma unroll
            for (int i = 0; i < NCT; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[i][v] = fmaf(p[(16 * i + v) * 64 + lane], f[w], o[i][v]);
            l_run = fmaf(p[(NCT * 16 + 1) * 64 + lane], f[w], l_run);
        }
    }
    float l_tot = l_run + __shfl_xor(l_run, 32);
    if (LIN && !a.norm_rowsum) l_tot += a.n_tokens;
    const float inv = 1.0f / l_tot;
    if (q >= a.L) return;
    float* Op = reinterpret_cast<float*>(a.O) + ((int64_t)b * a.L + q) * a.dq + h * dh;
#pragma unroll
    for (int i = 0; i < NCT; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int c = 32 * i + 8 * g + 4 * lh;
            const f32x4 v = {o[i][4 * g] * inv, o[i][4 * g + 1] * inv, o[i][4 * g + 2] * inv, o[i][4 * g + 3] * inv};
            if (vec) { if (c < dh) *reinterpret_cast<f32x4*>(Op + c) = v; }
            else {
#pragma unroll
                for (int e = 0; e < 4; ++e) if (c + e < dh) Op[c + e] = v[e];
            }
        }
}

// A few keys of wide heads: one wave per query, features spread over the lanes, key after key.  A tile of 32 keys and 128 queries takes the
// same time whatever is in it (12 µs at a head width of 256, with the loads before it and the sums after it in one chain); this kernel takes
// about 0.6 µs per key while the waves fit the chip.
template <bool LIN>
__global__ void __launch_bounds__(256) attn_f32_few_keys_kernel(AttnArgs a, int dh) {
    const int b = blockIdx.z, h = blockIdx.y, lane = threadIdx.x & 63;
    const int q = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (q >= a.L) return;
    const float* Qp = reinterpret_cast<const float*>(a.Q) + ((int64_t)b * a.L + q) * a.dq + h * dh;
    const float* Kp = reinterpret_cast<const float*>(a.K) + ((int64_t)b * a.nk) * a.dq + h * dh;
    const float* Vp = reinterpret_cast<const float*>(a.V) + ((int64_t)b * a.nk) * a.dq + h * dh;
    const float* csum = LIN ? a.colsum + (int64_t)b * a.nk_pad : nullptr;
    float qv[4], ov[4];   // features lane, lane + 64, ...
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = lane + 64 * i;
        qv[i] = c < dh ? Qp[c] * a.scale : 0.f;
        ov[i] = 0.f;
    }
    float m_run = -INFINITY, l_run = 0.f;
    for (int j = 0; j < a.nk; ++j) {
        const float *kr = Kp + (int64_t)j * a.dq, *vr = Vp + (int64_t)j * a.dq;
        float s = 0.f, p, keep = 1.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) if (lane + 64 * i < dh) s = fmaf(qv[i], kr[lane + 64 * i], s);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
        if constexpr (LIN) {
            p = csum[j] + s;
            l_run += a.norm_rowsum ? p : s * csum[j];
        } else {
            const float m_new = fmaxf(m_run, s), m_ref = m_new == -INFINITY ? 0.f : m_new;   // (no finite score so far: weights of zero)
            keep = expf(m_run - m_ref);
            p = expf(s - m_ref);
            l_run = l_run * keep + p;
            m_run = m_new;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) if (lane + 64 * i < dh) ov[i] = fmaf(p, vr[lane + 64 * i], ov[i] * keep);
    }
    if (LIN && !a.norm_rowsum) l_run += a.n_tokens;
    const float inv = 1.0f / l_run;
    float* Op = reinterpret_cast<float*>(a.O) + ((int64_t)b * a.L + q) * a.dq + h * dh;
#pragma unroll
    for (int i = 0; i < 4; ++i) if (lane + 64 * i < dh) Op[lane + 64 * i] = ov[i] * inv;
}

template <int DP, int KS>
hipError_t launch_attn_f32(hipStream_t st, const AttnArgs& a, int dh) {
    const dim3 grid((a.L + 128 / KS - 1) / (128 / KS), a.heads, a.batch);
    const int vec = dh % 4 == 0;   // bases are 16-byte aligned, rows and heads then start at multiples of 16 bytes
    if (a.linearised) hipLaunchKernelGGL((attn_f32_kernel<DP, KS, true>), grid, dim3(256), 0, st, a, dh, vec);
    else hipLaunchKernelGGL((attn_f32_kernel<DP, KS, false>), grid, dim3(256), 0, st, a, dh, vec);
    return hipGetLastError();
}

// out[b][j] = sum over the L rows of U[b][:, j]; one workgroup per (64 columns, item): thread (ry, cx)
// adds rows ry, ry+16, ... of column cx in a fixed order, then the sixteen partial sums are added in a
// fixed order.  Columns r .. ld_out-1 of out are zeroed.  Bound by load latency (r/64 workgroups), hence sixteen
// waves with eight loads in flight each: 123 -> 12 µs at L = 2048, r = 512 (four waves, one load at a time before).
template <typename T>
__global__ void __launch_bounds__(1024) colsum_kernel(const T* __restrict__ U, float* __restrict__ out, int L, int r,
                                                      int64_t ld_out) {
    __shared__ float part[16][64];
    const int b = blockIdx.y;
    const int cx = threadIdx.x & 63, ry = threadIdx.x >> 6;
    const int col = blockIdx.x * 64 + cx;
    float s = 0.f;
    if (col < r) {
        const T* p = U + (int64_t)b * L * r + col;
#pragma unroll 8
        for (int i = ry; i < L; i += 16) {
            if constexpr (sizeof(T) == 2) s += bf2f(p[(int64_t)i * r]);
            else s += p[(int64_t)i * r];
        }
    }
    part[ry][cx] = s;
    __syncthreads();
    if (ry == 0 && col < ld_out) {
        float t = 0.f;
#pragma unroll
        for (int q = 0; q < 16; ++q) t += part[q][cx];
        out[(int64_t)b * ld_out + col] = (col < r) ? t : 0.f;
    }
}

}  // namespace

hipError_t column_sums(hipStream_t st, const void* U, float* out, int L, int r, int64_t ld_out, int batch, int elem_bytes) {
    dim3 grid((unsigned)((ld_out + 63) / 64), batch);
    if (grid.y > 65535) return hipErrorInvalidValue;
    if (elem_bytes == 2)
        hipLaunchKernelGGL(colsum_kernel<bf16_t>, grid, dim3(1024), 0, st, (const bf16_t*)U, out, L, r, ld_out);
    else
        hipLaunchKernelGGL(colsum_kernel<float>, grid, dim3(1024), 0, st, (const float*)U, out, L, r, ld_out);
    return hipGetLastError();
}

hipError_t attention_bf16(hipStream_t st, const AttnArgs& a) {
    const int dh = a.dq / a.heads;
    const int64_t nwg = (int64_t)((a.L + QT - 1) / QT) * a.heads * a.batch;
    if (nwg > 0x7fffffff) return hipErrorInvalidValue;
    dim3 grid((unsigned)nwg);
    const float c = a.linearised ? a.scale : a.scale * 1.4426950408889634f;
    if (dh != 128 && dh != 64) return hipErrorInvalidValue;
#ifndef ATP_ATTN_KT
#define ATP_ATTN_KT 64
#endif
    if (a.linearised) {
        if (dh == 128) hipLaunchKernelGGL((attn_bf16_kernel<128, true, 64>), grid, dim3(256), 0, st, a, c);
        else hipLaunchKernelGGL((attn_bf16_kernel<64, true, 64>), grid, dim3(256), 0, st, a, c);
    } else {
        if (dh == 128) hipLaunchKernelGGL((attn_bf16_kernel<128, false, ATP_ATTN_KT>), grid, dim3(256), 0, st, a, c);
        else hipLaunchKernelGGL((attn_bf16_kernel<64, false, ATP_ATTN_KT>), grid, dim3(256), 0, st, a, c);
    }
    return hipGetLastError();
}

hipError_t attention_f32(hipStream_t st, const AttnArgs& a) {
    const int dh = a.dq / a.heads;
    if (dh > 256 || a.heads > 65535 || a.batch > 65535) return hipErrorInvalidValue;
    // A wave per query for a few keys (see the kernel), as far as it is ahead of the tiles.  Measured in µs, wave / tiles:
    // width 256, 8192 queries: 1 key 11.6 / 25.8, 16 keys 25.5 / 25.9; 16384: 8 keys 26.6 / 27.3; 131072: 2 keys 112 / 150, 4 keys 182 / 137;
    // width 128, 8192 queries: 8 keys 12.8 / 13.2, 12 keys 16 / 13.4; 16384: 2 keys 12.1 / 14.1, 4 keys 14.0 / 13.8; 131072: 1 key 48 / 53, 2 keys 67 / 54;
    // width 64, 131072 queries: 1 key 34.5 / 25.3; width 30 (rows at no multiple of 16 bytes), 65536: 1 key 16.9 / 19.4, 2 keys 22 / 19.
    const int64_t queries = (int64_t)a.L * a.heads * a.batch;
    const bool few = dh > 128 ? a.nk <= 2 || (a.nk <= 16 && queries <= 16384 && queries * a.nk <= 131072)
                   : dh > 64  ? a.nk == 1 || (a.nk <= 2 && queries <= 16384) || (a.nk <= 8 && queries <= 8192)
                              : a.nk == 1 && dh % 4 != 0;
    if (few) {
        const dim3 grid((a.L + 3) / 4, a.heads, a.batch);
        if (a.linearised) hipLaunchKernelGGL(attn_f32_few_keys_kernel<true>, grid, dim3(256), 0, st, a, dh);
        else hipLaunchKernelGGL(attn_f32_few_keys_kernel<false>, grid, dim3(256), 0, st, a, dh);
        return hipGetLastError();
    }
    // 128 queries per workgroup once that gives every second compute unit one, else 32 with the keys dealt to four waves
    const bool wide = (int64_t)((a.L + 127) / 128) * a.heads * a.batch >= 128 || a.nk <= 32;
    if (dh <= 64) return wide ? launch_attn_f32<64, 1>(st, a, dh) : launch_attn_f32<64, 4>(st, a, dh);
    if (dh <= 128) return wide ? launch_attn_f32<128, 1>(st, a, dh) : launch_attn_f32<128, 4>(st, a, dh);
    return launch_attn_f32<256, 1>(st, a, dh);   // (four shares of 256 features do not fit the LDS)
}

}  // namespace atp
