"""Kernels at the sizes where their tiling can go wrong: edges of tiles, remainders, the ends of a dispatch range.
Compared with the float64 oracle on the rounded inputs.

Tolerances.  fp32: a sum of K products carries at most about sqrt(K)·2^-24 relative error for inputs of random sign
(K = 4096: 4e-6).  bf16: the products are exact and the sums fp32, so the output rounding is what remains; with 8
significant bits half a unit in the last place is at most 2^-8 of an entry (a value just above a power of two)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from util import rel_fro, to_dev, to_host

pytestmark = pytest.mark.gpu

F32_TOL, BF16_TOL = 1e-5, 2.0 ** -8 * 1.05


@pytest.fixture(scope="module")
def atp():
    import paper_2403_02352_amd as m
    return m


def rnd(shape, seed, scale=1.0):
    return np.random.default_rng(seed).standard_normal(shape) * scale


# (batch, m, k, n): single elements, one short of / one past the 32-, 64- and 128-wide tiles and the k-tiles, K odd,
# even (4-byte pieces), a multiple of 4 and of 8, and one shape per tile size of the strided kernel
STRIDED = [(1, 1, 1, 1), (2, 31, 33, 65), (1, 33, 130, 31), (3, 64, 250, 96), (1, 127, 129, 128), (2, 128, 36, 132),
           (1, 300, 127, 260), (1, 1000, 62, 900), (2, 1100, 72, 1990)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("layout", ["kn", "nk"])
@pytest.mark.parametrize("epilogue", ["none", "swiglu"])
@pytest.mark.parametrize("case", STRIDED)
def test_strided_products(atp, dtype, layout, epilogue, case):
    batch, m, k, n = case
    n *= 2 if epilogue == "swiglu" else 1
    B = wl.round_to_dtype(rnd((batch, m, k), 1), dtype)
    W = wl.round_to_dtype(rnd((k, n), 2, 1 / np.sqrt(k)), dtype)
    ref = np.stack([oracle.lowrank_linear(B[b], W, *(["swiglu"] if epilogue == "swiglu" else [])) for b in range(batch)])
    Wd = to_dev(W if layout == "kn" else W.T, dtype)
    out = atp.lowrank_linear(to_dev(B, dtype), Wd, atp.ATP_W_KN if layout == "kn" else atp.ATP_W_NK,
                             atp.ATP_EPI_SWIGLU if epilogue == "swiglu" else atp.ATP_EPI_NONE)
    torch.cuda.synchronize()
    assert rel_fro(to_host(out), ref) <= (F32_TOL if dtype == "f32" else BF16_TOL)


def _fmaf():
    import ctypes
    f = ctypes.CDLL("libm.so.6").fmaf
    f.restype, f.argtypes = ctypes.c_float, [ctypes.c_float] * 3
    return f


# (batch, m, k, n): the three tiles of the strided kernel (the first wherever fewer than 192 tiles of 64×64 exist), k around its k-tiles
# (some tiles whole, rows of a multiple of 16 bytes and not)
CHAINS = [(1, 33, 70, 35), (2, 64, 259, 40), (50, 70, 65, 66), (200, 20, 33, 30), (1, 1800, 36, 1796), (1, 1801, 37, 1795)]


@pytest.mark.parametrize("layout", ["kn", "nk"])
@pytest.mark.parametrize("case", CHAINS)
def test_fp32_products_are_one_chain_over_k(atp, layout, case):
    """Every output of the fp32 path is fmaf over k = 0 .. K-1, bit for bit, whichever tile is taken (60 entries of each case)."""
    batch, m, k, n = case
    A, W = (rnd(shape, s).astype(np.float32) for s, shape in ((1, (batch, m, k)), (2, (batch, k, n))))
    Wd = W if layout == "kn" else np.ascontiguousarray(W.transpose(0, 2, 1))
    out = atp.lowrank_linear(to_dev(A, "f32"), to_dev(Wd, "f32"), atp.ATP_W_KN if layout == "kn" else atp.ATP_W_NK).cpu().numpy()
    fma, rng = _fmaf(), np.random.default_rng(3)
    for b, i, j in zip(rng.integers(batch, size=60), rng.integers(m, size=60), rng.integers(n, size=60)):
        acc = 0.0
        for t in range(k):
            acc = fma(float(A[b, i, t]), float(W[b, t, j]), acc)
        assert np.float32(acc) == out[b, i, j]


# (batch, m, k, n): one shape per tile of the asynchronous kernel (128×64, 128×128, 256×256), one past and one short of the tiles,
# columns a multiple of 8 and not, one k-tile, an odd and an even number of them; the middle tile with W as it lies; contractions split
# along k
ASYNC = [(1, 1, 64, 8), (1, 129, 128, 63), (3, 127, 192, 72), (1, 1100, 256, 1032), (2, 1025, 64, 1031), (1, 4097, 192, 3080),
         (1, 4100, 128, 3101), (2, 1025, 64, 1032), (1, 40, 4160, 136), (2, 130, 6272, 264)]


@pytest.mark.parametrize("layout", ["kn", "nk"])
@pytest.mark.parametrize("epilogue", ["none", "swiglu"])
@pytest.mark.parametrize("case", ASYNC)
def test_async_products(atp, layout, epilogue, case):
    batch, m, k, n = case
    n *= 2 if epilogue == "swiglu" else 1
    B = wl.round_to_dtype(rnd((batch, m, k), 1), "bf16")
    shared = epilogue == "swiglu"   # without the gate every sequence has weights of its own
    W = wl.round_to_dtype(rnd((1 if shared else batch, k, n), 2, 1 / np.sqrt(k)), "bf16")
    ref = np.stack([oracle.lowrank_linear(B[b], W[0 if shared else b], *(["swiglu"] if shared else [])) for b in range(batch)])
    Wd = W if layout == "kn" else W.transpose(0, 2, 1)
    out = atp.lowrank_linear(to_dev(B, "bf16"), to_dev(np.ascontiguousarray(Wd[0] if shared else Wd), "bf16"),
                             atp.ATP_W_KN if layout == "kn" else atp.ATP_W_NK, atp.ATP_EPI_SWIGLU if shared else atp.ATP_EPI_NONE)
    torch.cuda.synchronize()
    assert rel_fro(to_host(out), ref) <= BF16_TOL


# (batch, L, r, dq): both operands stored by columns in the asynchronous kernel (L a multiple of 64; 128×64 tiles three times, 128×128,
# 256×256), in the strided one, and turned first (columns no multiple of 8)
PROJECTED = [(1, 64, 8, 64), (2, 192, 72, 264), (1, 128, 1032, 1096), (1, 64, 1544, 1800), (1, 64, 3080, 4104), (2, 100, 40, 136), (1, 256, 33, 130), (1, 77, 9, 70)]


@pytest.mark.parametrize("case", PROJECTED)
def test_projection_onto_bases(atp, case):
    batch, L, r, dq = case
    U, Y = wl.round_to_dtype(rnd((batch, L, r), 3), "bf16"), wl.round_to_dtype(rnd((batch, L, dq), 4), "bf16")
    out = atp.project_onto_bases(to_dev(U, "bf16"), to_dev(Y, "bf16"))
    torch.cuda.synchronize()
    assert rel_fro(to_host(out), np.stack([oracle.project_onto_bases(U[b], Y[b]) for b in range(batch)])) <= BF16_TOL


# keys around the 64-key tile, both head widths, the last tile in either stage.  bf16 probabilities and outputs: two roundings of 2^-9
# relative, so 2^-8.  An infinite value makes its own feature infinite and no other.
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("r", [1, 15, 63, 64, 65, 127, 128, 129, 200])
def test_bf16_attention_key_tiles(atp, dh, r):
    Q, K, V = (wl.round_to_dtype(rnd((2, n, 2 * dh), 10 + i), "bf16") for i, n in enumerate((130, r, r)))
    dev = [to_dev(x, "bf16") for x in (Q, K, V)]
    out = to_host(atp.attention(*dev, 2))
    ref = np.stack([oracle.attention(Q[b], K[b], V[b], 2) for b in range(2)])
    assert rel_fro(out, ref) <= BF16_TOL
    dev[2][0, r - 1, 5] = float("inf")
    out2 = to_host(atp.attention(*dev, 2))
    assert np.isposinf(out2[0, :, 5]).all()
    out2[0, :, 5] = out[0, :, 5]
    assert np.array_equal(out, out2)


# (batch, L, d, r1, r2): rows of aligned 16-byte pieces and of single elements, pieces shared between few and many rows; copies are exact
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(1, 1, 8, 8, 8), (2, 65, 72, 16, 24), (2, 130, 2056, 40, 8), (1, 33, 70, 8, 12), (2, 40, 71, 5, 3), (1, 600, 64, 304, 280)])
def test_concatenated_blocks_and_norm(atp, dtype, case):
    batch, L, d, r1, r2 = case
    U1, C1, U2, C2 = (to_dev(rnd((batch, *shape), 20 + i), dtype) for i, shape in enumerate(((L, r1), (r1, d), (L, r2), (r2, d))))
    P, C = atp.concat_factors(U1, C1, U2, C2)
    assert torch.equal(P, torch.cat([U1, U2], 2)) and torch.equal(C, torch.cat([C1, C2], 1))
    gain = 1 + 0.1 * torch.randn(d, generator=torch.Generator().manual_seed(5))
    for center in (False, True):
        Pn, Cn = atp.norm_factored(P, C, gain.cuda(), 1e-6, center)
        for b in range(batch):
            Pr, Cr = oracle.norm_factored(to_host(P[b]), to_host(C[b]), gain.double().numpy(), 1e-6, center)
            # bf16: M and each factor rounded once
            assert rel_fro(to_host(Pn[b]), Pr) <= (1e-5 if dtype == "f32" else 2 * BF16_TOL)
            assert rel_fro(to_host(Cn[b]), Cr) <= (1e-5 if dtype == "f32" else 2 * BF16_TOL)


# (batch, L, heads, dh): several rows to a workgroup and one, a last workgroup with fewer, heads in one group, in groups of one and in uneven
# groups, head halves of 1, 3, 8, 32, 256 and more than the 256 of a workgroup.  fp32: angles up to 4096 rad carry 2^-24 of themselves, 2.5e-4 at most
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(1, 1, 1, 2), (2, 5, 3, 6), (1, 4093, 2, 16), (3, 700, 3, 64), (1, 2050, 1, 512), (2, 9, 1, 1040),
                                  (1, 1, 700, 8), (1, 60, 13, 128), (2, 130, 7, 6), (1, 1025, 5, 4)])
def test_rope_rows(atp, dtype, case):
    batch, L, heads, dh = case
    Y = wl.round_to_dtype(rnd((batch, L, heads * dh), 30), dtype)
    out = to_host(atp.rope(to_dev(Y, dtype), heads))
    ref = np.stack([oracle.rope(Y[b], heads) for b in range(batch)])
    assert np.abs(out - ref).max() <= (3e-4 if dtype == "f32" else 3e-4 + 2.0 ** -8) * np.abs(ref).max()


# (batch, L, r, dq, heads): fp32 attention with 128 queries per workgroup and with the keys dealt to four waves; heads of every
# padded width (64, 128, 256), widths that are no multiple of 4 (scalar loads); one short of / past the 32-key tile and the
# 128-key stage; a single key and a single query
F32_ATTENTION = [(1, 1, 1, 5, 1), (1, 33, 31, 64, 1), (2, 129, 33, 130, 2), (1, 127, 127, 128, 1), (1, 65, 129, 256, 2),
                 (1, 40, 300, 96, 1), (1, 130, 65, 200, 1), (1, 100, 257, 512, 2), (4, 500, 97, 640, 10), (3, 260, 129, 1408, 22),
                 (2, 512, 96, 8192, 64),
                 # few keys, a wave per query: one and the most it takes, one more, one query too many, ragged widths
                 (1, 1, 1, 128, 1), (2, 33, 8, 256, 2), (1, 33, 9, 130, 1), (1, 50, 16, 410, 2), (1, 50, 17, 410, 2), (2, 65, 2, 768, 3), (1, 16384, 3, 200, 1),
                 (1, 16385, 3, 200, 1), (1, 70, 1, 66, 2), (1, 70, 2, 66, 2)]


@pytest.mark.parametrize("variant", ["softmax", "taylor", "rowsum"])
@pytest.mark.parametrize("case", F32_ATTENTION)
def test_attention_f32(atp, case, variant):
    """The score sums carry sqrt(d_h)·2^-24 of their terms' size, which the exponential passes on: below 1e-5."""
    batch, L, r, dq, heads = case
    Q, K, V = (rnd((batch, n, dq), s).astype(np.float32) for s, n in ((3, L), (4, r), (5, r)))
    if variant == "softmax":
        ref = np.stack([oracle.attention(Q[b], K[b], V[b], heads) for b in range(batch)])
        out = atp.attention(to_dev(Q, "f32"), to_dev(K, "f32"), to_dev(V, "f32"), heads)
    else:
        # column sums c_j of about 0.8·sqrt(L) and scores s_j of about 0.1: Σ s_j·c_j is 0.08·sqrt(L·r) or less, a fraction of L, so
        # neither denominator (L + Σ s_j·c_j, Σ c_j + s_j) cancels and its relative error stays that of the sums
        U = (np.abs(rnd((batch, L, r), 6)) / np.sqrt(L)).astype(np.float32)
        Q *= np.float32(0.1)
        ref = np.stack([oracle.linearised_attention(Q[b], K[b], V[b], U[b], heads, norm=variant) for b in range(batch)])
        norm = atp.ATP_NORM_TAYLOR if variant == "taylor" else atp.ATP_NORM_ROWSUM
        out = atp.attention_linearised(to_dev(Q, "f32"), to_dev(K, "f32"), to_dev(V, "f32"), to_dev(U, "f32"), heads, norm=norm)
    torch.cuda.synchronize()
    err = rel_fro(to_host(out), ref)
    print(case, variant, err, flush=True)
    assert err <= F32_TOL


# (L, r, dh, standard deviation of the scores, bound in units of 2^-24)
@pytest.mark.parametrize("case", [(400, 33, 256, 1, 4.5), (200, 300, 256, 1, 8), (500, 500, 128, 3, 9.5), (300, 200, 64, 1, 5)])
def test_attention_f32_scores_are_short_sums(atp, case):
    """A sum of n terms of variance v in one chain carries 2^-24/sqrt(3)·sqrt(v·n^2/2), over 256 features 6.5 units at a standard deviation of
    1; sums of 8 or 16 features, added up, carry 2 of them (4.6 and 2 at 128 features, times 3 here).  The exponential hands that on to the
    weights, the sums over the keys add to it."""
    L, r, dh, sd, units = case
    Q, K, V = (rnd((1, n, 2 * dh), 70 + i).astype(np.float32) for i, n in enumerate((L, r, r)))
    Q *= np.float32(sd)
    err = rel_fro(to_host(atp.attention(*(to_dev(x, "f32") for x in (Q, K, V)), 2))[0], oracle.attention(Q[0], K[0], V[0], 2))
    print(case, err * 2 ** 24, flush=True)
    assert err <= units * 2.0 ** -24


# (batch, L, heads): keys dealt to four waves; 128 queries per workgroup
@pytest.mark.parametrize("case", [(1, 40, 1), (4, 1000, 4)])
@pytest.mark.parametrize("dead", [(32, 64), (0, 32), (0, 128), (96, 300)])
def test_attention_f32_keys_at_minus_infinity(atp, case, dead):
    """Keys whose score is -inf weigh nothing, whichever wave or tile they fill."""
    batch, L, heads = case
    Q, K, V = (rnd((batch, n, 64 * heads), 50 + i).astype(np.float32) for i, n in enumerate((L, 300, 300)))
    Q = np.abs(Q) + np.float32(0.1)
    K[:, dead[0]:dead[1]] = -np.inf
    out = to_host(atp.attention(*(to_dev(x, "f32") for x in (Q, K, V)), heads))
    live = np.r_[0:dead[0], dead[1]:300]
    ref = np.stack([oracle.attention(Q[b], K[b][live], V[b][live], heads) for b in range(batch)])
    assert rel_fro(out, ref) <= F32_TOL


@pytest.mark.parametrize("dead", [0, 2, 4])
def test_attention_f32_few_keys_at_minus_infinity(atp, dead):
    Q, K, V = (rnd((1, n, 200), 60 + i).astype(np.float32) for i, n in enumerate((30, 5, 5)))
    Q = np.abs(Q) + np.float32(0.1)
    K[:, dead] = -np.inf
    live = [j for j in range(5) if j != dead]
    out = to_host(atp.attention(*(to_dev(x, "f32") for x in (Q, K, V)), 1))
    assert rel_fro(out[0], oracle.attention(Q[0], K[0][live], V[0][live], 1)) <= F32_TOL


# r: one index, an odd one, one short of / at / past one block pair (64), block counts with padding blocks, several pairs
@pytest.mark.parametrize("r", [1, 2, 33, 63, 64, 65, 96, 97, 128, 129, 200])
def test_rayleigh_ritz_block_edges(atp, r):
    """sigma from 1 to 1/2: eigenvalues of T lie 0.5/r apart or more, so the fp32 rounding of T (a few 2^-24) turns its
    eigenvectors by a few 2^-24·2r."""
    batch, L, d = 2, 210, 230
    rng = np.random.default_rng(77 + r)
    U, B = np.empty((batch, L, r), np.float32), np.empty((batch, r, d), np.float32)
    for b in range(batch):
        M = np.linalg.qr(rng.standard_normal((r, r)))[0]
        U[b] = np.linalg.qr(rng.standard_normal((L, r)) + 0.2)[0] @ M
        B[b] = M.T @ (np.linspace(1.0, 0.5, r)[:, None] * np.linalg.qr(rng.standard_normal((d, r)))[0].T)
    Uo, Bo, sig, diag = atp.rayleigh_ritz(to_dev(U, "f32"), to_dev(B, "f32"), 10)
    torch.cuda.synchronize()
    tol = 20 * 2.0 ** -24 * 2 * r + 2e-6
    for b in range(batch):
        Ur, Br, sr = oracle.rayleigh_ritz(U[b].astype(np.float64), B[b].astype(np.float64))
        assert np.abs(sig[b].cpu().numpy() - sr).max() <= 5e-6
        # a column sum near zero leaves its sign to rounding
        clear = np.abs(Ur.sum(0)) > 1e-3
        eu, eb = rel_fro(to_host(Uo[b])[:, clear], Ur[:, clear]), rel_fro(to_host(Bo[b])[clear], Br[clear])
        orth = np.abs(to_host(Uo[b]).T @ to_host(Uo[b]) - np.eye(r)).max()
        print(r, b, eu, eb, orth, float(diag[b, 1]), flush=True)
        assert eu <= tol and eb <= tol and orth <= 2e-5
        assert float(diag[b, 1]) <= 1e-5
        assert abs(float(diag[b, 0]) - (sr ** 2).sum()) <= 1e-5 * (sr ** 2).sum()


# (batch, L, d, r, iters): each extent one short of, at and past the multiples that the extraction pads its rows to (64, 32 for r, 4 on
# the fp32 path), all of them odd, r = 1, and several 64-wide block columns with a padded last one
PADDED_BASES = [(1, 65, 63, 1, 1), (2, 127, 128, 31, 1), (1, 129, 100, 33, 0), (2, 191, 77, 66, 2), (1, 256, 192, 95, 2),
                (2, 301, 250, 97, 1), (1, 515, 384, 250, 2), (3, 128, 130, 64, 1)]


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", PADDED_BASES)
def test_principal_bases_padded_extents(atp, case, dtype, mode):
    """Spectrum without small values (1 to 1/2 over min(L, d)), so the basis is determined to rounding.  fp32: U itself against the
    oracle, 1e-4.  bf16: X·Omega and the iterates are products of bf16 operands, 2^-9 each, and a basis that they perturb still
    captures X to second order: the residual agrees to 1e-2 of the norm, U'U and B = U'X to the rounding of U (2^-9 per entry)."""
    batch, L, d, r, iters = case
    n = min(L, d)
    X = np.stack([wl.make_X(L, d, np.sqrt(L * d / n) * np.linspace(1.0, 0.5, n), 0.0, 40 + b) for b in range(batch)])
    X = wl.round_to_dtype(X, dtype)
    Om = wl.make_omega(d, r, 3)
    atp.set_factor_mode(mode)
    try:
        U, B, info, Um = atp.principal_bases(to_dev(X, dtype), r, iters, to_dev(Om, "f32"), want_master=True)
        torch.cuda.synchronize()
    finally:
        atp.set_factor_mode(True)
    assert (info == 0).all()
    for b in range(batch):
        Xb, Ub, Bb = X[b].astype(np.float64), to_host(U[b]), to_host(B[b])
        Uo, Bo = oracle.principal_bases(Xb, Om.astype(np.float64), iters)
        orth, coef = np.abs(to_host(Um[b]).T @ to_host(Um[b]) - np.eye(r)).max(), rel_fro(Bb, Ub.T @ Xb)
        recon = abs(np.linalg.norm(Xb - Ub @ Bb) - np.linalg.norm(Xb - Uo @ Bo)) / np.linalg.norm(Xb)
        print(case, dtype, mode, orth, coef, recon, rel_fro(to_host(Um[b]), Uo), flush=True)
        assert orth <= (1e-5 if dtype == "f32" else 1e-4) and coef <= (1e-5 if dtype == "f32" else 2.0 ** -8) and recon <= 1e-2
        if dtype == "f32":
            assert rel_fro(to_host(Um[b]), Uo) <= 1e-4


def _whole_numbers(n, seed):
    h = (np.arange(1, n + 1, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15) + np.uint64(seed << 60)) >> np.uint64(40)
    h = (h ^ (h >> np.uint64(11))) * np.uint64(2654435761) & np.uint64(0xFFFFFFFF)
    return ((h >> np.uint64(23)).astype(np.int64) - 256) / 256.0


# (dtype, batch, L, d, r, iters): digests of U, its fp32 master and B in the two factorisation modes, at extents that need no padding.
# Whole numbers below 2^8 over 2^8 as input, so nothing depends on a generator or a library.
DIGESTS = {("f32", 1, 128, 64, 32, 4): ("1229367ac83f665d", "1229367ac83f665d"),
           ("f32", 2, 192, 320, 96, 1): ("a65e093e6fabd748", "2b6774bf9d5dd660"),
           ("bf16", 2, 128, 256, 64, 2): ("458e5216b2709520", "458e5216b2709520"),
           ("bf16", 1, 512, 384, 128, 1): ("e4c095fd896ba470", "cd44cdbed4b3206e"),
           # three, four and five block rows: the tile before the last of the inverse is formed by another instruction than the others
           ("f32", 2, 320, 256, 160, 1): ("29fe5a667e119116", "cfc03f9069fb3883"),
           ("bf16", 2, 512, 384, 256, 1): ("1b59f43d5971c0cc", "d0d7b1716439c964"),
           ("bf16", 29, 640, 512, 320, 1): ("9efa08b04ccb3f6b", "1700362255381e74"),
           # six tiles per bulk workgroup, as many as the registers hold
           ("f32", 19, 768, 640, 448, 1): ("43f5221234f19134", "37294b199648131a")}


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("case", DIGESTS)
def test_extraction_keeps_its_bits(atp, case, mode):
    """A rounding that moves anywhere in the extraction (the order of a sum, a product and a sum that round once or twice) shows here.
    The trailing columns and everything behind them (softmax, a second extraction) magnify it, so it is to be meant when it happens:
    a new digest goes with a measured error against float64 that is no larger."""
    import hashlib
    dtype, batch, L, d, r, iters = case
    X = _whole_numbers(batch * L * d, 1).reshape(batch, L, d)
    atp.set_factor_mode(mode)
    try:
        U, B, info, Um = atp.principal_bases(to_dev(X, dtype), r, iters, to_dev(_whole_numbers(d * r, 2).reshape(d, r), "f32"), want_master=True)
        torch.cuda.synchronize()
    finally:
        atp.set_factor_mode(True)
    assert (info == 0).all()
    h = hashlib.sha256()
    for t in (U, Um, B):
        h.update(t.cpu().view(torch.uint8).numpy().tobytes())
    print(case, mode, h.hexdigest()[:16], flush=True)
    assert h.hexdigest()[:16] == DIGESTS[case][mode]


# ranks on both sides of the 16-column stages of a diagonal tile, of the 64-wide blocks, and one to eight block rows (the roles of the spine
# workgroups change up to the fourth)
@pytest.mark.parametrize("r", [1, 4, 15, 16, 17, 33, 48, 49, 64, 65, 81, 128, 129, 177, 193, 256, 257, 321, 449])
def test_factorisation_at_every_edge(atp, r):
    """One orthonormalisation against the oracle (fp32, conditioned like X·Omega of a flat spectrum: 1e-4), and the two forms of the factorisation
    against each other: a single block is the same chain of multiply-adds in both, so the same bits; more differ by rounding, 2^-24 per
    term of sums of up to r and the condition number of X·Omega that R^-1 magnifies it by (7 at r = 257, 82 at 449)."""
    batch, L, d = 3, 560, 470
    X = np.stack([wl.make_X(L, d, np.sqrt(L) * np.linspace(1.0, 0.5, d), 0.0, 60 + b) for b in range(batch)]).astype(np.float32)
    Om = wl.make_omega(d, r, 3)
    U = []
    for mode in (0, 1):
        atp.set_factor_mode(mode)
        try:
            u, _, info, _ = atp.principal_bases(to_dev(X, "f32"), r, 0, to_dev(Om, "f32"))
            torch.cuda.synchronize()
        finally:
            atp.set_factor_mode(True)
        assert (info == 0).all()
        U.append(to_host(u))
    for b in range(batch):
        Uo, _ = oracle.principal_bases(X[b].astype(np.float64), Om.astype(np.float64), 0)
        print(r, b, rel_fro(U[1][b], Uo), rel_fro(U[1][b], U[0][b]), flush=True)
        assert rel_fro(U[1][b], Uo) <= 1e-4
        cond = np.linalg.cond(X[b].astype(np.float64) @ Om)
        assert (U[0][b] == U[1][b]).all() if r <= 64 else rel_fro(U[1][b], U[0][b]) <= cond * np.sqrt(r) * 2.0 ** -24


# the largest batches that one launch takes: six tiles per bulk workgroup, 250, 256 (every compute unit) and 253 workgroups; one sequence more
# takes the other form
@pytest.mark.parametrize("batch,r,one_launch", [(25, 384, True), (16, 512, True), (11, 640, True), (17, 512, False)])
def test_factorisation_of_the_largest_batches(atp, batch, r, one_launch):
    """Modes 0 and 1 give the same bits exactly where mode 1 takes the launch per block column.  Otherwise U differs by rounding, 2^-24 per term of
    sums of up to r and the condition number that R^-1 magnifies it by.  |U'U - I| is 7.5 to 9.5 * 2^-24 per column in both forms
    (against float64); 15 is allowed."""
    L, d = 2 * r + 64, 2 * r
    X, Om = rnd((batch, L, d), 21).astype(np.float32), wl.make_omega(d, r, 3)
    cond = max(np.linalg.cond(X[b].astype(np.float64) @ Om) for b in range(batch))
    U = []
    for mode in (0, 1, 1):
        atp.set_factor_mode(mode)
        try:
            u, _, info, _ = atp.principal_bases(to_dev(X, "f32"), r, 0, to_dev(Om, "f32"))
            torch.cuda.synchronize()
        finally:
            atp.set_factor_mode(True)
        assert (info == 0).all()
        U.append(u)
    assert torch.equal(U[1], U[2]) and torch.equal(U[0], U[1]) != one_launch
    eye, worst = torch.eye(r, dtype=torch.float64, device="cuda"), 0.0
    for u in U[:2]:
        orth = max(torch.linalg.norm(u[b].double().T @ u[b].double() - eye).item() for b in range(batch))
        print(batch, r, cond, orth / np.sqrt(r) * 2 ** 24, flush=True)
        assert orth <= 15 * np.sqrt(r) * 2.0 ** -24
    for b in range(batch):
        worst = max(worst, rel_fro(to_host(U[1][b]), to_host(U[0][b])))
    print(worst, cond * np.sqrt(r) * 2.0 ** -24, flush=True)
    assert worst <= cond * np.sqrt(r) * 2.0 ** -24


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("r", [130, 200, 256, 330])
def test_factorisation_stays_within_the_workspace(atp, dtype, r):
    """The exchange slots are the last thing in the workspace: nothing behind it is written (three to six block rows, a megabyte looked at)."""
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    X, Om = to_dev(rnd((3, 400, 352), 8), dtype), to_dev(wl.make_omega(352, r, 3), "f32")
    need = atp.binding.principal_bases_workspace(3, 400, 352, r, 1, t)
    buf = torch.full((need + (1 << 20),), 0xA5, dtype=torch.uint8, device="cuda")
    out = atp.principal_bases(X, r, 1, Om, workspace=buf[:need])
    torch.cuda.synchronize()
    assert (buf[need:] == 0xA5).all() and (out[2] == 0).all()


@pytest.mark.parametrize("batch,r", [(5, 64), (44, 256), (33, 330)])
def test_factorisation_in_groups_stays_within_the_workspace(atp, batch, r):
    """Mode 2 with batches beyond one launch (42 and 32 sequences fit), and a single block column: flags and slots are those of one launch, taken
    over by the next, with nothing written behind them and the bits of the same sequences in one launch."""
    X, Om = to_dev(rnd((batch, 400, 352), 8), "f32"), to_dev(wl.make_omega(352, r, 3), "f32")
    need = atp.binding.principal_bases_workspace(batch, 400, 352, r, 1, torch.float32)
    buf = torch.full((need + (1 << 20),), 0xA5, dtype=torch.uint8, device="cuda")
    atp.set_factor_mode(2)
    try:
        U, B, info, _ = atp.principal_bases(X, r, 1, Om, workspace=buf[:need])
        one = atp.principal_bases(X[batch - 3:].contiguous(), r, 1, Om)
        torch.cuda.synchronize()
    finally:
        atp.set_factor_mode(True)
    assert (buf[need:] == 0xA5).all() and (info == 0).all()
    assert torch.equal(U[batch - 3:], one[0]) and torch.equal(B[batch - 3:], one[1])


@pytest.mark.parametrize("bits", [0xFFFFFFFF, 0x7FFFFFFF, 0x7FC00000, 0xFFC00000])
def test_every_nan_is_flagged(atp, bits):
    """The factorisation marks what has not been handed over yet with the NaN of all ones, so no other entry may look like it.  The fp32 products
    carry the bits of a NaN along: the workspace of one round shows that those of the input are the ones in the Gram matrix, and that set-up
    leaves the one NaN 0x7fc00000 in S' whatever came in.  The call flags the sequence, with and without iterations, and no other."""
    batch, L, d, r = 3, 300, 280, 260                     # (multiples of 4: the fp32 path pads nothing)
    X = rnd((batch, L, d), 5).astype(np.float32)
    X[0, 17, 33] = np.uint32(bits).view(np.float32)
    Xd, Om = to_dev(X, "f32"), to_dev(wl.make_omega(d, r, 3), "f32")
    assert Xd.view(torch.int32)[0, 17, 33].item() & 0xFFFFFFFF == bits
    ws = torch.zeros(atp.binding.principal_bases_workspace(batch, L, d, r, 0, torch.float32), dtype=torch.uint8, device="cuda")
    try:
        atp.set_qr_passes(2, 1, 1)
        _, _, info, _ = atp.principal_bases(Xd, r, 0, Om, workspace=ws)
        torch.cuda.synchronize()
    finally:
        atp.set_qr_passes(2, 1, 2)
    words = [batch * d * L, d * r, d * r] + 4 * [batch * L * r] + 4 * [batch * d * r] + [batch * r * L, batch * r * d]
    at = sum((4 * n + 255) // 256 * 256 for n in words)
    nans = []
    for n in (batch * r * r, batch * r * r):              # the Gram matrix (of eight places for parts, fp32 takes one) and S'
        v = ws[at:at + 4 * n].view(torch.int32).cpu().numpy().view(np.uint32)
        nans.append(set(v[np.isnan(v.view(np.float32))].tolist()))
        at += (8 * 4 * n + 255) // 256 * 256
    print(hex(bits), info.tolist(), [[hex(x) for x in n] for n in nans], flush=True)
    assert nans == [{bits}, {0x7FC00000}]
    assert info[0] > 0 and (info[1:] == 0).all()
    _, _, info, _ = atp.principal_bases(Xd, r, 1, Om)
    torch.cuda.synchronize()
    assert info[0] > 0 and (info[1:] == 0).all()


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("r", [1, 5, 64, 65, 193, 260])
def test_input_that_is_not_finite_gives_a_positive_info(atp, r, dtype, mode):
    """info = -1 is kept for a wait that gave up: an infinity or a NaN gives a positive number, in every form of the factorisation
    (the padding of the rank counts as columns here: infinity times its zeros is a NaN)."""
    X = rnd((3, 300, 280), 5)
    X[0, 17, 33], X[2, 299, 0] = np.inf, np.nan
    atp.set_factor_mode(mode)
    try:
        _, _, info, _ = atp.principal_bases(to_dev(X, dtype), r, 1, to_dev(wl.make_omega(280, r, 3), "f32"))
        torch.cuda.synchronize()
    finally:
        atp.set_factor_mode(True)
    print(r, dtype, mode, info.tolist(), flush=True)
    assert info[0] > 0 and info[1] == 0 and info[2] > 0


# (L, d, r, iters): extents that are no multiple of 32, alone and together
RAGGED_ORTH = [(300, 200, 64, 1), (161, 528, 20, 1), (515, 384, 250, 2), (1003, 440, 118, 1)]


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("case", RAGGED_ORTH)
def test_ragged_bases_are_orthonormal_to_fp32(atp, case, mode):
    """bf16 hi+lo planes hold about 17 bits.  A Gram matrix without the product of the lo planes misses sum(lo^2) of sum(x^2): lo is uniform
    within 2^-8 of the leading bit, 2.4e-6 to 3.5e-6 on average over a mantissa, and U comes out that much too long in every column.
    With it the mean of the diagonal of U'U - 1 has random errors only: 2^-17 per entry over L·r of them, far below 5e-7."""
    L, d, r, iters = case
    X = wl.make_X(L, d, np.sqrt(L * d / min(L, d)) * np.linspace(1.0, 0.5, min(L, d)), 0.0, 7)
    atp.set_factor_mode(mode)
    try:
        _, _, info, Um = atp.principal_bases(to_dev(X[None], "bf16"), r, iters, to_dev(wl.make_omega(d, r, 3), "f32"), want_master=True)
        torch.cuda.synchronize()
    finally:
        atp.set_factor_mode(True)
    assert (info == 0).all()
    U = to_host(Um[0])
    dev = U.T @ U - np.eye(r)
    print(case, mode, abs(np.diag(dev).mean()), np.abs(dev).max(), flush=True)
    assert abs(np.diag(dev).mean()) <= 5e-7


# eigenvalues of T at both ends of the fp32 range: 5e-35 (the entries that are still to be annihilated reach down to the smallest numbers
# that fp32 holds) and 2e37
@pytest.mark.parametrize("exponent", [-57, 62])
@pytest.mark.parametrize("r", [40, 130])
def test_rayleigh_ritz_at_the_ends_of_the_range(atp, r, exponent):
    """B scaled by a power of two: the same singular values and vectors, to the tolerance of the unscaled ones."""
    L, d = 210, 230
    rng = np.random.default_rng(177 + r)
    M = np.linalg.qr(rng.standard_normal((r, r)))[0]
    U = (np.linalg.qr(rng.standard_normal((L, r)) + 0.2)[0] @ M).astype(np.float32)
    B = (M.T @ (np.linspace(1.0, 0.5, r)[:, None] * np.linalg.qr(rng.standard_normal((d, r)))[0].T)).astype(np.float32)
    scale = 2.0 ** exponent
    Uo, Bo, sig, diag = atp.rayleigh_ritz(to_dev(U[None], "f32"), to_dev((B * scale)[None], "f32"), 10)
    sr = np.linalg.svd(B.astype(np.float64))[1]
    print(r, exponent, np.abs(sig[0].cpu().numpy() / scale - sr).max(), float(diag[0, 1]), flush=True)
    assert np.abs(sig[0].cpu().numpy() / scale - sr).max() <= 5e-6
    assert float(diag[0, 1]) <= 1e-5
    Uo, Bo = to_host(Uo[0]), to_host(Bo[0]) / scale
    assert rel_fro(Uo @ Bo, U.astype(np.float64) @ B) <= 2e-5
    G = Bo @ Bo.T
    assert np.linalg.norm(G - np.diag(np.diag(G))) <= 2e-5 * np.linalg.norm(G)


def _row_cyclic_off_diagonal(T, sweeps):
    """max |T_ij| / max T_ii after `sweeps` sweeps of Jacobi rotations, a round-robin over the indices (float64)."""
    r = len(T)
    n = r + r % 2
    A = np.zeros((n, n))
    A[:r, :r] = T
    for k in list(range(n - 1)) * sweeps:
        for x, y in [(n - 1, k)] + [((k + i) % (n - 1), (k - i + n - 1) % (n - 1)) for i in range(1, n // 2)]:
            p, q = min(x, y), max(x, y)
            if A[p, q] == 0.0:
                continue
            tau = (A[q, q] - A[p, p]) / (2 * A[p, q])
            t = (1.0 if tau >= 0 else -1.0) / (abs(tau) + np.hypot(1.0, tau))
            c = 1 / np.hypot(1.0, t)
            J = np.array([[c, -t * c], [t * c, c]])
            A[[p, q]] = J @ A[[p, q]]
            A[:, [p, q]] = A[:, [p, q]] @ J.T
    return np.abs(A - np.diag(np.diag(A))).max() / np.diag(A).max()


@pytest.mark.parametrize("r", [3, 4, 7, 16, 31, 33, 48, 64])
def test_rayleigh_ritz_small_r_sweeps_are_row_cyclic(atp, r):
    """Up to 64 indices a sweep is r-1 steps of a round-robin, whatever r: what it leaves after two is far above rounding and comparable
    to a hundredth (fp32 angles carry 1e-6 of it on, through 2·r rotations of every row)."""
    rng = np.random.default_rng(277 + r)
    M = np.linalg.qr(rng.standard_normal((r, r)))[0]
    U = np.linalg.qr(rng.standard_normal((80, r)) + 0.2)[0].astype(np.float32)
    B = (M.T @ (np.linspace(1.0, 0.5, r)[:, None] * np.linalg.qr(rng.standard_normal((90, r)))[0].T)).astype(np.float32)
    sweeps = 1 if r < 8 else 2
    off = float(atp.rayleigh_ritz(to_dev(U[None], "f32"), to_dev(B[None], "f32"), sweeps)[3][0, 1])
    ref = _row_cyclic_off_diagonal(B.astype(np.float64) @ B.astype(np.float64).T, sweeps)
    print(r, off, ref, flush=True)
    assert abs(off - ref) <= 1e-2 * ref


# three pairs of blocks, five, eight
@pytest.mark.parametrize("spectrum", ["steep", "clustered"])
@pytest.mark.parametrize("r", [130, 300, 500])
def test_rayleigh_ritz_converges_in_ten_sweeps(atp, r, spectrum):
    """Spectra whose eigenvalues of T fall below the rounding of the first (0.9^i) or stand in groups of eight.  What is left off the diagonal
    after ten sweeps is rounding: 64 products of 2^-24 in each pass over a tile, a few passes since the last large rotation."""
    rng = np.random.default_rng(377 + r)
    i = np.arange(r)
    s = 0.9 ** i if spectrum == "steep" else 1.0 - 0.1 * (i // 8) / (r // 8)
    M = np.linalg.qr(rng.standard_normal((r, r)))[0]
    U = (np.linalg.qr(rng.standard_normal((520, r)) + 0.2)[0] @ M).astype(np.float32)
    B = (M.T @ (s[:, None] * np.linalg.qr(rng.standard_normal((530, r)))[0].T)).astype(np.float32)
    Uo, Bo, sig, diag = atp.rayleigh_ritz(to_dev(U[None], "f32"), to_dev(B[None], "f32"), 10)
    print(r, spectrum, float(diag[0, 1]), flush=True)
    assert float(diag[0, 1]) <= 8 * 2.0 ** -24
    G = to_host(Bo[0]) @ to_host(Bo[0]).T
    assert np.linalg.norm(G - np.diag(np.diag(G))) <= 5e-6 * np.linalg.norm(G)


@pytest.mark.parametrize("level", [1, 2])
@pytest.mark.parametrize("case", RAGGED_ORTH)
def test_ragged_bases_with_single_conditioning_products(atp, case, level):
    """The passes before the last from the hi planes alone: the last one still certifies U, and the basis captures X as the oracle's does."""
    L, d, r, iters = case
    X = wl.round_to_dtype(wl.make_X(L, d, np.sqrt(L * d / min(L, d)) * np.linspace(1.0, 0.5, min(L, d)), 0.0, 7), "bf16")
    Om = wl.make_omega(d, r, 3)
    atp.set_conditioning_gram(level)
    try:
        U, B, info, Um = atp.principal_bases(to_dev(X[None], "bf16"), r, iters, to_dev(Om, "f32"), want_master=True)
        torch.cuda.synchronize()
    finally:
        atp.set_conditioning_gram(0)
    assert (info == 0).all()
    Ub, Bb, M = to_host(U[0]), to_host(B[0]), to_host(Um[0])
    Uo, Bo = oracle.principal_bases(X, Om, iters)
    assert abs(np.diag(M.T @ M - np.eye(r)).mean()) <= 5e-7 and np.abs(M.T @ M - np.eye(r)).max() <= 1e-4
    assert rel_fro(Bb, Ub.T @ X) <= 2.0 ** -8
    assert abs(np.linalg.norm(X - Ub @ Bb) - np.linalg.norm(X - Uo @ Bo)) / np.linalg.norm(X) <= 1e-2


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("call", ["bases", "norm", "linear", "ritz"])
def test_calls_stay_within_the_queried_workspace(atp, dtype, call):
    """Ragged extents, a workspace of exactly the queried size, and what lies behind it."""
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    code = atp.binding._dt(torch.empty(0, dtype=t))
    X, P = to_dev(rnd((2, 131, 70), 1), dtype), to_dev(rnd((2, 131, 33), 2), dtype)
    C = to_dev(rnd((2, 33, 70), 3), dtype)
    W = to_dev(rnd((2, 70, 40), 4), dtype)
    long_B, long_W = to_dev(rnd((1, 40, 4160), 5), dtype), to_dev(rnd((4160, 136), 6, 1 / 64), dtype)
    lib = atp.binding.lib
    runs = {"bases": [(atp.binding.principal_bases_workspace(2, 131, 70, 33, 1, t), lambda ws: atp.principal_bases(X, 33, 1, seed=1, workspace=ws)[:2])],
            "norm": [(lib.atp_norm_factored_workspace(2, 131, 70, 33, code), lambda ws, c=c: atp.norm_factored(P, C, torch.ones(70, device="cuda"), 1e-6, c, workspace=ws))
                     for c in (False, True)],
            "linear": [(atp.lowrank_linear_workspace(2, 131, 70, 40, 2800, atp.ATP_W_KN, t), lambda ws: [atp.lowrank_linear(X, W, atp.ATP_W_KN, workspace=ws)]),
                       (atp.lowrank_linear_workspace(1, 40, 4160, 136, 0, atp.ATP_W_KN, t), lambda ws: [atp.lowrank_linear(long_B, long_W, atp.ATP_W_KN, workspace=ws)])],
            "ritz": [(atp.rayleigh_ritz_workspace(2, 131, 70, 33, t), lambda ws: atp.rayleigh_ritz(P, C, 2, workspace=ws)[:3])]}
    for need, run in runs[call]:
        buf = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        ref = run(None)
        out = run(buf[:need] if need else None)
        torch.cuda.synchronize()
        assert (buf[need:] == 0xA5).all()
        assert all(torch.equal(a, b) for a, b in zip(out, ref))
