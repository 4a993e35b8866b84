// Scores and depth softmax of every read site of a pass for one token, on
// the matrix cores: shared by the all-sites forward and backward.  Internal
// to the library.
#pragma once

#include "route_common.h"

#include <algorithm>

namespace lrar {

constexpr int kAllMaxSources = 64;  // sources S, and sites T
constexpr int kAllMaxRank = 64;

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

constexpr int kAllSlab = 128;                     // columns per wave pass
constexpr int kAlphaRow = kAllMaxSources + 4;     // floats per LDS alpha row
constexpr int kKeyRow = kAllMaxRank + 8;          // bf16 per LDS key row

// 8 fp32 values as hi + lo bf16 (relative 2^-17).
__device__ __forceinline__ void split2(const float (&v)[8], bf16x8_t &hi, bf16x8_t &lo)
{
    u32x4_t h, l;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        h[k] = pack_bf16x2(v[2 * k], v[2 * k + 1]);
        l[k] = pack_bf16x2(v[2 * k] - bf16_lo(h[k]), v[2 * k + 1] - bf16_hi(h[k]));
    }
    hi = __builtin_bit_cast(bf16x8_t, h);
    lo = __builtin_bit_cast(bf16x8_t, l);
}

struct AllArgs {
    const void *V;       // [S][N][d]
    const void *keys;    // projected: K [S][N][r]; sliced: V
    const float *Q;      // [T][r]
    void *H;             // [T][N][d]
    float *neff;         // [T][N] or NULL
    int S, d, r, krow, koff, first, T;
    int64_t N;
    float eps;
    bool kvec;           // bf16 keys readable as 16-byte vectors
};

// Scores, softmax and N_eff of one token.  Wave w owns the sites of tile w
// (16 w .. 16 w + 15) and computes their scores against all sources on the
// matrix cores: s_{j,i} rho_i = Q_j . k_i is a [16 x r] x [r x S] product per
// tile.  The MFMA's B operand is the keys as stored (lane l: source
// 16 nt + (l mod 16), key elements kb .. kb + 7 of its k-slice), so rho_i
// comes from the same loads: each lane squares its elements and the four
// k-slices of a source are summed with two exchanges.  The result tile has
// sites on rows 4 (l / 16) + e and sources on column l mod 16, so a site's
// softmax is a reduction over the 16 lanes of its row group.
// Writes alpha (fp32 [64][kAlphaRow], zero past each prefix and for absent
// sites) to LDS and N_eff to global; ends with a workgroup barrier (LDS only).
//
// bf16 storage: v_mfma_f32_16x16x32_bf16, 32 key elements per step; the keys
// are exact in bf16 and Q enters as hi + lo bf16 (two MFMAs), so the dot
// product has fp32-level accuracy.  fp32 storage: v_mfma_f32_16x16x4_f32,
// 4 key elements per step, operands as they are.
//
// SAVE (bf16 storage only): wave 0 also leaves every source's key (bf16,
// [64][kKeyRow], zero past r and past S) and rho_i ([64]) in LDS, for the
// backward's key-path terms.
//
// bf16 storage can take the keys already loaded (kpre, from load_site_keys,
// so that they can be issued ahead of other loads) and the queries from LDS
// (qlds, Q [T][r]); by default both are read here from global memory.
// Sum over the 16 lanes of each row of the wave, returned to all 16: four DPP
// moves (group_sum over groups of 16).
__device__ __forceinline__ float row16_sum(float x) { return group_sum(x, 16); }

// Whether site `site` reads source i.
__device__ __forceinline__ bool read_by(const AllArgs &a, int site, int i)
{
    return site < a.T && i < a.first + site;
}

// Softmax over depth of the 16 sites of tile `wave`, from the score products
// D[nt][e] = rho_i Q_j . kbar_i: lane l holds sites j = 16 wave + 4 (l / 16) + e
// against sources i = 16 nt + (l mod 16), irho[nt] = 1 / rho_i.  Leaves the
// scores (-inf past a site's prefix) and the weights (0 there and for absent
// sites), and writes N_eff if asked for.  STRICT: a NaN or infinite score of
// a source that the site reads makes the site's weights NaN, as in the
// single-site kernels; otherwise such a source drops out.  Source tiles from
// NT on hold no source (a compile-time bound that saves their zeros).  GL: the
// lanes that share a token's sources, col the lane's place among them (fewer
// than 16 only with one tile).
template <bool STRICT, int NT = 4, int GL = 16>
__device__ __forceinline__ void site_softmax(const AllArgs &a, int64_t n, int wave, int col,
                                             int ks, const f32x4_t (&D)[4],
                                             const float (&irho)[4], float (&s)[4][4],
                                             float (&al)[4][4])
{
    // No contraction: the same operations, hence the same bits, in every
    // kernel that calls it.
#pragma clang fp contract(off)
    float m[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int i = 16 * nt + col;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int site = 16 * wave + 4 * ks + e;
            // STRICT: irho holds rho itself (one rounding less than with its
            // reciprocal).
            s[nt][e] = !read_by(a, site, i) ? -INFINITY
                       : STRICT             ? D[nt][e] / irho[nt]
                                            : D[nt][e] * irho[nt];
            m[e] = fmaxf(m[e], s[nt][e]);
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        m[e] = group_max(m[e], GL);
    float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool in = STRICT ? read_by(a, 16 * wave + 4 * ks + e, 16 * nt + col)
                                   : s[nt][e] > -INFINITY;
            al[nt][e] = in ? expf(s[nt][e] - m[e]) : 0.0f;
            z[e] += al[nt][e];
        }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        z[e] = group_sum(z[e], GL);
    float sa[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float inv = (STRICT ? z[e] != 0.0f : z[e] > 0.0f) ? 1.0f / z[e] : 0.0f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const bool some = STRICT ? al[nt][e] != 0.0f : al[nt][e] > 0.0f;
            const float ex = al[nt][e];
            al[nt][e] *= inv;
            if (some)
                sa[e] = fmaf(STRICT ? ex : al[nt][e], s[nt][e] - m[e], sa[e]);
        }
    }
    if (a.neff) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            sa[e] = group_sum(sa[e], GL);
            const int site = 16 * wave + 4 * ks + e;
            // STRICT: z exp(-t / z) with the sums of the exponentials, as
            // route_neff forms it (half the error of the other form).
            if (col == 0 && site < a.T)
                a.neff[(size_t)site * a.N + n] =
                    STRICT ? z[e] * expf(-sa[e] / z[e]) : expf(logf(z[e]) - sa[e]);
        }
    }
}

template <int RP>
__device__ __forceinline__ void load_site_keys(const AllArgs &a, int64_t n, u32x4_t *kraw)
{
    constexpr int KK = RP / 32;
    const int lane = threadIdx.x % kWaveSize;
    const int col = lane & 15, ks = lane >> 4;
    const uint16_t *keys = static_cast<const uint16_t *>(a.keys) + n * a.krow + a.koff;
    const size_t kplane = (size_t)a.N * a.krow;
    if (a.kvec) {
        // Sources past S and elements past r load a valid address; they are
        // zeroed where the keys are used.
        // One 64-bit row address per lane; the other rows are 16 planes on.
        const uint16_t *k0 = keys + (size_t)(unsigned)col * kplane + 8 * ks;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                const int i = 16 * nt + col, c = 32 * kk + 8 * ks;
                const bool ok = i < a.S && c < a.r;
                kraw[nt * KK + kk] = load_raw<uint16_t, 8>(ok ? k0 + 16 * nt * kplane + 32 * kk : keys);
            }
    } else {
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                const int i = 16 * nt + col, c = 32 * kk + 8 * ks;
                u32x4_t kr = {0u, 0u, 0u, 0u};
                if (i < a.S && c < a.r) {
                    const uint16_t *kp = keys + i * kplane + c;
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        const unsigned x0 = c + 2 * h < a.r ? kp[2 * h] : 0u;
                        const unsigned x1 = c + 2 * h + 1 < a.r ? kp[2 * h + 1] : 0u;
                        kr[h] = x0 | (x1 << 16);
                    }
                }
                kraw[nt * KK + kk] = kr;
            }
    }
}

template <typename T, int RP, bool SAVE = false>
__device__ __forceinline__ void all_site_weights(const AllArgs &a, int64_t n, float *alpha,
                                                 float *rho_out = nullptr,
                                                 uint16_t *key_out = nullptr,
                                                 const u32x4_t *kpre = nullptr,
                                                 const float *qlds = nullptr)
{
    // The lane's indices are formed here, each call, instead of being held
    // across a persistent caller's token loop (where they would take
    // registers for the kernel's lifetime).
    unsigned tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid % kWaveSize, wave = tid / kWaveSize;
    const int col = lane & 15, ks = lane >> 4;
    const int qsite = 16 * wave + col;  // site of this lane's A-operand row
    const T *keys = static_cast<const T *>(a.keys) + n * a.krow + a.koff;
    const size_t kplane = (size_t)a.N * a.krow;

    f32x4_t D[4];
    float ss[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        D[nt] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        ss[nt] = 0.0f;
    }
    if constexpr (std::is_same<T, uint16_t>::value) {
        constexpr int KK = RP / 32;
        bf16x8_t Ahi[KK], Alo[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            float qv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int c = 32 * kk + 8 * ks + e;
                qv[e] = (qsite < a.T && c < a.r)
                            ? (qlds ? qlds[qsite * a.r + c] : a.Q[(size_t)qsite * a.r + c])
                            : 0.0f;
            }
            u32x4_t hi, lo;
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const unsigned hw = pack_bf16x2(qv[2 * h], qv[2 * h + 1]);
                hi[h] = hw;
                lo[h] = pack_bf16x2(qv[2 * h] - bf16_lo(hw), qv[2 * h + 1] - bf16_hi(hw));
            }
            Ahi[kk] = __builtin_bit_cast(bf16x8_t, hi);
            Alo[kk] = __builtin_bit_cast(bf16x8_t, lo);
        }
        u32x4_t kown[4 * KK];
        if (!kpre)
            load_site_keys<RP>(a, n, kown);
        const u32x4_t *kraw = kpre ? kpre : kown;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const int i = 16 * nt + col;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                const int c = 32 * kk + 8 * ks;
                const u32x4_t kr = (i < a.S && c < a.r) ? kraw[nt * KK + kk]
                                                        : u32x4_t{0u, 0u, 0u, 0u};
                if (SAVE && wave == 0)
                    *reinterpret_cast<u32x4_t *>(key_out + i * kKeyRow + c) = kr;
                float x[8];
                widen(kr, x);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    ss[nt] = fmaf(x[e], x[e], ss[nt]);
                const bf16x8_t B = __builtin_bit_cast(bf16x8_t, kr);
                D[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ahi[kk], B, D[nt], 0, 0, 0);
                D[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Alo[kk], B, D[nt], 0, 0, 0);
            }
        }
    } else {
        constexpr int KK = RP / 4;
        float A[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const int c = 4 * kk + ks;
            A[kk] = (qsite < a.T && c < a.r) ? a.Q[(size_t)qsite * a.r + c] : 0.0f;
        }
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const int i = 16 * nt + col;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                const int c = 4 * kk + ks;
                const float x = (i < a.S && c < a.r)
                                    ? reinterpret_cast<const float *>(keys)[i * kplane + c]
                                    : 0.0f;
                ss[nt] = fmaf(x, x, ss[nt]);
                D[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[kk], x, D[nt], 0, 0, 0);
            }
        }
    }

    // One reciprocal per key instead of a division per score.
    float irho[4];
    const float inv_r = 1.0f / (float)a.r;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        float t = ss[nt];
        t += __shfl_xor(t, 16, kWaveSize);
        t += __shfl_xor(t, 32, kWaveSize);
        const float rho = sqrtf(fmaf(t, inv_r, a.eps));
        irho[nt] = 1.0f / rho;
        if (SAVE && wave == 0 && ks == 0)
            rho_out[16 * nt + col] = rho;
    }
    float s[4][4], al[4][4];
    site_softmax<false>(a, n, wave, col, ks, D, irho, s, al);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
            alpha[(16 * wave + 4 * ks + e) * kAlphaRow + 16 * nt + col] = al[nt][e];
    lds_barrier();
}

// ---------------------------------------------------------------------------
// Keys wider than kAllMaxRank columns (sliced or full rank), bf16 storage.
// ---------------------------------------------------------------------------

// 8 fp32 values as three bf16 operands whose sum is exact to fp32's 24 bits
// (hi = RNE(v), mid = RNE(v - hi), lo = RNE(v - hi - mid)): products with
// bf16 values then lose nothing that fp32 would keep.
__device__ __forceinline__ void split3(const float (&v)[8], bf16x8_t &hi, bf16x8_t &mid,
                                       bf16x8_t &lo)
{
    u32x4_t h, m, l;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const unsigned hw = pack_bf16x2(v[2 * k], v[2 * k + 1]);
        const float r0 = v[2 * k] - bf16_lo(hw), r1 = v[2 * k + 1] - bf16_hi(hw);
        const unsigned mw = pack_bf16x2(r0, r1);
        h[k] = hw;
        m[k] = mw;
        l[k] = pack_bf16x2(r0 - bf16_lo(mw), r1 - bf16_hi(mw));
    }
    hi = __builtin_bit_cast(bf16x8_t, h);
    mid = __builtin_bit_cast(bf16x8_t, m);
    lo = __builtin_bit_cast(bf16x8_t, l);
}

// Arguments of the wide-key kernels.  Sources past the last site's prefix are
// left out: no site reads them.
inline AllArgs all_wide_args(const AllProblem &p)
{
    AllArgs a;
    a.V = a.keys = p.V;
    a.Q = p.Q;
    a.H = p.H;
    a.neff = p.neff;
    a.S = (int)std::min<int64_t>(p.S, p.first + p.T - 1);
    a.d = a.krow = (int)p.d;
    a.r = (int)p.r;
    a.koff = (int)(p.d - p.r);
    a.first = (int)p.first;
    a.T = (int)p.T;
    a.N = p.N;
    a.eps = p.eps;
    a.kvec = true;
    return a;
}

// sum[nt] += A * v[nt]^T over one step of 32 columns, A as TERMS bf16 terms
// (smallest first).  The step's products start from zero and are then added
// with an fp32 addition: the matrix cores round a long chain of their own
// coarsely and downwards (measured 0.6 - 0.9 of 2^-24 a step against 0.3; over
// rows of 2048 columns dq lost a factor 2 to it).
template <int TERMS, int NT = 4>
__device__ __forceinline__ void step_product(const bf16x8_t *A, const u32x4_t (&v)[NT],
                                             f32x4_t (&sum)[4])
{
    f32x4_t t[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
        t[nt] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < TERMS; ++k)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            t[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                A[k], __builtin_bit_cast(bf16x8_t, v[nt]), t[nt], 0, 0, 0);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
        sum[nt] += t[nt];
}

// Units of 64 columns that each wave of wide_products takes of `ncol`.
__device__ __forceinline__ int wide_units(int ncol)
{
    return ((ncol + 63) / 64 + kWaves - 1) / kWaves;
}

// LDS exchange of wide_products, in bytes: one accumulator set per wave.
template <int MT> constexpr int wide_exchange_bytes() { return kWaves * MT * 4 * kWaveSize * 16; }

// The waves' shares of the products, added in wave order: sum k^2 (ss[nt],
// this lane's columns of source 16 nt + (l mod 16)), then D, then G.  Returns
// what wide_products does.
template <int MT, bool GRAD>
__device__ __forceinline__ void wide_meet(const AllArgs &a, unsigned char *exchange,
                                          float (&ss)[4], const f32x4_t (&pd)[MT][4],
                                          const f32x4_t (&pg)[MT][4], float *rho, f32x4_t (&D)[4],
                                          f32x4_t (&G)[4], float (&rho_l)[4])
{
#pragma clang fp contract(off)
    const int lane = threadIdx.x % kWaveSize;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const int lc = lane & 15, ks = lane >> 4;
    f32x4_t *ex = reinterpret_cast<f32x4_t *>(exchange);
    float *exs = reinterpret_cast<float *>(exchange);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        ss[nt] += __shfl_xor(ss[nt], 16, kWaveSize);
        ss[nt] += __shfl_xor(ss[nt], 32, kWaveSize);
        if (ks == 0)
            exs[wave * kAllMaxSources + 16 * nt + lc] = ss[nt];
    }
    lds_barrier();
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
            t += exs[w * kAllMaxSources + 16 * nt + lc];
        rho_l[nt] = sqrtf(t / (float)a.r + a.eps);
        if (wave == 0 && ks == 0)
            rho[16 * nt + lc] = rho_l[nt];
    }
    lds_barrier();
    auto meet = [&](const f32x4_t (&part)[MT][4], f32x4_t (&sum)[4]) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
                ex[((wave * MT + mt) * 4 + nt) * kWaveSize + lane] = part[mt][nt];
        lds_barrier();
        const int tile = min(wave, MT - 1);  // waves past the tiles: masked later
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            sum[nt] = ex[(tile * 4 + nt) * kWaveSize + lane];
#pragma unroll
            for (int w = 1; w < kWaves; ++w)
                sum[nt] += ex[((w * MT + tile) * 4 + nt) * kWaveSize + lane];
        }
        lds_barrier();
    };
    meet(pd, D);
    if (GRAD)
        meet(pg, G);
}

// The products of one token that contract whole rows: D = Q [16 MT x r] * K^T
// [r x 64] (Q as three bf16 terms), and with GRAD also G = dH [16 MT x d] *
// V^T [d x 64].  On return wave w holds tile w's rows: D[nt], G[nt] of sites
// 16 w + 4 (l / 16) + e against source 16 nt + (l mod 16); rho_l[nt] = rho of
// those sources, and rho (LDS, 64 floats) of all.
// Without GRAD the columns are those of the key; with it those of the whole
// row, first the ones before the key, then the key's.  The waves share the
// columns, a run of whole 64-column units each, so that each line of the
// token's rows is read once: with a tile of sites per wave, and so every row read by all four,
// the rows came from beyond the L2 each time (the planes of a stack lie a
// power of two apart and share the L2's sets) and the backward took 333 us
// instead of 256 (49 sources, 48 sites, d = 1024, r = 256, 2048 tokens).  The waves'
// partial sums meet in LDS and are added in wave order.  Steps of 32 columns,
// AHEAD of them in flight.  No load sits behind a branch, so that the
// compiler's wait counts leave the later steps in flight: rows past the
// sources or sites re-read the last one, which reaches only entries that are
// masked later, and columns past a range's end re-read its last ones against
// zeros in the other operand.  nsrc: sources that some site reads.
template <int MT, bool GRAD>
__device__ __forceinline__ void wide_products(const AllArgs &a, int64_t n, const uint16_t *dH,
                                              int nsrc, unsigned char *exchange, float *rho,
                                              f32x4_t (&D)[4], f32x4_t (&G)[4], float (&rho_l)[4])
{
#pragma clang fp contract(off)
    // Steps of source rows in flight, and of the sites' rows (which take MT
    // times the registers: one step, refilled as soon as it has been used,
    // where two waves per SIMD leave no room for more).  Four steps at MT = 2
    // and 3 were slower (301 us instead of 239, as above: a wave often has
    // fewer than eight).
    constexpr int AHEAD = MT == 1 ? 4 : 2, HA = MT <= 2 ? AHEAD : 1;
    const int lane = threadIdx.x % kWaveSize;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const int lc = lane & 15, ks = lane >> 4;
    const int key0 = GRAD ? a.koff : 0;  // the key's first column, from `base` on
    const uint16_t *base = static_cast<const uint16_t *>(a.keys) + n * a.krow + (GRAD ? 0 : a.koff);
    const size_t plane = (size_t)a.N * a.krow;
    const uint16_t *rows[4], *hrow[MT];
    const float *qrow[MT];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
        rows[nt] = base + (size_t)min(16 * nt + lc, nsrc - 1) * plane;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int site = min(16 * mt + lc, a.T - 1);
        qrow[mt] = a.Q + (size_t)site * a.r - key0;
        hrow[mt] = GRAD ? dH + ((size_t)site * a.N + n) * a.d : nullptr;
    }
    f32x4_t pd[MT][4], pg[MT][4];
    float ss[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        ss[nt] = 0.0f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            pd[mt][nt] = pg[mt][nt] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    }

    // Columns [beg, end), KEY: of the key.
    auto range = [&](auto keyc, int beg, int end) {
        constexpr bool KEY = decltype(keyc)::value;
        u32x4_t v[AHEAD][4], h[HA][MT];
        f32x4_t q[HA][MT][2];
        // The wave's share: `per` units of 64 columns, two steps each.  Column of
        // its step s (this lane's 8).
        const int per = wide_units(end - beg);
        auto column = [&](int s) { return beg + 64 * wave * per + 32 * s + 8 * ks; };
        auto load_v = [&](int s, int u) {
            const int c = min(column(s), end - 8);
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
                v[u][nt] = load_raw<uint16_t, 8>(rows[nt] + c);
        };
        auto load_h = [&](int s, int u, int mt) {
            if (GRAD)
                h[u][mt] = load_raw<uint16_t, 8>(hrow[mt] + min(column(s), end - 8));
        };
        auto load_q = [&](int s, int u, int mt) {
            if (KEY) {
                const float *p = qrow[mt] + min(column(s), end - 8);
                q[u][mt][0] = *reinterpret_cast<const f32x4_t *>(p);
                q[u][mt][1] = *reinterpret_cast<const f32x4_t *>(p + 4);
            }
        };
        auto use = [&](int s, int u) {
            // Past the wave's share (the last round of steps) or the columns.
            const bool ok = s < 2 * per && column(s) < end;
            if (GRAD) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const bf16x8_t A =
                        __builtin_bit_cast(bf16x8_t, ok ? h[u % HA][mt] : u32x4_t{0u, 0u, 0u, 0u});
                    load_h(s + HA, u % HA, mt);
                    step_product<1>(&A, v[u], pg[mt]);
                }
            }
            if (KEY) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    float x[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        x[e] = ok ? q[u % HA][mt][e / 4][e % 4] : 0.0f;
                    bf16x8_t A[3];
                    split3(x, A[2], A[1], A[0]);
                    load_q(s + HA, u % HA, mt);
                    step_product<3>(A, v[u], pd[mt]);
                }
#pragma unroll
                for (int nt = 0; nt < 4; ++nt) {
                    float y[8], t = 0.0f;
                    widen(v[u][nt], y);
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        t = fmaf(y[e], y[e], t);
                    ss[nt] += ok ? t : 0.0f;
                }
            }
        };
        // Steps of this wave that hold any column.
        const int steps = min(2 * per, (end - beg - 64 * wave * per + 31) / 32);
        if (steps <= 0)
            return;
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            if (u < HA)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    load_h(u, u, mt);
                    load_q(u, u, mt);
                }
            load_v(u, u);
        }
        for (int s = 0; s < steps; s += AHEAD)
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                __builtin_amdgcn_sched_barrier(0);
                use(s + u, u);
                __builtin_amdgcn_sched_barrier(0);
                load_v(s + u + AHEAD, u);
            }
    };
    if (key0 > 0)
        range(std::false_type{}, 0, key0);
    range(std::true_type{}, key0, key0 + a.r);

    wide_meet<MT, GRAD>(a, exchange, ss, pd, pg, rho, D, G, rho_l);
}

// The softmax gradient of the 16 sites of tile `wave` from the value dots
// G[nt][e] = dH_j . o_i, in the layout of site_softmax:
//     ds = alpha (G - sum alpha G),  cq = ds / rho,
// and skk[nt] = sum over the lane's 4 sites of ds s (the RMSNorm term of the
// sources' key gradients).  Entries past a site's prefix are 0.
template <int NT = 4, int GL = 16>
__device__ __forceinline__ void wide_softmax_grad(const AllArgs &a, int wave, int col, int ks,
                                                  const f32x4_t (&G)[4], const float (&rho_l)[4],
                                                  const float (&s)[4][4],
                                                  const float (&al)[4][4], float (&cq)[4][4],
                                                  float (&skk)[4])
{
#pragma clang fp contract(off)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
        skk[nt] = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int site = 16 * wave + 4 * ks + e;
        float gb = 0.0f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            if (read_by(a, site, 16 * nt + col))
                gb = fmaf(al[nt][e], G[nt][e], gb);
        gb = group_sum(gb, GL);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            cq[nt][e] = 0.0f;
            if (read_by(a, site, 16 * nt + col)) {
                const float ds = al[nt][e] * (G[nt][e] - gb);
                cq[nt][e] = ds / rho_l[nt];
                skk[nt] = fmaf(ds, s[nt][e], skk[nt]);
            }
        }
    }
}

// Pairs of bf16 from two packed words: the low halves (lo_pair) or the
// high halves (hi_pair) of x and y, x's in the low half of the result.  An
// 8 x 8 block of bf16 (8 rows of 8 consecutive columns, one 16-byte row per
// register quad) is transposed with these into MFMA operands that hold one
// column of 8 rows.
// Each is one byte permute (v_perm_b32: selector bytes 0-3 pick bytes of the
// second operand, 4-7 of the first).
__device__ __forceinline__ unsigned lo_pair(unsigned x, unsigned y)
{
    return __builtin_amdgcn_perm(y, x, 0x05040100u);  // (x & 0xffff) | (y << 16)
}
__device__ __forceinline__ unsigned hi_pair(unsigned x, unsigned y)
{
    return __builtin_amdgcn_perm(y, x, 0x07060302u);  // (x >> 16) | (y & 0xffff0000)
}

}  // namespace

}  // namespace lrar
