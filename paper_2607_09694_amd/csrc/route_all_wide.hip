// Backward of the read sites of a pass for keys wider than kAllMaxRank
// columns: sliced keys (the last r columns of each value) and full-rank keys
// (sliced keys with r = d, of any width), bf16 storage, S and T up to 64.  The equations
// are those of the all-sites backward of narrow keys; what differs is that a
// token's keys and queries no longer fit the LDS and the dQ of a token no
// longer fits the registers of a persistent workgroup, so the work is two
// kernels:
//
//   route_all_bwd_wide (one token per workgroup, 4 waves)
//     1. the waves contract whole rows on the matrix cores (wide_products):
//        D = Q K^T and G = dH V^T from one read of the rows; wave w then
//        holds the sites of tile w; softmax and softmax gradient in registers;
//        alpha and cq = ds / rho to LDS as three bf16 terms each (all of fp32's
//        24 bits), [source][site], and cq to the workspace in fp32;
//     2. each wave takes 64-column slabs of all 64 sources:
//            dV = alpha^T dH + (key columns) cq^T Q - ck k
//        with the upstream rows transposed in registers as in the forward
//        and Q as three terms (the six products of cq Q down to 2^-24: 5 us of
//        299 at r = 256 as below, 30 of 451 at full rank, against two terms),
//        ck_i = sum_j ds s / (rho_i^2 r).
//   wide_dq (one 64-column slab of the keys and one share of the tokens per
//     wave): dQ += cq K over its tokens in registers, on the fp32 matrix
//     cores, then a fixed-order sum of the shares in fp64.
//
// The single-site backward of full-rank keys is the same for one site, with
// its rows in registers (route_bwd_full_rows) and its dQ on the vector units
// (wide_dq_one): the same operations in the same order for every element of D,
// G, the softmax, cq and dQ, whichever sites are computed beside it, so that
// row j of an all-sites dQ is bit for bit the single-site dq of site j where
// that takes this form (full_rows).
//
// Measured at 49 sources, d = 1024.  48 sites, 2048 tokens: sliced r = 256, 48
// x (77 + dq 5) us site by site before; now 265 + 44 + 6 us (0.61 GB of rows
// in and out at least).  Full rank: 48 x (212 + dq 5) us before; now 335 + 131
// + 5 us: the fp32 matrix cores bound wide_dq, rows read again in part 2 and
// its short phases the rest.  One full-rank site, 4096 tokens: 447 + 5 us
// before (two reads of the rows at 256 workgroups); now 220 + 86 + 5 us (0.82
// GB in and out, then 0.41 GB again for dq).
#include "route_all_weights.h"

#include <algorithm>

namespace lrar {

namespace {

constexpr int kDqSlab = 64;                 // key columns per workgroup of the dQ product
constexpr int kDqAhead = 3;                 // source groups in flight in the dQ product
constexpr int kDqOneSlab = 256;             // columns per workgroup of the one-site dQ product
constexpr int kWideSlab = 64;               // columns per wave pass of the value gradient
constexpr int kOpRow = kAllMaxSources + 8;  // bf16 per LDS row of an operand [source][site]
constexpr int kOp = kAllMaxSources * kOpRow;

struct WideBwdArgs {
    AllArgs f;           // V, Q, sizes; f.S: sources that some site reads
    int sources;         // sources of the stack (rows of dV)
    const uint16_t *dH;  // [T][N][d]
    uint16_t *dV;        // [sources][N][d]
    float *cq;           // [N][T][64] ds / rho
    int64_t n0 = 0, n1 = 0;  // route_bwd_full_rows: its tokens (cq from the first on)
};

// One slab of dV (or its key term) summed over the reading sites only, on the
// vector units: taken when the matrix form gave a non-finite value, since an
// infinite or NaN upstream value of a site that doesn't read a source enters
// that source's product as 0 * value.  Lanes: 4 columns, sources 4 ks + e of
// every tile.
template <bool ACC>
__device__ __forceinline__ void wide_dv_prefixes(const WideBwdArgs &b, int64_t n,
                                              const uint16_t *at, const float *ck, int c0, int ks)
{
    const AllArgs &a = b.f;
    if (c0 >= a.d)
        return;
    const size_t plane = (size_t)a.N * a.d;
#pragma unroll 1
    for (int t = 0; t < 16; ++t) {
        const int i = 16 * (t / 4) + 4 * ks + t % 4;
        if (i >= b.sources)
            continue;
        float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
        for (int j = max(0, i + 1 - a.first); j < a.T && i < a.S; ++j) {
            const uint16_t *o = at + i * kOpRow + j;
            const float w = load_elem(o) + (load_elem(o + kOp) + load_elem(o + 2 * kOp));
            float x[4];
            widen(load_raw<uint16_t, 4>(b.dH + j * plane + n * a.d + c0), x);
            const float cq = b.cq[((size_t)n * a.T + j) * kAllMaxSources + i];
            const float *q = a.Q + (size_t)j * a.r + (c0 - a.koff);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = fmaf(w, x[e], v[e]);
                if (c0 >= a.koff)
                    v[e] = fmaf(cq, q[e], v[e]);
            }
        }
        const size_t o = i * plane + n * a.d + c0;
        if (c0 >= a.koff && i < a.S) {
            float x[4];
            widen(load_raw<uint16_t, 4>(static_cast<const uint16_t *>(a.V) + o), x);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] = fmaf(-ck[i], x[e], v[e]);
        }
        if (ACC)
            add_stored(v, load_raw<uint16_t, 4>(b.dV + o));
        store_raw<uint16_t, 4>(b.dV + o, Narrow<uint16_t, 4>::run(v));
    }
}

// The next bf16 term of four values (nearest even), taken off them.
__device__ __forceinline__ u32x2_t next_term(f32x4_t &v)
{
    const u32x2_t w = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    v -= f32x4_t{bf16_lo(w[0]), bf16_hi(w[0]), bf16_lo(w[1]), bf16_hi(w[1])};
    return w;
}

template <int MT, bool ACC>
__global__ __launch_bounds__(kBlock, 2) void route_all_bwd_wide(WideBwdArgs b)
{
    constexpr int KG = (MT + 1) / 2;  // groups of 32 sites in the contractions over sites
    // The exchange of the products, then the operands of the value gradient.
    __shared__ __align__(16)
        unsigned char lds[std::max<int>(wide_exchange_bytes<MT>(), 6 * kOp * sizeof(uint16_t))];
    // alpha and cq in three bf16 terms each, the largest first.
    uint16_t *const at = reinterpret_cast<uint16_t *>(lds), *const ct = at + 3 * kOp;
    __shared__ float rho[kAllMaxSources], ck[kAllMaxSources], part[kWaves * kAllMaxSources];
    const AllArgs &a = b.f;
    const int64_t n = xcd_block().x;  // each XCD a range of tokens (up to 8% faster)
    const int lane = threadIdx.x % kWaveSize;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const int lc = lane & 15, ks = lane >> 4;
    const size_t plane = (size_t)a.N * a.d;
    {
        f32x4_t D[4], G[4];
        float rho_l[4], s[4][4], al[4][4], cq[4][4], skk[4];
        wide_products<MT, true>(a, n, b.dH, a.S, lds, rho, D, G, rho_l);
        site_softmax<true>(a, n, wave, lc, ks, D, rho_l, s, al);
        wide_softmax_grad(a, wave, lc, ks, G, rho_l, s, al, cq, skk);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const int i = 16 * nt + lc;
            // Four consecutive sites of source i: one 8-byte write per term.
            const int o = i * kOpRow + 16 * wave + 4 * ks;
            f32x4_t x = {al[nt][0], al[nt][1], al[nt][2], al[nt][3]};
            f32x4_t y = {cq[nt][0], cq[nt][1], cq[nt][2], cq[nt][3]};
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                *reinterpret_cast<u32x2_t *>(at + t * kOp + o) = next_term(x);
                *reinterpret_cast<u32x2_t *>(ct + t * kOp + o) = next_term(y);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int site = 16 * wave + 4 * ks + e;
                if (site < a.T)
                    b.cq[((size_t)n * a.T + site) * kAllMaxSources + i] = cq[nt][e];
            }
            float t = skk[nt];
            t += __shfl_xor(t, 16, kWaveSize);
            t += __shfl_xor(t, 32, kWaveSize);
            if (ks == 0)
                part[wave * kAllMaxSources + i] = t;
        }
    }
    lds_barrier();
    if (threadIdx.x < kAllMaxSources) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
            t += part[w * kAllMaxSources + threadIdx.x];
        const float rr = rho[threadIdx.x];
        ck[threadIdx.x] = t / (rr * rr * (float)a.r);
    }
    __syncthreads();  // cq is read back from memory where a slab is done again

    // Slabs of 64 columns, 4 per lane: the accumulators of all source tiles
    // then leave room to have the next group's rows in flight.  The slabs
    // before the key and the key's run as two loops, each without a branch
    // around its loads.
    auto slabs = [&](auto keyc, int beg, int end) {
        constexpr bool KEY = decltype(keyc)::value;
        u32x2_t w[8];
        f32x4_t q[8];
        // The lane's 8 sites of group kg at its columns of slab `slab`; sites
        // past T re-read the last one (their weights are 0), columns past the
        // row its start, columns before the key the queries' start.
        auto load = [&](int slab, int kg) {
            const int c = slab * kWideSlab + 4 * lc;
            const uint16_t *h = b.dH + n * a.d + (c < a.d ? c : 0);
            // Row offsets are formed at each use: held across the loop they
            // would take the registers that the prefetch needs.
            int k8 = 8 * ks;
            asm volatile("" : "+v"(k8));
#pragma unroll
            for (int e = 0; e < 8; ++e)
                w[e] = load_raw<uint16_t, 4>(h + (unsigned)min(32 * kg + k8 + e, a.T - 1) * plane);
            if (KEY) {
                const float *qc = a.Q + (c >= a.koff && c < a.d ? c - a.koff : 0);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    q[e] = *reinterpret_cast<const f32x4_t *>(
                        qc + min(32 * kg + k8 + e, a.T - 1) * a.r);
            }
        };
        if (beg < end)
            load(beg, 0);
        for (int slab = beg; slab < end; slab += kWaves) {
            const int c0 = slab * kWideSlab + 4 * lc;
            const bool ok = c0 < a.d, kok = ok && c0 >= a.koff;
            f32x4_t acc[4][4];
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    acc[nt][p] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kg = 0; kg < KG; ++kg) {
                // Operands: one column of the lane's 8 sites each.
                bf16x8_t B[4], Q[3][4];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    u32x4_t x;
#pragma unroll
                    for (int h = 0; h < 4; ++h)
                        x[h] = (p & 1) ? hi_pair(w[2 * h][p / 2], w[2 * h + 1][p / 2])
                                       : lo_pair(w[2 * h][p / 2], w[2 * h + 1][p / 2]);
                    B[p] = __builtin_bit_cast(bf16x8_t, x);
                }
                if (KEY) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        float v[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            v[e] = kok ? q[e][p] : 0.0f;
                        split3(v, Q[0][p], Q[1][p], Q[2][p]);
                    }
                }
                // The next group, or the next slab's first (the last slab's
                // again at the end).
                load(kg + 1 < KG ? slab : slab + kWaves < end ? slab + kWaves : slab,
                     kg + 1 < KG ? kg + 1 : 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int nt = 0; nt < 4; ++nt) {
                    if (16 * nt >= a.S)
                        continue;  // wave-uniform
                    const int o = (16 * nt + lc) * kOpRow + 32 * kg + 8 * ks;
                    // Smallest terms first; of cq Q the products down to 2^-24.
#pragma unroll
                    for (int t = 2; t >= 0; --t) {
                        const bf16x8_t A = *reinterpret_cast<const bf16x8_t *>(at + t * kOp + o);
#pragma unroll
                        for (int p = 0; p < 4; ++p)
                            acc[nt][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, B[p], acc[nt][p], 0, 0, 0);
                    }
                    if (KEY) {
#pragma unroll
                        for (int t = 2; t >= 0; --t) {
                            const bf16x8_t C = *reinterpret_cast<const bf16x8_t *>(ct + t * kOp + o);
#pragma unroll
                            for (int u = 2 - t; u >= 0; --u)
#pragma unroll
                                for (int p = 0; p < 4; ++p)
                                    acc[nt][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(C, Q[u][p], acc[nt][p], 0, 0, 0);
                        }
                    }
                }
            }
            float bad = 0.0f;
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                for (int p = 0; p < 4; ++p)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        bad = fmaf(acc[nt][p][e], 0.0f, bad);
            if (__any(bad != 0.0f)) {
                wide_dv_prefixes<ACC>(b, n, at, ck, c0, ks);
                continue;
            }
            u32x2_t vk[4][4];
            if (KEY) {
                // The key rows of the lane's sources, for the norm's term.
                const uint16_t *v0 = static_cast<const uint16_t *>(a.V) + n * a.d + (ok ? c0 : 0);
                int k4 = 4 * ks;
                asm volatile("" : "+v"(k4));
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        vk[nt][e] = load_raw<uint16_t, 4>(
                            v0 + (unsigned)min(16 * nt + k4 + e, a.S - 1) * plane);
            }
            // Lane: sources 16 nt + 4 ks + e, columns c0 .. c0 + 3.
            uint16_t *d0 = b.dV + (size_t)(unsigned)(4 * ks) * plane + n * a.d + c0;
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = 16 * nt + 4 * ks + e;
                    float v[4];
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        v[p] = acc[nt][p][e];
                    if (KEY) {
                        float x[4];
                        widen(vk[nt][e], x);
                        const float c = kok && i < a.S ? -ck[i] : 0.0f;
#pragma unroll
                        for (int p = 0; p < 4; ++p)
                            v[p] = c != 0.0f ? fmaf(c, x[p], v[p]) : v[p];
                    }
                    if (ok && i < b.sources) {
                        uint16_t *dst = d0 + (16 * nt + e) * plane;
                        if (ACC)
                            add_stored(v, load_raw<uint16_t, 4>(dst));
                        store_stream<uint16_t, 4, kNtStore>(dst, Narrow<uint16_t, 4>::run(v));
                    }
                }
        }
    };
    const int nslab = (a.d + kWideSlab - 1) / kWideSlab, kslab = a.koff / kWideSlab;
    slabs(std::false_type{}, wave, kslab);
    slabs(std::true_type{}, kslab + wave, nslab);
}

// The same for one site of full-rank keys (the single-site backward), rows of
// up to 128 HS columns and up to 16 NT sources: the token's rows stay in
// registers (a quarter of the row is HS steps of 32 columns), so that every
// row is read once for the products and the gradient, and the gradient is
// formed on the vector units (one site would use 1 of 32 rows of the matrix
// form's contraction).  cq is what route_all_bwd_wide gives for the site, bit
// for bit: the same products in the same order, quarter by quarter.
// A token has a workgroup, a quarter of the row per wave (TOK = 0); or, where
// whole rows of few sources meet many tokens, a wave, which takes the quarters
// one after the other and needs no exchange (TOK = 1), or a share of a wave
// (TOK = 2, 4: up to 8, 4 sources; a tile's 16 columns are then the sources of
// 2, 4 tokens, and row t of the G product is token t's).
template <int HS, int NT, int TOK, bool ACC>
__global__ __launch_bounds__(kBlock, 2) void route_bwd_full_rows(WideBwdArgs b)
{
#pragma clang fp contract(off)
    constexpr bool WAVE = TOK > 0;
    constexpr int P = WAVE ? TOK : 1, GL = 16 / P;  // tokens per wave, lanes per token
    static_assert(P == 1 || NT == 1, "tokens share one tile of sources");
    constexpr int QW = WAVE ? kWaves : 1;  // quarters of the row per wave
    constexpr int kCols = 128 * HS;
    __shared__ __align__(16) unsigned char exchange[WAVE ? 16 : wide_exchange_bytes<1>()];
    __shared__ __align__(16) uint16_t hall[(WAVE ? kWaves * P : 1) * kCols];
    __shared__ __align__(16) float qs[kCols];
    __shared__ __align__(16) uint16_t qt3[3 * kCols];
    __shared__ float rho[kAllMaxSources];
    AllArgs a = b.f;
    a.T = 1;  // known to the compiler: rows 1 .. 15 of the products fold away
    a.neff = nullptr;
    const int lane = threadIdx.x % kWaveSize;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const int lc = lane & 15, ks = lane >> 4;
    // Each XCD a range of tokens (3-5% faster).
    // The lane's token (the wave's first for P = 1) and its source in a tile;
    // lanes past the tokens re-read the last one and store nothing.
    const int tl = lc / GL, il = lc % GL;
    const int64_t nw =
        b.n0 + (WAVE ? ((int64_t)xcd_block().x * kWaves + wave) * P : xcd_block().x);
    const bool live = nw + tl < b.n1;
    const int64_t n = min(nw + tl, b.n1 - 1);
    uint16_t *const hs = hall + (WAVE ? wave * P * kCols : 0);
    const size_t plane = (size_t)a.N * a.d;
    // This lane's columns of step s of quarter k; a quarter has 2 per <= HS
    // steps (what follows is another quarter's).
    const int per = wide_units(a.d);
    auto column = [&](int k, int s) { return 64 * (WAVE ? k : wave) * per + 32 * s + 8 * ks; };
    const uint16_t *rows[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
        rows[nt] = static_cast<const uint16_t *>(a.V) + n * a.d +
                   (unsigned)min(16 * nt + il, a.S - 1) * plane;
    // The upstream row and the query into LDS (all lanes with one ks need the
    // same 8 columns a step), zeros past the row; their loads go first, so that
    // the LDS writes don't wait for the rows.
    constexpr int kHl = WAVE ? (kCols + 4 * kWaveSize - 1) / (4 * kWaveSize) : 1;
    const int t4 = 4 * threadIdx.x, h4 = WAVE ? 4 * lane : t4;
    u32x2_t ht[P][kHl];
    f32x4_t qt = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int t = 0; t < P; ++t)
#pragma unroll
        for (int k = 0; k < kHl; ++k) {
            const int c = h4 + 4 * kWaveSize * k;
            ht[t][k] = load_raw<uint16_t, 4>(b.dH + min(nw + t, b.n1 - 1) * a.d + min(c, a.d - 4));
            if (c >= a.d)
                ht[t][k] = u32x2_t{0u, 0u};
        }
    if (t4 < a.d)
        qt = *reinterpret_cast<const f32x4_t *>(a.Q + t4);
    // The lines of a row one after the other, and the two halves of a line
    // (steps 2 k and 2 k + 1) next to each other here and in the stores: the
    // planes of a stack often lie a power of two apart, their lines then share
    // one set of the L2 and don't outlive the other rows of the token (with
    // the steps outermost and the waves taking columns in turn: 253 us instead
    // of 202 at 49 sources, d = 1024, 4096 tokens).
    u32x4_t v[QW][HS][NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int k = 0; k < QW; ++k)
#pragma unroll
            for (int s = 0; s < HS; ++s)
                v[k][s][nt] = load_raw<uint16_t, 8>(rows[nt] + min(column(k, s), a.d - 8));
#pragma unroll
    for (int t = 0; t < P; ++t)
#pragma unroll
        for (int k = 0; k < kHl; ++k)
            if (h4 + 4 * kWaveSize * k < kCols)
                *reinterpret_cast<u32x2_t *>(hs + t * kCols + h4 + 4 * kWaveSize * k) = ht[t][k];
    if (t4 < kCols) {
        // The query as it is, for the gradient, and as the products' three
        // bf16 terms (as split3 forms them), once for all waves and lanes.
        *reinterpret_cast<f32x4_t *>(qs + t4) = qt;
        float r[4] = {qt.x, qt.y, qt.z, qt.w};
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            u32x2_t w;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                w[k] = pack_bf16x2(r[2 * k], r[2 * k + 1]);
                r[2 * k] -= bf16_lo(w[k]);
                r[2 * k + 1] -= bf16_hi(w[k]);
            }
            *reinterpret_cast<u32x2_t *>(qt3 + (2 - t) * kCols + t4) = w;  // smallest first
        }
    }
    lds_barrier();
    auto query = [&](int c, float (&x)[8]) {
        const f32x4_t q0 = *reinterpret_cast<const f32x4_t *>(qs + c);
        const f32x4_t q1 = *reinterpret_cast<const f32x4_t *>(qs + c + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x[e] = q0[e];
            x[4 + e] = q1[e];
        }
    };
    f32x4_t D[4], G[4];
    float rho_l[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        D[nt] = G[nt] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        rho_l[nt] = 0.0f;  // WAVE: sum k^2 at first
    }
#pragma unroll
    for (int k = 0; k < QW; ++k) {
        f32x4_t pd[1][4], pg[1][4];
        float ss[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
            pd[0][nt] = pg[0][nt] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < HS; ++s) {
            __builtin_amdgcn_sched_barrier(0);
            if (s >= 2 * per)
                break;  // wave-uniform
            const int c = column(k, s);
            // Row t of the G operand: token t's upstream row.
            const bf16x8_t Ah =
                *reinterpret_cast<const bf16x8_t *>(hs + (P > 1 ? lc % P * kCols : 0) + c);
            step_product<1, NT>(&Ah, v[k][s], pg[0]);
            bf16x8_t A[3];
#pragma unroll
            for (int t = 0; t < 3; ++t)
                A[t] = *reinterpret_cast<const bf16x8_t *>(qt3 + t * kCols + c);
            step_product<3, NT>(A, v[k][s], pd[0]);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                float y[8], t = 0.0f;
                widen(v[k][s][nt], y);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    t = fmaf(y[e], y[e], t);
                ss[nt] += c < a.d ? t : 0.0f;
            }
        }
        if constexpr (WAVE) {
            // The sums of wide_meet, in its order.
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                ss[nt] += __shfl_xor(ss[nt], 16, kWaveSize);
                ss[nt] += __shfl_xor(ss[nt], 32, kWaveSize);
                rho_l[nt] += ss[nt];
                D[nt] = k == 0 ? pd[0][nt] : D[nt] + pd[0][nt];
                G[nt] = k == 0 ? pg[0][nt] : G[nt] + pg[0][nt];
            }
        } else {
            wide_meet<1, true>(a, exchange, ss, pd, pg, rho, D, G, rho_l);
        }
    }
    if constexpr (WAVE)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            rho_l[nt] = sqrtf(rho_l[nt] / (float)a.r + a.eps);
    float al_i[NT], cq_i[NT], ck_i[NT];
    {
        // Every wave of a token forms the one site's weights and coefficients;
        // they are on the lanes of row 0 (l < 16), and go to all from there.
        float s[4][4], al[4][4], cq[4][4], skk[4];
        if constexpr (P > 1)  // a token's dots are in its own row
#pragma unroll
            for (int t = 1; t < P; ++t)
                G[0][0] = tl == t ? G[0][t] : G[0][0];
        site_softmax<true, NT, GL>(a, n, 0, il, ks, D, rho_l, s, al);
        wide_softmax_grad<NT, GL>(a, 0, il, ks, G, rho_l, s, al, cq, skk);
        if ((WAVE ? live : wave == 0) && ks == 0)
#pragma unroll
            for (int k = 0; k < kAllMaxSources / GL; ++k)
                b.cq[(size_t)(n - b.n0) * kAllMaxSources + GL * k + il] = k < NT ? cq[k < NT ? k : 0][0] : 0.0f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            al_i[nt] = __shfl(al[nt][0], lc, kWaveSize);
            cq_i[nt] = __shfl(cq[nt][0], lc, kWaveSize);
            ck_i[nt] = __shfl(skk[nt], lc, kWaveSize) / (rho_l[nt] * rho_l[nt] * (float)a.d);
        }
    }
    // The rows as raw bits again, the query and dH from LDS: what the products
    // made of them would otherwise be kept for here, in registers that do not
    // exist.
    asm volatile("" ::: "memory");
#pragma unroll
    for (int k = 0; k < QW; ++k)
#pragma unroll
        for (int s = 0; s < HS; ++s)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                asm volatile("" : "+v"(v[k][s][nt]));
    // Lane: sources 16 nt + lc, 8 columns a step.
    uint16_t *d0 = b.dV + n * a.d + (size_t)(unsigned)il * plane;
#pragma unroll
    for (int k = 0; k < QW; ++k)
#pragma unroll
        for (int s = 0; s < HS; s += 2) {
            if (s >= 2 * per)
                break;  // wave-uniform
            __builtin_amdgcn_sched_barrier(0);
            float x[2][8], y[2][8];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                query(column(k, s + u), x[u]);
                widen(*reinterpret_cast<const u32x4_t *>(hs + tl * kCols + column(k, s + u)), y[u]);
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                u32x4_t o[2];
                uint16_t *dst = d0 + 16 * nt * plane + column(k, s);
                const bool src = 16 * nt + il < a.S && live;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    float g[8];
                    widen(v[k][s + u][nt], g);
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        g[e] = fmaf(al_i[nt], y[u][e], fmaf(cq_i[nt], x[u][e], -ck_i[nt] * g[e]));
                    if (ACC && src && column(k, s + u) < a.d)
                        add_stored(g, load_raw<uint16_t, 8>(dst + 32 * u));
                    o[u] = Narrow<uint16_t, 8>::run(g);
                }
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    if (src && column(k, s + u) < a.d)
                        store_raw<uint16_t, 8>(dst + 32 * u, o[u]);
            }
        }
}

// dQ shares.  Wave `id` of the grid's y dimension sums
//     share[j][c] = sum_n sum_i cq[n][j][i] k[n][i][c]
// over its tokens n = id, id + waves, ... in order, for the 64 key columns of
// slab blockIdx.x, on the fp32 matrix cores: a lane's 8-byte row pieces,
// widened, are the operands as they stand (16 sources a group, four a step,
// lane group ks taking sources 4 ks .. 4 ks + 3 of the group, so that its cq
// come as one 16-byte vector).  The sum of a group starts from zero, a token's
// groups add up on their own, then the tokens, then the 4 waves of a workgroup:
// short chains of fp32 additions, so that dQ is 0.76 - 0.96 times as far from
// 64 bits as the site-by-site calls (1 to 7000 tokens, 5 to 64 sources; up to
// 1.06 times with one chain over a token and the shares summed in fp32).
// The bf16 matrix cores with cq as three terms took 27 us against 44 (49
// sources, 48 sites, r = 256, 2048 tokens), but round long sums coarsely: in
// one chain, the error grew with the tokens, to 1.6 times at 2048.
struct WideDqArgs {
    const uint16_t *V;  // [S][N][d]
    const float *cq;    // [N][T][64]
    float *partial;     // [gridDim.y][T][r]
    int S, d, r, first, T;
    int64_t N;
    // wide_dq_one: its tokens (cq from the first on), and where the waves' sums
    // [gridDim.y][4][r] pass from one range of tokens to the next (NULL for one
    // range).
    int64_t n0 = 0, n1 = 0;
    float *carry = nullptr;
};

// The same share over each site's prefix only, on the vector units (a
// non-finite source value past a site's prefix met cq = 0).
__device__ __forceinline__ void wide_dq_prefix(const WideDqArgs &a, int64_t n0, int64_t step,
                                            int site, int c, f32x4_t &v)
{
    v = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    const size_t plane = (size_t)a.N * a.d;
#pragma unroll 1
    for (int64_t n = n0; n < a.N; n += step)
#pragma unroll 1
        for (int i = 0; i < min(a.S, a.first + site); ++i) {
            const float w = a.cq[((size_t)n * a.T + site) * kAllMaxSources + i];
            float x[4];
            widen(load_raw<uint16_t, 4>(a.V + i * plane + n * a.d + (a.d - a.r) + c), x);
#pragma unroll
            for (int p = 0; p < 4; ++p)
                v[p] = fmaf(w, x[p], v[p]);
        }
}

template <int MT>
__global__ __launch_bounds__(kBlock, 2) void wide_dq(WideDqArgs a)
{
    __shared__ __align__(16) float red[16 * kDqSlab * (kWaves - 1)];
    const int lane = threadIdx.x % kWaveSize;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const int lc = lane & 15, ks = lane >> 4;
    const int c0 = blockIdx.x * kDqSlab + 4 * lc;
    const bool ok = c0 < a.r;
    const size_t plane = (size_t)a.N * a.d;
    const uint16_t *key = a.V + (a.d - a.r) + (ok ? c0 : 0);
    const int64_t n0 = (int64_t)blockIdx.y * kWaves + wave, step = (int64_t)gridDim.y * kWaves;
    const int ngroups = (a.S + 15) / 16;
    f32x4_t acc[MT][4], tok[MT][4];  // over the tokens, and of the current one
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int p = 0; p < 4; ++p)
            acc[mt][p] = tok[mt][p] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    // kDqAhead groups in flight.  A wave's groups in order: those of its first
    // token, of its next, ...; past the last one, the last again.
    u32x2_t raw[kDqAhead][4];
    f32x4_t q[kDqAhead][MT];
    auto load = [&](int64_t n, int g, int u) {
        // Sources past S re-read the last one; their cq is 0.  Sites past T
        // re-read the last one; their rows are not stored.
        const uint16_t *r0 = key + n * a.d;
        int s0 = 16 * g + 4 * ks;
        asm volatile("" : "+v"(s0));
#pragma unroll
        for (int e = 0; e < 4; ++e)
            raw[u][e] = load_raw<uint16_t, 4>(r0 + (unsigned)min(s0 + e, a.S - 1) * plane);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            q[u][mt] = *reinterpret_cast<const f32x4_t *>(
                a.cq + ((size_t)n * a.T + min(16 * mt + lc, a.T - 1)) * kAllMaxSources + 16 * g + 4 * ks);
    };
    auto use = [&](int g, int u) {
        float x[4][4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            widen(raw[u][e], x[e]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            if (16 * g >= a.first + 16 * mt + 15)
                continue;  // wave-uniform: no site of the tile reads the group
            f32x4_t t[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    t[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                        q[u][mt][e], x[e][p], e == 0 ? f32x4_t{0.0f, 0.0f, 0.0f, 0.0f} : t[p], 0, 0, 0);
#pragma unroll
            for (int p = 0; p < 4; ++p)
                tok[mt][p] += t[p];
        }
        if (g + 1 == ngroups)  // wave-uniform
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    acc[mt][p] += tok[mt][p];
                    tok[mt][p] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
                }
    };
    const int64_t total = n0 < a.N ? ((a.N - n0 + step - 1) / step) * ngroups : 0;
    int64_t nl = n0;  // token and group of the next load
    int gl = 0;
    auto advance = [&]() {
        if (++gl == ngroups) {
            gl = 0;
            nl += step;
        }
        if (nl >= a.N) {
            nl -= step;
            gl = ngroups - 1;
        }
    };
    if (total > 0) {
#pragma unroll
        for (int u = 0; u < kDqAhead; ++u) {
            load(nl, gl, u);
            advance();
        }
    }
    int g = 0;
    for (int64_t k = 0; k < total; k += kDqAhead)
#pragma unroll
        for (int u = 0; u < kDqAhead; ++u) {
            __builtin_amdgcn_sched_barrier(0);
            if (k + u < total)  // wave-uniform
                use(g, u);
            g = g + 1 == ngroups ? 0 : g + 1;
            __builtin_amdgcn_sched_barrier(0);
            load(nl, gl, u);
            advance();
        }
    // Lane: sites 16 mt + 4 ks + e, columns c0 .. c0 + 3; one site tile of
    // every wave meets in LDS at a time.
    float *part = a.partial + (size_t)blockIdx.y * a.T * a.r;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        f32x4_t v[4];
        float bad = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                v[e][p] = acc[mt][p][e];
                bad = fmaf(v[e][p], 0.0f, bad);
            }
        if (__any(bad != 0.0f)) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (ok && 16 * mt + 4 * ks + e < a.T)
                    wide_dq_prefix(a, n0, step, 16 * mt + 4 * ks + e, c0, v[e]);
        }
        if (wave > 0)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                *reinterpret_cast<f32x4_t *>(red + ((wave - 1) * 16 + 4 * ks + e) * kDqSlab + 4 * lc) =
                    v[e];
        __syncthreads();
        if (wave == 0 && ok)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int site = 16 * mt + 4 * ks + e;
                if (site >= a.T)
                    continue;
#pragma unroll
                for (int w = 0; w < kWaves - 1; ++w)
                    v[e] += *reinterpret_cast<const f32x4_t *>(red + (w * 16 + 4 * ks + e) * kDqSlab + 4 * lc);
                *reinterpret_cast<f32x4_t *>(part + (size_t)site * a.r + c0) = v[e];
            }
        __syncthreads();
    }
}

// The shares of one site, on the vector units: the matrix form would use one
// of its 16 rows, and is then bound by the matrix cores (110 us instead of
// 82 at 49 sources, d = r = 1024, 4096 tokens).  The same operations in the same order:
// v_mfma_f32_16x16x4_f32 is a chain of four fused multiply-adds, k ascending
// (measured against such chains, bit for bit), here sources 16 g + e, + 4,
// + 8, + 12 for e = 0 .. 3.  A lane owns 4 columns; AHEAD groups in flight.  K4: the
// fours of sources that a group holds (4, or fewer where S <= 8 leaves one
// group mostly empty; cq is 0 there).
template <int K4>
__global__ __launch_bounds__(kBlock) void wide_dq_one(WideDqArgs a)
{
    constexpr int AHEAD = 8 / K4;
    __shared__ __align__(16) float red[(kWaves - 1) * kDqOneSlab];
    const BlockXY blk = xcd_block();  // the slabs of one share on one XCD
    const int lane = threadIdx.x % kWaveSize;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const int c0 = blk.x * kDqOneSlab + 4 * lane;
    const bool ok = c0 < a.r;
    const size_t plane = (size_t)a.N * a.d;
    const uint16_t *key = a.V + (a.d - a.r) + (ok ? c0 : 0);
    const int64_t n0 = a.n0 + (int64_t)blk.y * kWaves + wave, step = (int64_t)gridDim.y * kWaves;
    const int ngroups = (a.S + 15) / 16;
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f}, tok[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    u32x2_t raw[AHEAD][4 * K4];
    auto load = [&](int64_t n, int g, int u) {
        const uint16_t *r0 = key + n * a.d;
#pragma unroll
        for (int i = 0; i < 4 * K4; ++i)  // sources past S re-read the last one; their cq is 0
            raw[u][i] = load_stream<uint16_t, 4, true>(r0 + (size_t)min(16 * g + i, a.S - 1) * plane);
    };
    auto use = [&](int64_t n, int g, int u) {
        const float *c = a.cq + (size_t)(n - a.n0) * kAllMaxSources + 16 * g;  // wave-uniform
        float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int k = 0; k < K4; ++k) {
                float x[4];
                widen(raw[u][4 * k + e], x);
                const float w = c[4 * k + e];
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    t[p] = fmaf(w, x[p], t[p]);
            }
#pragma unroll
        for (int p = 0; p < 4; ++p)
            tok[p] += t[p];
        if (g + 1 == ngroups)  // wave-uniform
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                acc[p] += tok[p];
                tok[p] = 0.0f;
            }
    };
    const int64_t total = n0 < a.n1 ? ((a.n1 - n0 + step - 1) / step) * ngroups : 0;
    int64_t nl = n0, nu = n0;  // token and group of the next load and of the next use
    int gl = 0, gu = 0;
    auto advance = [&]() {
        if (++gl == ngroups) {
            gl = 0;
            nl += step;
        }
        if (nl >= a.n1) {
            nl -= step;
            gl = ngroups - 1;
        }
    };
    f32x4_t *carry =
        reinterpret_cast<f32x4_t *>(a.carry + ((size_t)blk.y * kWaves + wave) * a.r + c0);
    if (a.carry && a.n0 > 0 && ok) {
        const f32x4_t v = *carry;
#pragma unroll
        for (int p = 0; p < 4; ++p)
            acc[p] = v[p];
    }
    if (total > 0) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            load(nl, gl, u);
            advance();
        }
    }
    for (int64_t k = 0; k < total; k += AHEAD)
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            __builtin_amdgcn_sched_barrier(0);
            if (k + u < total) {  // wave-uniform
                use(nu, gu, u);
                if (++gu == ngroups) {
                    gu = 0;
                    nu += step;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            load(nl, gl, u);
            advance();
        }
    if (a.carry && a.n1 < a.N) {  // uniform: more tokens follow
        if (ok)
            *carry = f32x4_t{acc[0], acc[1], acc[2], acc[3]};
        return;
    }
    if (wave > 0)
        *reinterpret_cast<f32x4_t *>(red + (wave - 1) * kDqOneSlab + 4 * lane) =
            f32x4_t{acc[0], acc[1], acc[2], acc[3]};
    __syncthreads();
    if (wave == 0 && ok) {
#pragma unroll
        for (int w = 0; w < kWaves - 1; ++w)
#pragma unroll
            for (int p = 0; p < 4; ++p)
                acc[p] += red[w * kDqOneSlab + 4 * lane + p];
        *reinterpret_cast<f32x4_t *>(a.partial + (size_t)blk.y * a.r + c0) =
            f32x4_t{acc[0], acc[1], acc[2], acc[3]};
    }
}

// dQ[x] (+)= the shares of element x: a workgroup takes 64 elements, its wave
// w the w-th quarter of the shares, eight interleaved chains of them, summed
// pairwise, and the quarters add up in order (coalesced over the elements;
// zeros without tokens).  Sums in fp64, which the kernel's time doesn't show
// (it waits for its loads): the shares keep what they have.
template <bool ACC>
__global__ __launch_bounds__(kBlock) void wide_dq_sum(const float *__restrict__ partial,
                                                      float *__restrict__ dQ, int shares, int n)
{
    __shared__ double red[kWaves][kWaveSize];
    const int lane = threadIdx.x % kWaveSize, wave = threadIdx.x / kWaveSize;
    const int x = blockIdx.x * kWaveSize + lane;
    const int per = (shares + kWaves - 1) / kWaves;
    const int beg = wave * per, end = min(shares, beg + per);
    double s[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (x < n) {
        int k = beg;
        for (; k + 8 <= end; k += 8) {
            float t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                t[u] = partial[(size_t)(k + u) * n + x];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                s[u] += t[u];
        }
#pragma unroll
        for (int u = 0; u < 7; ++u)
            if (k + u < end)
                s[u] += partial[(size_t)(k + u) * n + x];
    }
#pragma unroll
    for (int h = 4; h >= 1; h >>= 1)
#pragma unroll
        for (int u = 0; u < h; ++u)
            s[u] += s[u + h];
    red[wave][lane] = s[0];
    __syncthreads();
    if (wave == 0 && x < n) {
        const double t = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
        dQ[x] = (float)(ACC ? dQ[x] + t : t);
    }
}

template <int MT>
void launch_wide_mt(const WideBwdArgs &b, const WideDqArgs &q, dim3 qgrid, bool accumulate,
                    hipStream_t st)
{
    const dim3 grid((unsigned)b.f.N), block(kBlock);
    if (accumulate)
        hipLaunchKernelGGL((route_all_bwd_wide<MT, true>), grid, block, 0, st, b);
    else
        hipLaunchKernelGGL((route_all_bwd_wide<MT, false>), grid, block, 0, st, b);
    hipLaunchKernelGGL(wide_dq<MT>, qgrid, block, 0, st, q);
}

void launch_dq_one(const WideDqArgs &q, int64_t shares, hipStream_t st)
{
    const dim3 grid((unsigned)((q.r + kDqOneSlab - 1) / kDqOneSlab), (unsigned)shares), block(kBlock);
    if (q.S <= 4)
        hipLaunchKernelGGL(wide_dq_one<1>, grid, block, 0, st, q);
    else if (q.S <= 8)
        hipLaunchKernelGGL(wide_dq_one<2>, grid, block, 0, st, q);
    else
        hipLaunchKernelGGL(wide_dq_one<4>, grid, block, 0, st, q);
}

// Token shares of wide_dq: about four workgroups per CU over all key slabs,
// at least one token per wave.  Depends on N and r only (not on the sites or
// sources), so that the order of every dQ sum does too.
int64_t wide_shares(int64_t N, int64_t r)
{
    const int64_t nslab = (r + kDqSlab - 1) / kDqSlab;
    return std::max<int64_t>(1, std::min<int64_t>(1024 / nslab, (N + kWaves - 1) / kWaves));
}

}  // namespace

// cq, then the dQ shares, from a 16-byte boundary of the workspace on.
size_t wide_bwd_workspace_bytes(int64_t N, int64_t T, int64_t r)
{
    return 16 + ((size_t)N * T * kAllMaxSources + (size_t)wide_shares(N, r) * T * r) * sizeof(float);
}

namespace {

// Tokens above which few sources take a wave per token: the quarters of its
// rows then run one after the other, which costs a call of few tokens more
// than the idle lanes of a workgroup per token do.  Workgroup per token ->
// wave: one tile of sources, 2 of d = 1024: 256 tokens 16 -> 19 us, 400
// level, 2048 50 -> 23; 16 of d = 512: 256 14 -> 14, 512 17 -> 16, 2048 46 ->
// 26.  More tiles, 32 of d = 512: 800 tokens 25 -> 27, 1024 26 -> 28, 2048 52
// -> 42; 64 of d = 256: 800 30 -> 28, 2048 51 -> 41.
constexpr int64_t kFullWaveTokens = 320, kFullWaveTokensTiles = 1024;

template <int HS, int NT, int TOK, bool ACC>
void launch_rows(const WideBwdArgs &b, hipStream_t st)
{
    constexpr int per = TOK > 0 ? TOK * kWaves : 1;  // tokens per workgroup
    hipLaunchKernelGGL((route_bwd_full_rows<HS, NT, TOK, ACC>),
                       dim3((unsigned)((b.n1 - b.n0 + per - 1) / per)), dim3(kBlock), 0, st, b);
}

// HS for the row width; a wave holds at most 32 vectors a lane of its rows, so
// a whole token's (4 HS NT) only where these are as few.
template <int HS, bool ACC>
void launch_rows_hs(const WideBwdArgs &b, hipStream_t st)
{
    const int nt = (b.f.S + 15) / 16;
    const bool many = b.f.N > (nt == 1 ? kFullWaveTokens : kFullWaveTokensTiles);
    if (many && b.f.S <= 4)
        return launch_rows<HS, 1, 4, ACC>(b, st);
    if (many && b.f.S <= 8)
        return launch_rows<HS, 1, 2, ACC>(b, st);
    if (many && nt == 1)
        return launch_rows<HS, 1, 1, ACC>(b, st);
    if constexpr (HS <= 4)
        if (many && nt == 2)
            return launch_rows<HS, 2, 1, ACC>(b, st);
    if constexpr (HS <= 2) {
        if (many)
            return launch_rows<HS, 4, 1, ACC>(b, st);
    } else {
        if (nt == 2)
            return launch_rows<HS, 2, 0, ACC>(b, st);
        if (nt == 3)
            return launch_rows<HS, 3, 0, ACC>(b, st);
    }
    launch_rows<HS, 4, 0, ACC>(b, st);
}

// The single site of full-rank keys with its rows in registers, up to
// kFullRowsMax columns.
template <bool ACC>
void launch_full_rows(const WideBwdArgs &b, hipStream_t st)
{
    if (b.f.d <= 256)
        launch_rows_hs<2, ACC>(b, st);
    else if (b.f.d <= 512)
        launch_rows_hs<4, ACC>(b, st);
    else
        launch_rows_hs<8, ACC>(b, st);
}

}  // namespace

// Rows of 1024 columns, which route_bwd_full takes without column masks, leave
// the register form level with it at 32 sources and behind with fewer from
// about 16384 tokens on (route_bwd_full -> this: 16001 tokens, 4 sources 103 ->
// 101 us, 16: 357 -> 317; 24000 tokens, 2: 84 -> 107, 16: 411 -> 460, 32: 898 ->
// 898; 60001 tokens, 16: 986 -> 1115).  Rows of 1000 columns gain throughout
// (60001 tokens, 2: 285 -> 283, 16: 1463 -> 1251).  Up to that line the form is
// kept for few sources too, where it costs up to 15% (8192 tokens, 2 sources),
// for the bits that it shares with the all-sites form.
bool full_rows(const Problem &p)
{
    return p.mode == LRAR_MODE_FULL && p.dtype == LRAR_DTYPE_BF16 && p.d % 8 == 0 &&
           p.d <= kFullRowsMax && (p.d < kFullRowsMax || p.N <= 16384) &&
           p.N * kBlock < ((int64_t)1 << 32);
}

// Adding to the gradients, rows of 512 columns fall behind too, and all wide
// ones earlier (route_bwd_full / this, 2, 4, 16, 32 or 49 sources): d = 1024: 4096
// tokens 0.96, 1.00, 1.42, 1.16, 8192: 0.79, 0.88, 0.86, 0.86; d = 512: 8192 1.09,
// 1.05, 1.28, 1.11, 16384: 0.86, 0.81, 0.88, 0.96; d = 1000: 6000 0.99, 1.07, 1.37,
// 1.28, 12288: 0.72, 0.84, 0.86, 0.88, 24000: 0.76, 0.83, 0.88; d = 776: 8000 0.92,
// 1.02, 1.17, 1.14, 24000 0.76, 0.96, 0.88, 0.88.
bool full_rows_adding(const Problem &p)
{
    const int64_t most = p.d % 512 == 0 ? 1 << 22 : 6 << 20;  // tokens x columns
    return full_rows(p) && (p.d < 512 || p.N * p.d <= most);
}

int launch_wide_bwd(const AllProblem &p, const void *dH, void *dV, float *dQ, void *ws,
                    size_t ws_bytes, bool accumulate, hipStream_t st, std::string *err)
{
    const int64_t shares = wide_shares(p.N, p.r);
    float *cq = reinterpret_cast<float *>((reinterpret_cast<uintptr_t>(ws) + 15) / 16 * 16);
    float *partial = nullptr;
    if (p.N > 0) {
        // The tokens go in one range where the workspace holds their cq.  For
        // one site (the only caller with less, the allocation-free backward)
        // they go in ranges of whole rounds over the shares, and the waves'
        // sums pass on in between: the same additions in the same order.
        const bool one = p.T == 1;
        int64_t range = p.N;
        size_t carry = 0;
        if (one && ws_bytes < wide_bwd_workspace_bytes(p.N, 1, p.r)) {
            const int64_t round = shares * kWaves;
            carry = (size_t)round * p.r;
            const int64_t room = (int64_t)((ws_bytes - 16) / sizeof(float)) -
                                 (int64_t)(carry + (size_t)shares * p.r);
            range = room / kAllMaxSources / round * round;
            if (range <= 0) {
                *err = "workspace too small for the full-rank backward";
                return LRAR_EINVAL;
            }
        }
        partial = cq + (size_t)range * p.T * kAllMaxSources;
        WideBwdArgs b;
        b.f = all_wide_args(p);
        b.f.H = nullptr;
        b.f.neff = nullptr;
        b.sources = (int)p.S;
        b.dH = static_cast<const uint16_t *>(dH);
        b.dV = static_cast<uint16_t *>(dV);
        b.cq = cq;
        WideDqArgs q{static_cast<const uint16_t *>(p.V), cq, partial, b.f.S, (int)p.d,
                     (int)p.r, b.f.first, b.f.T, p.N};
        if (carry)
            q.carry = partial + (size_t)shares * p.r;
        const dim3 qgrid((unsigned)((p.r + kDqSlab - 1) / kDqSlab), (unsigned)shares);
        for (int64_t n = 0; one && n < p.N; n += range) {
            b.n0 = q.n0 = n;
            b.n1 = q.n1 = std::min(p.N, n + range);
            accumulate ? launch_full_rows<true>(b, st) : launch_full_rows<false>(b, st);
            launch_dq_one(q, shares, st);
        }
        switch (one ? 0 : (b.f.T + 15) / 16) {
        case 0: break;
        case 1: launch_wide_mt<1>(b, q, qgrid, accumulate, st); break;
        case 2: launch_wide_mt<2>(b, q, qgrid, accumulate, st); break;
        case 3: launch_wide_mt<3>(b, q, qgrid, accumulate, st); break;
        default: launch_wide_mt<4>(b, q, qgrid, accumulate, st); break;
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return hip_status(e, "route_all_bwd_wide", err);
    }
    const int n = (int)(p.T * p.r), ns = p.N > 0 ? (int)shares : 0;
    const dim3 grid((unsigned)((n + kWaveSize - 1) / kWaveSize));
    if (accumulate)
        hipLaunchKernelGGL(wide_dq_sum<true>, grid, dim3(kBlock), 0, st, partial, dQ, ns, n);
    else
        hipLaunchKernelGGL(wide_dq_sum<false>, grid, dim3(kBlock), 0, st, partial, dQ, ns, n);
    return hip_status(hipGetLastError(), "route_all_bwd_wide dQ sum", err);
}

}  // namespace lrar
