// Backward of the read sites of a pass for keys wider than kAllMaxRank
// columns: sliced keys (the last r columns of each value), bf16 storage, S and
// T up to 64.  The equations
// are those of the all-sites backward of narrow keys; what differs is that a
// token's keys and queries no longer fit the LDS and the dQ of a token no
// longer fits the registers of a persistent workgroup, so the work is two
// kernels:
//
//   route_all_bwd_wide (one token per workgroup, 4 waves)
//     1. the waves contract whole rows on the matrix cores (wide_products):
//        D = Q K^T and G = dH V^T from one read of the rows; wave w then
//        holds the sites of tile w; softmax and softmax gradient in registers; alpha and cq = ds / rho to LDS as hi + lo bf16,
//        [source][site], and cq to the workspace in fp32;
//     2. each wave takes 64-column slabs of all 64 sources:
//            dV = alpha^T dH + (key columns) cq^T Q - ck k
//        with the upstream rows transposed in registers as in the forward
//        and Q as hi + lo (three MFMAs), ck_i = sum_j ds s / (rho_i^2 r).
//   wide_dq (one 128-column slab of the keys and one share of the tokens per
//     wave): dQ += cq K over its tokens in registers, on the fp32 matrix
//     cores, then a fixed-order sum of the shares.
//
// Measured (49 sources, 48 sites, d = 1024, sliced r = 256, 2048 tokens; site
// by site before: 48 x (bwd 77 + dq 5) us): route_all_bwd_wide 239 us (0.61 GB
// of rows in and out, 0.1 GB of them read twice), wide_dq 34 us, the sum 5 us.
#include "route_all_weights.h"

#include <algorithm>

namespace lrar {

namespace {

constexpr int kWideSlab = 64;               // columns per wave pass of the value gradient
constexpr int kOpRow = kAllMaxSources + 8;  // bf16 per LDS row of an operand [source][site]

struct WideBwdArgs {
    AllArgs f;           // V, Q, sizes; f.S: sources that some site reads
    int sources;         // sources of the stack (rows of dV)
    const uint16_t *dH;  // [T][N][d]
    uint16_t *dV;        // [sources][N][d]
    float *cq;           // [N][T][64] ds / rho
};

// 8 rows of 8 consecutive columns (one 16-byte row per register quad) as 8
// operands that hold one column of the 8 rows.
__device__ __forceinline__ void transpose8(const u32x4_t (&w)[8], bf16x8_t (&b)[8])
{
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        u32x4_t q;
#pragma unroll
        for (int h = 0; h < 4; ++h)
            q[h] = (p & 1) ? hi_pair(w[2 * h][p / 2], w[2 * h + 1][p / 2])
                           : lo_pair(w[2 * h][p / 2], w[2 * h + 1][p / 2]);
        b[p] = __builtin_bit_cast(bf16x8_t, q);
    }
}

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

// One slab of dV (or its key term) summed over the reading sites only, on the
// vector units: taken when the matrix form gave a non-finite value, since an
// infinite or NaN upstream value of a site that doesn't read a source enters
// that source's product as 0 * value.  Lanes: 4 columns, sources 4 ks + e of
// every tile.
template <bool ACC>
__device__ __forceinline__ void wide_dv_prefixes(const WideBwdArgs &b, int64_t n,
                                              const uint16_t *ahi, const uint16_t *alo,
                                              const float *ck, int c0, int ks)
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
            const float w = load_elem(ahi + i * kOpRow + j) + load_elem(alo + i * kOpRow + j);
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

template <int MT, bool ACC>
__global__ __launch_bounds__(kBlock, 2) void route_all_bwd_wide(WideBwdArgs b)
{
    constexpr int KG = (MT + 1) / 2;  // groups of 32 sites in the contractions over sites
    // The exchange of the products, then the operands of the value gradient.
    constexpr int kOp = kAllMaxSources * kOpRow;
    __shared__ __align__(16)
        unsigned char lds[std::max<int>(wide_exchange_bytes<MT>(), 4 * kOp * sizeof(uint16_t))];
    uint16_t *const ahi = reinterpret_cast<uint16_t *>(lds), *const alo = ahi + kOp;
    uint16_t *const chi = alo + kOp, *const clo = chi + kOp;
    __shared__ float rho[kAllMaxSources], ck[kAllMaxSources], part[kWaves * kAllMaxSources];
    const AllArgs &a = b.f;
    const int64_t n = blockIdx.x;
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
            // Four consecutive sites of source i: one 8-byte write per array.
            u32x2_t h, l;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                h[k] = pack_bf16x2(al[nt][2 * k], al[nt][2 * k + 1]);
                l[k] = pack_bf16x2(al[nt][2 * k] - bf16_lo(h[k]), al[nt][2 * k + 1] - bf16_hi(h[k]));
            }
            const int o = i * kOpRow + 16 * wave + 4 * ks;
            *reinterpret_cast<u32x2_t *>(ahi + o) = h;
            *reinterpret_cast<u32x2_t *>(alo + o) = l;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                h[k] = pack_bf16x2(cq[nt][2 * k], cq[nt][2 * k + 1]);
                l[k] = pack_bf16x2(cq[nt][2 * k] - bf16_lo(h[k]), cq[nt][2 * k + 1] - bf16_hi(h[k]));
            }
            *reinterpret_cast<u32x2_t *>(chi + o) = h;
            *reinterpret_cast<u32x2_t *>(clo + o) = l;
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
                bf16x8_t B[4], Qh[4], Ql[4];
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
                        split2(v, Qh[p], Ql[p]);
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
                    const bf16x8_t Ah = *reinterpret_cast<const bf16x8_t *>(ahi + o);
                    const bf16x8_t Al = *reinterpret_cast<const bf16x8_t *>(alo + o);
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        acc[nt][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Al, B[p], acc[nt][p], 0, 0, 0);
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        acc[nt][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ah, B[p], acc[nt][p], 0, 0, 0);
                    if (KEY) {
                        const bf16x8_t Ch = *reinterpret_cast<const bf16x8_t *>(chi + o);
                        const bf16x8_t Cl = *reinterpret_cast<const bf16x8_t *>(clo + o);
#pragma unroll
                        for (int p = 0; p < 4; ++p)
                            acc[nt][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Cl, Qh[p], acc[nt][p], 0, 0, 0);
#pragma unroll
                        for (int p = 0; p < 4; ++p)
                            acc[nt][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ch, Ql[p], acc[nt][p], 0, 0, 0);
#pragma unroll
                        for (int p = 0; p < 4; ++p)
                            acc[nt][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ch, Qh[p], acc[nt][p], 0, 0, 0);
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
                wide_dv_prefixes<ACC>(b, n, ahi, alo, ck, c0, ks);
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

// dQ shares.  Wave `id` of the grid's y dimension sums
//     share[j][c] = sum_n sum_i cq[n][j][i] k[n][i][c]
// over its tokens n = id, id + waves, ... in order, for the 128 key columns
// of slab blockIdx.x, on the fp32 matrix cores: a lane's 16-byte row pieces,
// widened, are the operands as they stand (16 sources a group, four a step,
// lane group ks taking sources 4 ks .. 4 ks + 3 of the group, so that its cq
// come as one 16-byte vector).  The bf16 matrix cores with cq as three terms
// took 27 us against 34 (49 sources, 48 sites, r = 256, 2048 tokens), but
// their sums are biased: the error of dQ grew with the tokens, from 1.8e-7 to
// 3.4e-7 at 2048, where these reach 2.4e-7 (site by site: 2.1e-7).  The 4
// waves of a workgroup then add up in wave order.
struct WideDqArgs {
    const uint16_t *V;  // [S][N][d]
    const float *cq;    // [N][T][64]
    float *partial;     // [gridDim.y][T][r]
    int S, d, r, first, T;
    int64_t N;
};

// The same share over each site's prefix only, on the vector units (a
// non-finite source value past a site's prefix met cq = 0).
__device__ __forceinline__ void wide_dq_prefix(const WideDqArgs &a, int64_t n0, int64_t step,
                                            int site, int c, float (&v)[8])
{
#pragma unroll
    for (int p = 0; p < 8; ++p)
        v[p] = 0.0f;
    const size_t plane = (size_t)a.N * a.d;
#pragma unroll 1
    for (int64_t n = n0; n < a.N; n += step)
#pragma unroll 1
        for (int i = 0; i < min(a.S, a.first + site); ++i) {
            const float w = a.cq[((size_t)n * a.T + site) * kAllMaxSources + i];
            float x[8];
            widen(load_raw<uint16_t, 8>(a.V + i * plane + n * a.d + (a.d - a.r) + c), x);
#pragma unroll
            for (int p = 0; p < 8; ++p)
                v[p] = fmaf(w, x[p], v[p]);
        }
}

template <int MT>
__global__ __launch_bounds__(kBlock, 2) void wide_dq(WideDqArgs a)
{
    __shared__ __align__(16) float red[16 * kAllSlab * (kWaves - 1)];
    const int lane = threadIdx.x % kWaveSize;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const int lc = lane & 15, ks = lane >> 4;
    const int c0 = blockIdx.x * kAllSlab + 8 * lc;
    const bool ok = c0 < a.r;
    const size_t plane = (size_t)a.N * a.d;
    const uint16_t *key = a.V + (a.d - a.r) + (ok ? c0 : 0);
    const int64_t n0 = (int64_t)blockIdx.y * kWaves + wave, step = (int64_t)gridDim.y * kWaves;
    const int ngroups = (a.S + 15) / 16;
    f32x4_t acc[MT][8];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int p = 0; p < 8; ++p)
            acc[mt][p] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    u32x4_t raw[4];
    f32x4_t q[MT];
    auto load = [&](int64_t n, int g) {
        // Sources past S re-read the last one; their cq is 0.  Sites past T
        // re-read the last one; their rows are not stored.
        const uint16_t *r0 = key + n * a.d;
        int s0 = 16 * g + 4 * ks;
        asm volatile("" : "+v"(s0));
#pragma unroll
        for (int e = 0; e < 4; ++e)
            raw[e] = load_raw<uint16_t, 8>(r0 + (unsigned)min(s0 + e, a.S - 1) * plane);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            q[mt] = *reinterpret_cast<const f32x4_t *>(
                a.cq + ((size_t)n * a.T + min(16 * mt + lc, a.T - 1)) * kAllMaxSources + 16 * g + 4 * ks);
    };
    if (n0 < a.N)
        load(n0, 0);
    for (int64_t n = n0; n < a.N; n += step)
        for (int g = 0; g < ngroups; ++g) {
            u32x4_t now[4];
            f32x4_t w[MT];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                now[e] = raw[e];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                w[mt] = q[mt];
            // The next group, or the next token's first (the last again at
            // the end).
            const bool more = g + 1 < ngroups;
            load(more ? n : n + step < a.N ? n + step : n, more ? g + 1 : 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float x[8];
                widen(now[e], x);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    if (16 * g >= a.first + 16 * mt + 15)
                        continue;  // wave-uniform: no site of the tile reads the group
#pragma unroll
                    for (int p = 0; p < 8; ++p)
                        acc[mt][p] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[mt][e], x[p], acc[mt][p], 0, 0, 0);
                }
            }
        }
    // Lane: sites 16 mt + 4 ks + e, columns c0 .. c0 + 7; one site tile of
    // every wave meets in LDS at a time.
    float *part = a.partial + (size_t)blockIdx.y * a.T * a.r;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        float v[4][8];
        float bad = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int p = 0; p < 8; ++p) {
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
            for (int e = 0; e < 4; ++e) {
                float *dst = red + ((wave - 1) * 16 + 4 * ks + e) * kAllSlab + 8 * lc;
                *reinterpret_cast<f32x4_t *>(dst) = f32x4_t{v[e][0], v[e][1], v[e][2], v[e][3]};
                *reinterpret_cast<f32x4_t *>(dst + 4) = f32x4_t{v[e][4], v[e][5], v[e][6], v[e][7]};
            }
        __syncthreads();
        if (wave == 0 && ok)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int site = 16 * mt + 4 * ks + e;
                if (site >= a.T)
                    continue;
#pragma unroll
                for (int w = 0; w < kWaves - 1; ++w) {
                    const float *src = red + (w * 16 + 4 * ks + e) * kAllSlab + 8 * lc;
#pragma unroll
                    for (int p = 0; p < 8; ++p)
                        v[e][p] += src[p];
                }
                float *dst = part + (size_t)site * a.r + c0;
                *reinterpret_cast<f32x4_t *>(dst) = f32x4_t{v[e][0], v[e][1], v[e][2], v[e][3]};
                *reinterpret_cast<f32x4_t *>(dst + 4) = f32x4_t{v[e][4], v[e][5], v[e][6], v[e][7]};
            }
        __syncthreads();
    }
}

// dQ[x] (+)= the shares of element x: a workgroup takes 64 elements, its wave
// w the w-th quarter of the shares, eight interleaved chains of them, summed
// pairwise, and the quarters add up in order (coalesced over the elements;
// long chains of fp32 additions would lose a bit that the shares still have;
// zeros without tokens).
template <bool ACC>
__global__ __launch_bounds__(kBlock) void wide_dq_sum(const float *__restrict__ partial,
                                                      float *__restrict__ dQ, int shares, int n)
{
    __shared__ float red[kWaves][kWaveSize];
    const int lane = threadIdx.x % kWaveSize, wave = threadIdx.x / kWaveSize;
    const int x = blockIdx.x * kWaveSize + lane;
    const int per = (shares + kWaves - 1) / kWaves;
    const int beg = wave * per, end = min(shares, beg + per);
    float s[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
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
        const float t = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
        dQ[x] = ACC ? dQ[x] + t : t;
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

// Token shares of wide_dq: about two workgroups per CU over all key slabs,
// at least one token per wave.  Depends on N and r only (not on the sites or
// sources), so that the order of every dQ sum does too.
int64_t wide_shares(int64_t N, int64_t r)
{
    const int64_t nslab = (r + kAllSlab - 1) / kAllSlab;
    return std::max<int64_t>(1, std::min<int64_t>(512 / nslab, (N + kWaves - 1) / kWaves));
}

}  // namespace

// cq, then the dQ shares, from a 16-byte boundary of the workspace on.
size_t wide_bwd_workspace_bytes(int64_t N, int64_t T, int64_t r)
{
    return 16 + ((size_t)N * T * kAllMaxSources + (size_t)wide_shares(N, r) * T * r) * sizeof(float);
}

int launch_wide_bwd(const AllProblem &p, const void *dH, void *dV, float *dQ, void *ws,
                    bool accumulate, hipStream_t st, std::string *err)
{
    const int64_t shares = wide_shares(p.N, p.r);
    float *cq = reinterpret_cast<float *>((reinterpret_cast<uintptr_t>(ws) + 15) / 16 * 16);
    float *partial = cq + (size_t)p.N * p.T * kAllMaxSources;
    if (p.N > 0) {
        WideBwdArgs b;
        b.f = all_wide_args(p);
        b.f.H = nullptr;
        b.f.neff = nullptr;
        b.sources = (int)p.S;
        b.dH = static_cast<const uint16_t *>(dH);
        b.dV = static_cast<uint16_t *>(dV);
        b.cq = cq;
        const WideDqArgs q{static_cast<const uint16_t *>(p.V), cq, partial, b.f.S, (int)p.d,
                           (int)p.r, b.f.first, b.f.T, p.N};
        const dim3 qgrid((unsigned)((p.r + kAllSlab - 1) / kAllSlab), (unsigned)shares);
        switch ((b.f.T + 15) / 16) {
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
