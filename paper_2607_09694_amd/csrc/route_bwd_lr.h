// The backward of projected and sliced keys (the gradient of Sec. 3.2 Eqs.
// lr_key_norm, lr_attnres_weight, lr_attnres_output): kernel and launch
// template, shared by the translation units that instantiate its forms.
// Internal to the library.
#pragma once

#include "route_common.h"

namespace lrar {

// ---------------------------------------------------------------------------
// Backward kernels (gradient of L = sum_n dH[n] . h[n]; see the header)
// ---------------------------------------------------------------------------

// Key-pass geometry of the projected / sliced backward.  The key pass covers
// `ncols` columns per source: projected keys, the r key columns; sliced keys,
// the value columns from the vector-aligned tail start to d (the tail dV is
// written only here, with the key gradient added).  They are `nkv` vectors of
// KV elements.  A lane owns one vector slot v of one source of a group of
// 64 / LPS sources (LPS = lanes per source, a power of two), so its dq
// partial always belongs to the same columns; rows wider than 64 vectors are
// covered in chunks of 64.
template <int KV> struct KeyChunks { static constexpr int value = KV == 8 ? 1 : KV == 4 ? 2 : 4; };

// Projected / sliced keys.  Each token wave:
//   recomputes s, rho, alpha;  streams the S rows once, forming the partial
//   dots g_i = dH . o_i (one batched reduction per 8 sources) and writing
//   dV_i = alpha_i dH for every column before the key tail;
//   forms ds_i = alpha_i (g_i - sum_l alpha_l g_l);
//   then, lanes over (source, key vector), writes dK (projected) or the last
//   columns of dV including the key gradient (sliced), and accumulates dq.
// dq is reduced per workgroup in a fixed order into partial[blockIdx.x][r].
// T is the storage of V, K, dV and dK; TH that of dH (the same except for
// block sources, whose fp32 summary slots meet the model's bf16 gradient).
// DEFER (block sources, deferred form): only the last source (the block in
// progress) receives gradients, added into the single rows dV [N][d] and
// dK [N][r]; for every other source i the wave writes the three per-token
// coefficients of its gradient instead,
//     coef[i][0][n] = alpha_i,  coef[i][1][n] = ds_i / rho_i,
//     coef[i][2][n] = ds_i s_i / (rho_i r),
// from which dV_i = alpha_i dH + (key columns) coef1 q - coef2 kbar_i.  The
// site's member then retires in the same pass (DeferOut): its gradient is
// the new running row (dO, dK in the model dtype), and it leaves the slot
// (Bp -= o_new, KBp -= k_new) once the slot row has been read for the last
// time (the key columns after the key pass).
// SPLIT (few tokens): one token per workgroup, its sources cut into kWaves
// ranges, one per wave.  A wave scores, streams and differentiates its own
// range; the scores and the value dots of all of them meet in LDS, and every
// wave takes the softmax and its mean over all sources by itself.  The chain of
// dependent loads per wave, which bounds a launch with few tokens, is a
// quarter as long, with more rows of it in flight.
// DALL (every source deferred): the coefficients of every source, the last
// one included, are written, and no gradient row at all; each source's
// gradient is then gathered once from the sites that read it (the
// full-source reverse pass).
struct DeferOut {
    float *coef;
    const void *o_new, *k_new;  // model dtype
    void *dO, *dK;              // model dtype
    float *Bp, *KBp;            // the slot of the block in progress
};

template <typename T, typename TH, int VEC, int NCH, bool FULLCOLS, int KV, bool ACC,
          bool DEFER = false, bool DALL = false, bool SPLIT = false>
__global__ void __launch_bounds__(kBlock)
route_bwd_lr(const T *__restrict__ V, const T *__restrict__ keys, const float *__restrict__ q,
             const TH *__restrict__ dH, T *__restrict__ dV, T *__restrict__ dK,
             float *__restrict__ partial, int S, int N, int d, int r, int krow, int koff,
             int sliced, int tail_start, float eps, int s_pad, int r_pad, int tpw, int lps,
             DeferOut dfo = DeferOut{})
{
    float *__restrict__ coef = dfo.coef;
    extern __shared__ float lds[];
    const int lane = threadIdx.x & (kWaveSize - 1);
    // wave-uniform (scalar): the stream's buffer descriptors depend on it
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    // Per wave, or (SPLIT) s, rho and g of the workgroup, a wave's own alpha.
    const int slice = SPLIT ? 0 : 4 * wave;
    float *s = lds + (slice + 0) * s_pad;
    float *rho = lds + (slice + 1) * s_pad;
    float *g = lds + (slice + 2) * s_pad;
    float *alpha = lds + (slice + 3 + (SPLIT ? wave : 0)) * s_pad;
    float *stage = lds + 4 * kWaves * s_pad;  // [kWaves][r_pad]
    // The wave's sources.
    const int per = SPLIT ? (S + kWaves - 1) / kWaves : S;
    const int ib = SPLIT ? min(S, wave * per) : 0, ie = SPLIT ? min(S, ib + per) : S;
    auto meet = [&]() {  // the LDS writes above are visible to every reader below
        if constexpr (SPLIT)
            __syncthreads();
        else
            wave_lds_sync();
    };

    constexpr int KC = KeyChunks<KV>::value;
    const int kbase = sliced ? tail_start : 0;   // first column of the key pass
    const int kshift = sliced ? d - r : 0;       // column of key element 0
    const int nkv = (sliced ? d - tail_start : r) / KV;
    const int isub = lane / lps;                 // source within a group
    const int spi = kWaveSize / lps;             // sources per group
    const int vl = lane % lps;
    const float inv_r = 1.0f / (float)r;

    // Per-lane key-pass constants: q at the lane's key columns.
    float qk[KC][KV], dq_acc[KC][KV];
#pragma unroll
    for (int k = 0; k < KC; ++k)
#pragma unroll
        for (int e = 0; e < KV; ++e) {
            const int v = k * kWaveSize + vl;
            const int j = kbase + v * KV + e - kshift;
            qk[k][e] = (v < nkv && j >= 0) ? q[j] : 0.0f;
            dq_acc[k][e] = 0.0f;
        }

    const int col = lane * VEC;
    bool ok[NCH], wr[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        ok[c] = col + c * kWaveSize * VEC < d;
        wr[c] = col + c * kWaveSize * VEC < tail_start;
    }
    const size_t plane = (size_t)N * d;

    const int bx = blockIdx.x;
    for (int t = 0; t < tpw; ++t) {
        // (SPLIT: tpw = 1, one token of the grid's N per workgroup.)
        const int n = SPLIT ? bx : (bx * tpw + t) * kWaves + wave;
        if (n >= N)
            break;  // wave-uniform; the workgroup barrier below is outside the loop
        if (ie > ib)
            lr_scores<T, VEC, std::is_same<T, float>::value>(keys + (size_t)ib * N * krow, q,
                                                              ie - ib, N, r, krow, koff, eps, n,
                                                              lane, s + ib, rho + ib);
        if constexpr (SPLIT)
            meet();
        depth_softmax<std::is_same<T, float>::value>(s, alpha, S, lane);

        typedef typename Raw<T, VEC>::type raw_t;
        float dh[NCH][VEC];
        const TH *dhrow = dH + (size_t)n * d + col;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if (FULLCOLS || ok[c]) {
                widen(load_raw<TH, VEC>(dhrow + c * kWaveSize * VEC), dh[c]);
            } else {
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    dh[c][e] = 0.0f;
            }
        }
        const T *vbase = V + (size_t)n * d + col;
        T *dvbase = dV + (size_t)n * d + col;
        constexpr int L = SPLIT ? BwdInflightSplit<NCH>::value : BwdInflight<NCH>::value;
        // With 16-byte vectors every access of the stream goes through a
        // per-row buffer resource: source i's value row (no bytes past the
        // last source) and its gradient row (bytes up to the key tail, none
        // when the source takes no gradient row here).  Lanes past the row
        // end and sources past S read zeros and store nothing, with no branch
        // around any access, so the compiler's wait counts let the stores and
        // the next loads stay in flight.  Scalar rows keep guarded accesses.
        constexpr bool BUF = VEC > 1;
        for (int i0 = ib; i0 < ie; i0 += 8) {
            float part[8];
#pragma unroll
            for (int h = 0; h < 8; h += L) {
                raw_t raw[L][NCH], old[ACC ? L : 1][NCH];
                __amdgpu_buffer_rsrc_t rv[L], rd[L];
#pragma unroll
                for (int u = 0; u < L; ++u) {
                    const int i = i0 + h + u;
                    const bool live = i < ie;
                    const bool takes = live && (!DEFER || (!DALL && i == S - 1));
                    if constexpr (BUF) {
                        const size_t ic = (size_t)min(i, S - 1);  // in-range base
                        rv[u] = row_rsrc(V + (ic * N + n) * d, live ? d * (int)sizeof(T) : 0);
                        // every source of a fully deferred step takes no row (dV may be NULL)
                        rd[u] = row_rsrc(DALL ? nullptr : dV + (DEFER ? (size_t)n : ic * N + n) * d,
                                         takes ? tail_start * (int)sizeof(T) : 0);
#pragma unroll
                        for (int c = 0; c < NCH; ++c) {
                            const int off = (col + c * kWaveSize * VEC) * (int)sizeof(T);
                            raw[u][c] = buffer_load16<T, VEC, kBwdNtLoad>(rv[u], off);
                            if constexpr (ACC)
                                old[u][c] = buffer_load16<T, VEC, kBwdNtLoad>(rd[u], off);
                        }
                    } else if (live) {
#pragma unroll
                        for (int c = 0; c < NCH; ++c)
                            if (FULLCOLS || ok[c]) {
                                const size_t off = (size_t)i * plane + c * kWaveSize * VEC;
                                raw[u][c] = load_stream<T, VEC, kNtLoad>(vbase + off);
                                if constexpr (ACC)
                                    if (wr[c] && takes)
                                        old[u][c] = load_stream<T, VEC, kNtLoad>(
                                            dvbase + (DEFER ? c * kWaveSize * VEC : off));
                            }
                    }
                }
#pragma unroll
                for (int u = 0; u < L; ++u) {
                    float p = 0.0f;
                    const int i = i0 + h + u;
                    if (BUF || i < ie) {
                        const float a = i < ie ? alpha[min(i, S - 1)] : 0.0f;
#pragma unroll
                        for (int c = 0; c < NCH; ++c) {
                            if (BUF || FULLCOLS || ok[c]) {
                                float x[VEC], y[VEC];
                                widen(raw[u][c], x);
#pragma unroll
                                for (int e = 0; e < VEC; ++e) {
                                    p = fmaf(dh[c][e], x[e], p);
                                    y[e] = a * dh[c][e];
                                }
                                const bool wdv = wr[c] && i < ie && (!DEFER || (!DALL && i == S - 1));
                                if constexpr (BUF) {
                                    if constexpr (ACC)
                                        add_stored(y, old[u][c]);
                                    buffer_store16<T, VEC, kBwdNtStore>(
                                        rd[u], (col + c * kWaveSize * VEC) * (int)sizeof(T),
                                        Narrow<T, VEC>::run(y));
                                } else {
                                    if constexpr (ACC)
                                        if (wdv)
                                            add_stored(y, old[u][c]);
                                    if (wdv)
                                        store_stream<T, VEC, kNtStore>(
                                            dvbase + (DEFER ? 0 : (size_t)i * plane) + c * kWaveSize * VEC,
                                            Narrow<T, VEC>::run(y));
                                }
                                if constexpr (DEFER && !DALL) {
                                    if (wdv) {
                                        // retire: dO = the new running row;
                                        // the member leaves the slot
                                        const size_t ro = (size_t)n * d + col + c * kWaveSize * VEC;
                                        store_stream<TH, VEC, kNtStore>(
                                            static_cast<TH *>(dfo.dO) + ro, Narrow<TH, VEC>::run(y));
                                        float o[VEC];
                                        widen(load_raw<TH, VEC>(static_cast<const TH *>(dfo.o_new) + ro), o);
#pragma unroll
                                        for (int e = 0; e < VEC; ++e)
                                            x[e] -= o[e];
                                        store_raw<float, VEC>(dfo.Bp + ro, Narrow<float, VEC>::run(x));
                                    }
                                }
                            }
                        }
                    }
                    part[h + u] = p;
                }
                // One step of L sources at a time: the dots of this step are
                // formed before the next step's loads go out, so at most one
                // step's rows are in flight per wave.
#pragma unroll
                for (int u = 0; u < L; ++u)
                    asm volatile("" : "+v"(part[h + u])::"memory");
            }
            const float tot = multi_sum<8>(part, lane);
            const int idx = multi_sum_index<8>(lane);
            if (multi_sum_writer<8>(lane) && i0 + idx < ie)
                g[i0 + idx] = tot;
        }
        meet();
        float gb = 0.0f;
        for (int i = lane; i < S; i += kWaveSize)
            gb = fmaf(alpha[i], g[i], gb);
        gb = wave_sum_t<std::is_same<T, float>::value>(gb);
        if constexpr (SPLIT)
            meet();  // every wave has read the dots
        for (int i = ib + lane; i < ie; i += kWaveSize)
            g[i] = alpha[i] * (g[i] - gb);  // g now holds ds
        wave_lds_sync();

        // Key pass: lanes over (source, key vector).
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const int v = k * kWaveSize + vl;
            if (k * kWaveSize >= nkv)
                break;  // wave-uniform
            const bool vok = v < nkv;
            const int c0 = kbase + v * KV;  // projected: key index; sliced: value column
            float dhk[KV];
            if (sliced && vok) {
                widen(load_raw<TH, KV>(dH + (size_t)n * d + c0), dhk);
            } else {
#pragma unroll
                for (int e = 0; e < KV; ++e)
                    dhk[e] = 0.0f;
            }
#pragma unroll 4
            for (int i0 = ib; i0 < ie; i0 += spi) {
                const int i = i0 + isub;
                if (!vok || i >= ie)
                    continue;
                const size_t row = (size_t)i * N + n;
                const float ri = 1.0f / rho[i];
                const float dsi = g[i];
                const float cq = dsi * ri;              // ds_i / rho_i
                const float ck = cq * s[i] * inv_r;     // ds_i s_i / (rho_i r)
                const bool defer_i = DEFER && (DALL || i < S - 1);
                const size_t orow = DEFER ? (size_t)n : row;  // output row of source i
                if (defer_i && k == 0 && vl == 0) {
                    coef[((size_t)i * 3 + 0) * N + n] = alpha[i];
                    coef[((size_t)i * 3 + 1) * N + n] = cq;
                    coef[((size_t)i * 3 + 2) * N + n] = ck;
                }
                float x[KV], y[KV];
                if (!sliced) {
                    widen(load_raw<T, KV>(keys + row * krow + c0), x);
#pragma unroll
                    for (int e = 0; e < KV; ++e) {
                        const float kb = x[e] * ri;
                        y[e] = fmaf(cq, qk[k][e], -ck * kb);
                        dq_acc[k][e] = fmaf(dsi, kb, dq_acc[k][e]);
                    }
                    if (defer_i)
                        continue;
                    if constexpr (ACC)
                        add_stored(y, load_raw<T, KV>(dK + orow * r + c0));
                    store_raw<T, KV>(dK + orow * r + c0, Narrow<T, KV>::run(y));
                    if constexpr (DEFER && !DALL) {
                        // retire the member's key: dK = the new running key
                        // row; the key leaves the slot's key summary
                        const size_t ro = (size_t)n * r + c0;
#pragma unroll
                        for (int e = 0; e < KV; ++e) {
                            store_elem(static_cast<TH *>(dfo.dK) + ro + e, y[e]);
                            dfo.KBp[ro + e] =
                                x[e] - load_elem(static_cast<const TH *>(dfo.k_new) + ro + e);
                        }
                    }
                } else {
                    widen(load_raw<T, KV>(V + row * d + c0), x);
                    const float a = alpha[i];
#pragma unroll
                    for (int e = 0; e < KV; ++e) {
                        y[e] = a * dhk[e];
                        if (c0 + e >= kshift) {
                            const float kb = x[e] * ri;
                            y[e] += fmaf(cq, qk[k][e], -ck * kb);
                            dq_acc[k][e] = fmaf(dsi, kb, dq_acc[k][e]);
                        }
                    }
                    if (defer_i)
                        continue;
                    if constexpr (ACC)
                        add_stored(y, load_raw<T, KV>(dV + orow * d + c0));
                    store_raw<T, KV>(dV + orow * d + c0, Narrow<T, KV>::run(y));
                    if constexpr (DEFER && !DALL) {
                        // retire the member's columns of the key pass: its
                        // gradient, and the slot without it (the slot row
                        // was read here for the last time)
                        const size_t ro = (size_t)n * d + c0;
#pragma unroll
                        for (int e = 0; e < KV; ++e) {
                            store_elem(static_cast<TH *>(dfo.dO) + ro + e, y[e]);
                            dfo.Bp[ro + e] =
                                x[e] - load_elem(static_cast<const TH *>(dfo.o_new) + ro + e);
                        }
                    }
                }
            }
        }
        wave_lds_sync();  // LDS of this token is reused by the next one
    }

    // Fixed-order reduction of dq: over the source groups of the wave
    // (butterfly over the lane bits above the vector slot), then over the
    // waves of the workgroup in wave order.
#pragma unroll
    for (int k = 0; k < KC; ++k)
#pragma unroll
        for (int e = 0; e < KV; ++e)
            for (int m = lps; m < kWaveSize; m <<= 1)
                dq_acc[k][e] += __shfl_xor(dq_acc[k][e], m, kWaveSize);
    float *my = stage + wave * r_pad;
    for (int j = lane; j < r; j += kWaveSize)
        my[j] = 0.0f;
    wave_lds_sync();
    if (isub == 0) {
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const int v = k * kWaveSize + vl;
            if (v < nkv) {
#pragma unroll
                for (int e = 0; e < KV; ++e) {
                    const int j = kbase + v * KV + e - kshift;
                    if (j >= 0)
                        my[j] = dq_acc[k][e];
                }
            }
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < r; j += kBlock) {
        float sum = 0.0f;
        for (int w = 0; w < kWaves; ++w)
            sum += stage[w * r_pad + j];
        partial[(size_t)bx * r + j] = sum;
    }
}

namespace {

// Key-pass vector width and lanes per source of the projected / sliced
// backward: 16-byte vectors when the key rows allow it, else scalars.
struct KeyPass {
    int kv, lps, nkv;
};

KeyPass key_pass(const Problem &p, const Plan &pl)
{
    const bool sliced = p.mode == LRAR_MODE_SLICED;
    const int tail_start = sliced ? (int)((p.d - p.r) / pl.vec * pl.vec) : (int)p.d;
    KeyPass k;
    k.kv = pl.vec > 1 && (sliced || p.r % pl.vec == 0) ? pl.vec : 1;
    k.nkv = (int)(sliced ? p.d - tail_start : p.r) / k.kv;
    k.lps = 1;
    while (k.lps < k.nkv && k.lps < kWaveSize)
        k.lps <<= 1;
    return k;
}

template <typename T, typename TH, int VEC, bool ACC, bool DEFER = false, bool DALL = false>
hipError_t launch_bwd_t(const Problem &p, const Plan &pl, const void *dH, void *dV, void *dK,
                        float *partial, hipStream_t st, const DeferOut &dfo = DeferOut{})
{
    const T *V = static_cast<const T *>(p.V);
    const int tail_start = p.mode == LRAR_MODE_SLICED ? (int)((p.d - p.r) / pl.vec * pl.vec)
                                                      : (int)p.d;
    const T *keys = p.mode == LRAR_MODE_PROJECTED ? static_cast<const T *>(p.K) : V;
    const int krow = p.mode == LRAR_MODE_PROJECTED ? (int)p.r : (int)p.d;
    const int koff = p.mode == LRAR_MODE_SLICED ? (int)(p.d - p.r) : 0;
    const KeyPass kp = key_pass(p, pl);
    // Block sources (mixed storage; their plans never split either) have too
    // few slots for it: 1.6 ms against 3.2 for a pass of 49 sites at 1024 tokens.
    constexpr bool kSplits = std::is_same<T, TH>::value && (!DEFER || DALL);
    return dispatch_chunks<VEC>(pl, [&](auto nch, auto fc) -> hipError_t {
        constexpr int NCH = decltype(nch)::value;
        constexpr bool FC = decltype(fc)::value;
        auto launch_as = [&](auto kvc, auto splitc) {
            constexpr int KV = decltype(kvc)::value;
            constexpr bool SPLIT = decltype(splitc)::value;
            hipLaunchKernelGGL((route_bwd_lr<T, TH, VEC, NCH, FC, KV, ACC, DEFER, DALL, SPLIT>),
                               dim3(pl.nblocks), dim3(kBlock), pl.lds, st, V, keys, p.q,
                               static_cast<const TH *>(dH), static_cast<T *>(dV),
                               static_cast<T *>(dK), partial, (int)p.S, (int)p.N, (int)p.d,
                               (int)p.r, krow, koff, p.mode == LRAR_MODE_SLICED ? 1 : 0,
                               tail_start, p.eps, pl.s_pad, pl.r_pad, pl.tpw, kp.lps, dfo);
        };
        auto launch = [&](auto kvc) {
            if constexpr (kSplits) {
                if (pl.wg_split)
                    return launch_as(kvc, std::true_type{});
            }
            launch_as(kvc, std::false_type{});
        };
        if constexpr (VEC > 1) {
            if (kp.kv == VEC)
                launch(std::integral_constant<int, VEC>{});
            else
                launch(std::integral_constant<int, 1>{});
        } else {
            launch(std::integral_constant<int, 1>{});
        }
        return hipGetLastError();
    });
}

}  // namespace

}  // namespace lrar
