// Backward kernels of the LR-AttnRes depth routing (the gradient of Sec. 3.2
// Eqs. lr_key_norm, lr_attnres_weight, lr_attnres_output), the fixed-order
// dq reduction, and their launcher.
#include "route_bwd_lr.h"

#include <mutex>

namespace lrar {

// Full-rank AttnRes backward: pass 1 reads the rows once for sum(o^2), q.o
// and dH.o (one batched reduction per 4 sources); pass 2 re-reads them to
// write dV_i = alpha_i dH + (ds_i/rho_i)(q - o_i s_i/(rho_i d)) and to
// accumulate dq = sum ds_i o_i / rho_i per lane column.
template <typename T, int VEC, int NCH, bool FULLCOLS, bool ACC>
__global__ void __launch_bounds__(kBlock)
route_bwd_full(const T *__restrict__ V, const float *__restrict__ q, const T *__restrict__ dH,
               T *__restrict__ dV, float *__restrict__ partial, int S, int N, int d, float eps,
               int s_pad, int tpw)
{
    extern __shared__ float lds[];
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x / kWaveSize;
    float *ss = lds + (4 * wave + 0) * s_pad;     // sum o^2, then rho
    float *sc = lds + (4 * wave + 1) * s_pad;     // q.o, then the score
    float *g = lds + (4 * wave + 2) * s_pad;      // dH.o, then ds
    float *alpha = lds + (4 * wave + 3) * s_pad;
    float *stage = lds + 4 * kWaves * s_pad;      // [d]

    const int col = lane * VEC;
    bool ok[NCH];
    float qv[NCH][VEC], dqa[NCH][VEC];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        ok[c] = col + c * kWaveSize * VEC < d;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            qv[c][e] = (FULLCOLS || ok[c]) ? q[col + c * kWaveSize * VEC + e] : 0.0f;
            dqa[c][e] = 0.0f;
        }
    }
    const size_t plane = (size_t)N * d;
    const float inv_d = 1.0f / (float)d;

    const int bx = blockIdx.x;
    for (int t = 0; t < tpw; ++t) {
        const int n = (bx * tpw + t) * kWaves + wave;
        if (n >= N)
            break;  // wave-uniform; the workgroup barriers are after the loop
        float dh[NCH][VEC];
        const T *vbase = V + (size_t)n * d + col;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if (FULLCOLS || ok[c]) {
                widen(load_raw<T, VEC>(dH + (size_t)n * d + col + c * kWaveSize * VEC), dh[c]);
            } else {
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    dh[c][e] = 0.0f;
            }
        }
        for (int i0 = 0; i0 < S; i0 += 4) {
            float part[16];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float a = 0.0f, b = 0.0f, p = 0.0f;
                if (i0 + u < S) {
#pragma unroll
                    for (int c = 0; c < NCH; ++c) {
                        if (FULLCOLS || ok[c]) {
                            float x[VEC];
                            widen(load_raw<T, VEC>(vbase + (size_t)(i0 + u) * plane +
                                                   c * kWaveSize * VEC), x);
#pragma unroll
                            for (int e = 0; e < VEC; ++e) {
                                a = fmaf(x[e], x[e], a);
                                b = fmaf(qv[c][e], x[e], b);
                                p = fmaf(dh[c][e], x[e], p);
                            }
                        }
                    }
                }
                part[u] = a;
                part[4 + u] = b;
                part[8 + u] = p;
                part[12 + u] = 0.0f;
            }
            const float tot = multi_sum<16>(part, lane);
            const int idx = multi_sum_index<16>(lane);
            const int i = i0 + (idx & 3);
            if (multi_sum_writer<16>(lane) && idx < 12 && i < S)
                (idx < 4 ? ss : idx < 8 ? sc : g)[i] = tot;
        }
        wave_lds_sync();
        for (int i = lane; i < S; i += kWaveSize) {
            const float rho = sqrtf(ss[i] / (float)d + eps);
            ss[i] = rho;
            sc[i] = sc[i] / rho;
        }
        depth_softmax(sc, alpha, S, lane);
        float gb = 0.0f;
        for (int i = lane; i < S; i += kWaveSize)
            gb = fmaf(alpha[i], g[i], gb);
        gb = wave_sum(gb);
        for (int i = lane; i < S; i += kWaveSize)
            g[i] = alpha[i] * (g[i] - gb);
        wave_lds_sync();

        T *dvbase = dV + (size_t)n * d + col;
        for (int i = 0; i < S; ++i) {
            const float a = alpha[i];
            const float c1 = g[i] / ss[i];                  // ds_i / rho_i
            const float c2 = c1 * sc[i] / ss[i] * inv_d;    // ds_i s_i / (rho_i^2 d)
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                if (FULLCOLS || ok[c]) {
                    float x[VEC], y[VEC];
                    widen(load_raw<T, VEC>(vbase + (size_t)i * plane + c * kWaveSize * VEC), x);
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        y[e] = fmaf(a, dh[c][e], fmaf(c1, qv[c][e], -c2 * x[e]));
                        dqa[c][e] = fmaf(c1, x[e], dqa[c][e]);
                    }
                    if constexpr (ACC)
                        add_stored(y, load_raw<T, VEC>(dvbase + (size_t)i * plane +
                                                       c * kWaveSize * VEC));
                    store_raw<T, VEC>(dvbase + (size_t)i * plane + c * kWaveSize * VEC,
                                      Narrow<T, VEC>::run(y));
                }
            }
        }
        wave_lds_sync();
    }

    // Fixed-order workgroup reduction of dq: waves add their columns in turn.
    for (int w = 0; w < kWaves; ++w) {
        if (wave == w) {
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                if (FULLCOLS || ok[c]) {
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        float *p = stage + col + c * kWaveSize * VEC + e;
                        *p = (w == 0 ? 0.0f : *p) + dqa[c][e];
                    }
                }
            }
        }
        __syncthreads();
    }
    for (int j = threadIdx.x; j < d; j += kBlock)
        partial[(size_t)bx * d + j] = stage[j];
}

// dq[j] = sum_b partial[b][j] in a fixed order: one workgroup per column;
// thread t sums rows t, t+256, ... in order, then a fixed pairwise tree over
// the 256 thread sums.  Writes zeros when nblocks = 0.  Bound by latency: four
// rows' loads are in flight together, and the tree's last six steps are one
// wave's lane exchanges.
template <bool ACC>
__global__ void __launch_bounds__(256)
dq_reduce(const float *__restrict__ partial, float *__restrict__ dq, int nblocks, int ncols)
{
    __shared__ float red[256];
    const int t = threadIdx.x;
    const int j = blockIdx.x;
    float s = 0.0f;
    for (int b = t; b < nblocks; b += 1024) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            v[u] = partial[(size_t)min(b + 256 * u, nblocks - 1) * ncols + j];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            s += b + 256 * u < nblocks ? v[u] : 0.0f;
    }
    red[t] = s;
    lds_barrier();
    if (t >= 64)
        return;
    s = (red[t] + red[t + 128]) + (red[t + 64] + red[t + 192]);
#pragma unroll
    for (int w = 32; w >= 1; w >>= 1)
        s += __shfl_down(s, w, kWaveSize);
    if (t == 0)
        dq[j] = ACC ? dq[j] + s : s;
}

hipError_t launch_dq_reduce(const float *partial, float *dq, int nblocks, int ncols,
                            bool accumulate, hipStream_t st)
{
    if (accumulate)
        hipLaunchKernelGGL(dq_reduce<true>, dim3(ncols), dim3(256), 0, st, partial, dq, nblocks,
                           ncols);
    else
        hipLaunchKernelGGL(dq_reduce<false>, dim3(ncols), dim3(256), 0, st, partial, dq, nblocks,
                           ncols);
    return hipGetLastError();
}

namespace {

template <typename T, int VEC, bool ACC>
hipError_t launch_bwd_full_t(const Problem &p, const Plan &pl, const void *dH, void *dV,
                             float *partial, hipStream_t st)
{
    return dispatch_chunks<VEC>(pl, [&](auto nch, auto fc) -> hipError_t {
        constexpr int NCH = decltype(nch)::value;
        constexpr bool FC = decltype(fc)::value;
        hipLaunchKernelGGL((route_bwd_full<T, VEC, NCH, FC, ACC>), dim3(pl.nblocks), dim3(kBlock),
                           pl.lds, st, static_cast<const T *>(p.V), p.q,
                           static_cast<const T *>(dH), static_cast<T *>(dV), partial, (int)p.S,
                           (int)p.N, (int)p.d, p.eps, pl.s_pad, pl.tpw);
        return hipGetLastError();
    });
}

// The routing backward (accumulating dV / dK when ACC) and the dq reduction
// (accumulating when ACCQ).  Mixed storage (fp32 values, bf16 dH) exists only
// for the accumulating form used by block sources.
template <bool ACC, bool ACCQ>
hipError_t launch_bwd_acc(const Problem &p, const Plan &pl, const void *dH, void *dV, void *dK,
                          float *dq, float *partial, hipStream_t st)
{
    hipError_t e = hipSuccess;
    if (p.N > 0) {
        const bool mixed = p.dtype == LRAR_DTYPE_F32 && p.dh_dtype == LRAR_DTYPE_BF16;
        if (p.mode == LRAR_MODE_FULL && p.dtype == LRAR_DTYPE_BF16)
            e = pl.vec > 1 ? launch_bwd_full_t<uint16_t, 8, ACC>(p, pl, dH, dV, partial, st)
                           : launch_bwd_full_t<uint16_t, 1, ACC>(p, pl, dH, dV, partial, st);
        else if (p.mode == LRAR_MODE_FULL)
            e = pl.vec > 1 ? launch_bwd_full_t<float, 4, ACC>(p, pl, dH, dV, partial, st)
                           : launch_bwd_full_t<float, 1, ACC>(p, pl, dH, dV, partial, st);
        else if (p.dtype == LRAR_DTYPE_BF16)
            e = pl.vec > 1 ? launch_bwd_t<uint16_t, uint16_t, 8, ACC>(p, pl, dH, dV, dK, partial, st)
                           : launch_bwd_t<uint16_t, uint16_t, 1, ACC>(p, pl, dH, dV, dK, partial, st);
        else if (!mixed)
            e = pl.vec > 1 ? launch_bwd_t<float, float, 4, ACC>(p, pl, dH, dV, dK, partial, st)
                           : launch_bwd_t<float, float, 1, ACC>(p, pl, dH, dV, dK, partial, st);
        else if constexpr (ACC)
            e = pl.vec > 1 ? launch_bwd_t<float, uint16_t, 4, ACC>(p, pl, dH, dV, dK, partial, st)
                           : launch_bwd_t<float, uint16_t, 1, ACC>(p, pl, dH, dV, dK, partial, st);
        else
            e = hipErrorInvalidValue;
        if (e != hipSuccess)
            return e;
    }
    const int ncols = (int)(p.mode == LRAR_MODE_FULL ? p.d : p.r);
    const int nb = p.N > 0 ? pl.nblocks : 0;
    hipLaunchKernelGGL(dq_reduce<ACCQ>, dim3(ncols), dim3(256), 0, st, partial, dq, nb, ncols);
    return hipGetLastError();
}

}  // namespace

int launch_bwd(const Problem &p, const void *dH, void *dV, void *dK, float *dq, void *ws,
               size_t ws_bytes, bool accumulate, hipStream_t st, std::string *err)
{
    Plan pl;
    if (!make_plan(p, true, &pl, err))
        return LRAR_EUNSUPPORTED;
    // One site of full-rank keys: the all-sites form for one (the same bits in
    // dq).  The rows are read once for the dots and dV and once more for dq, by
    // workgroups per token (step with its forward, 49 sources, d = 1024: 304 ->
    // 35 us at 64 tokens, 488 -> 353 at 4096).  Wider rows don't fit its
    // registers; there route_bwd_full is ahead from about 4000 tokens on (1292
    // against 1938 us at 50 sources, d = 2048, 8192 tokens).
    const AllProblem one{p.V, p.K, p.q, nullptr, nullptr, p.S, p.N, p.d, p.r, p.S, 1,
                         p.mode, p.dtype, p.eps};
    if (p.N > 0 && p.S > 1 && (accumulate ? full_rows_adding(p) : full_rows(p)) && all_wide(one))
        return launch_wide_bwd(one, dH, dV, dq, ws, ws_bytes, accumulate, st, err);
    float *partial = static_cast<float *>(ws);
    const hipError_t e =
        accumulate ? launch_bwd_acc<true, true>(p, pl, dH, dV, dK, dq, partial, st)
                   : launch_bwd_acc<false, false>(p, pl, dH, dV, dK, dq, partial, st);
    return hip_status(e, "route_bwd launch", err);
}

// Block sources, one site of the reverse pass: accumulate the slot gradients
// (fp32) from the model-dtype dH, write dq, then retire the site (the
// member's gradient is its slot's gradient so far; the member leaves its
// slot).
int launch_block_bwd(const Problem &p, const BlockRetire &br, const void *dH, void *dB,
                     void *dKB, float *dq, void *ws, hipStream_t st, std::string *err)
{
    Plan pl;
    if (!make_plan(p, true, &pl, err, false))
        return LRAR_EUNSUPPORTED;
    hipError_t e = launch_bwd_acc<true, false>(p, pl, dH, dB, dKB, dq, static_cast<float *>(ws),
                                               st);
    if (e == hipSuccess && p.N > 0)
        e = launch_block_retire(br, st);
    return hip_status(e, "block_route_bwd launch", err);
}

// ---------------------------------------------------------------------------
// Allocation-free backward: the dq partials in a file-scope device array
// ---------------------------------------------------------------------------

// The per-workgroup dq partials of lr_attnres_route_bwd_noalloc live here
// instead of in a caller workspace.  Every device the library runs on holds
// its own copy until the process ends; all calls on one device share it, and
// each launch overwrites the rows it later reads, so nothing has to start at
// zero.  Host code never passes this name to a kernel: it stands for a host
// shadow, and the device address comes from hipGetSymbolAddress.
static __device__ __align__(256) float scratch[kNoAllocScratchBytes / sizeof(float)];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
float *g_scratch_addr[kMaxDevices];

// Device address of `scratch` on device `dev`, looked up once per device
// with that device current.
int scratch_address(int dev, float **out, std::string *err)
{
    if (dev < 0 || dev >= kMaxDevices) {
        *err = "device index " + std::to_string(dev) + " beyond the allocation-free backward's " +
               std::to_string(kMaxDevices) + " devices";
        return LRAR_EUNSUPPORTED;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_addr[dev]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess)
            return hip_status(e, "hipGetDevice", err);
        if (cur != dev && (e = hipSetDevice(dev)) != hipSuccess)
            return hip_status(e, "hipSetDevice", err);
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != dev) {
            const hipError_t back = hipSetDevice(cur);
            if (e == hipSuccess)
                e = back;
        }
        if (e != hipSuccess)
            return hip_status(e, "hipGetSymbolAddress(scratch)", err);
        g_scratch_addr[dev] = static_cast<float *>(p);
    }
    *out = g_scratch_addr[dev];
    return LRAR_OK;
}

}  // namespace

int launch_bwd_noalloc(const Problem &p, const void *dH, void *dV, void *dK, float *dq,
                       hipStream_t st, std::string *err)
{
    const size_t need = bwd_partial_bytes(p);
    if (need > kNoAllocScratchBytes) {
        *err = "the allocation-free backward needs " + std::to_string(need) +
               " bytes of dq partials; its device array holds " +
               std::to_string(kNoAllocScratchBytes);
        return LRAR_EUNSUPPORTED;
    }
    int dev = -1;
    hipError_t e = st ? hipStreamGetDevice(st, &dev) : hipGetDevice(&dev);
    if (e != hipSuccess)
        return hip_status(e, st ? "hipStreamGetDevice" : "hipGetDevice", err);
    float *ws = nullptr;
    const int rc = scratch_address(dev, &ws, err);
    if (rc != LRAR_OK)
        return rc;
    return launch_bwd(p, dH, dV, dK, dq, ws, kNoAllocScratchBytes, false, st, err);
}

}  // namespace lrar
