// The deferred forms of the low-rank backward: per-site coefficients instead of
// gradient rows (route_bwd_lr's DEFER and DALL).
#include "route_bwd_lr.h"

namespace lrar {

int launch_block_bwd_deferred(const Problem &p, const BlockRetire &br, const void *dH, float *dP,
                              float *dKP, float *coef, float *dq, void *ws, hipStream_t st,
                              std::string *err)
{
    Plan pl;
    if (!make_plan(p, true, &pl, err, false))
        return LRAR_EUNSUPPORTED;
    float *partial = static_cast<float *>(ws);
    // The retire step runs inside the backward kernel (DeferOut).
    const size_t plane = (size_t)p.N * p.d, kplane = (size_t)p.N * p.r;
    DeferOut dfo;
    dfo.coef = coef;
    dfo.o_new = br.o_new;
    dfo.k_new = br.k_new;
    dfo.dO = br.dO;
    dfo.dK = br.dK;
    dfo.Bp = br.B + br.j * plane;
    dfo.KBp = br.KB ? br.KB + br.j * kplane : nullptr;
    hipError_t e = hipSuccess;
    if (p.N > 0) {
        if (p.dh_dtype == LRAR_DTYPE_BF16)
            e = pl.vec > 1
                    ? launch_bwd_t<float, uint16_t, 4, true, true>(p, pl, dH, dP, dKP, partial, st, dfo)
                    : launch_bwd_t<float, uint16_t, 1, true, true>(p, pl, dH, dP, dKP, partial, st, dfo);
        else
            e = pl.vec > 1
                    ? launch_bwd_t<float, float, 4, true, true>(p, pl, dH, dP, dKP, partial, st, dfo)
                    : launch_bwd_t<float, float, 1, true, true>(p, pl, dH, dP, dKP, partial, st, dfo);
    }
    if (e == hipSuccess) {
        const int ncols = (int)p.r;
        e = launch_dq_reduce(partial, dq, p.N > 0 ? pl.nblocks : 0, ncols, false, st);
    }
    return hip_status(e, "block_route_bwd_deferred launch", err);
}

int launch_bwd_deferred_all(const Problem &p, const void *dH, float *coef, float *dq, void *ws,
                            hipStream_t st, std::string *err)
{
    if (p.mode == LRAR_MODE_FULL) {
        *err = "the deferred backward takes projected or sliced keys";
        return LRAR_EUNSUPPORTED;
    }
    Plan pl;
    if (!make_plan(p, true, &pl, err))
        return LRAR_EUNSUPPORTED;
    float *partial = static_cast<float *>(ws);
    DeferOut dfo;
    dfo.coef = coef;
    hipError_t e = hipSuccess;
    if (p.N > 0) {
        if (p.dtype == LRAR_DTYPE_BF16)
            e = pl.vec > 1 ? launch_bwd_t<uint16_t, uint16_t, 8, false, true, true>(
                                 p, pl, dH, nullptr, nullptr, partial, st, dfo)
                           : launch_bwd_t<uint16_t, uint16_t, 1, false, true, true>(
                                 p, pl, dH, nullptr, nullptr, partial, st, dfo);
        else
            e = pl.vec > 1 ? launch_bwd_t<float, float, 4, false, true, true>(
                                 p, pl, dH, nullptr, nullptr, partial, st, dfo)
                           : launch_bwd_t<float, float, 1, false, true, true>(
                                 p, pl, dH, nullptr, nullptr, partial, st, dfo);
    }
    if (e == hipSuccess)
        e = launch_dq_reduce(partial, dq, p.N > 0 ? pl.nblocks : 0, (int)p.r, false, st);
    return hip_status(e, "route_bwd_deferred launch", err);
}

}  // namespace lrar
