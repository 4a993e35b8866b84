// Launch plans of the routing kernels: which kernel instance, grid and LDS
// size serve a validated problem, and the limits beyond which none does.
// Host code only.
#include "route_common.h"

#include <algorithm>

namespace lrar {

namespace {

constexpr int kMaxSourcesFwd = 1024;
constexpr int kMaxSourcesBwd = 512;
constexpr int kMaxRankBwd = 256;

// Token counts up to which the forward splits each token's sources over the
// four waves of a workgroup (measured on MI355X at 49 sources, d = 1024: the
// split is ahead up to these counts, level with or behind one wave per token
// above them).  LRAR_WG_SPLIT_MAX_TOKENS overrides both.
#ifdef LRAR_WG_SPLIT_MAX_TOKENS
constexpr int64_t kWgSplitLowRank = LRAR_WG_SPLIT_MAX_TOKENS;
constexpr int64_t kWgSplitFull = LRAR_WG_SPLIT_MAX_TOKENS;
#else
constexpr int64_t kWgSplitLowRank = 2048;
constexpr int64_t kWgSplitFull = 1024;
#endif

// Tokens up to which the low-rank backward splits each token's sources over a
// workgroup, from this many sources on: up to 8 are one batch of loads for a
// wave, so that a quarter of them each wins nothing and the meeting costs.
// One wave per token / split: 2 to 8 sources of d = 1024, r = 128 0.90 to 1.0 up
// to 256 tokens, 0.77 to 0.87 at 512; 9 and more at least 0.98 everywhere.  Step
// of forward and backward, one wave per token -> split: 49 sources, d = 1024, r
// = 16: 46 -> 27 us at 128 tokens, 52 -> 39 at 512, 67 -> 68 at 1024; 64
// sources, d = 2048: 81 -> 39, 103 -> 91, 146 -> 156.
constexpr int64_t kWgSplitBwd = 512;
constexpr int64_t kWgSplitBwdSources = 9;

// Workgroups below which a backward gives its waves fewer tokens (two per CU).
// Full-rank rows, read twice by a wave with many loads of its own, gain from it
// only below one per CU (rows above 2 KiB) or one and a half: four tokens a
// wave / two, 2 and 24 sources: bf16, d = 1280: 5000 tokens 0.94, 1.01, 7000
// 0.87, 1.00; d = 2048: 5000 0.91, 0.92; fp32, d = 512: 5000 1.34, 1.39; bf16, d =
// 1024: 6000 1.25, 1.21, 7000 0.94, 0.87.
constexpr int64_t kFewBlocks = 512;
constexpr int64_t kFewBlocksFull = 384, kFewBlocksWide = 256;

int round_up(int x, int m) { return (x + m - 1) / m * m; }

}  // namespace

void plan_wg_split(const Problem &p, Plan *pl)
{
    if (p.N > (p.mode == LRAR_MODE_FULL ? kWgSplitFull : kWgSplitLowRank) || p.S < 2)
        return;
    pl->wg_split = true;
    pl->nblocks = (int)p.N;
    const size_t row = (size_t)pl->nch * kWaveSize * pl->vec;
    // Scores in LDS (low-rank keys only), per-wave statistics, the
    // accumulators of waves 1..kWaves-1.
    pl->s_pad = round_up((int)((p.S + kWaves - 1) / kWaves), 4);
    const size_t scores = p.mode == LRAR_MODE_FULL ? 0 : (size_t)kWaves * pl->s_pad;
    pl->lds = (scores + 2 * kWaves + (kWaves - 1) * row) * sizeof(float);
}

bool make_plan(const Problem &p, bool bwd, Plan *pl, std::string *why, bool split)
{
    const int vmax = p.dtype == LRAR_DTYPE_BF16 ? 8 : 4;
    pl->vec = p.d % vmax == 0 ? vmax : 1;
    const int width = kWaveSize * pl->vec;
    const int64_t need = (p.d + width - 1) / width;
    static const int vec_list[] = {1, 2, 4, 8};
    static const int sc_list[] = {1, 2, 4, 8, 16};
    const int *list = pl->vec > 1 ? vec_list : sc_list;
    const int nlist = pl->vec > 1 ? 4 : 5;
    const int maxch = list[nlist - 1];
    if (p.N > (1 << 30)) {
        *why = "N exceeds 2^30 tokens";
        return false;
    }
    if (p.S > (bwd ? kMaxSourcesBwd : kMaxSourcesFwd)) {
        *why = bwd ? "backward supports at most 512 sources" : "forward supports at most 1024 sources";
        return false;
    }
    if (bwd && p.mode != LRAR_MODE_FULL && p.r > kMaxRankBwd) {
        *why = "backward with projected or sliced keys supports r <= 256";
        return false;
    }
    if (need > maxch) {
        if (bwd || p.mode == LRAR_MODE_FULL) {
            *why = "row width d too large for the backward / full-rank kernels";
            return false;
        }
        pl->nch = maxch;
        pl->ysplit = (int)((need + maxch - 1) / maxch);
    } else {
        for (int k = 0; k < nlist; ++k)
            if (list[k] >= need) {
                pl->nch = list[k];
                break;
            }
    }
    pl->fullcols = pl->vec > 1 && p.d % ((int64_t)width * pl->nch) == 0;
    pl->s_pad = round_up((int)p.S, 4);
    pl->r_pad = round_up((int)p.r, 4);
    if (!bwd) {
        pl->nblocks = (int)((p.N + kWaves - 1) / kWaves);
        // The low-rank forward keeps the weights in LDS; the full-rank one
        // holds its online-softmax state in registers.  (The plan is that of
        // one token per wave; route_fwd_lr's launch scales it to its TW.)
        pl->lds = p.mode == LRAR_MODE_FULL ? 0 : (size_t)kWaves * pl->s_pad * sizeof(float);
    } else {
        pl->tpw = p.mode == LRAR_MODE_FULL ? 4 : bwd_tokens_per_wave(pl->nch);
        // Fewer tokens per wave where there are too few workgroups to keep the
        // memory busy (step of forward and backward: fp32, 17 sources, d = 768,
        // 1000 tokens 62 -> 44 us; bf16 rows of 1020 columns, 49 sources, 2048
        // tokens 986 -> 634; full rank, 20 sources, d = 1280, 2000 tokens 333 ->
        // 127; at twice kFewBlocks level or 1% slower).  The dq partials, one
        // row a workgroup, stay within what a caller without a workspace has.
        const int64_t ncols = p.mode == LRAR_MODE_FULL ? p.d : p.r;
        const int64_t few = p.mode != LRAR_MODE_FULL ? kFewBlocks
                            : p.d * (p.dtype == LRAR_DTYPE_BF16 ? 2 : 4) > 2048 ? kFewBlocksWide
                                                                                : kFewBlocksFull;
        const bool fewer = p.N < few * kWaves * pl->tpw;
        while (fewer && pl->tpw > 1 && p.N < kFewBlocks * kWaves * pl->tpw &&
               (p.N / (kWaves * (pl->tpw / 2)) + 1) * ncols * (int64_t)sizeof(float) <=
                   (int64_t)kNoAllocScratchBytes)
            pl->tpw /= 2;
        pl->wg_split = split && p.mode != LRAR_MODE_FULL && p.S >= kWgSplitBwdSources &&
                       p.N <= kWgSplitBwd;
        const int64_t per_block = pl->wg_split ? 1 : (int64_t)kWaves * pl->tpw;
        if (pl->wg_split)
            pl->tpw = 1;
        pl->nblocks = (int)((p.N + per_block - 1) / per_block);
        pl->lds = (size_t)kWaves * 4 * pl->s_pad * sizeof(float);
        pl->lds += p.mode == LRAR_MODE_FULL ? (size_t)round_up((int)p.d, 4) * sizeof(float)
                                            : (size_t)kWaves * pl->r_pad * sizeof(float);
    }
    return true;
}


int hip_status(hipError_t e, const char *what, std::string *err)
{
    if (e == hipSuccess)
        return LRAR_OK;
    *err = std::string(what) + ": " + hipGetErrorString(e);
    return LRAR_EHIP;
}


int check_supported(const Problem &p, bool bwd, std::string *why)
{
    Plan pl;
    return make_plan(p, bwd, &pl, why) ? LRAR_OK : LRAR_EUNSUPPORTED;
}

size_t bwd_partial_bytes(const Problem &p)
{
    // Of a site of many sources: few may need fewer rows (their tokens are not
    // split), but a buffer sized for the first site of a pass serves them all.
    Problem q = p;
    q.S = std::max(p.S, kWgSplitBwdSources);
    Plan pl;
    std::string why;
    if (!make_plan(q, true, &pl, &why))
        return 0;
    const int64_t ncols = p.mode == LRAR_MODE_FULL ? p.d : p.r;
    return (size_t)pl.nblocks * (size_t)ncols * sizeof(float);
}

size_t bwd_workspace_bytes(const Problem &p)
{
    // The register form of full-rank keys where the call can take it, whatever
    // the number of sources (as the partials: the same for every site).
    const size_t need = bwd_partial_bytes(p);
    return need > 0 && full_rows(p) ? std::max(need, wide_bwd_workspace_bytes(p.N, 1, p.d)) : need;
}

}  // namespace lrar
