// Autotuner for the all-pairs launch shape: times every supported variant on
// the caller's mesh and keeps the fastest per (N, M, half_domain, precision) and, in FP64,
// form of the kernel: with the S2 sums formed on their own (one problem) or with the
// pairs (a batch and the mixed solves' outer residual), whose fastest shapes differ.
#include <hip/hip_runtime.h>

#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "bim_common.h"

namespace bim {

namespace {
using Key = std::tuple<int, int, int, int, bool>;  // last: FP64 with the S2 sums formed with the pairs
std::mutex g_mu;
std::map<Key, bim_pair_config> g_best;
}  // namespace

namespace {
inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }
}  // namespace

PairLaunch pair_launch(const Dims &d, int tpl, int unroll, int chunks) {
    PairLaunch pl;
    pl.tpl = (tpl == 2) ? 2 : 1;
    pl.unroll = (unroll == 2 || unroll == 8) ? unroll : 4;
    pl.row_groups = cdiv(d.M, pl.tpl);
    pl.tiles_per_bnd = cdiv(pl.row_groups * (d.N - 1), 64);
    pl.target_tiles = 2 * pl.tiles_per_bnd;
    pl.src_rows = 2 * d.M;
    pl.chunks = (int)std::max(1L, std::min((long)chunks, (long)pl.src_rows * d.N));
    pl.blocks = cdiv((long)pl.target_tiles * pl.chunks, 4);
    return pl;
}

int chunks_for_waves(const Dims &d, int tpl, int unroll, long want_waves) {
    const PairLaunch base = pair_launch(d, tpl, unroll, 1);
    return (int)std::max(1L, (want_waves + base.target_tiles / 2) / base.target_tiles);
}

PairLaunch pair_launch_cfg(const Dims &d, int prec, const bim_pair_config &cfg) {
    int chunks = cfg.chunks;
    if (chunks <= 0 && cfg.rows_per_chunk > 0) chunks = cdiv(2 * d.M, cfg.rows_per_chunk);
    // default wave count.  FP32C: about 32 waves per SIMD (1024 SIMDs), the best
    // count measured at 181 x 61.  FP64: 3 per mesh node, between 1 and 48 per SIMD
    // (fewer hide less latency, more cost the reduction of their partial sums;
    // measured optima: 31 x 11 1.7 thousand waves, 61 x 21 4.1, 91 x 31 8.2, 121 x 41
    // 16, 181 x 61 33, full 71 x 71 16, full 151 x 151 49 thousand)
    if (chunks <= 0) {
        const long want = prec == BIM_FP64 ? std::max(1024L, std::min(49152L, 3L * d.nnode)) : 32768;
        chunks = chunks_for_waves(d, cfg.targets_per_lane, cfg.unroll, want);
    }
    return pair_launch(d, cfg.targets_per_lane, cfg.unroll, chunks);
}

static bool tuned_launch(const bim_problem *p, int prec, bool s2_with_pairs, bim_pair_config *cfg) {
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_best.find(Key(p->N, p->M, p->half_domain ? 1 : 0, prec, s2_with_pairs && prec == BIM_FP64));
    if (it == g_best.end()) return false;
    *cfg = it->second;
    return true;
}

PairLaunch pair_launch_for(const bim_problem *p, int prec) {
    const Dims d(p);
    bim_pair_config cfg;
    if (tuned_launch(p, prec, false, &cfg)) return pair_launch_cfg(d, prec, cfg);
    // untuned defaults, the fastest shapes measured: FP64 4-way unroll, two rows per
    // lane on a full domain of some size, where the shared record work is half of a
    // pair's (151 x 151: 1242 us with one row, 1119 with two; 71 x 71: 109 / 106; 41 x 41:
    // 44 / 44; on a half domain the images share it already: 488 / 489 at 181 x 61);
    // FP32C 2-way unroll
    const bool two = prec == BIM_FP64 && d.nimg == 1 && d.nnode >= 4096;
    cfg = {two ? 2 : 1, prec == BIM_FP32C ? 2 : 4, 0, 0};
    return pair_launch_cfg(d, prec, cfg);
}

PairLaunch pair_launch_batch(const bim_problem *p, int prec) {
    const Dims d(p);
    bim_pair_config cfg;
    if (!tuned_launch(p, prec, true, &cfg)) {
        cfg = {1, prec == BIM_FP32C ? 2 : 4, 0, 0};
        // about 24 waves per SIMD in FP64, the best count of these kernels at 181 x 61
        if (prec == BIM_FP64) cfg.chunks = chunks_for_waves(d, 1, 4, 24576);
    }
    PairLaunch pl = pair_launch_cfg(d, prec, cfg);
    pl.s2_with_pairs = true;
    return pl;
}

}  // namespace bim

using namespace bim;

extern "C" int bim_tune_residual(const bim_problem *prob, const double *u, int prec, void *stream,
                                 bim_pair_config *best, double *best_ms) {
    int rc = validate(prob);
    if (rc) return rc;
    if (!u) return fail(BIM_EINVAL, "u must be a device pointer");
    if (prec != BIM_FP64 && prec != BIM_FP32C) return fail(BIM_EINVAL, "unknown precision");
    const Dims d(prob);
    hipStream_t s = (hipStream_t)stream;
    double *F = nullptr;
    if ((rc = hip_check(hipMallocAsync((void **)&F, sizeof(double) * d.nvec, s), "hipMallocAsync"))) return rc;
    // every variant at its default chunk count and those giving 8 to 48 waves per SIMD
    // (1024 SIMDs); the form with the pairs at 24 and 32, its best counts (a batch takes only the
    // variant from the choice)
    const int forms = prec == BIM_FP64 ? 2 : 1;
    bim_pair_config pick[2] = {};
    double pick_ms[2] = {1e30, 1e30};
    for (int f = 0; f < forms && !rc; ++f) {
        std::vector<bim_pair_config> cands;
        const std::vector<long> wants = f ? std::vector<long>{24576, 32768}
                                          : std::vector<long>{0, 8192, 16384, 24576, 32768, 49152};
        for (int tpl : {1, 2})
            for (int unr : {2, 4, 8})
                for (long want : wants) {
                    const int chunks = want ? pair_launch(d, tpl, unr, chunks_for_waves(d, tpl, unr, want)).chunks
                                            : pair_launch_cfg(d, prec, {tpl, unr, 0, 0}).chunks;
                    bim_pair_config c{tpl, unr, 0, chunks};
                    bool dup = false;
                    for (auto &o : cands)
                        dup |= (o.targets_per_lane == tpl && o.unroll == unr && o.chunks == chunks);
                    if (!dup) cands.push_back(c);
                }
        for (auto &c : cands) {
            PairLaunch pl = pair_launch_cfg(d, prec, c);
            pl.s2_with_pairs = f == 1;
            double kms = 0, tms = 0;
            if ((rc = residual_timed(prob, u, F, prec, 3, pl, s, &kms, &tms))) break;
            if (kms < pick_ms[f]) {
                pick_ms[f] = kms;
                pick[f] = c;
            }
        }
    }
    (void)hipFreeAsync(F, s);
    if (rc) return rc;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        for (int f = 0; f < forms; ++f) g_best[Key(prob->N, prob->M, prob->half_domain ? 1 : 0, prec, f == 1)] = pick[f];
    }
    if (best) *best = pick[0];
    if (best_ms) *best_ms = pick_ms[0];
    return BIM_OK;
}
