// iod_plan.h -- the host's rules for how a launch divides its work: lanes per
// particle of the FP64 propagations, waves to a SIMD of a batch's swarms, and
// the pipelined sensitivity sweeps. Host code without HIP calls; sizes only.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <functional>
#include <utility>
#include <vector>

#include "iod_internal.h"

namespace iodk {

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Lanes per particle of the FP64 propagations. A wave of one, two or four
// lanes per particle holds 64, 32 or 16 of them, and its steps take about
// SPLIT_COST times those of one lane per particle (measured on 500 steps to
// 10 observations: 243, 184 and 165 us). So more lanes shorten a launch while
// its waves have a SIMD each, and lengthen it once they share them: take the
// number with the shortest estimate; several lanes must gain 5%. The estimate
// is the largest of the longest wave, the SIMDs' mean load, and, since a wave
// is not divided, n times the n-th wave that some SIMD must take: the
// ((n - 1) simds + 1)-th longest (32,769 particles of one problem on 1,024
// SIMDs: 316 us with two lanes each, 252 us with one).
constexpr double SPLIT_COST[3] = {1.0, 0.76, 0.68};

using Load = std::pair<int64_t, int64_t>;   // (steps, particles) of a problem

inline Load load_of(int64_t m, int64_t steps) { return {std::max<int64_t>(steps, 1), m}; }

// work[0 .. n): the problems, longest first.
inline double split_estimate(const Load *work, size_t n, int l, int simds)
{
    double total = 0.0, t = 0.0;
    int64_t waves = 0;
    for (size_t p = 0; p < n; ++p) {
        const int64_t nw = ceil_div(work[p].second, 64 >> l);
        // waves waves + 1 .. waves + nw are of this length
        t = std::max(t, (double)((waves + nw - 1) / simds + 1) * (double)work[p].first);
        waves += nw;
        total += (double)nw * (double)work[p].first;
    }
    return SPLIT_COST[l] * std::max(t, total / simds);
}

// two: whether two lanes per particle are to be had
inline int split_lanes(const Load *work, size_t n, int simds, bool two = true)
{
    int best = 1;
    double t0 = 0.95 * split_estimate(work, n, 0, simds);
    for (int l = two ? 1 : 2; l < 3; ++l) {
        const double t = split_estimate(work, n, l, simds);
        if (t < t0) {
            best = 1 << l;
            t0 = t;
        }
    }
    return best;
}

struct SplitLoad {
    std::vector<Load> work;   // each problem
    void add(int64_t m, int64_t steps)
    {
        if (m > 0) work.push_back(load_of(m, steps));
    }
    // Estimates for at most two workgroups of bs threads to their SIMDs, longest
    // first (work in that order; INFINITY if there are more). alone: one after
    // the other, the second ones, longest first, where the first ends first, and
    // 10% longer, since nothing fills a wave's waits. Else side by side in the
    // order of dispatch, so that the longest has the longest of the second ones
    // beside it.
    double paired(int l, int bs, int simds, bool alone) const
    {
        const size_t places = (size_t)std::max(1, simds / (bs / 64));
        std::vector<int64_t> len;
        for (const auto &w : work) {
            const int64_t n = ceil_div(w.second, bs >> l);
            if (len.size() + (size_t)n > 2 * places) return INFINITY;
            len.insert(len.end(), (size_t)n, w.first);
        }
        if (len.empty()) return INFINITY;
        if (len.size() <= places) return SPLIT_COST[l] * (double)len[0];
        if (!alone) return SPLIT_COST[l] * (double)(len[0] + len[places]);
        int64_t t = len[0];
        for (size_t j = places; j < len.size(); ++j) t = std::max(t, len[j] + len[2 * places - 1 - j]);
        return 1.1 * SPLIT_COST[l] * (double)t;
    }
    // Lanes of a batch's FP64 swarm launches, whose workgroups of one lane per
    // particle have bs threads; solo: they run one wave to a SIMD.
    int swarm_lanes(int bs, int simds, bool &solo)
    {
        int best = lanes(simds);
        const double side = paired(best >> 1, best > 1 ? SPLIT_BS : bs, simds, false);
        double t0 = side < INFINITY ? side : split_estimate(work.data(), work.size(), best >> 1, simds);
        solo = false;
        for (int l = 0; l < 3; ++l) {
            const double t = paired(l, l ? SPLIT_BS : bs, simds, true);
            if (t <= t0) {
                best = 1 << l;
                t0 = t;
                solo = true;
            }
        }
        return best;
    }
    int lanes(int simds, bool two = true)
    {
        std::sort(work.begin(), work.end(), std::greater<Load>());
        return split_lanes(work.data(), work.size(), simds, two);
    }
};

// Most scratch for which the trials' checkpoints are the closest.
constexpr int64_t TRIAL_CKPT_BYTES = (int64_t)2 << 30;

// The problems of a sensitivity launch, and which of its sweeps are pipelined.
// The pipelined form shortens a step about four times (normal equations) or
// three times (gradient) while its workgroups (PIPE_P particles of one
// problem) have a compute unit each, and the launch grows with every further
// one to a unit: the normal equations by about half, the gradient by a third
// if their LDS lets several share a unit, else by its whole time.
// Over 2,000 steps the normal equations take 0.84, 1.20, 1.87, 2.29, 2.78 and
// 3.27 ms with one to six workgroups to a unit against 4.1 ms otherwise; the
// gradient 1.59, 3.14 and 4.7 ms against 4.7 ms, and over 500 steps (two share a
// unit) 0.45, 0.60 and 0.95 ms against 1.2 ms.
struct PipePlan {
    int64_t groups = 0, steps = 0, grid = 0;
    int32_t sub = 1, seg = PIPE_SUB;
    bool tan = false, adj = false;
    bool ckpt = false;   // the refinement's trials leave checkpoints
    void add(int64_t m, int64_t s)
    {
        if (m < 1) return;
        groups += ceil_div(m, PIPE_P);
        steps = std::max(steps, s);
        if (s <= PIPE_MAX_STEPS) seg = std::max(seg, pipe_segment((int32_t)s));
    }
    // the most workgroups for which the gradient's sweep is pipelined
    int64_t adj_limit(int simds, bool tan_too = false) const
    {
        const int64_t shared = (160 << 10) / pipe_lds_bytes(seg, tan_too, true);
        return (shared > 1 ? 3 : 2) * (simds / 4);
    }
    void decide(int simds)
    {
        if (steps > PIPE_MAX_STEPS) return;
        tan = groups <= 6 * (simds / 4);
        adj = groups <= adj_limit(simds);
    }
    // Scratch of the batched refinement and the segments of its trials'
    // checkpoints: states every seg steps and after the last one, in the rows
    // (of row_bytes) that the one-thread adjoint has `rows` of. The shortest
    // segments are the fastest (two workgroups share a compute unit's LDS); longer
    // ones where many problems' checkpoints would take gigabytes, and where the
    // scratch cannot be had: fits(n) says whether there is memory for n rows. The
    // last resort is the adjoint's own rows, without checkpoints. Returns
    // whether something fitted. seg is a power of two whatever the outcome (the
    // trials' kernel needs one), not what add() found for the adjoint's own.
    template <class Fits>
    bool trial_scratch(int64_t rows, int64_t row_bytes, Fits fits)
    {
        const auto ckpt_rows = [&] { return ceil_div(steps, seg) + 1; };
        seg = PIPE_SUB;
        ckpt = steps <= PIPE_MAX_STEPS;
        if (ckpt) {
            while (seg < PIPE_MAX_SEG && ckpt_rows() * row_bytes > TRIAL_CKPT_BYTES) seg *= 2;
            for (; seg <= PIPE_MAX_SEG; seg *= 2)
                if (fits(std::max(rows, ckpt_rows()))) return true;
            seg = PIPE_SUB;
            ckpt = false;
        }
        return fits(rows);
    }
};

}  // namespace iodk
