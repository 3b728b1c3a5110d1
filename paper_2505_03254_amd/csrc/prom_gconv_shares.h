// How many workgroups each layer of one shared grouped-convolution launch gets.
#pragma once

#include <algorithm>

namespace prom {

// One layer of a shared launch: `blocks` channel blocks that each take `units` units of work, and
// what a workgroup needs for one unit.
struct GconvShareLayer {
    int blocks, units;
    double unit_cost;
};

// A layer's workgroups per channel block that end by `time` (at least one unit of work each), and
// what it takes them by: with several channel blocks and enough workgroups a multiple of 8, for
// the XCD-aware order.  That order comes before the end where the layer has too few units for the
// next multiple (ResNeXt-50's layers at batch 2, one of 14 units: 20.0 us with eight workgroups per
// channel block, 21.3 with 14 in plain order).
inline int gconv_share_by(const GconvShareLayer &l, double time, int *step)
{
    const double fit = time / l.unit_cost * (1 + 1e-9);
    const int each = fit >= l.units ? l.units : fit < 1 ? 1 : (int)fit;
    const int need = (l.units - 1) / each + 1;
    *step = l.blocks > 1 && need >= 8 ? 8 : 1;
    return *step == 8 ? std::min((need + 7) / 8, l.units / 8) * 8 : need;
}

// Shares `slots` workgroups out so that the last one ends as early as it can, then hands out what
// is left.  A workgroup ends after a whole number of units: a layer of 32 units has 16 workgroups
// of two units each or 32 of one, and what lies between does not end it sooner, so shares in
// proportion to the cost spend workgroups where they gain nothing.  The end is found by halving between a time
// at which the shares fit and one at which they don't; what remains goes, a step at a time, to the
// layer with the most cost per workgroup (the estimate ends no sooner for it, but fewer wavefronts are
// idle meanwhile: without it RegNetX-400MF's layers take 43.5 instead of 41.9 us at batch 48, 73.7
// instead of 72.6 at batch 96).  Where even one workgroup per channel block does not fit, each has one.
inline void gconv_shares(const GconvShareLayer *layers, int n, int slots, int *per_block, int *step)
{
    auto plan = [&](double time) {
        long long used = 0;
        for (int k = 0; k < n; ++k) {
            per_block[k] = gconv_share_by(layers[k], time, &step[k]);
            used += (long long)per_block[k] * layers[k].blocks;
        }
        return used;
    };
    double total = 0, longest = 0, late = 0;  // nothing ends before a mean share or one unit
    for (int k = 0; k < n; ++k) {
        total += (double)layers[k].blocks * layers[k].units * layers[k].unit_cost;
        longest = std::max(longest, layers[k].unit_cost);
        late = std::max(late, layers[k].units * layers[k].unit_cost);
    }
    double early = std::max(total / slots, longest);
    long long used = plan(early);
    if (used > slots) {
        for (double t = early * 1.25; t < late; t *= 1.25) {
            if (plan(t) <= slots) {
                late = t;
                break;
            }
            early = t;
        }
        while (late - early > early * 1e-4) {
            const double t = 0.5 * (early + late);
            (plan(t) <= slots ? late : early) = t;
        }
        used = plan(late);
    }
    for (;;) {
        int best = -1;
        double best_cost = 0;
        for (int k = 0; k < n; ++k) {
            const GconvShareLayer &l = layers[k];
            if (per_block[k] + step[k] > l.units || used + (long long)step[k] * l.blocks > slots) continue;
            const double cost = l.unit_cost * l.units / per_block[k];
            if (best < 0 || cost > best_cost) {
                best = k;
                best_cost = cost;
            }
        }
        if (best < 0) break;
        per_block[best] += step[best];
        used += (long long)step[best] * layers[best].blocks;
    }
}

}  // namespace prom
