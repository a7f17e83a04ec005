// Which form of the FP64 contraction is the faster: a model of the launches of
// each (host only).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "kernels.hpp"
#include "tables.hpp"

namespace pufe {

// Time of the FP64 contraction (with its chunk sums and element matrices) for a
// given choice of form per element, in cycles of the chip.  Each launch takes the
// work of its groups over the slots of the chip (256 groups of eight waves, 512 of
// four, or 256 where their stage leaves room for one per CU), and half its longest
// group for the uneven end: the launches follow each other, so a few elements in
// another form than the rest cost a whole such span.  The constants (cycles of a
// SIMD where not said otherwise) are fitted to 360 problems of 27 to 13,824
// elements (8 to 283 functions, 3 to 12 Gauss points, levels 0 to 2, orders 1 and
// 2, sheared, tabulated and Bloch-periodic ones), each timed with the direct
// kernels, with the moment form and with both: 80 to 40,000 us, off by 11 % (rms).
struct FormElem {
    double pts, leaves, fill, per_point, ff, tiles, pairs, chunks;
    int nloc, nt, nfun, items, stages, buffers;   // items: work groups per chunk (0: no moment form); stages per leaf
};
struct FormModel {
    std::vector<FormElem> el;
    int n3 = 0, nfun = 0, nimg = 0;
    // over mom_cost_of, for groups of four and of eight waves: with the mixed terms
    // of sheared cells, or the spline and weights of the general variants, more
    double moment[2] = {1.41, 1.41};

    static double span(double sum, double longest, double slots) { return std::max(longest, sum / slots + 0.5 * longest); }
    static constexpr double kLaunch = 3300.0;
    // one direct work item over pts points: tile pairs, rows, evaluations of the functions
    static double direct_item(double pts, double pairs, double rows, double fill) {
        return pts * (42.0 * pairs + 6.4 * rows + fill + 308.0) + 47000.0;
    }
    static double narrow(const FormElem &e) { return direct_item(e.pts / e.chunks, e.pairs, e.nloc, 7.3 * e.fill); }
    template <class F>
    static void wide(const FormElem &e, F &&f) {   // per block of kWideTiles tiles
        const int T = (int)e.tiles, nb = (T + kWideTiles - 1) / kWideTiles;
        for (int j = 0; j < nb; ++j)
            for (int i = 0; i <= j; ++i) {
                const int ti = std::min(kWideTiles, T - i * kWideTiles), tj = std::min(kWideTiles, T - j * kWideTiles);
                f(direct_item(e.pts / e.chunks, i == j ? 0.5 * ti * (ti + 1) : ti * tj, 16.0 * (i == j ? ti : ti + tj),
                              31.0 * e.fill));
            }
    }
    // K-chunks of an element in moment form and cycles of one of its work groups on a SIMD
    static double share(const FormElem &e) { return e.nt <= 3 ? 2.0 : 4.0; }
    static double mom_chunks(const FormElem &e, double dur) {
        return std::max(1.0, std::min(e.leaves, std::ceil(e.per_point * e.pts / e.items / share(e) / dur)));
    }
    double group(const FormElem &e, double chunks) const {
        return moment[e.nt > 3] * e.per_point * e.pts / e.items / share(e) / chunks + 25300.0 +
               e.stages * e.leaves / chunks * (e.buffers == 1 ? 7500.0 : 5300.0);
    }
    double dur(const std::vector<char> &mom) const {
        double total = 0.0;
        for (size_t k = 0; k < el.size(); ++k)
            if (mom[k]) total += (el[k].per_point + el[k].ff) * el[k].pts;
        return std::max(total / 4096.0, 40000.0);
    }
    // expansion groups of an element, and what one takes of the chip (cycles)
    static double expand(const FormElem &e) { return (e.nt > 0 ? mom_quads_ae(e.nt) : 0) + (e.nfun + 1) / 2 + 1; }
    static constexpr double kExpand = 84.0, kSlot = 10.8;

    // where an element's own work is least
    bool cheaper(const FormElem &e, double d) const {
        double direct = 0.0;
        if (e.tiles <= kWholeMaxTiles) direct = e.chunks * narrow(e);
        else wide(e, [&](double c) { direct += e.chunks * c; });
        const double nch = e.nt > 0 ? mom_chunks(e, d) : 0.0, slots = nch > 1.0 ? nch * mom_slots(e.nt) : 0.0;
        const double mine = (e.nt > 0 ? nch * e.items * share(e) * group(e, nch) : 0.0) + 4900.0 * std::ceil(e.leaves / 16.0) +
                            0.8 * e.pts + 1024.0 * (kExpand * expand(e) + kSlot * slots);
        return mine < direct;
    }
    double time(const std::vector<char> &mom) const {
        struct Sum {
            double sum = 0.0, longest = 0.0;
            void add(double d, double count) {
                sum += d * count;
                longest = std::max(longest, d);
            }
        };
        Sum nar, wid, m4, m8;
        double reduce = 0.0, slots = 0.0, groups = 0.0, fe = 0.0, chain = 0.0, leaves = 1.0;
        int rows = 0;
        const double d = dur(mom);
        bool any = false;
        for (size_t k = 0; k < el.size(); ++k) {
            const FormElem &e = el[k];
            if (!mom[k]) {
                if (e.tiles <= kWholeMaxTiles) {
                    nar.add(narrow(e), e.chunks);
                    rows = std::max(rows, 16 * (int)e.tiles);
                    leaves = std::max(leaves, std::ceil(e.leaves / e.chunks));
                } else {
                    wide(e, [&](double c) { wid.add(c / 4.0, e.chunks); });
                }
                if (e.chunks > 1.0) reduce += e.chunks * e.pairs;
                continue;
            }
            any = true;
            const double ch = std::ceil(e.leaves / 16.0);
            fe += 4900.0 * ch + 0.8 * e.pts;
            chain = std::max(chain, std::min(4.0, std::ceil(e.leaves / ch / 4.0)) * 135.0 * n3);
            groups += expand(e);
            if (e.nt == 0) continue;
            const double nch = mom_chunks(e, d);
            (e.nt <= 3 ? m4 : m8).add(group(e, nch), nch * e.items);
            if (nch > 1.0) slots += nch * mom_slots(e.nt);
        }
        double t = 0.0;
        if (nar.sum > 0.0) {   // two groups share a CU, or one has it and hides less latency
            const bool two = 2 * contract_lds_bytes(24, rows, std::max(nfun, 1), nimg, (int)leaves, n3) <= (size_t)160 * 1024;
            t += kLaunch + (two ? span(nar.sum / 2.0, nar.longest / 2.0, 512.0)
                                : span(1.74 * nar.sum / 4.0, 1.74 * nar.longest / 4.0, 256.0));
        }
        if (wid.sum > 0.0) t += kLaunch + span(wid.sum, wid.longest, 256.0);
        if (reduce > 0.0) t += 12000.0 + 1.6 * reduce;
        if (!any) return t;
        if (m8.sum > 0.0) t += kLaunch + span(m8.sum, m8.longest, 256.0);
        if (m4.sum > 0.0) t += kLaunch + span(m4.sum, m4.longest, 512.0);
        if (slots > 0.0) t += 34000.0 + kSlot * slots;
        return t + kLaunch + std::max(fe / 1024.0, chain) + 25000.0 + kExpand * groups;
    }
};

}  // namespace pufe
