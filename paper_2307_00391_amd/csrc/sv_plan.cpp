// Cuts a gate list into windows: the gates of one window run together (in one
// pass over the state, or in one matrix block).
//
// A window starts from the earliest gate left and grows one gate's need at a
// time, each time by the need that lets it run the most ops; then it takes
// every gate it can.  Taking the earliest gates until the window is full
// instead fills it with one layer of a layered circuit: 20 layers of U3 and a
// CNOT ladder on 33 qubits came out at 66 windows of 13 qubits that way (the
// lowest 5 in each), and at 41 this way (27 with the lowest 4), since a window
// of neighbouring qubits runs a slanted stack of layers.
#include <string.h>

#include "sv_fused.h"

namespace sv {

namespace {

constexpr int MAX_CAND = 8;

struct Scan {
    int ops;
    uint64_t cand[MAX_CAND];   // needs that would unblock a gate
    int ncand;
};

// what a window with the qubits `set` can run of the gates left (packed in
// program order); `take`: their places in `left`
void scan(const std::vector<PlanItem> &left, uint64_t set, int cap, int item_out, int window_out, int max_ops,
          bool want_cand, Scan &r, std::vector<int> *take) {
    uint64_t blocked = 0, ext = 0;
    r.ops = 0;
    r.ncand = 0;
    const PlanItem *it = left.data();
    const int n = (int)left.size();
    for (int i = 0; i < n; ++i) {
        const PlanItem &g = it[i];
        if (g.order & blocked) {
            blocked |= g.order;
        } else {
            const uint64_t out = g.ext | (g.order & ~set);
            const bool near = item_out < 0 || popcount64(out) <= item_out;
            if (!(g.need & ~set) && near && r.ops + g.ops <= max_ops &&
                (window_out < 0 || popcount64(ext | out) <= window_out)) {
                ext |= out;
                r.ops += g.ops;
                if (take) take->push_back(i);
                continue;
            }
            if (want_cand && r.ncand < MAX_CAND) {
                const uint64_t m = (near ? g.need : g.need | g.order) & ~set;
                if (m && popcount64(set | m) <= cap) {
                    bool seen = false;
                    for (int j = 0; j < r.ncand; ++j) seen |= r.cand[j] == m;
                    if (!seen) r.cand[r.ncand++] = m;
                }
            }
            blocked |= g.order;
        }
        // Once every qubit of the window waits, only gates that need none of
        // them (phases on other qubits) are left: they are taken, not counted.
        if (!take && set && !(set & ~blocked)) break;
    }
}

}  // namespace

void plan_windows(const std::vector<PlanItem> &items, int cap, uint64_t base, int item_out, int window_out,
                  int max_ops, std::vector<PlanWindow> &out) {
    out.clear();
    std::vector<PlanItem> left(items);
    std::vector<int> where(items.size()), take;
    for (size_t i = 0; i < where.size(); ++i) where[i] = (int)i;
    Scan r, t;
    while (!left.empty()) {
        const PlanItem &f = left[0];
        uint64_t set = base | f.need;
        if (item_out >= 0 && popcount64(f.ext | (f.order & ~set)) > item_out) set |= f.order;
        while (popcount64(set) < cap) {
            scan(left, set, cap, item_out, window_out, max_ops, true, r, nullptr);
            if (!r.ncand) break;
            int best = -1, at = 0;
            for (int j = 0; j < r.ncand && r.ncand > 1; ++j) {
                scan(left, set | r.cand[j], cap, item_out, window_out, max_ops, false, t, nullptr);
                if (t.ops > best) {
                    best = t.ops;
                    at = j;
                }
            }
            set |= r.cand[at];
        }
        out.emplace_back();
        PlanWindow &w = out.back();
        w.set = set;
        take.clear();
        scan(left, set, cap, item_out, window_out, max_ops, false, r, &take);
        // the rest moves up
        size_t q = 0, e = 0;
        w.take.reserve(take.size());
        for (size_t i = 0; i < left.size(); ++i) {
            if (e < take.size() && take[e] == (int)i) {
                w.take.push_back(where[i]);
                ++e;
            } else {
                left[q] = left[i];
                where[q++] = where[i];
            }
        }
        left.resize(q);
        where.resize(q);
    }
}

void plan_earliest(const std::vector<PlanItem> &items, int cap, uint64_t base, int max_ops,
                   std::vector<PlanWindow> &out) {
    out.clear();
    std::vector<int> left(items.size()), rest;
    for (size_t i = 0; i < left.size(); ++i) left[i] = (int)i;
    while (!left.empty()) {
        out.emplace_back();
        PlanWindow &w = out.back();
        w.set = base;
        uint64_t blocked = 0;
        int ops = 0;
        rest.clear();
        for (int i : left) {
            const PlanItem &g = items[i];
            if (!(g.order & blocked) && popcount64(w.set | g.need) <= cap && ops + g.ops <= max_ops) {
                w.set |= g.need;
                ops += g.ops;
                w.take.push_back(i);
            } else {
                blocked |= g.order;
                rest.push_back(i);
            }
        }
        left.swap(rest);
    }
}

}  // namespace sv
