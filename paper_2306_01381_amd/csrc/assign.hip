// Bit-width assignment for the next period (Sec. 4.2): host code, no GPU work.
//
// The paper builds a bi-objective problem from the traced beta values - Eq. 8, the variance a message adds to the
// weight gradients, against Eq. 7, the time of the slowest device pair - scalarises it with a weight lambda
// (Eq. 9) and hands it to a MILP solver, with the messages of a pair sorted by beta and cut into groups that
// share a width.  Here the solver is replaced by a greedy search that needs no library: every group starts at
// 2 bits; per pair the upgrades 2->4 and 4->8 are ordered by variance removed per extra transferred bit (the
// order in which the relaxed problem would take them); for every pair time that such a prefix can reach, each
// pair takes the longest prefix that fits under it, and the time with the smallest Eq. 9 value wins.  With one
// pair this is the exact optimum; with several, a pair misses its best packing by less than one upgrade.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <memory>
#include <numeric>
#include <vector>

#include "adaqp.h"
#include "host_sort.hpp"

namespace {

struct Upgrade {
    double efficiency;      // variance removed per extra bit on the wire
    int32_t group;
    int32_t step;           // 0: 2 -> 4 bits, 1: 4 -> 8 bits
    double gain;
    int64_t cost;           // extra bits on the wire
};

struct PairPath {
    size_t begin, end;                          // the pair's messages in the list sorted by (pair, descending beta)
    std::vector<Upgrade> upgrades;              // in the order they are taken
    std::vector<double> time;                   // [m]: pair time with the first m upgrades applied
    std::vector<double> variance;               // [m]: Eq. 8 share of this pair
};

double inv_levels_sq(int b)
{
    const double levels = (double)((1 << b) - 1);
    return 1.0 / (levels * levels);
}

float beta_of(uint32_t key)
{
    const uint32_t bits = ~key;
    float f;
    memcpy(&f, &bits, sizeof(f));
    return f;
}

template <typename Index>
void assign(int64_t n, const float *beta_host, const int32_t *peer_of_slot_host, int32_t n_peers, int32_t dim,
            int32_t group_size, double lambda, const double *theta_host, const double *gamma_host, uint8_t *bits_out,
            double *objective_out)
{
    const double w2 = inv_levels_sq(2), w4 = inv_levels_sq(4), w8 = inv_levels_sq(8);
    const double step_weight[2] = {w2 - w4, w4 - w8};
    const int64_t step_bits[2] = {2, 4};

    // ---- the messages of each pair by descending beta (non-negative floats order as their bits do), ties by slot ----
    // slots mostly come peer by peer: counted and placed in runs of one peer
    std::vector<size_t> first((size_t)n_peers + 1, 0);
    auto for_runs = [&](auto &&f) {
        for (int64_t k = 0; k < n;) {
            const int32_t peer = peer_of_slot_host[k];
            int64_t e = k + 1;
            while (e < n && peer_of_slot_host[e] == peer) ++e;
            f((size_t)peer, k, e);
            k = e;
        }
    };
    for_runs([&](size_t peer, int64_t k, int64_t e) { first[peer + 1] += (size_t)(e - k); });
    size_t most = 0;
    for (int32_t i = 0; i < n_peers; ++i) {
        most = std::max(most, first[(size_t)i + 1]);
        first[(size_t)i + 1] += first[(size_t)i];
    }
    // not initialised: every item is written before it is read
    std::unique_ptr<adaqp::KeyedIndex<Index>[]> sorted(new adaqp::KeyedIndex<Index>[(size_t)n]), other(new adaqp::KeyedIndex<Index>[most]);
    {
        std::vector<size_t> next(first.begin(), first.end() - 1);
        for_runs([&](size_t peer, int64_t k, int64_t e) {
            adaqp::KeyedIndex<Index> *to = sorted.get() + next[peer];
            next[peer] += (size_t)(e - k);
            for (; k < e; ++k) {
                const float beta = beta_host[k] + 0.0f;             // -0 counts as 0
                uint32_t bits;
                memcpy(&bits, &beta, sizeof(bits));
                *to++ = {~bits, (Index)k};
            }
        });
    }
    for (int32_t i = 0; i < n_peers; ++i)
        adaqp::sort_by_key(sorted.get() + first[(size_t)i], other.get(), first[(size_t)i + 1] - first[(size_t)i]);

    // ---- per pair: groups, upgrade order, reachable (time, variance) points ----
    std::vector<PairPath> pairs;
    std::vector<int32_t> pair_id;
    for (int32_t i = 0; i < n_peers; ++i) {
        PairPath path;
        path.begin = first[(size_t)i];
        path.end = first[(size_t)i + 1];
        const size_t n_slots = path.end - path.begin;
        if (n_slots == 0) continue;                                 // a pair that exchanges nothing takes no time
        const size_t n_groups = (n_slots + (size_t)group_size - 1) / (size_t)group_size;
        const adaqp::KeyedIndex<Index> *messages = sorted.get() + path.begin;
        // a group's sum is a chain of additions in the order of its messages; four whole groups at a time, as an addition takes as long as four
        // (with the merges below: 0.27 of the time of one after the other and three sorts; the whole assignment of 100 000 messages 491 -> 423 us)
        std::vector<double> betas(n_groups, 0.0);
        size_t g = 0;
        for (; (g + 4) * (size_t)group_size <= n_slots; g += 4) {
            const adaqp::KeyedIndex<Index> *of = messages + g * (size_t)group_size;
            double sum[4] = {0.0, 0.0, 0.0, 0.0};
            for (size_t q = 0; q < (size_t)group_size; ++q)
                for (int k = 0; k < 4; ++k) sum[k] += (double)beta_of(of[(size_t)k * (size_t)group_size + q].key);
            std::copy(sum, sum + 4, betas.begin() + (std::ptrdiff_t)g);
        }
        for (; g < n_groups; ++g)
            for (size_t q = g * (size_t)group_size; q < std::min(n_slots, (g + 1) * (size_t)group_size); ++q) betas[g] += (double)beta_of(messages[q].key);
        double variance_at_2 = 0.0;
        for (g = 0; g < n_groups; ++g) variance_at_2 += betas[g] * w2;
        // By descending efficiency, ties by group and step.  Betas descend, so that the upgrades of a step mostly do as well and the two steps
        // are merged; the last group may be smaller and another place its own.
        auto before = [](const Upgrade &a, const Upgrade &b) {
            if (a.efficiency != b.efficiency) return a.efficiency > b.efficiency;
            if (a.group != b.group) return a.group < b.group;
            return a.step < b.step;
        };
        path.upgrades.resize(2 * n_groups);
        for (int32_t step = 0; step < 2; ++step) {
            const auto begin = path.upgrades.begin() + (std::ptrdiff_t)(step * n_groups), end = begin + (std::ptrdiff_t)n_groups;
            for (g = 0; g < n_groups; ++g) {
                Upgrade &u = begin[(std::ptrdiff_t)g];
                u.group = (int32_t)g;
                u.step = step;
                u.gain = betas[g] * step_weight[step];
                u.cost = step_bits[step] * (int64_t)(std::min(n_slots, (g + 1) * (size_t)group_size) - g * (size_t)group_size) * dim;
                u.efficiency = u.gain / (double)u.cost;
            }
            if (!std::is_sorted(begin, end, before)) std::sort(begin, end, before);
        }
        std::inplace_merge(path.upgrades.begin(), path.upgrades.begin() + (std::ptrdiff_t)n_groups, path.upgrades.end(), before);
        const int64_t base_bits = 2 * (int64_t)dim * (int64_t)n_slots;
        path.time.push_back(theta_host[i] * (double)base_bits + gamma_host[i]);
        path.variance.push_back(variance_at_2);
        int64_t cost = 0;
        double gain = 0.0;
        for (const Upgrade &u : path.upgrades) {
            cost += u.cost;
            gain += u.gain;
            path.time.push_back(theta_host[i] * (double)(base_bits + cost) + gamma_host[i]);
            path.variance.push_back(variance_at_2 - gain);
        }
        pairs.push_back(std::move(path));
        pair_id.push_back(i);
    }

    // ---- the candidate times: every point any pair can reach, not below the all-2-bit time of the slowest ----
    std::vector<size_t> taken(pairs.size(), 0);
    if (!pairs.empty()) {
        double z_min = pairs[0].time[0];
        for (const PairPath &p : pairs) z_min = std::max(z_min, p.time[0]);
        // Each pair's times ascend: merged, not sorted (400 000 messages of 1 000 pairs in groups of 4: 528 ms sorted, 563 merged pair by pair into one
        // list, 517 so; of 64 in groups of 20 16.2, 12.3, 12.3).
        std::vector<double> candidates;
        std::vector<size_t> ends;
        for (const PairPath &p : pairs) {
            candidates.insert(candidates.end(), std::lower_bound(p.time.begin(), p.time.end(), z_min), p.time.end());
            ends.push_back(candidates.size());
        }
        adaqp::merge_runs(candidates, std::move(ends));
        candidates.erase(std::unique(candidates.begin(), candidates.end()), candidates.end());
        bool have = false;
        double best = 0.0;
        std::vector<size_t> m(pairs.size(), 0);
        for (double z : candidates) {                               // ascending: the prefixes only grow
            double variance = 0.0, worst = 0.0;
            for (size_t q = 0; q < pairs.size(); ++q) {
                const std::vector<double> &t = pairs[q].time;           // non-decreasing (theta >= 0)
                while (m[q] + 1 < t.size() && t[m[q] + 1] <= z) ++m[q];
                variance += pairs[q].variance[m[q]];
                worst = q == 0 ? t[m[q]] : std::max(worst, t[m[q]]);
            }
            const double f = lambda * variance + (1.0 - lambda) * worst;
            if (!have || f < best) {
                have = true;
                best = f;
                taken = m;
            }
        }
    }

    // ---- widths per slot, and the objective of the result from its definition ----
    double variance = 0.0, worst = 0.0;
    for (size_t q = 0; q < pairs.size(); ++q) {
        const PairPath &p = pairs[q];
        const size_t n_slots = p.end - p.begin, n_groups = (n_slots + (size_t)group_size - 1) / (size_t)group_size;
        std::vector<int> width(n_groups, 2);
        for (size_t j = 0; j < taken[q]; ++j) width[(size_t)p.upgrades[j].group] += p.upgrades[j].step == 0 ? 2 : 4;
        int64_t payload = 0;
        for (size_t g = 0; g < n_groups; ++g) {
            const size_t s = g * (size_t)group_size, e = std::min(n_slots, s + (size_t)group_size);
            for (size_t k = s; k < e; ++k) bits_out[sorted[p.begin + k].index] = (uint8_t)width[g];
            payload += (int64_t)(e - s) * dim * width[g];
        }
        const double t = theta_host[pair_id[q]] * (double)payload + gamma_host[pair_id[q]];
        worst = q == 0 ? t : std::max(worst, t);
    }
    if (objective_out) {
        const double weight[9] = {0, 0, w2, 0, w4, 0, 0, 0, w8};
        for (int64_t k = 0; k < n; ++k) variance += (double)beta_host[k] * weight[bits_out[k]];
        objective_out[0] = lambda * variance + (1.0 - lambda) * worst;
        objective_out[1] = variance;
        objective_out[2] = worst;
    }
}

}  // namespace

extern "C" int adaqp_assign_bits(int64_t n, const float *beta_host, const int32_t *peer_of_slot_host,
                                 int32_t n_peers, int32_t dim, int32_t group_size, double lambda,
                                 const double *theta_host, const double *gamma_host, uint8_t *bits_out,
                                 double *objective_out)
{
    if (n < 0 || n_peers <= 0 || dim <= 0 || group_size <= 0 || !(lambda >= 0.0 && lambda <= 1.0))
        return ADAQP_EINVAL;
    if (!theta_host || !gamma_host) return ADAQP_EINVAL;
    if (n > 0 && (!beta_host || !peer_of_slot_host || !bits_out)) return ADAQP_EINVAL;
    if (n > ((int64_t)1 << 40) / dim) return ADAQP_ESIZE;           // bit counts stay far inside int64
    for (int32_t i = 0; i < n_peers; ++i)
        if (!(theta_host[i] >= 0.0) || !std::isfinite(theta_host[i]) || !std::isfinite(gamma_host[i]))
            return ADAQP_EINVAL;
    bool ok = true;
    for (int64_t k = 0; k < n; ++k)
        ok &= (uint32_t)peer_of_slot_host[k] < (uint32_t)n_peers & beta_host[k] >= 0.0f & beta_host[k] <= FLT_MAX;
    if (!ok) return ADAQP_EINVAL;

    if (n <= INT32_MAX)
        assign<int32_t>(n, beta_host, peer_of_slot_host, n_peers, dim, group_size, lambda, theta_host, gamma_host, bits_out,
                        objective_out);
    else
        assign<int64_t>(n, beta_host, peer_of_slot_host, n_peers, dim, group_size, lambda, theta_host, gamma_host, bits_out,
                        objective_out);
    return ADAQP_OK;
}
