// Stable sorts of index lists by 32-bit keys for the host planners.
#pragma once

#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <utility>
#include <vector>

namespace adaqp {

template <typename Index> struct KeyedIndex { uint32_t key; Index index; };

// Sorts by ascending key, equal keys in their present order: least significant digit first, in as few digits of up to eleven bits as the keys'
// range needs, all of about the same width.  A comparison sort through an index spends its time on mispredicted branches and
// scattered reads; digits no wider than needed leave a cache line per value of a digit in the first-level cache (100 000 floats of 27 bits,
// three digits of nine bits instead of eleven: 0.95 of the time).  `other`: scratch of n items.
template <typename Index>
void sort_by_key(KeyedIndex<Index> *items, KeyedIndex<Index> *other, size_t n)
{
    constexpr int kMostBits = 11;
    if (n < 256) {
        std::stable_sort(items, items + n,
                         [](const KeyedIndex<Index> &x, const KeyedIndex<Index> &y) { return x.key < y.key; });
        return;
    }
    uint32_t lo = items[0].key, hi = lo;
    for (size_t i = 1; i < n; ++i) {
        lo = std::min(lo, items[i].key);
        hi = std::max(hi, items[i].key);
    }
    int range_bits = 0;
    while (range_bits < 32 && ((hi - lo) >> range_bits) != 0) ++range_bits;
    const int digits = (range_bits + kMostBits - 1) / kMostBits;
    if (digits == 0) return;
    const int bits = (range_bits + digits - 1) / digits;
    const uint32_t mask = (1u << bits) - 1;
    auto passes = [&](auto *counts) {
        for (size_t i = 0; i < n; ++i) {
            const uint32_t key = items[i].key - lo;
            for (int d = 0; d < digits; ++d) ++counts[((size_t)d << bits) + ((key >> (d * bits)) & mask)];
        }
        KeyedIndex<Index> *from = items, *to = other;
        for (int d = 0; d < digits; ++d) {
            auto *at = counts + ((size_t)d << bits);
            size_t sum = 0;
            for (uint32_t b = 0; b <= mask; ++b) {
                const size_t c = at[b];
                at[b] = sum;
                sum += c;
            }
            for (size_t i = 0; i < n; ++i) to[at[((from[i].key - lo) >> (d * bits)) & mask]++] = from[i];
            std::swap(from, to);
        }
        if (from != items) memcpy(items, from, n * sizeof(*items));
    };
    std::vector<uint32_t> count(n <= UINT32_MAX ? (size_t)digits << bits : 0);
    std::vector<uint64_t> count64(n <= UINT32_MAX ? 0 : (size_t)digits << bits);
    if (n <= UINT32_MAX) passes(count.data());
    else passes(count64.data());
}

// order_out[k] = position of the k-th smallest value, ties by position (n up to 2^31 - 1).
inline void order_by_value(int64_t n, const int32_t *values, int32_t *order_out)
{
    int32_t lo = values[0], hi = values[0];
    bool sorted = true;
    for (int64_t i = 1; i < n; ++i) {
        sorted = sorted && values[i - 1] <= values[i];
        lo = std::min(lo, values[i]);
        hi = std::max(hi, values[i]);
    }
    if (sorted) {
        for (int64_t i = 0; i < n; ++i) order_out[i] = (int32_t)i;
        return;
    }
    const int64_t range = (int64_t)hi - lo + 1;
    try {
        if (range <= 4 * n) {                               // rows of one partition: one counter each
            std::vector<int32_t> at((size_t)range, 0);
            for (int64_t i = 0; i < n; ++i) ++at[(size_t)((int64_t)values[i] - lo)];
            int32_t sum = 0;
            for (int32_t &c : at) {
                const int32_t here = c;
                c = sum;
                sum += here;
            }
            for (int64_t i = 0; i < n; ++i) order_out[at[(size_t)((int64_t)values[i] - lo)]++] = (int32_t)i;
            return;
        }
        std::vector<KeyedIndex<int32_t>> items((size_t)n), other((size_t)n);
        for (int64_t i = 0; i < n; ++i) items[(size_t)i] = {(uint32_t)values[i] ^ 0x80000000u, (int32_t)i};
        sort_by_key(items.data(), other.data(), (size_t)n);
        for (int64_t k = 0; k < n; ++k) order_out[k] = items[(size_t)k].index;
    } catch (const std::bad_alloc &) {
        // no room for the scratch, and nothing may be thrown through a C entry: a comparison sort does without
        for (int64_t i = 0; i < n; ++i) order_out[i] = (int32_t)i;
        std::stable_sort(order_out, order_out + n, [values](int32_t x, int32_t y) { return values[x] < values[y]; });
    }
}

}  // namespace adaqp
