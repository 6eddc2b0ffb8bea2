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

// The passes of sort_by_key.  A loop over a number of digits that is not known to the compiler takes up to 1.5 times as long.
template <int DIGITS, typename Index, typename Count>
void sort_by_digits(KeyedIndex<Index> *items, KeyedIndex<Index> *other, size_t n, uint32_t lo, int bits, Count *counts)
{
    const uint32_t mask = (1u << bits) - 1;
    for (size_t i = 0; i < n; ++i) {
        const uint32_t key = items[i].key - lo;
#pragma unroll
        for (int d = 0; d < DIGITS; ++d) ++counts[((size_t)d << bits) + ((key >> (d * bits)) & mask)];
    }
    KeyedIndex<Index> *from = items, *to = other;
#pragma unroll
    for (int d = 0; d < DIGITS; ++d) {
        Count *at = counts + ((size_t)d << bits);
        const int shift = d * bits;
        if (at[((items[0].key - lo) >> shift) & mask] == n) continue;
        Count sum = 0;
        for (uint32_t b = 0; b <= mask; ++b) {
            const Count c = at[b];
            at[b] = sum;
            sum += c;
        }
        for (size_t i = 0; i < n; ++i) to[at[((from[i].key - lo) >> shift) & mask]++] = from[i];
        std::swap(from, to);
    }
    if (from != items) memcpy(items, from, n * sizeof(*items));
}

// Sorts by ascending key, equal keys in their present order: least significant digit first, in as few digits of up to eleven bits as the keys'
// range needs, all of about the same width, and digits in which all keys agree left out (100 000 floats that came from 16 bits: 1.05 -> 0.83
// ms).  A comparison sort through an index spends its time on mispredicted branches and
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
    auto passes = [&](auto count) {
        std::vector<decltype(count)> counts((size_t)digits << bits);
        if (digits == 1) sort_by_digits<1>(items, other, n, lo, bits, counts.data());
        else if (digits == 2) sort_by_digits<2>(items, other, n, lo, bits, counts.data());
        else sort_by_digits<3>(items, other, n, lo, bits, counts.data());
    };
    if (n <= UINT32_MAX) passes(uint32_t());
    else passes(uint64_t());
}

// Sorts a list of ascending runs, the q-th of which ends before ends[q]: neighbours are merged until one is left, so that an item is moved once
// per doubling of the number of runs.
template <typename T>
void merge_runs(std::vector<T> &items, std::vector<size_t> ends)
{
    while (ends.size() > 1) {
        size_t kept = 0, begin = 0;
        for (size_t q = 0; q < ends.size(); q += 2) {
            const size_t end = ends[std::min(q + 1, ends.size() - 1)];
            std::inplace_merge(items.begin() + (std::ptrdiff_t)begin, items.begin() + (std::ptrdiff_t)ends[q], items.begin() + (std::ptrdiff_t)end);
            ends[kept++] = begin = end;
        }
        ends.resize(kept);
    }
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
