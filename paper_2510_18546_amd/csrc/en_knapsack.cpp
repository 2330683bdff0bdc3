// The retrieval knapsack of Section 3.4 Eq. (1), arXiv 2510.18546: host code only.
//
// Exact 0/1 knapsack over token capacity with a total order on the solutions: largest summed value,
// then fewest tokens, then the lexicographically smallest list of ids. It sits in front of every
// planning step that retrieves its groups, so it is host time that the GPU waits for.
//
// The dynamic programme over all candidates costs candidates x budget cells (256 groups of 192 .. 256
// tokens under a budget of 7 K tokens: 0.9 M cells, 470 us of a step whose kernels take 150). Nearly
// all candidates are decided without it: sorted by value per token, the greedy order's first ones are
// in every optimal set and its last ones in none, and the linear relaxation proves it item by item.
// So: (1) a good solution from a small programme over the items around the point where the greedy
// order fills the budget; (2) every item whose relaxation bound, when its decision is reversed, falls
// below that solution is fixed (strictly below: all optimal sets survive, so the tie rules hold);
// (3) the programme over the few items that are left (10 - 25 of 128 in such instances).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>
#include <vector>

#include <immintrin.h>

#include "en_internal.h"

// (the library is compiled without NaN semantics: finiteness is read from the bits)
static inline bool finite_bits(float x)
{
    uint32_t u;
    std::memcpy(&u, &x, sizeof u);
    return (u & 0x7f800000u) != 0x7f800000u;
}

namespace {

// Value and tokens of a set in one number, value * 2^shift - tokens with 2^shift above all tokens:
// the larger number is the better set under the first two rules.
template <typename K>
struct Item {
    int id;
    int w;
    K key;
};

// One item's row of the programme, in place: row[c] held the best number with capacity c over the items behind
// this one and gets this one too; bit c of `bits`: taking it is optimal there, ties included. Columns
// 64 * first_word .. 64 * end_word - 1, from the last down: what a column reads lies in front of it (w > 0).
template <typename K>
void knapsack_row_scalar(K *row, uint64_t *bits, size_t first_word, size_t end_word, size_t w, K key)
{
    for (size_t wd = end_word; wd-- > first_word;) {
        uint64_t m = 0;
        for (size_t c = wd * 64 + 64; c-- > wd * 64;) {
            if (c < w)
                break;
            const K with = row[c - w] + key;
            if (with >= row[c]) {
                row[c] = with;
                m |= uint64_t(1) << (c & 63);
            }
        }
        bits[wd] = m;
    }
}

// The same on 64-bit numbers, four at a time (about 0.2 ns per cell instead of 0.6).
__attribute__((target("avx2"))) void knapsack_row_avx2(int64_t *row, uint64_t *bits, size_t first_word,
                                                        size_t end_word, size_t w, int64_t key)
{
    const size_t whole = std::max(first_word, std::min(end_word, (w + 63) / 64));      // words with c >= w throughout
    const __m256i k4 = _mm256_set1_epi64x(key);
    for (size_t wd = end_word; wd-- > whole;) {
        uint64_t skip = 0;
        for (int i = 15; i >= 0; --i) {
            const size_t c = wd * 64 + 4 * i;
            const __m256i old = _mm256_loadu_si256(reinterpret_cast<const __m256i *>(row + c));
            const __m256i with =
                _mm256_add_epi64(_mm256_loadu_si256(reinterpret_cast<const __m256i *>(row + c - w)), k4);
            const __m256i worse = _mm256_cmpgt_epi64(old, with);
            _mm256_storeu_si256(reinterpret_cast<__m256i *>(row + c), _mm256_blendv_epi8(with, old, worse));
            skip |= uint64_t(unsigned(_mm256_movemask_pd(_mm256_castsi256_pd(worse)))) << (4 * i);
        }
        bits[wd] = ~skip;
    }
    knapsack_row_scalar(row, bits, first_word, whole, w, key);
}

void knapsack_row(int64_t *row, uint64_t *bits, size_t first, size_t end, size_t w, int64_t key)
{
    static const bool avx2 = __builtin_cpu_supports("avx2");
    if (avx2)
        knapsack_row_avx2(row, bits, first, end, w, key);
    else
        knapsack_row_scalar(row, bits, first, end, w, key);
}
void knapsack_row(__int128 *row, uint64_t *bits, size_t first, size_t end, size_t w, __int128 key)
{
    knapsack_row_scalar(row, bits, first, end, w, key);
}

// Best number over items[0 .. m) with capacity W. With `taken` non-null the optimal set that prefers
// the items in front is returned in it.
template <typename K>
K solve(const Item<K> *items, int m, int64_t W, std::vector<int> *taken)
{
    int64_t all_w = 0;
    K all_key = 0;
    for (int a = 0; a < m; ++a) {
        all_w += items[a].w;
        all_key += items[a].key;
    }
    if (all_w <= W) {
        for (int a = 0; taken && a < m; ++a)
            taken->push_back(items[a].id);
        return all_key;
    }
    const size_t words = size_t(W) / 64 + 1;
    std::vector<K> row(words * 64, K(0));
    std::vector<uint64_t> bits(taken ? size_t(m) * words : words);
    int64_t before = all_w;              // tokens of the items in front of a
    for (int a = m - 1; a >= 0; --a) {
        before -= items[a].w;
        // whatever the items in front take, at least W - before is left when it is a's turn
        const size_t first = size_t(std::max<int64_t>(0, W - before)) / 64;
        knapsack_row(row.data(), bits.data() + (taken ? size_t(a) * words : 0), first, words, size_t(items[a].w),
                     items[a].key);
    }
    if (taken) {
        int64_t c = W;
        for (int a = 0; a < m; ++a)
            if (bits[size_t(a) * words + size_t(c >> 6)] >> (c & 63) & 1) {
                taken->push_back(items[a].id);
                c -= items[a].w;
            }
    }
    return row[size_t(W)];
}

// items: positive lengths of at most W, ids ascending, together longer than W.
template <typename K>
void choose(std::vector<Item<K>> &items, int64_t W, std::vector<int32_t> &chosen)
{
    const int m = int(items.size());
    // by value per token, best first
    std::vector<std::pair<double, int>> order(m);
    for (int a = 0; a < m; ++a)
        order[a] = {-double(items[a].key) / double(items[a].w), a};
    std::sort(order.begin(), order.end());
    std::vector<int64_t> w_sum(m + 1, 0);
    std::vector<double> k_sum(m + 1, 0.0);
    K head_key = 0;
    for (int j = 0; j < m; ++j) {
        const Item<K> &it = items[order[j].second];
        w_sum[j + 1] = w_sum[j] + it.w;
        k_sum[j + 1] = k_sum[j] + double(it.key);
    }
    // items 0 .. brk-1 of the order fit, with item brk they do not
    const int brk = int(std::upper_bound(w_sum.begin(), w_sum.end(), W) - w_sum.begin()) - 1;
    // (1) the items before the window taken, the best of the window. Six on either side: wider ones
    // cost more than the few items that they fix in addition.
    constexpr int HALF = 6;
    const int w0 = std::max(0, brk - HALF), w1 = std::min(m, brk + HALF);
    std::vector<Item<K>> window;
    for (int j = w0; j < w1; ++j)
        window.push_back(items[order[j].second]);
    for (int j = 0; j < w0; ++j)
        head_key += items[order[j].second].key;
    const double found = double(head_key + solve<K>(window.data(), int(window.size()), W - w_sum[w0], nullptr));
    // (2) the relaxation without item `skip` in capacity `cap`: the order's items as long as they fit and
    // a fraction of the next one. Sums of at most a few thousand doubles: their relative error is far
    // below the margin that the comparison leaves.
    constexpr double MARGIN = 1.0 + 1e-9;
    auto relaxed = [&](int64_t cap, int skip) {
        const int64_t sw = w_sum[skip + 1] - w_sum[skip];
        const double sk = k_sum[skip + 1] - k_sum[skip];
        // prefix lengths with the item cut out: w_sum[j] up to skip, w_sum[j + 1] - sw behind it
        int j;
        if (w_sum[skip] > cap) {
            j = int(std::upper_bound(w_sum.begin(), w_sum.begin() + skip + 1, cap) - w_sum.begin()) - 1;
            return k_sum[j] - order[j].first * double(cap - w_sum[j]);
        }
        j = int(std::upper_bound(w_sum.begin() + skip + 1, w_sum.end(), cap + sw) - w_sum.begin()) - 1;
        const double whole = k_sum[j] - sk;
        return j < m ? whole - order[j].first * double(cap + sw - w_sum[j]) : whole;
    };
    std::vector<Item<K>> core;
    std::vector<char> state(m);          // 0 out, 1 in, 2 open
    int64_t left = W;
    for (int j = 0; j < m; ++j) {
        const Item<K> &it = items[order[j].second];
        const double other = j < brk ? relaxed(W, j) : double(it.key) + relaxed(W - it.w, j);
        const bool fixed = other * MARGIN < found;
        state[order[j].second] = !fixed ? 2 : j < brk ? 1 : 0;
    }
    for (int a = 0; a < m; ++a) {
        if (state[a] == 2) {
            core.push_back(items[a]);
        } else if (state[a] == 1) {
            chosen.push_back(items[a].id);
            left -= items[a].w;
        }
    }
    // (3)
    std::vector<int> taken;
    solve<K>(core.data(), int(core.size()), left, &taken);
    chosen.insert(chosen.end(), taken.begin(), taken.end());
}

struct Candidate {
    int id;
    int w;
    int64_t v;
};

template <typename K>
void choose_from(const std::vector<Candidate> &cand, int64_t W, int shift, int unit, std::vector<int32_t> &chosen)
{
    std::vector<Item<K>> items;
    items.reserve(cand.size());
    for (const Candidate &c : cand) {
        if (c.w == 0)
            chosen.push_back(c.id);      // costs nothing: in every optimal set
        else if (c.w <= W)
            items.push_back({c.id, c.w / unit, (K(c.v) << shift) - K(c.w)});
    }
    const int64_t cap = W / unit;
    int64_t sum = 0;
    for (const Item<K> &it : items)
        sum += it.w;
    if (sum <= cap) {
        for (const Item<K> &it : items)
            chosen.push_back(it.id);
    } else {
        choose<K>(items, cap, chosen);
    }
    std::sort(chosen.begin(), chosen.end());
}

}  // namespace

int en_knapsack(const float *p_host, const int32_t *len, int G, float threshold, int64_t budget_tokens,
                std::vector<int32_t> &chosen)
{
    chosen.clear();
    if (!finite_bits(threshold)) {
        en_set_error("retrieval knapsack: the threshold is not finite");
        return EN_ERR_INVALID_ARG;
    }
    std::vector<Candidate> cand;
    int64_t wsum = 0;
    double vsum = 0.0;
    int unit = 0;                        // common divisor of the lengths
    for (int g = 0; g < G; ++g) {
        if (len[g] < 0)
            continue;                       // not a candidate (a store group never put)
        if (!finite_bits(p_host[g])) {
            en_set_error("retrieval knapsack: score of group %d is not finite", g);
            return EN_ERR_INVALID_ARG;
        }
        const double d = double(p_host[g]) - double(threshold);
        const int64_t v = (int64_t)std::nearbyint(d * 4294967296.0);   // ties to even
        if (v > 0) {
            cand.push_back({g, len[g], v});
            wsum += len[g];
            vsum += double(v);
            unit = std::gcd(unit, len[g]);
        }
    }
    const int m = int(cand.size());
    if (wsum <= budget_tokens) {
        for (const Candidate &c : cand)
            chosen.push_back(c.id);
        return EN_OK;
    }
    const int64_t W = budget_tokens;
    {
        // One bit per (item, capacity) and 24 bytes per capacity: refused beyond a stated size. The programme holds
        // the bits and one row of 8 or 16 bytes per capacity, so no instance that is accepted needs more.
        const size_t cols = size_t(W) + 1;
        const size_t need = size_t(m) * ((cols + 63) / 64) * 8 + cols * 24;
        if (need > EN_KNAPSACK_MAX_BYTES) {
            en_set_error("retrieval knapsack: %d candidates x %lld tokens of budget need a table of %zu bytes (limit "
                         "%zu)", m, (long long)W, need, EN_KNAPSACK_MAX_BYTES);
            return EN_ERR_CAPACITY;
        }
    }
    int shift = 1;
    while ((int64_t(1) << shift) <= wsum)
        ++shift;
    // 64-bit numbers wherever the sum of all values leaves room for the tokens: 256 groups of 256 tokens do up to
    // scores of 2^4 each; other instances take 128-bit ones (one cell at a time: where nothing can be fixed either,
    // 256 groups under 7 K tokens take 2.1 ms)
    if (std::ldexp(vsum, shift) < 0x1p61)
        choose_from<int64_t>(cand, W, shift, unit, chosen);
    else
        choose_from<__int128>(cand, W, shift, unit, chosen);
    return EN_OK;
}
