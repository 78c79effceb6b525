// Tables of the LDS-resident decoder and training (decode_lds.hip,
// train_lds.hip), host code run once per graph at build time.
//
// Rows and bits are sorted by degree (stable, descending) and cut into groups
// of 64, one lane each.  A group of rows lists the posterior slots of its
// edges, a group of bits the positions of its messages in ascending check
// order, as pairs of 16-bit indices; entries past a row's (bit's) own degree
// name slot n, which holds +infinity (position npos, which holds 0).
#include <algorithm>
#include <numeric>

#include "ldpc_internal.h"

namespace ldpc {
namespace {

// The row degree that the kernel unrolls for a group whose largest row has d edges.
int row_bucket(int d) { return d <= 2 ? 2 : d <= 16 ? d : (d + 3) / 4 * 4; }

// Chooses which bit of a degree sits in which slot.  A wavefront gathers, per
// edge number k, the posteriors of 64 rows and, per column entry u, the
// messages of 64 bits; the LDS serves 32 lanes at a time without conflict when
// their words differ modulo 32 (a message's word is its row's lane modulo 32).
// Random swaps of two bits of one degree are kept while they lower the sum over
// the 32-lane halves of the squared numbers of lanes per bank.  Rows keep their
// lanes and their edges' order (training breaks ties by it).
void spread_banks(const std::vector<int32_t> &rowptr, const std::vector<int32_t> &col, const std::vector<int32_t> &rows,
                  const std::vector<int32_t> &colptr, std::vector<int32_t> &bits) {
    constexpr int kBanks = 32, kTrials = 48; // trials per bit: 1 to 60 ms for the codes in range
    const int32_t n = (int32_t)bits.size();
    if (n < 2) return;
    // of every bit's messages, by ascending check: the half of rows and edge number, and the row's lane
    struct Use {
        int32_t hist; // first bin of (row half, k)
        int32_t lane;
    };
    std::vector<int32_t> place(rowptr.size(), -1);
    for (size_t p = 0; p < rows.size(); ++p) place[rows[p]] = (int32_t)p;
    std::vector<Use> use(col.size());
    std::vector<int32_t> fill(colptr.begin(), colptr.end() - 1);
    const size_t halves = (rows.size() + 31) / 32;
    for (size_t i = 0; i + 1 < rowptr.size(); ++i)
        for (int32_t e = rowptr[i]; e < rowptr[i + 1]; ++e)
            use[fill[col[e]]++] = Use{(int32_t)(((size_t)place[i] / 32 * kLdsMaxDegree + (e - rowptr[i])) * kBanks),
                                      place[i] % kBanks};
    std::vector<int16_t> rh(halves * kLdsMaxDegree * kBanks, 0); // check pass
    // bit pass: bins for the largest degree of each half (its first slot's), so that one long column costs its
    // own half only
    std::vector<size_t> bit_half((size_t)(n + 31) / 32);
    size_t bins = 0;
    for (size_t h = 0; h < bit_half.size(); ++h) {
        bit_half[h] = bins;
        bins += (size_t)(colptr[bits[32 * h] + 1] - colptr[bits[32 * h]]) * kBanks;
    }
    std::vector<int16_t> bh(bins, 0);
    auto put = [&](int32_t j, int32_t p, int s) { // adds (takes) bit j at slot p; the change of the sums
        int32_t d = 0;
        for (int32_t q = colptr[j]; q < colptr[j + 1]; ++q) {
            int16_t &a = rh[(size_t)use[q].hist + p % kBanks];
            int16_t &b = bh[bit_half[p / 32] + (size_t)(q - colptr[j]) * kBanks + use[q].lane];
            d += 2 * s * (a + b) + 2;
            a += (int16_t)s;
            b += (int16_t)s;
        }
        return d;
    };
    for (int32_t p = 0; p < n; ++p) put(bits[p], p, 1);
    uint32_t seed = 12345u;
    auto rnd = [&](uint32_t below) {
        seed = seed * 1664525u + 1013904223u;
        return (int32_t)(((uint64_t)seed * below) >> 32);
    };
    for (int32_t lo = 0; lo < n;) { // the slots of one degree
        int32_t hi = lo;
        const int32_t d = colptr[bits[lo] + 1] - colptr[bits[lo]];
        while (hi < n && colptr[bits[hi] + 1] - colptr[bits[hi]] == d) ++hi;
        if (d > 0 && hi - lo > 1)
            for (int64_t t = 0; t < (int64_t)kTrials * (hi - lo); ++t) {
                const int32_t p = lo + rnd((uint32_t)(hi - lo)), q = lo + rnd((uint32_t)(hi - lo));
                if (p == q) continue;
                const int32_t a = bits[p], b = bits[q];
                const int32_t change = put(a, p, -1) + put(b, q, -1) + put(a, q, 1) + put(b, p, 1);
                if (change <= 0) {
                    std::swap(bits[p], bits[q]);
                } else {
                    put(a, q, -1);
                    put(b, p, -1);
                    put(a, p, 1);
                    put(b, q, 1);
                }
            }
        lo = hi;
    }
}

} // namespace

bool lds_tables(const std::vector<int32_t> &rowptr, const std::vector<int32_t> &col,
                const std::vector<int32_t> &row_class, int32_t m, int32_t n, LdsHostTables *out, size_t lds_max) {
    std::vector<int32_t> rows, colptr(n + 1, 0);
    int32_t dmax = 0;
    for (int32_t i = 0; i < m; ++i) {
        const int32_t d = rowptr[i + 1] - rowptr[i];
        dmax = std::max(dmax, d);
        if (d > 0) rows.push_back(i); // rows of degree 0 are always satisfied
    }
    if (dmax > kLdsMaxDegree || n > 16 * kLdsMaxThreads || rows.empty()) return false;
    auto deg = [&](int32_t i) { return rowptr[i + 1] - rowptr[i]; };
    std::stable_sort(rows.begin(), rows.end(), [&](int32_t a, int32_t b) { return deg(a) > deg(b); });
    // The message positions, and whether a frame's state fits at all (n = 15000, rows of up to 16, which does not: a
    // graph build of 30 ms with the search below, 5 without).
    size_t positions = 0;
    for (size_t p = 0; p < rows.size(); p += 64) positions += 64 * (size_t)row_bucket(deg(rows[p]));
    if (positions + 1 > 65535 || 4 * ((size_t)n + positions + 2) > lds_max) return false;
    for (int32_t j : col) ++colptr[j + 1];
    std::partial_sum(colptr.begin(), colptr.end(), colptr.begin());
    std::vector<int32_t> bits(n);
    std::iota(bits.begin(), bits.end(), 0);
    auto cdeg = [&](int32_t j) { return colptr[j + 1] - colptr[j]; };
    std::stable_sort(bits.begin(), bits.end(), [&](int32_t a, int32_t b) { return cdeg(a) > cdeg(b); });
    spread_banks(rowptr, col, rows, colptr, bits);
    LdsHostTables T;
    T.slot_of.resize(n);
    T.bit_of.resize(n);
    for (int32_t p = 0; p < n; ++p) {
        T.slot_of[bits[p]] = (uint16_t)p;
        T.bit_of[p] = (uint16_t)bits[p];
    }
    // rows: groups of 64, positions group by group
    std::vector<int32_t> edge_pos(col.size());
    const int32_t rg = ((int32_t)rows.size() + 63) / 64;
    T.row_class.assign((size_t)rg * 64, 0);
    for (int32_t g = 0; g < rg; ++g) {
        LdsGroup G{};
        G.degree = row_bucket(deg(rows[(size_t)g * 64]));
        G.first = T.npos;
        G.table = (int32_t)T.rows.size();
        const int32_t words = (G.degree + 1) / 2;
        T.rows.resize(T.rows.size() + (size_t)words * 64, (uint32_t)n | (uint32_t)n << 16);
        for (int32_t l = 0; l < 64 && g * 64 + l < (int32_t)rows.size(); ++l) {
            const int32_t i = rows[(size_t)g * 64 + l];
            T.row_class[(size_t)g * 64 + l] = row_class[i];
            for (int32_t k = 0; k < deg(i); ++k) {
                const int32_t e = rowptr[i] + k, sh = 16 * (k & 1);
                uint32_t &word = T.rows[(size_t)G.table + 64 * (k / 2) + l];
                word = (word & ~(0xffffu << sh)) | (uint32_t)T.slot_of[col[e]] << sh;
                edge_pos[e] = G.first + 64 * k + l;
            }
        }
        T.npos += 64 * G.degree;
        T.row_group.push_back(G);
    }
    T.rows.resize(T.rows.size() + kLdsMaxDegree / 2 * 64, 0u); // read, but not used, past the last group
    std::vector<int32_t> fill(colptr.begin(), colptr.end() - 1), csc(col.size());
    for (size_t e = 0; e < col.size(); ++e) csc[fill[col[e]]++] = (int32_t)e; // ascending row in every column
    const int32_t bg = (n + 63) / 64;
    for (int32_t g = 0; g < bg; ++g) {
        LdsGroup G{};
        G.degree = cdeg(bits[(size_t)g * 64]);
        G.table = (int32_t)T.bits.size();
        const int32_t words = (G.degree + 1) / 2;
        T.bits.resize(T.bits.size() + (size_t)words * 64, (uint32_t)T.npos | (uint32_t)T.npos << 16);
        for (int32_t l = 0; l < 64 && g * 64 + l < n; ++l) {
            const int32_t j = bits[(size_t)g * 64 + l];
            for (int32_t u = 0; u < cdeg(j); ++u) {
                const int32_t sh = 16 * (u & 1);
                uint32_t &word = T.bits[(size_t)G.table + 64 * (u / 2) + l];
                word = (word & ~(0xffffu << sh)) | (uint32_t)edge_pos[csc[colptr[j] + u]] << sh;
            }
        }
        T.bit_group.push_back(G);
    }
    T.bits.resize(T.bits.size() + kLdsMaxDegree / 2 * 64, 0u);
    *out = std::move(T);
    return true;
}

} // namespace ldpc
