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

} // namespace

bool lds_tables(const std::vector<int32_t> &rowptr, const std::vector<int32_t> &col,
                const std::vector<int32_t> &row_class, int32_t m, int32_t n, LdsHostTables *out) {
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
    for (int32_t j : col) ++colptr[j + 1];
    std::partial_sum(colptr.begin(), colptr.end(), colptr.begin());
    std::vector<int32_t> bits(n);
    std::iota(bits.begin(), bits.end(), 0);
    auto cdeg = [&](int32_t j) { return colptr[j + 1] - colptr[j]; };
    std::stable_sort(bits.begin(), bits.end(), [&](int32_t a, int32_t b) { return cdeg(a) > cdeg(b); });
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
    if (T.npos + 1 > 65535) return false;
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
