// Checks the LDS-resident decoder's tables (csrc/lds_tables.hip) on one graph
// read from stdin ("m n" then, per row, its degree and bits): bits have
// distinct slots; every edge has a message position of its own below npos, at
// first + 64 k + lane of its row's group; every bit lists its messages in
// ascending check order; the entries past a row's or bit's degree name slot n
// and position npos; group degrees are ones that the kernel unrolls and
// everything stays inside the tables.  Prints "ok" or a failure.
#include <algorithm>
#include <cstdio>
#include <map>
#include <vector>

#include "ldpc_internal.h"

static int fail(const char *what) {
    std::printf("FAIL %s\n", what);
    return 1;
}

int main() {
    int m, n;
    if (std::scanf("%d %d", &m, &n) != 2) return fail("input");
    std::vector<int32_t> rowptr(m + 1, 0), col, cls(m);
    for (int i = 0; i < m; ++i) {
        int d;
        if (std::scanf("%d", &d) != 1) return fail("input");
        for (int k = 0; k < d; ++k) {
            int x;
            if (std::scanf("%d", &x) != 1) return fail("input");
            col.push_back(x);
        }
        rowptr[i + 1] = (int32_t)col.size();
        cls[i] = i; // (the row itself, to recognise it)
    }
    LdsHostTables T;
    if (!ldpc::lds_tables(rowptr, col, cls, m, n, &T)) {
        std::printf("refused\n");
        return 0;
    }
    std::vector<int> bit_in(n, -1);
    for (int j = 0; j < n; ++j) {
        const int p = T.slot_of[j];
        if (p >= n || bit_in[p] >= 0) return fail("slots");
        bit_in[p] = j;
    }
    auto entry = [](const std::vector<uint32_t> &t, size_t at, int k, int lane) {
        return (int)((t[at + 64 * (size_t)(k / 2) + lane] >> (16 * (k % 2))) & 0xffffu);
    };
    const size_t pad = (size_t)ldpc::kLdsMaxDegree / 2 * 64; // read past the last group's words
    std::map<int, std::pair<int, int>> edge_at;              // position -> (row, bit)
    std::vector<int> seen(m, 0);
    int next = 0;
    for (size_t g = 0; g < T.row_group.size(); ++g) {
        const LdsGroup &G = T.row_group[g];
        const int d = G.degree;
        if (!((d >= 2 && d <= 16) || (d <= 32 && d % 4 == 0)) || G.first != next) return fail("row group");
        next += 64 * d;
        if ((size_t)G.table + pad > T.rows.size() || (size_t)G.table + 64 * ((d + 1) / 2) + pad > T.rows.size())
            return fail("row table size");
        for (int l = 0; l < 64; ++l) {
            std::vector<int> bits;
            for (int k = 0; k < d + d % 2; ++k) {
                const int p = entry(T.rows, G.table, k, l);
                if (p > n) return fail("slot range");
                if (p == n) continue;
                if (k >= d || (int)bits.size() != k) return fail("padding inside a row");
                bits.push_back(bit_in[p]);
            }
            if (bits.empty()) continue;
            const int i = T.row_class[64 * g + l];
            if (i < 0 || i >= m || seen[i]++ ||
                std::vector<int>(col.begin() + rowptr[i], col.begin() + rowptr[i + 1]) != bits)
                return fail("row");
            for (size_t k = 0; k < bits.size(); ++k) edge_at[G.first + 64 * (int)k + l] = {i, bits[k]};
        }
    }
    if (next != T.npos || edge_at.size() != col.size()) return fail("positions");
    for (int i = 0; i < m; ++i)
        if ((rowptr[i + 1] > rowptr[i]) != (seen[i] == 1)) return fail("rows");
    if (64 * T.bit_group.size() < (size_t)n) return fail("bit groups");
    size_t listed = 0;
    for (size_t g = 0; g < T.bit_group.size(); ++g) {
        const LdsGroup &G = T.bit_group[g];
        if ((size_t)G.table + 64 * ((G.degree + 1) / 2) + pad > T.bits.size()) return fail("bit table size");
        for (int l = 0; l < 64; ++l) {
            int last = -1;
            bool ended = false;
            for (int u = 0; u < G.degree + G.degree % 2; ++u) {
                const int p = entry(T.bits, G.table, u, l);
                if (p == T.npos) {
                    ended = true;
                    continue;
                }
                auto it = edge_at.find(p);
                if (ended || u >= G.degree || it == edge_at.end() || 64 * (int)g + l >= n ||
                    it->second.second != bit_in[64 * g + l] || it->second.first <= last)
                    return fail("bit list");
                last = it->second.first;
                ++listed;
            }
        }
    }
    if (listed != col.size()) return fail("bit lists incomplete");
    // mean largest number of lanes per bank over the 32-lane halves of both passes' gathers
    double load = 0.0, gathers = 0.0;
    auto half = [&](const std::vector<uint32_t> &t, const LdsGroup &G, int h, int k, int none, int base) {
        int bank[32] = {}, most = 0;
        for (int l = 32 * h; l < 32 * h + 32; ++l) {
            const int p = entry(t, G.table, k, l);
            if (p != none) most = std::max(most, ++bank[(p - base) % 32]);
        }
        if (most) load += most, gathers += 1.0;
    };
    for (const LdsGroup &G : T.row_group)
        for (int h = 0; h < 2; ++h)
            for (int k = 0; k < G.degree; ++k) half(T.rows, G, h, k, n, 0);
    for (const LdsGroup &G : T.bit_group)
        for (int h = 0; h < 2; ++h)
            for (int u = 0; u < G.degree; ++u) half(T.bits, G, h, u, T.npos, 0);
    std::printf("ok %.3f\n", load / gathers);
    return 0;
}
