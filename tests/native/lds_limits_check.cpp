// Host cost of the LDS-resident decoder's tables (csrc/lds_tables.hip).
//   column M N   M rows of two bits, the first bit in all of them: prints the
//                host memory in MB that building the tables took at its peak
//   limit LDS    the (4,8) shape of 16,000 bits: prints whether the tables are
//                built with no limit and with LDS bytes
#include <sys/resource.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "ldpc_internal.h"

static long peak_kb() {
    rusage u{};
    getrusage(RUSAGE_SELF, &u);
    return u.ru_maxrss;
}

int main(int argc, char **argv) {
    std::vector<int32_t> rowptr{0}, col;
    LdsHostTables T;
    if (argc == 4 && !std::strcmp(argv[1], "column")) {
        const int32_t m = std::atoi(argv[2]), n = std::atoi(argv[3]);
        for (int32_t i = 0; i < m; ++i) {
            col.push_back(0);
            col.push_back(1 + i % (n - 1));
            rowptr.push_back((int32_t)col.size());
        }
        const long before = peak_kb();
        if (!ldpc::lds_tables(rowptr, col, std::vector<int32_t>(m, 0), m, n, &T, 160 * 1024)) return 1;
        std::printf("%.1f\n", (peak_kb() - before) / 1024.0);
        return 0;
    }
    if (argc == 3 && !std::strcmp(argv[1], "limit")) {
        const int32_t n = 16000, m = 8000;
        for (int32_t i = 0; i < m; ++i) {
            for (int32_t k = 0; k < 8; ++k) col.push_back(2000 * k + i % 2000); // ascending
            rowptr.push_back((int32_t)col.size());
        }
        const std::vector<int32_t> cls(m, 0);
        const bool all = ldpc::lds_tables(rowptr, col, cls, m, n, &T);
        std::printf("%d %d\n", all, ldpc::lds_tables(rowptr, col, cls, m, n, &T, (size_t)std::atol(argv[2])));
        return 0;
    }
    return 2;
}
