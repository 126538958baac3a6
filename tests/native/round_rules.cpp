// Host-only checks of rules on a round's shape (built and run by
// tests/test_round_rules.py; no kernel is launched).
#include <cstdio>

#include "engine.h"
#include "sssp_internal.h"

using namespace sssp;

static int failures = 0;
#define CHECK(c)                                                        \
    do {                                                                \
        if (!(c)) {                                                     \
            std::fprintf(stderr, "FAILED line %d: %s\n", __LINE__, #c); \
            ++failures;                                                 \
        }                                                               \
    } while (0)

int main() {
    // rows are read by groups only while the groups' lines are fewer bytes than the rows'
    // parts, whatever the number of rows and partitions
    for (uint32_t bytes : {64u, 128u, 256u, 528u, 1024u, 16384u})
        for (int P : {1, 4, 16, 64})
            for (uint32_t m : {1u, 64u, 65u, 1000u, 25613u, 65536u})
                for (uint32_t ng = 0; ng <= 64; ++ng)
                    CHECK(!sparse_round(ng, m, P, bytes) || (ng * 128u <= bytes && m > 64u && ng <= kSparseGroups));
    // the stragglers of large dense graphs still are
    CHECK(sparse_round(1, 20628, 16, 1024) && sparse_round(8, 60421, 16, 1024));
    CHECK(sparse_round(4, 25613, 16, 528) && !sparse_round(5, 25613, 16, 528));
    // threads of the one-workgroup solve: literal steps take the fewest that hold the columns
    for (int n : {1, 128, 129, 300, 768, 769, 1000, 1024}) CHECK(single_threads(n, true) == 256);
    CHECK(single_threads(128, false) == 256 && single_threads(129, false) == 512);
    CHECK(single_threads(768, false) == 512 && single_threads(769, false) == 1024);
    for (int n : {1025, 5000, 16384}) CHECK(single_threads(n, true) == 1024 && single_threads(n, false) == 1024);
    if (failures) return 1;
    std::printf("round rules ok\n");
    return 0;
}
