// CPU driver of the launch rules (paper_1005_5198_amd/csrc/rs_launch.h), built with
// AddressSanitizer and UndefinedBehaviorSanitizer by tests/test_launch_rules.py.
// Reads one query per line from standard input and prints its answer.
#include "rs_launch.h"

#include <cinttypes>
#include <cstdio>
#include <cstring>

using namespace rs;

int main() {
    char what[32];
    while (scanf("%31s", what) == 1) {
        if (!strcmp(what, "queue_blocks")) {
            int64_t entries, per_block, cap;
            if (scanf("%" SCNd64 " %" SCNd64 " %" SCNd64, &entries, &per_block, &cap) != 3) return 1;
            printf("%" PRId64 "\n", queue_blocks(entries, per_block, cap));
        } else {
            return 1;
        }
    }
    return 0;
}
