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
        } else if (!strcmp(what, "recheck_in_one")) {
            int64_t rays, n_lens;
            int several, is_crowded;
            if (scanf("%" SCNd64 " %" SCNd64 " %d %d", &rays, &n_lens, &several, &is_crowded) != 4) return 1;
            printf("%d\n", recheck_in_one(rays, n_lens, several != 0, is_crowded != 0) ? 1 : 0);
        } else if (!strcmp(what, "default_shape")) {
            int mixed;
            int64_t patches, cus;
            if (scanf("%d %" SCNd64 " %" SCNd64, &mixed, &patches, &cus) != 3) return 1;
            printf("%d\n", default_shape(mixed != 0, patches, cus));
        } else if (!strcmp(what, "tune_sample")) {
            int64_t W, H, n_lens, rays;
            if (scanf("%" SCNd64 " %" SCNd64 " %" SCNd64 " %" SCNd64, &W, &H, &n_lens, &rays) != 4) return 1;
            const TuneSample s = tune_sample(W, H, n_lens, rays);
            printf("%" PRId64 " %" PRId64 "\n", s.rows, s.lenses);
        } else if (!strcmp(what, "first_patch")) {
            uint32_t block, n_blocks;
            int turn;
            if (scanf("%" SCNu32 " %" SCNu32 " %d", &block, &n_blocks, &turn) != 3) return 1;
            printf("%" PRId64 "\n", first_patch(block, n_blocks, turn));
        } else if (!strcmp(what, "ticket_patch")) {
            uint32_t ticket, n_blocks;
            if (scanf("%" SCNu32 " %" SCNu32, &ticket, &n_blocks) != 2) return 1;
            printf("%" PRId64 "\n", ticket_patch(ticket, n_blocks));
        } else if (!strcmp(what, "crowded")) {
            int64_t nx, ny, n_lens;
            if (scanf("%" SCNd64 " %" SCNd64 " %" SCNd64, &nx, &ny, &n_lens) != 3) return 1;
            printf("%d\n", crowded(nx, ny, n_lens) ? 1 : 0);
        } else if (!strcmp(what, "entry_run")) {
            uint32_t entries, n_waves;
            if (scanf("%" SCNu32 " %" SCNu32, &entries, &n_waves) != 2) return 1;
            printf("%" PRIu32 "\n", entry_run(entries, n_waves));
        } else {
            return 1;
        }
    }
    return 0;
}
