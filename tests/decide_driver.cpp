// CPU driver of the far-field ray kernel's pixel decision (paper_1005_5198_amd/csrc/rs_decide.h),
// built with UndefinedBehaviorSanitizer, conversions of floating-point values that do not fit
// among its checks, by tests/test_decide.py. Reads lines of u v Mu Mv npx npy and prints the pixel.
#include "rs_decide.h"

#include <cinttypes>
#include <cstdio>
#include <cstdlib>

int main() {
    char w[4][64];
    int64_t npx, npy;
    while (scanf("%63s %63s %63s %63s %" SCNd64 " %" SCNd64, w[0], w[1], w[2], w[3], &npx, &npy) == 6)
        printf("%d\n", rs::pixel_inside(strtod(w[0], nullptr), strtod(w[1], nullptr), strtod(w[2], nullptr),
                                        strtod(w[3], nullptr), npx, npy));
    return 0;
}
