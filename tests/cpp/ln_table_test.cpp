// Host test of the heatmap kernels' logarithm table: ln c within 0.6e-16 (half
// a unit of the last place at the table's end is 0.56e-16) and 1 / c correctly
// rounded, against the 80-bit logarithm.
#include <cmath>
#include <cstdio>

#include "ln_table.h"

int main() {
    constexpr flock::LnTable t = flock::make_ln_table();
    for (int k = 0; k < flock::kLnBuckets; ++k) {
        const long double c = 1.0L + ((long double)k + 0.5L) / flock::kLnBuckets;
        if (std::fabs(t.ln_c[k] - std::log(c)) > 0.6e-16L || t.inv_c[k] != 1.0 / (double)c) {
            std::printf("bucket %d: ln off by %Lg\n", k, t.ln_c[k] - std::log(c));
            return 1;
        }
    }
    std::puts("ln table ok");
    return 0;
}
