// ln_table.h - bucket centres of the heatmap kernels' natural logarithm: for m
// in [1, 2) and k the bucket of width 1 / kLnBuckets that holds it, c = 1 +
// (k + 1/2) / kLnBuckets, as ln c and 1 / c.
#pragma once

#include <cstdint>

namespace flock {

constexpr int kLnBuckets = 128;
struct LnTable {
    double ln_c[kLnBuckets], inv_c[kLnBuckets];
};

// The table is a constant of the program: ln c = 2 atanh(z), z = (c - 1) /
// (c + 1), by its series (z < 1/3: the terms fall by 9 each, 20 of them pass
// below 2^-65) in integers with 64 fractional bits, a few units of 2^-64 off
// and rounded once (the series in fp64 was up to 1.3e-16 off).  Filling it with
// the library's log in every workgroup took about 1.5 us of each.
constexpr LnTable make_ln_table() {
    static_assert(kLnBuckets == 128, "z below");
    using u128 = unsigned __int128;
    LnTable t{};
    for (int k = 0; k < kLnBuckets; ++k) {
        const int n = 2 * k + 1;  // c = 1 + n / 256
        const u128 z = ((u128)n << 64) / (512 + n), z2 = (z * z) >> 64;
        u128 sum = 0;
        for (int i = 19; i >= 0; --i) sum = ((sum * z2) >> 64) + ((u128)1 << 64) / (2 * i + 1);
        t.ln_c[k] = (double)(uint64_t)((z * sum) >> 63) * 0x1p-64;
        t.inv_c[k] = 256.0 / (256 + n);
    }
    return t;
}

}  // namespace flock
