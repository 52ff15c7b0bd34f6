// Division of page and block numbers by a divisor that is fixed for a whole call, as one multiplication: the
// quotient is made per lane in the decoder, where the compiler's own 32-bit division costs about 20 vector
// instructions and the multiplication three.
#pragma once
#include <stdint.h>

namespace kvc {

struct FastDiv {
    uint32_t mul, shift;
};

// n / d == mulhi(2 n, mul) >> shift for every n < 2^31 and 1 <= d <= 2^31: with 2^(L-1) < d <= 2^L and
// mul = ceil(2^(31+L) / d) the product n * mul / 2^(31+L) exceeds n / d by less than n / (d * 2^31) < 1 / d.
inline FastDiv make_fast_div(uint32_t d) {
    uint32_t L = 0;
    while ((1ull << L) < d) ++L;
    FastDiv r;
    r.mul = (uint32_t)(((1ull << (31 + L)) + d - 1) / d);
    r.shift = L;
    return r;
}

#ifdef __HIPCC__
__host__ __device__
#endif
inline uint32_t fast_div(uint32_t n, FastDiv f) {
    return (uint32_t)(((uint64_t)(n << 1) * f.mul) >> 32) >> f.shift;
}

}  // namespace kvc
