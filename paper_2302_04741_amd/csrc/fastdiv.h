// Index arithmetic of the kernels: unsigned 32-bit division by a divisor fixed at
// launch, the periodic wrap of a streaming shift and quotients by a common divisor; no
// HIP dependency (CPU tests check them).
#pragma once

#include <stdint.h>

namespace lbm {

// n / d as a multiply-high and two shifts (Granlund and Montgomery, "Division
// by invariant integers using multiplication", 1994, Fig. 4.1): for d >= 1,
// l = ceil(log2 d), m = floor(2^32 (2^l - d) / d) + 1, and every n < 2^32
// gives n / d = (t + ((n - t) >> min(l, 1))) >> max(l - 1, 0) with
// t = mulhi(n, m).  On a uniform n all of it runs on the scalar unit (an
// integer division would expand into vector-unit reciprocal code).
struct DivU32 {
    uint32_t m, s1, s2;
};

// d >= 1 (grid extents are validated before; 0 is taken as 1)
inline DivU32 make_divu32(uint32_t d)
{
    if (d == 0) d = 1;
    uint32_t l = 0;
    while ((uint64_t(1) << l) < d) ++l;
    const uint64_t m = ((uint64_t(1) << 32) * ((uint64_t(1) << l) - d)) / d + 1;
    return DivU32{uint32_t(m), l < 1 ? l : 1u, l > 1 ? l - 1 : 0u};
}

__host__ __device__ inline uint32_t divu(const DivU32 &q, uint32_t n)
{
    const uint32_t t = uint32_t((uint64_t(n) * q.m) >> 32);  // mulhi(n, m)
    return (t + ((n - t) >> q.s1)) >> q.s2;
}

// d mod n for a shift d of 1..3 nodes and any n >= 1
__host__ __device__ inline uint32_t shift_mod(uint32_t d, uint32_t n)
{
    return d < n ? d : (n == 2 ? d & 1u : 0u);
}

// (v - d) mod n for v in [0, n), |d| <= 3, 1 <= n <= 2^31: the shift is taken
// modulo n first (on the scalar unit), so one correction is left, and of its two
// candidates the unsigned smaller is the one in [0, n).  No branch: a loop or a
// test on n < 4 here cost a wavefront some 40 instructions for each of 14 shifts.
__host__ __device__ inline uint32_t wrap_back(uint32_t v, int d, uint32_t n)
{
    if (d == 0) return v;
    const uint32_t m = shift_mod(uint32_t(d < 0 ? -d : d), n);
    const uint32_t s = d > 0 ? v - m : v + m;
    const uint32_t t = d > 0 ? s + n : s - n;
    return s < t ? s : t;
}

// m / d, correctly rounded, for several m over one d: inv is 1.0 / d, correctly rounded,
// and one correction of m inv with the exact remainder gives the rounded quotient
// (Markstein, "Computation of elementary functions on the IBM RISC System/6000
// processor", 1990).  Finite m and d, d and the quotient normal.
__host__ __device__ inline double quotient(double m, double d, double inv)
{
    const double q = m * inv;
    return __builtin_fma(__builtin_fma(-q, d, m), inv, q);
}

}  // namespace lbm
