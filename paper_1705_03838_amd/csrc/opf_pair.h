// Unevaluated sums of two doubles (Dekker 1971; products by multiply-add):
// about 106 bits.
//
// Every function turns contraction off: with it, which is hipcc's default, the
// sum of a product and its rounding error becomes one multiply-add, and the
// error is then counted twice (a product right to 53 bits).
#pragma once
#include <cmath>

#include <hip/hip_runtime.h>

namespace opf {

struct dd {
    double hi, lo;
};
__host__ __device__ inline dd two_sum(double a, double b) {
#pragma clang fp contract(off)
    const double s = a + b, t = s - a;
    return {s, (a - (s - t)) + (b - t)};
}
// s + a b, not renormalised: the low part takes the errors of the product and
// of the sum, so that a chain of these waits for one addition each.
__host__ __device__ inline dd madd(dd s, dd a, double b) {
#pragma clang fp contract(off)
    const double p = a.hi * b;
    const dd t = two_sum(s.hi, p);
    return {t.hi, t.lo + (s.lo + fma(a.lo, b, fma(a.hi, b, -p)))};
}

}  // namespace opf
