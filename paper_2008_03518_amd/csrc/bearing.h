// bearing.h -- horizontal distance to the goal and direction of the bearing
// from one approximate reciprocal square root (internal; plain arithmetic,
// also compiled for the host).
//
// The states of a run follow one behind the other, each behind a square root
// and two divisions; one chain from one seed, without their scaling, is
// shorter than the three.  The results are rounded as theirs are:
// Goldschmidt's iteration and two exact remainders give the square root; the
// reciprocal of the rounded distance, refined once more against it, is the
// correctly rounded one (but for a chance of about 2^-37), and with such a
// reciprocal one exact remainder rounds a quotient correctly (Markstein 1990).
// (With the iteration's own 1 / br, good to about 2^-45, a quotient within
// 2^-90 of the middle between two doubles could round to the other side.)
// The caller sees to it that r2 is far from the ends of the exponent range.
#pragma once

namespace fmdp {

struct Bearing {
    double br, inv;                                    // sqrt(r2), 1 / br
};

// y: 1 / sqrt(r2) to about 2^-22.  (F: double; a constexpr template is a
// function of the host and the device.)
template <typename F>
constexpr Bearing bearing(F r2, F y) {
    F a = r2 * y, h = 0.5 * y;
    const F e = __builtin_fma(-h, a, 0.5);
    a = __builtin_fma(a, e, a);
    h = __builtin_fma(h, e, h);
    a = __builtin_fma(__builtin_fma(-a, a, r2), h, a);
    const F br = __builtin_fma(__builtin_fma(-a, a, r2), h, a);
    const F inv = h + h;
    return Bearing{br, __builtin_fma(__builtin_fma(-br, inv, 1.0), inv, inv)};
}

// b / br, |b| <= br.
template <typename F>
constexpr F bearing_quotient(F b, const Bearing &v) {
    const F q = b * v.inv;
    return __builtin_fma(__builtin_fma(-v.br, q, b), v.inv, q);
}

}  // namespace fmdp
