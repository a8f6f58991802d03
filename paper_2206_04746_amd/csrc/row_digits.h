// Elements of class rows as signed digits of 8 bits (row_dots.hip); also compiled on its own by the CPU tests.
#pragma once

#include <math.h>
#include <stdint.h>
#include <string.h>

#if defined(__HIPCC__)
#define HDC_BOTH __host__ __device__
#else
#define HDC_BOTH
#endif

namespace hdc {

// The signed digits of v, |v| < 2^54, a float times a power of two: byte k of (lo, hi) is digit k, seven of them; all of v if it is a
// whole number.  A double that is a whole number k more than 1.5 x 2^52 has the bits of that and k more, in 64 bits: so the halves are
// put together whichever way the upper one was rounded.  (Converting a lower half of +2^31 to 32 bits, as ties leave it, is not defined.)
HDC_BOTH inline void digits_of(double v, uint32_t &lo, uint32_t &hi) {
    const double big = 0x1.8p52, upper = fma(v, 0x1p-32, big), lower = fma(upper - big, -0x1p32, v) + big;
    uint64_t u, l;
    memcpy(&u, &upper, 8);
    memcpy(&l, &lower, 8);
    const uint64_t whole = (u << 32) + l + (0x80808080808080ull - 0x4338000000000000ull);   // byte k less 128 is digit k
    lo = (uint32_t)whole ^ 0x80808080u;
    hi = (uint32_t)(whole >> 32) ^ 0x808080u;
}

// An element x (its bits) relative to the largest of its slice, whose exponent field is `top`: below 2^54.
HDC_BOTH inline double digits_scale(uint32_t top) { return ldexp(1.0, 54 + 126 - (top > 1 ? (int)top : 1)); }
// Whether the digits hold every element for sure: `least` is the smallest of (x & 0x7FFFFFFF) - 1, zeros last.  Then each is
// at least 2^-31 of the largest one's power of two, and its 24 bits are whole.
HDC_BOTH inline bool digits_hold(uint32_t least, uint32_t top) { return top <= 31 || least + 1 >= (top - 30) << 23 || least == 0xFFFFFFFFu; }

// Digits 2 k and 2 k + 1 of a sum of up to 512 products together, the four pairs put together: a whole number below 2^63, rounded once.
HDC_BOTH inline double sum_of_digits(int32_t s01, int32_t s23, int32_t s45, int32_t s6) {
    return fma(fma(fma((double)s6, 65536.0, (double)s45), 65536.0, (double)s23), 65536.0, (double)s01);
}

}  // namespace hdc
