// CPU check of the digits that row_dots.hip makes of a row's elements: every element of 24 significant bits whose last one is a
// whole number is the sum of its digits again, elements that are not are told apart, and sums of products are put together with one rounding.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "row_digits.h"

static uint64_t rng_state = 0x243F6A8885A308D3ull;
static uint32_t rnd() {
    rng_state ^= rng_state << 13;
    rng_state ^= rng_state >> 7;
    rng_state ^= rng_state << 17;
    return (uint32_t)(rng_state >> 16);
}

static int64_t value_of(uint32_t lo, uint32_t hi, int digit[7]) {
    int64_t v = 0;
    for (int k = 6; k >= 0; --k) {
        digit[k] = (int8_t)((k < 4 ? lo >> 8 * k : hi >> 8 * (k - 4)) & 0xFF);
        v = v * 256 + digit[k];
    }
    return v;
}

int main() {
    long checked = 0;
    int digit[7];
    uint32_t lo, hi;
    // mantissas of 24 bits whose last one stands at `shift`: all that are 0 to 15 modulo 16, beside the smallest and largest
    // ones, at random and next to half a digit's carry
    for (int shift = -30; shift <= 30; ++shift)
        for (int i = 0; i < 4000; ++i) {
            uint32_t m = i < 64 ? 0x800000u + (uint32_t)i : i < 128 ? 0xFFFFFFu - (uint32_t)(i - 64) : i < 192 ? 0xC00000u - 32 + (uint32_t)(i - 128)
                       : i < 256 ? (uint32_t)(i - 192) : (rnd() & 0xFFFFFFu);
            for (int sign = -1; sign <= 1; sign += 2) {
                const double v = sign * ldexp((double)m, shift);
                const bool whole = v == floor(v);
                hdc::digits_of(v, lo, hi);
                if (whole && (value_of(lo, hi, digit) != (int64_t)v || digit[6] < -64 || digit[6] > 64)) {
                    printf("shift %d mantissa %x sign %d: %lld\n", shift, m, sign, (long long)(value_of(lo, hi, digit) - (int64_t)v));
                    return 1;
                }
                ++checked;
            }
        }
    // floats beside a largest one, subnormal ones and zeros too: those that digits_hold says are whole numbers are
    for (int i = 0; i < 2000000; ++i) {
        uint32_t top_bits = rnd() & 0x7FFFFFFFu, x = rnd() & 0x7FFFFFFFu;
        if (i % 2) x = (top_bits >> 23 << 23) - (rnd() % 36 << 23) + (rnd() & 0x7FFFFFu);   // within 36 binades
        if (i % 5 == 0) x &= 0x807FFFFFu;
        if (i % 64 == 0) x = 0;
        if (i % 7 == 0) top_bits &= 0x10FFFFFFu;
        x &= 0x7FFFFFFFu;
        if (top_bits >= 0x7F800000u || x > top_bits) continue;
        float f;
        memcpy(&f, &x, 4);
        const uint32_t top = top_bits >> 23;
        const double v = (double)f * hdc::digits_scale(top);
        const bool holds = hdc::digits_hold(x - 1, top);
        if (v >= 0x1p54 || (holds && v != floor(v)) || (!holds && top >> 1 && v >= 0x1p24 && v == floor(v))) {
            printf("element %08x beside %08x: %g, said to %s\n", x, top_bits, v, holds ? "hold" : "not to");
            return 1;
        }
        ++checked;
    }
    // sums of 512 products with 1 and -1, of elements of one binade, of several and of one value alone
    for (int trial = 0; trial < 3000; ++trial) {
        int sum[7] = {};
        __int128 want = 0;
        for (int d = 0; d < 512; ++d) {
            const uint32_t m = trial % 3 == 2 ? 0xFFFFFFu : (rnd() & 0xFFFFFFu) | 0x800000u;
            const double v = ldexp((double)m, 30 - (trial % 3 == 1 ? (int)(rnd() % 31) : 0)) * (rnd() & 1 ? 1 : -1);
            hdc::digits_of(v, lo, hi);
            value_of(lo, hi, digit);
            const int s = trial % 5 == 0 ? (v < 0 ? -1 : 1) : (rnd() & 1 ? 1 : -1);
            for (int k = 0; k < 7; ++k) sum[k] += s * digit[k];
            want += s * (__int128)(int64_t)v;
        }
        const double got = hdc::sum_of_digits(sum[0] + 256 * sum[1], sum[2] + 256 * sum[3], sum[4] + 256 * sum[5], sum[6]);
        if (got != (double)want) {
            printf("trial %d: %.0f, not %.0f\n", trial, got, (double)want);
            return 1;
        }
        ++checked;
    }
    printf("OK %ld\n", checked);
    return 0;
}
