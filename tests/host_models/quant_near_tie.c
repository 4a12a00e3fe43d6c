/* Host model of the quantiser's route for values near a tie: y = x * r, r a reciprocal of the scale that is up to one ulp off
 * R = fl32(1 / scale), corrected to y + (x - y * scale) * r with two FMAs, must be the IEEE quotient x / scale.  Every
 * bf16 amax in [lo, hi], every bf16 x in (0, amax] down to 2^-10 amax (the quotients below that are less than 1/8: code 0
 * by either route, and no tie is near).
 * out[0] = cases, out[1] = those within the guard of a tie, out[2] = cases whose quotient or code differs. */
#include <math.h>
#include <stdint.h>
#include <string.h>

static float bf16_bits_to_float(uint16_t b) {
    uint32_t u = (uint32_t)b << 16;
    float f;
    memcpy(&f, &u, 4);
    return f;
}

int model_near_tie_sweep(float lo, float hi, float guard, long *out) {
    long cases = 0, near_ties = 0, bad = 0;
#pragma omp parallel for schedule(dynamic, 16) reduction(+ : cases, near_ties, bad)
    for (int ab = 1; ab < 0x7f80; ++ab) {
        const float amax = bf16_bits_to_float((uint16_t)ab);
        if (!(amax >= lo && amax <= hi)) continue;
        const float scale = amax / 127.0f, R = 1.0f / scale;
        const float rs[3] = {nextafterf(R, 0.0f), R, nextafterf(R, INFINITY)};
        for (int xb = ab > 10 * 128 ? ab - 10 * 128 : 1; xb <= ab; ++xb) {
            const float x = bf16_bits_to_float((uint16_t)xb), want = x / scale;
            for (int k = 0; k < 3; ++k) {
                const float y = x * rs[k];
                const float got = fmaf(fmaf(-y, scale, x), rs[k], y);
                cases++;
                if (!(fabsf(y - rintf(y)) < 0.5f - guard)) near_ties++;
                if (got != want || (got + 12582912.0f) - 12582912.0f != rintf(want)) bad++;
            }
        }
    }
    out[0] = cases;
    out[1] = near_ties;
    out[2] = bad;
    return 0;
}
