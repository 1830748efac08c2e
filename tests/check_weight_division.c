/* Host check of the weight quantizer's quotient: v is any float and s > 0 an fp16 value, r = fl(1/s),
 *     q0 = fl(v * r),  rem = fma(-q0, s, v),  q = fma(rem, r, q0)
 * equals the IEEE quotient fl(v / s), and so does the code it rounds to.  Tried for every s: the
 * floats within four places of every (n + 0.5) s, where a wrong last bit would change a code, and
 * seeded random v of either sign from far below s to 33 s.  Where v / s underflows only the code
 * is compared (it is 0).  Prints the numbers of pairs and of mismatches; exit status 1 on any. */
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

static float half_value(int bits)
{
    const int e = (bits >> 10) & 31, m = bits & 1023;
    return e == 0 ? ldexpf((float)m, -24) : ldexpf((float)(m + 1024), e - 25);
}

static int code(float q)
{
    const float c = rintf(q);
    return (int)(c < -32.0f ? -32.0f : c > 31.0f ? 31.0f : c);
}

static int differs(float v, float s, float r)
{
    const float q0 = v * r;
    const float rem = fmaf(-q0, s, v);
    const float q = fmaf(rem, r, q0), want = v / s;
    return code(q) != code(want) || (fabsf(want) >= 1e-30f && q != want);
}

static float bits_float(uint32_t b)
{
    float f;
    memcpy(&f, &b, 4);
    return f;
}

int main(void)
{
    long pairs = 0, wrong = 0;
#pragma omp parallel for reduction(+ : pairs, wrong) schedule(dynamic, 64)
    for (int sb = 1; sb <= 0x7bff; ++sb) {
        const float s = half_value(sb), r = 1.0f / s;
        for (int n = -33; n <= 32; ++n) {
            const float middle = ((float)n + 0.5f) * s;
            uint32_t b;
            memcpy(&b, &middle, 4);
            for (int d = -4; d <= 4; ++d) {
                ++pairs;
                wrong += differs(bits_float(b + (uint32_t)d), s, r);
            }
        }
        uint64_t x = 0x9E3779B97F4A7C15ull * (uint64_t)sb + 1;
        for (int i = 0; i < 1000; ++i) {
            x ^= x << 13;
            x ^= x >> 7;
            x ^= x << 17;
            /* 24 random bits scaled to 33 s, every eighth value down to 2^-40 of that and below */
            float v = (float)(int32_t)(uint32_t)x * 0x1p-31f * 33.0f * s;
            if ((x >> 32) % 8 == 0) v = ldexpf(v, -(int)((x >> 40) % 140));
            ++pairs;
            wrong += differs(v, s, r);
        }
    }
    printf("%ld %ld\n", pairs, wrong);
    return wrong != 0;
}
