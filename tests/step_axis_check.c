/* The propagation kernel's step of one axis (step_axis) over its whole domain:
 * metres left 1 <= r < 2^16, rates 0 <= q <= 2^30, n >= 1 minutes left.  The
 * minute of arrival t = trunc(r * rcp(max(q, 1))), then t += (umul24(t, q) < r),
 * where umul24 multiplies the low 24 bits and the reciprocal is the correctly
 * rounded one or a neighbour; it counts if q > 0 and t <= n, else r loses
 * umul24(q, n).  Compared with whole-number arithmetic in 64 bits.  Prints the
 * cases checked and the failures. */
#include <math.h>
#include <stdint.h>
#include <stdio.h>

static uint32_t umul24(uint32_t a, uint32_t b) { return (uint32_t)((uint64_t)(a & 0xFFFFFFu) * (b & 0xFFFFFFu)); }

static long n_checked = 0, bad = 0;

static void check(int64_t r, int64_t q, int64_t n) {
    const int64_t want_t = q > 0 ? (r + q - 1) / q : 0;
    const int64_t want = q > 0 && want_t <= n ? want_t : 0;
    const int64_t want_left = want ? 0 : r - q * n;
    const uint32_t d = q > 1 ? (uint32_t)q : 1u;
    const float c = 1.0f / (float)d, rc[3] = {c, nextafterf(c, 0.0f), nextafterf(c, 2.0f)};
    for (int k = 0; k < 3; ++k) {
        uint32_t t = (uint32_t)((float)r * rc[k]);
        t += umul24(t, d) < (uint32_t)r;
        const int reach = q > 0 && (int64_t)t <= n;
        const int64_t got = reach ? (int64_t)t : 0;
        const int64_t left = reach ? 0 : (int64_t)(int32_t)((uint32_t)r - umul24((uint32_t)q, (uint32_t)n));
        ++n_checked;
        bad += got != want || left != want_left;
    }
}

int main(void) {
    const int64_t big[] = {65535, 65536, 65537, 131071, 131072, (1 << 24) - 1, 1 << 24, (1 << 24) + 1, (1 << 24) + 2,
                           (1 << 25) - 1, (1 << 25) + 65535, 123456789, (1 << 30) - 64, 1 << 30};
    const int64_t ns[] = {1, 2, 59, 60, 1440, 65535, (1 << 20) - 2};
    uint64_t s = 0x9E3779B97F4A7C15ull;
    for (int64_t r = 1; r < 65536; ++r) {
        for (unsigned k = 0; k < sizeof ns / sizeof *ns; ++k) {
            check(r, 0, ns[k]);
            check(r, 1, ns[k]);
            check(r, r - 1, ns[k]);
            check(r, r, ns[k]);
            check(r, r + 1, ns[k]);
            check(r, 2 * r - 1, ns[k]);
            check(r, 2 * r, ns[k]);
        }
        for (unsigned k = 0; k < sizeof big / sizeof *big; ++k) check(r, big[k], 1 + (int64_t)(r % 61));
        for (int k = 0; k < 40; ++k) {
            s ^= s << 13; s ^= s >> 7; s ^= s << 17;
            check(r, (int64_t)(s % ((1u << 30) + 1u)) >> (s >> 59), 1 + (int64_t)((s >> 33) % 1440));
        }
    }
    printf("%ld %ld\n", n_checked, bad);
    return 0;
}
