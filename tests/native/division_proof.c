/* That the short division of the step kernels (reciprocal estimate, one Newton step on it, the quotient, one correction by its
 * residual; csrc/eco_device.hpp, div_rn_midrange) is correctly rounded for every pair of significands, checked pair by pair
 * where it could fail.
 *
 * The reciprocal estimate y0 is taken to be within 2 units in the last place of 1/d (the instruction is specified to 1): every
 * float that close is tried.  y1 = fma(fma(-d, y0, 1), y0, y0) is then within 2^-24 (1 + 2^-20) of 1/d relatively, q0 = RN(n y1)
 * within 1.6 units of n/d, and the sum q0 + RN(n - d q0) y1 before its last rounding within 1.6 (2^-24 + 2^-24) (1 + ...) < 2^-22
 * units: it can only round to the wrong side if n/d lies within 2^-22 units of the middle between two floats.  (Operands are
 * scaled by powers of two inside the kernels' ranges, where nothing under- or overflows: n, d in [1, 2) stand for all.)
 *
 * With d = D 2^-23 and n = N 2^-23 (D, N in [2^23, 2^24)) the middles are M 2^-24 (n >= d) or M 2^-25 (n < d), M odd, and
 *   | N 2^s - M D | = | j | <= 2 D 2^-22 < 8,   s = 24 or 25,
 * so the pairs in question are the solutions of N 2^s = j (mod D) for | j | <= 8: about one N in a million for each D.  The
 * program runs the sequence and the division on all of them and prints the pairs on which some estimate that close would give
 * a wrong quotient: what the instruction's estimate gives for those is for a test on the device to say. */
#include <math.h>
#include <stdint.h>
#include <stdio.h>

static int64_t inverse(int64_t a, int64_t m) {              /* a^-1 mod m, gcd(a, m) = 1 */
  int64_t r0 = m, r1 = a % m, t0 = 0, t1 = 1;
  while (r1) { const int64_t q = r0 / r1, r = r0 - q * r1, t = t0 - q * t1; r0 = r1; r1 = r; t0 = t1; t1 = t; }
  return t0 < 0 ? t0 + m : t0;
}

static float divide(float n, float d, float y1) {
  const float q0 = n * y1;
  const float r0 = fmaf(-d, q0, n);
  return fmaf(r0, y1, q0);
}

int main(void) {
  const int64_t LO = 1 << 23, HI = 1 << 24;
  int64_t pairs = 0, wrong = 0, worst = 0;
#pragma omp parallel for schedule(dynamic, 4096) reduction(+ : pairs, wrong) reduction(max : worst)
  for (int64_t D = LO; D < HI; ++D) {
    const float d = (float)D * 0x1p-23f;
    /* the reciprocals that may come out of the Newton step */
    float y1[8];
    int ny = 0;
    const float near = 1.0f / d;
    float y0 = near;
    for (int k = 0; k < 3; ++k) y0 = nextafterf(y0, 0.0f);
    for (int k = 0; k < 7; ++k, y0 = nextafterf(y0, 2.0f)) {
      const float unit = D == LO ? 0x1p-23f : 0x1p-24f;      /* of 1/d, in (1/2, 1] */
      if (fabs((double)y0 - 1.0 / (double)d) > 2 * (double)unit) continue;
      const float y = fmaf(fmaf(-d, y0, 1.0f), y0, y0);
      /* its distance from 1/d in units of 2^-24 / d, to the nearest thousandth: the bound above allows 1 */
      const double off = fabs((double)y * (double)d - 1.0) * 0x1p24;
      const int64_t thousandths = (int64_t)(off * 1000 + 0.5);
      if (thousandths > worst) worst = thousandths;
      int known = 0;
      for (int i = 0; i < ny; ++i) known |= y1[i] == y;
      if (!known) y1[ny++] = y;
    }
    int64_t odd = D, two = 1;
    while (odd % 2 == 0) { odd /= 2; two *= 2; }
    for (int s = 24; s <= 25; ++s) {
      /* N 2^s = j (mod D): two divides j, and N is fixed modulo `odd` */
      const int64_t inv = odd == 1 ? 0 : inverse((1ll << s) % odd, odd);
      for (int64_t j = -8; j <= 8; ++j) {
        if (j == 0 || j % two) continue;
        int64_t N = odd == 1 ? 0 : (((j % odd) + odd) % odd) * inv % odd;
        N += (LO - N + odd - 1) / odd * odd;
        for (; N < HI; N += odd) {
          if ((s == 24) != (N >= D)) continue;
          if ((((N << s) - j) / D) % 2 == 0 || ((N << s) - j) % D) continue;      /* M odd: a middle, not a float */
          const float n = (float)N * 0x1p-23f, want = n / d;
          for (int i = 0; i < ny; ++i) {
            ++pairs;
            if (divide(n, d, y1[i]) != want) {
              ++wrong;
#pragma omp critical
              printf("open %lld %lld\n", (long long)N, (long long)D);
            }
          }
        }
      }
    }
  }
  printf("%lld pairs, %lld open, reciprocal off by %.3f\n", (long long)pairs, (long long)wrong, (double)worst / 1000);
  return worst > 1001;                                       /* the bound that the choice of pairs rests on */
}
