// Arithmetic that kernels rely on and that is checked on the CPU as well: plain C, no device types.
#pragma once
#include <math.h>
#include <stdint.h>

#ifdef __HIPCC__
#define VLQ_HD __attribute__((host)) __attribute__((device, always_inline)) static inline
#else
#define VLQ_HD static inline
#endif

// ---- places of k_scan_wide (scan_wide.hip) ----
// The points of a workgroup's lists are laid end to end and handed out in turns of SW_TURN places.  A workgroup can
// meet every stored point, up to 2^31 - 1, so the places one past the last turn need the 32nd bit.
#define SW_NT 512              // threads of a workgroup
#define SW_U 4                 // chunks of 64 points per wave and turn
#define SW_TURN (SW_NT * SW_U) // points per workgroup and turn
typedef uint32_t sw_place_t;

VLQ_HD sw_place_t sw_wave_base(sw_place_t turn, int wave) { return turn + (sw_place_t)wave * (64u * SW_U); }
VLQ_HD sw_place_t sw_place(sw_place_t base, int u, int lane) { return base + 64u * (sw_place_t)u + (sw_place_t)lane; }

// How far the one-table distance of k_scan_wide can be from the 2m-lookup one (k_scan) of the same point.  Upper bounds:
// R2 of a = ||y - c_i||^2, Y2 of ||y - mu||^2, Q2 of ||q2||^2, e2 of c = ||s_ij - c_i||^2 over what the workgroup meets,
// L of |l|.  With u = 2^-24, by Cauchy's inequality and |q1 - mu| <= Y + R + L e, summand by summand:
//   a and c are sums of D squares, (D + 2) u each, c with weight L^2 + L inside s_x;
//   l is rounded three times in fp32 and once in fp64 (s_x): 3 L (2 L + 1) e^2 + 6 L e Q;
//   s_x, s_x - ts, b - a, l (b - a), a + l (b - a), their sum, and the two thresholds it is compared with: 8 roundings of
//   values of at most M1;
//   ts: y - mu rounded, D/m products a sub-space, m sub-spaces: 2 (D/m + m + 1) Y Q;
//   2m-lookup form: (D/m + m + 4) (R + Q)^2 of the sum of A, 2 L (D/m + m + 1) e Q of the sum of B, and 3 roundings of
//   values of at most M2.
// g is the same number in both.  (One per cent more for the roundings of the bounds themselves, and what denormal
// results may lose.)
VLQ_HD float scan_wide_slack(float R2, float Y2, float Q2, float e2, float L, int D, int m)
{
    const float R = sqrtf(R2), Y = sqrtf(Y2), Q = sqrtf(Q2), e = sqrtf(e2), k = (float)(D / m + m);
    const float M1 = Q2 + 2.f * (2.f * Y + R + L * e) * Q + (L * L + 2.f * L) * e2 + 2.f * L * R * e + R2;
    const float M2 = (R + Q) * (R + Q) + L * L * e2 + 2.f * L * e * (Q + R);
    const float sum = (float)(D + 2) * (R2 + (L * L + L) * e2) + 3.f * L * (2.f * L + 1.f) * e2 + 6.f * L * e * Q + 8.f * M1 +
                      2.f * (k + 1.f) * Y * Q + (k + 4.f) * (R + Q) * (R + Q) + 2.f * L * (k + 1.f) * e * Q + 3.f * M2;
    return 1.01f * 5.9604645e-8f * sum + (float)(D + m + 16) * 4.7e-38f;
}
