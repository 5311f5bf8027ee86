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

// ---- the encoder's fp16 product (coarse_half.hip) ----
// Exponent of the power of two that brings mx to [2^14, 2^15); at most 2^+-60, so that the product of two inverse scales
// stays in range (beyond that the squared norms of the rows overflow or vanish in fp32 as well).
VLQ_HD int half_exponent(float mx)
{
    uint32_t bits;
    __builtin_memcpy(&bits, &mx, 4);
    const int ex = mx > 0.f ? 14 - ((int)(bits >> 23) - 127) : 0;
    return ex < -60 ? -60 : (ex > 60 ? 60 : ex);
}
// Rows up to this many binades below their block's largest keep 18 binades of their own before a component is flushed, and
// their residual is that of the rounding alone; beyond, every row of the block gets a scale of its own.
#define HALF_GAP 10
// A column's residual counts relative to its norm up to this share, beyond it as it is (the two words of the header).
#define HALF_REL_MAX 5e-4f
// Bits of a key that hold the tile, and what planting them costs: a key moves by less than 2^(bits - 23) of its own size,
// and a key e = d - ||a||^2 is at most ||a||^2 + d in size; minimum and candidate both carry it.
VLQ_HD int half_idx_bits(int tiles)
{
    int bits = 1;
    while ((1 << bits) < tiles) ++bits;
    return bits;
}
VLQ_HD float half_band_dist(int bits) { return 2.5f * ldexpf(1.f, bits - 23); }

// Width of the band around the smallest distance dmin of a row a, xn = ||a||^2, res = ||a - a'||, for columns with
// ||b - b'|| <= max(rho ||b||, big).  One value ||b||^2 - 2 <a', b'> is off by at most
//   2 (res ||b|| + ||a'|| max(rho ||b||, big))      rounding to fp16 (Cauchy-Schwarz), ||a'|| <= 1.002 ||a||
//   + 4 D 2^-24 s^2                                 fp32 accumulation of D products onto half the column's norm (D roundings
//                                                   of at most ||b||^2 / 2 + |a||b|, doubled: 3 D 2^-24 s^2) and the
//                                                   norms' own rounding, |a|, |b| <= s
// and a comparison involves two.  ||b|| <= ||a|| + sqrt(d) <= s for the columns that matter: their distance exceeds dmin by
// no more than the values' error, for which s has a tenth to spare (and the term in big).  A row that lost more than 2^-9
// of its norm (squares at the ends of fp32's range) gets every column.
VLQ_HD float nn_half_band(float xn, float res, float rho, float big, float dmin, float band_dist, int D)
{
    const float na = sqrtf(xn);
    if (!(res <= 0x1p-9f * na)) return INFINITY;
    const float s = 1.1f * (na + sqrtf(dmin)) + 1.5f * sqrtf(na * big);
    return 4.f * ((res + 1.01f * rho * na) * s + 1.01f * na * big) + 8.f * (float)(D + 8) * 0x1p-24f * s * s +
           band_dist * (xn + dmin);
}
