// Nearest of up to 256 codewords for the 64 vectors of a wave, on the fp32 matrix cores (Lloyd iterations of the codebooks of
// the product quantiser).
//
// A direct distance costs two vector instructions a dimension, 36 with the comparison for 16 dimensions.  Here the matrix
// cores form ||c||^2 / 2 - <x, c> in fp32 (v_mfma_f32_16x16x4_f32: rows = 16 codewords, columns = 16 vectors, the norms
// being what the products are added to), a lane sees four codewords of its vector at a time and keeps the two smallest of
// the fours' minima: six vector instructions for four codewords.  The four codewords of the smallest are then compared by
// their direct distances; where the second smallest is so close that another one could have the smallest direct distance,
// the vector's codewords are all compared directly.  So the choice is that of the direct fp32 distances, ties to the smaller
// index.  Bound by the MFMAs (32 clocks for four dimensions of 16 x 16 pairs).
#pragma once
#include "common.h"

// Vectors and codewords are taken relative to a point among the codewords (`mu`; each difference is rounded once, relative to
// itself), so that the error does not grow with their distance from the origin.
//
// How far the second smallest value has to lie above the smallest, v, in halves of squared distances, for a vector of squared
// norm xn = x^2 and codewords of norms up to c: twice the error of a value (DS + 2 roundings of at most c^2 / 2 + x c, and
// the norm's own DS of c^2 / 2), what the direct distances (DS + 1 roundings of (x + c)^2 each) can differ by, and the
// rounding of the differences (one of (x + c)^2 in each value).  Below the normal range roundings are no longer relative to
// the values: up to 2^-126 an operation, where the matrix cores flush, times the 2 (3 DS + 4) operations of two values and
// two distances.
// c is the largest norm that matters, not the largest there is (with that, one codeword at 30 times the usual norm left 9 % of
// the vectors undecided, at 100 times 64 %): d being the distance of v's codeword, its norm is at most x + d, and
// s = x + sqrt(2 v + x^2) differs from that by the root of v's error, 4e-3 s at most.  A codeword beyond 1.1 s is 0.09 s
// farther from the vector than d: it is not the nearest, whatever its value.
__device__ __forceinline__ float codeword_band(int ds, float xn, float v, float cmax)
{
    // (the hardware's root: what it is off by at most, and what it flushes, is far below the slack of s and of the band)
    const float x = __builtin_amdgcn_sqrtf(xn), s = x + __builtin_amdgcn_sqrtf(fmaxf(fmaf(2.f, v, xn), 0.f));
    const float c = fminf(cmax, 1.1f * s);
    return 4.f * (float)(ds + 8) * 0x1p-24f * (x + c) * (x + c) + 0x1p-119f;
}

// a row of DS floats, in 16-byte pieces where `vec` says that it lies on 16 bytes
template <int DS>
__device__ __forceinline__ void load_row(const float *w, bool vec, float (&r)[DS])
{
    if (DS % 4 == 0 && vec) {
#pragma unroll
        for (int d = 0; d + 3 < DS; d += 4) {
            const f32x4 v = *(const f32x4 *)(w + d);
#pragma unroll
            for (int e = 0; e < 4; ++e) r[d + e] = v[e];
        }
    } else {
#pragma unroll
        for (int d = 0; d < DS; ++d) r[d] = w[d];
    }
}

// half[256]: ||W_t||^2 / 2 of the codewords, CODEWORD_NONE for those that do not count (beyond k, or with a component that
// is not finite); cmax: largest norm of the others, infinite where a squared norm overflows.  Then the products say nothing
// (the direct distances to such a codeword may be finite all the same), and nor do they where all coincide or their squares
// are below the normal range: every vector is compared directly.
#define CODEWORD_NONE 3e38f
// Undecided vectors of a wave up to which they are compared one by one, all lanes a vector, instead of every lane walking all
// codewords.  One pass over 262 144 vectors, k = 256, at 12 / 24 / 36 / 50, us: D = 16, whole-number vectors 134 / 125 / 121 /
// 124, a sixteenth of the codewords there twice 141 / 124 / 124 / 125, groups of eight close codewords 161 / 161 / 161 / 192;
// D = 8, those groups 135 / 136 / 157 / 169.
#define CODEWORD_OPEN 24
// Wt: the codewords component by component, `stride` floats a component, 16 ceil(k / 16) of them readable (codeword by
// codeword a wave's load touched 64 places, and those loads took three times as long as the products).
// mu(d): component d of the point.  x(v, d): component d of the wave's vector v (0 .. 63).  exact(v, t): direct distance of vector v to codeword t, by any lane.
// all(v): the nearest codeword of vector v among all (v uniform, all lanes take part); walk(): the same for vector `lane`, for
// when more than CODEWORD_OPEN of the 64 are undecided.  Returns the codeword of vector `lane`.
template <int DS, typename Mu, typename X, typename Exact, typename All, typename Walk>
__device__ __forceinline__ int nearest_codeword64(const float *Wt, int stride, int k, const float *half, float cmax, int lane, Mu mu, X x,
                                                  Exact exact, All all, Walk walk)
{
    if (!(cmax < INFINITY && cmax > 0x1p-50f)) return walk();
    constexpr int KS = (DS + 3) / 4, NB = 4; // blocks of 16 vectors
    const int col = lane & 15, grp = lane >> 4;
    float xb[NB][KS], b1[NB], b2[NB], xs[NB];
    int four[NB];
    float ms[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) ms[s] = mu(min(4 * s + grp, DS - 1));
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        float xn = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int d = 4 * s + grp;
            const float v = DS % 4 == 0 || d < DS ? x(16 * i + col, min(d, DS - 1)) - ms[s] : 0.f;
            xb[i][s] = -v;
            xn = fmaf(v, v, xn);
        }
        xn += __shfl_xor(xn, 16, 64);
        xn += __shfl_xor(xn, 32, 64);
        xs[i] = xn;
        b1[i] = b2[i] = INFINITY;
        four[i] = 0;
    }
    const int blocks = (k + 15) / 16;
    auto fetch = [&](int j, float (&a)[KS]) {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int d = 4 * s + grp;
            a[s] = Wt[min(d, DS - 1) * stride + 16 * j + col] - ms[s];
            if (DS % 4 && d >= DS) a[s] = 0.f;
        }
    };
    float a[KS], an[KS];
    fetch(0, a);
#pragma unroll 1
    for (int j = 0; j < blocks; ++j) {
        fetch(min(j + 1, blocks - 1), an);
        const f32x4 c = *(const f32x4 *)(half + 16 * j + 4 * grp);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            f32x4 acc = c;
#pragma unroll
            for (int s = 0; s < KS; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], xb[i][s], acc, 0, 0, 0);
            const float m = __builtin_elementwise_minimum(__builtin_elementwise_minimum(__builtin_elementwise_minimum(acc[0], acc[1]), acc[2]), acc[3]);
            four[i] = m < b1[i] ? j : four[i];
            b2[i] = __builtin_amdgcn_fmed3f(b1[i], b2[i], m);
            b1[i] = fminf(b1[i], m);
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) a[s] = an[s];
    }
    int mine = 0;
    uint64_t open = 0; // vectors that are not decided, 16 a block
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        // over the four lanes of a vector: the smallest, whose it is, and the second smallest
        int at = 4 * four[i] + grp;
#pragma unroll
        for (int o = 16; o <= 32; o <<= 1) {
            const float p1 = __shfl_xor(b1[i], o, 64), p2 = __shfl_xor(b2[i], o, 64);
            const int pa = __shfl_xor(at, o, 64);
            b2[i] = fminf(fmaxf(b1[i], p1), fminf(b2[i], p2));
            at = p1 < b1[i] ? pa : at;
            b1[i] = fminf(b1[i], p1);
        }
        const bool clear = b2[i] - b1[i] > codeword_band(DS, xs[i], b1[i], cmax); // (false for values that are not numbers)
        // (where two are equal the lanes may name different fours, but then it is not clear)
        const int t = 4 * at + grp;
        const float d = exact(16 * i + col, min(t, k - 1));
        uint64_t key = t < k && d < INFINITY ? make_key(d, (uint32_t)t) : KEY_MAX;
        uint64_t other = shfl_xor_u64(key, 16);
        key = other < key ? other : key;
        other = shfl_xor_u64(key, 32);
        key = other < key ? other : key;
        const int best = key == KEY_MAX ? 0 : (int)(uint32_t)key;
        open |= (__ballot(!clear) & 0xFFFFull) << (16 * i);
        if (grp == i) mine = best;
        __builtin_amdgcn_sched_barrier(0); // (one block's rows in registers at a time)
    }
    if (__popcll(open) > CODEWORD_OPEN) return walk();
    while (open) {
        const int v = __ffsll((unsigned long long)open) - 1;
        open &= open - 1;
        const int got = all(v);
        if (lane == v) mine = got;
    }
    return mine;
}
