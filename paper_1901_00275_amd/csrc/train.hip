// Lloyd iterations (k-means) for the codebooks of Sec. 2.1 / Sec. 3.1: the update half.
// The assignment half is the nearest-centroid search of the encoder (coarse_bf16.hip /
// coarse.hip + k_encode_finish in nearest-only mode); small codebooks of few dimensions (the
// sub-spaces of the product quantiser) take k_lloyd_lanes, which does both halves in one pass.
//
// Member sums are accumulated in 64-bit fixed point, so the result does not depend on the
// order in which the atomics land: x is scaled by 2^shift / s, s = the smallest power of two
// >= max |x| over the sample, shift = 62 - ceil(log2(points)); the sum of all members cannot
// overflow and the resolution is s * 2^-shift (2^-38 s for 16 M points).
#include "codeword.h"
#include <type_traits>

// One atomic per workgroup at most, and only if the workgroup has something larger to report than what is
// there already: an atomic per wave on the one address took 0.20 ms for a sample of 16 MB.
__global__ __launch_bounds__(256) void k_absmax(const float *__restrict__ X, int64_t count, uint32_t *__restrict__ out)
{
    __shared__ uint32_t part[4];
    uint32_t m = 0;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += stride) {
        const uint32_t u = __float_as_uint(X[i]) & 0x7FFFFFFFu;
        if (u < 0x7F800000u) m = max(m, u); // finite values only
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, 64));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        m = max(max(part[0], part[1]), max(part[2], part[3]));
        if (m > *(volatile uint32_t *)out) atomicMax(out, m);
    }
}

void launch_absmax(const float *X, int64_t count, uint32_t *out_bits, hipStream_t st)
{
    if (count <= 0) return;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 2048) blocks = 2048; // eight workgroups per compute unit
    hipLaunchKernelGGL(k_absmax, dim3((unsigned)blocks), dim3(256), 0, st, X, count, out_bits);
}

// power of two >= the largest magnitude (1 for an all-zero sample)
__device__ __forceinline__ double scale_of(uint32_t absmax_bits)
{
    const float m = __uint_as_float(absmax_bits);
    if (!(m > 0.f)) return 1.0;
    int e;
    frexpf(m, &e); // m = f * 2^e, 0.5 <= f < 1
    return ldexp(1.0, e);
}

// one thread per (vector, dimension)
__global__ __launch_bounds__(256) void k_kmeans_accumulate(const float *__restrict__ X, int64_t nb, int D,
                                                           const int32_t *__restrict__ assign,
                                                           const uint32_t *__restrict__ absmax_bits, int shift,
                                                           long long *__restrict__ sums, int32_t *__restrict__ cnt)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= nb * D) return;
    const int64_t row = i / D;
    const int d = (int)(i - row * D);
    const int c = assign[row];
    if (c < 0) return;
    const double f = ldexp(1.0, shift) / scale_of(*absmax_bits);
    const float x = X[i];
    if (__float_as_uint(x) << 1 < 0xFF000000u) // finite
        atomicAdd((unsigned long long *)&sums[(int64_t)c * D + d], (unsigned long long)llrint((double)x * f));
    if (d == 0) atomicAdd(&cnt[c], 1);
}

void launch_kmeans_accumulate(const float *X, int64_t nb, int D, const int32_t *assign, const uint32_t *absmax_bits,
                              int shift, long long *sums, int32_t *cnt, hipStream_t st)
{
    const int64_t n = nb * D;
    if (n <= 0) return;
    hipLaunchKernelGGL(k_kmeans_accumulate, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, X, nb, D, assign,
                       absmax_bits, shift, sums, cnt);
}

// a centroid with members moves to their mean; one without stays
__global__ __launch_bounds__(256) void k_kmeans_update(float *__restrict__ C, int k, int D,
                                                       const long long *__restrict__ sums,
                                                       const int32_t *__restrict__ cnt,
                                                       const uint32_t *__restrict__ absmax_bits, int shift)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)k * D) return;
    const int c = (int)(i / D);
    const int n = cnt[c];
    if (n <= 0) return;
    const double inv = scale_of(*absmax_bits) / ldexp(1.0, shift);
    C[i] = (float)((double)sums[i] * inv / (double)n);
}

void launch_kmeans_update(float *C, int k, int D, const long long *sums, const int32_t *cnt,
                          const uint32_t *absmax_bits, int shift, hipStream_t st)
{
    const int64_t n = (int64_t)k * D;
    hipLaunchKernelGGL(k_kmeans_update, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, C, k, D, sums, cnt,
                       absmax_bits, shift);
}

// ---------------------------------------------------------------------------
// Lloyd iteration of a small codebook with few dimensions, both halves in one pass: a lane is a
// vector and keeps it in registers, the k centroids come in one after the other through uniform
// loads, and every lane keeps its own running (distance, index) minimum: exact fp32 distances, added
// up in the order of the encoder's (four components per partial sum, then pairwise), strict "<" in
// ascending order.  The member sums go to an LDS image [k][D + 1] of 64-bit words (the last one
// counts; an odd row length spreads the banks), and every workgroup writes its image out once for
// k_lloyd_reduce.  Sums are integers, so neither the order nor the split over workgroups shows.
// Bound by vector-ALU issue: about 2 D + 6 instructions per vector and centroid.  262 144 x 16 against
// 256 centroids: 90 us an iteration instead of 740 us for norms, centring, fp32 contraction, exact pass and
// global atomics (4.2 M on 4 096 addresses: 300 us of them).
// ---------------------------------------------------------------------------
#define LLOYD_NT 512
#define LLOYD_BLOCKS 512     // two workgroups per compute unit
#define LLOYD_LDS 65536      // limit of a workgroup's image: two fit beside each other
typedef const float __attribute__((address_space(4))) cfloat;

// squared distance of r to w in the order of the exact pass of the encoder
template <int DS>
__device__ __forceinline__ float lloyd_dist(const float (&r)[DS], const float *w)
{
    constexpr bool QUADS = DS % 4 == 0;
    constexpr int PARTS = QUADS ? DS / 4 : DS;
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < PARTS; ++i) {
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < (QUADS ? 4 : 1); ++e) {
            const float t = r[QUADS ? 4 * i + e : i] - w[QUADS ? 4 * i + e : i];
            acc = fmaf(t, t, acc);
        }
        v[i] = acc;
    }
    float s = PARTS > 1 ? v[0] + v[1] : v[0];
    if (PARTS > 2) s += PARTS > 3 ? v[2] + v[3] : v[2];
    if (PARTS > 4) s += v[4] + v[5];
    return s;
}

// One pass by the walk, of a whole workgroup.
template <int DS>
__device__ __forceinline__ void lloyd_lanes(const float *__restrict__ X, int64_t nt, int k, const float *__restrict__ C,
                                            const uint32_t *__restrict__ absmax_bits, int shift, int want_sums, int vec,
                                            unsigned long long *__restrict__ part, int32_t *__restrict__ assign, unsigned long long *img)
{
    const int tid = threadIdx.x;
    for (int i = tid; i < k * (DS + 1); i += LLOYD_NT) img[i] = 0;
    __syncthreads();
    const double f = ldexp(1.0, shift) / scale_of(*absmax_bits);
    // never written while the kernel runs: the constant address space takes the scalar path
    const cfloat *w = (const cfloat *)(uintptr_t)C;
    constexpr int CB = DS >= 12 ? 2 : (DS >= 6 ? 4 : 8); // centroids per batch of uniform loads
    const int64_t stride = (int64_t)gridDim.x * LLOYD_NT;
    for (int64_t base = (int64_t)blockIdx.x * LLOYD_NT; base < nt; base += stride) { // (uniform trip count)
        const int64_t row = base + tid;
        const bool live = row < nt;
        const float *x = X + (live ? row : nt - 1) * DS;
        float r[DS];
        if (DS % 4 == 0 && vec) {
#pragma unroll
            for (int d = 0; d + 3 < DS; d += 4) {
                const f32x4 v = *(const f32x4 *)(x + d);
                r[d] = v.x;
                r[d + 1] = v.y;
                r[d + 2] = v.z;
                r[d + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int d = 0; d < DS; ++d) r[d] = x[d];
        }
        float best = INFINITY;
        int bt = 0;
        float wc[CB * DS], wn[CB * DS];
        const int kb = k - k % CB;
        if (kb > 0) {
#pragma unroll
            for (int i = 0; i < CB * DS; ++i) wc[i] = w[i];
        }
        for (int t = 0; t < kb; t += CB) {
            const int tn = t + CB < kb ? t + CB : t;
#pragma unroll
            for (int i = 0; i < CB * DS; ++i) wn[i] = w[tn * DS + i];
#pragma unroll
            for (int u = 0; u < CB; ++u) {
                const float s = lloyd_dist<DS>(r, wc + u * DS);
                if (s < best) {
                    best = s;
                    bt = t + u;
                }
            }
#pragma unroll
            for (int i = 0; i < CB * DS; ++i) wc[i] = wn[i];
        }
        for (int t = kb; t < k; ++t) {
            float wt[DS];
#pragma unroll
            for (int d = 0; d < DS; ++d) wt[d] = w[t * DS + d];
            const float s = lloyd_dist<DS>(r, wt);
            if (s < best) {
                best = s;
                bt = t;
            }
        }
        if (live) {
            unsigned long long *row_img = img + bt * (DS + 1);
            if (want_sums) {
#pragma unroll
                for (int d = 0; d < DS; ++d)
                    if (__float_as_uint(r[d]) << 1 < 0xFF000000u) // finite
                        atomicAdd(&row_img[d], (unsigned long long)llrint((double)r[d] * f));
            }
            atomicAdd(&row_img[DS], 1ull);
            if (assign) assign[row] = bt;
        }
    }
    __syncthreads();
    unsigned long long *out = part + (int64_t)blockIdx.x * k * (DS + 1);
    for (int i = tid; i < k * (DS + 1); i += LLOYD_NT) out[i] = img[i];
}

template <int DS>
__global__ __launch_bounds__(LLOYD_NT) void k_lloyd_lanes(const float *__restrict__ X, int64_t nt, int k,
                                                          const float *__restrict__ C,
                                                          const uint32_t *__restrict__ absmax_bits, int shift, int want_sums,
                                                          int vec, unsigned long long *__restrict__ part,
                                                          int32_t *__restrict__ assign)
{
    extern __shared__ unsigned long long img[]; // [k][DS + 1]
    lloyd_lanes<DS>(X, nt, k, C, absmax_bits, shift, want_sums, vec, part, assign, img);
}

// The nearest of k centroids to the lane's vector, the first of equal ones; 0 where no distance is finite.  (The loop of
// k_lloyd_lanes.  That kernel has it written out: as a call its scalar registers are copied from batch to batch, and ten
// iterations of 262 144 x 8, k = 800 take 1 640 us instead of 1 280.)
template <int DS>
__device__ __forceinline__ int walk_centroids(const float *C, int k, const float (&r)[DS])
{
    // never written while the kernel runs: the constant address space takes the scalar path
    const cfloat *w = (const cfloat *)(uintptr_t)C;
    constexpr int CB = DS >= 12 ? 2 : (DS >= 6 ? 4 : 8); // centroids per batch of uniform loads
    float best = INFINITY;
    int bt = 0;
    float wc[CB * DS], wn[CB * DS];
    const int kb = k - k % CB;
    if (kb > 0) {
#pragma unroll
        for (int i = 0; i < CB * DS; ++i) wc[i] = w[i];
    }
    for (int t = 0; t < kb; t += CB) {
        const int tn = t + CB < kb ? t + CB : t;
#pragma unroll
        for (int i = 0; i < CB * DS; ++i) wn[i] = w[tn * DS + i];
#pragma unroll
        for (int u = 0; u < CB; ++u) {
            const float s = lloyd_dist<DS>(r, wc + u * DS);
            if (s < best) {
                best = s;
                bt = t + u;
            }
        }
#pragma unroll
        for (int i = 0; i < CB * DS; ++i) wc[i] = wn[i];
    }
    for (int t = kb; t < k; ++t) {
        float wt[DS];
#pragma unroll
        for (int d = 0; d < DS; ++d) wt[d] = w[t * DS + d];
        const float s = lloyd_dist<DS>(r, wt);
        if (s < best) {
            best = s;
            bt = t;
        }
    }
    return bt;
}

// the mean of the middle two of four finite values (halves are added, so that nothing overflows)
__device__ __forceinline__ float middle_of_four(float a, float b, float c, float d)
{
    return 0.5f * fmaxf(fminf(a, b), fminf(c, d)) + 0.5f * fminf(fmaxf(a, b), fmaxf(c, d));
}
// the same over four lanes, those that the two steps reach
template <int STEP1, int STEP2>
__device__ __forceinline__ float middle_of_lanes(float v)
{
    auto from = [](float x, auto step) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(step)::value, 0xF, 0xF, true));
    };
    const float w = from(v, std::integral_constant<int, STEP1>{}), lo = fminf(v, w), hi = fmaxf(v, w);
    return 0.5f * fmaxf(lo, from(lo, std::integral_constant<int, STEP2>{})) + 0.5f * fminf(hi, from(hi, std::integral_constant<int, STEP2>{}));
}

// The same iteration for up to 256 centroids with the nearest one from the matrix cores (codeword.h), 64 vectors a
// wave.  262 144 x 16 against 256 centroids: 73 us with the lanes' walk over the centroids, 46 so (66 with
// the centroids read from their rows): the products 14, the rest loads and the LDS additions of the sums.
// Where too many vectors are not decided by the products (groups of centroids closer to each other than the products resolve at
// their distance from the point), they are left out of the next three iterations, then tried again, and left out of fifteen ..: ten
// iterations of 262 144 vectors in 64 tight groups, k = 256, us, by the walk alone / with the products each time / so: D = 8 615 / 913 /
// 653, D = 16 1 000 / 1 247 / 1 032.  Every vector gets the same centroid either way.
#define LLOYD_CT 272 // floats a component: the four that a wave reads at once start 16 banks apart
template <int DS>
__global__ __launch_bounds__(LLOYD_NT, 4) void k_lloyd_cores(const float *__restrict__ X, int64_t nt, int k,
                                                             const float *__restrict__ C,
                                                             const uint32_t *__restrict__ absmax_bits, int shift, int want_sums,
                                                             int vec, unsigned long long *__restrict__ part,
                                                             int32_t *__restrict__ assign, int *__restrict__ turns)
{
    extern __shared__ unsigned long long img[]; // [k][DS + 1]
    __shared__ __align__(16) float half[256];
    __shared__ float ct[DS * LLOYD_CT]; // the centroids component by component
    __shared__ float mu[DS];
    __shared__ int sh_cmax, sh_compared;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (__builtin_amdgcn_readfirstlane(turns[LLOYD_WAIT]) > 0) {
        lloyd_lanes<DS>(X, nt, k, C, absmax_bits, shift, want_sums, vec, part, assign, img);
        return;
    }
    for (int i = tid; i < k * (DS + 1); i += LLOYD_NT) img[i] = 0;
    if (tid == 0) sh_cmax = sh_compared = 0;
    __syncthreads();
    if (tid < 256) {
#pragma unroll
        for (int d = 0; d < DS; ++d) ct[d * LLOYD_CT + tid] = tid < k ? C[(int64_t)tid * DS + d] : 0.f;
    }
    __syncthreads();
    // The point: component by component the mean of the middle two of four values, of four such means, and so on over all
    // centroids (from k on they begin anew).  The plain mean would do as well, but for centroids far from the others, which take
    // it along; a median by bisection is 1 us an iteration slower.
    for (int d = wave; d < DS; d += LLOYD_NT / 64) {
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int t = lane + 64 * j;
            t -= t >= k ? k : 0;
            t -= t >= k ? k : 0; // (k >= 96)
            v[j] = ct[d * LLOYD_CT + t];
            if (!(fabsf(v[j]) < INFINITY)) v[j] = 0.f;
        }
        float m = middle_of_four(v[0], v[1], v[2], v[3]);
        m = middle_of_lanes<0xB1, 0x4E>(m);   // quad_perm [1, 0, 3, 2] and [2, 3, 0, 1]: the four lanes of a quad
        m = middle_of_lanes<0x141, 0x140>(m); // row_half_mirror and row_mirror: the four quads of a row
        const int mi = __float_as_int(m);
        m = middle_of_four(__int_as_float(__builtin_amdgcn_readlane(mi, 0)), __int_as_float(__builtin_amdgcn_readlane(mi, 16)),
                           __int_as_float(__builtin_amdgcn_readlane(mi, 32)), __int_as_float(__builtin_amdgcn_readlane(mi, 48)));
        if (lane == 0) mu[d] = m;
    }
    __syncthreads();
    if (tid < 256) {
        float h = 0.f;
        bool there = tid < k; // (a centroid with a component that is not finite is nobody's nearest)
#pragma unroll
        for (int d = 0; d < DS; ++d) {
            const float c = ct[d * LLOYD_CT + tid], v = c - mu[d];
            there = there && fabsf(c) < INFINITY;
            h = fmaf(v, v, h);
        }
        half[tid] = there ? 0.5f * h : CODEWORD_NONE; // (the half of a finite sum of squares is smaller, an overflowed one infinite)
        if (there) atomicMax(&sh_cmax, (int)__float_as_uint(h < INFINITY ? sqrtf(h) : INFINITY));
        if (!there)
#pragma unroll
            for (int d = 0; d < DS; ++d) ct[d * LLOYD_CT + tid] = mu[d]; // (at the largest "norm", and never the nearest)
    }
    __syncthreads();
    int compared = 0; // vectors of the wave that were compared one by one; the walk takes the time of CODEWORD_OPEN of them
    const float cmax = __uint_as_float((uint32_t)sh_cmax);
    const double f = ldexp(1.0, shift) / scale_of(*absmax_bits);
    const int64_t stride = (int64_t)gridDim.x * LLOYD_NT;
    for (int64_t row0 = (int64_t)blockIdx.x * LLOYD_NT + wave * 64; row0 < nt; row0 += stride) {
        auto row_of = [&](int v) { return X + min(row0 + v, nt - 1) * DS; };
        auto exact = [&](int v, int t) {
            float r[DS], w[DS];
            if (half[t] == CODEWORD_NONE) return INFINITY;
            load_row<DS>(row_of(v), vec, r);
#pragma unroll
            for (int d = 0; d < DS; ++d) w[d] = ct[d * LLOYD_CT + t];
            return lloyd_dist<DS>(r, w);
        };
        auto all = [&](int v) {
            ++compared;
            uint64_t key = KEY_MAX;
            for (int t = lane; t < k; t += 64) {
                const float s = exact(v, t);
                const uint64_t tk = make_key(s, (uint32_t)t);
                if (s < INFINITY && tk < key) key = tk;
            }
            key = wave_min_u64(key);
            return key == KEY_MAX ? 0 : (int)(uint32_t)key;
        };
        auto walk = [&]() {
            float r[DS];
            load_row<DS>(row_of(lane), vec, r);
            compared += CODEWORD_OPEN;
            return walk_centroids<DS>(C, k, r);
        };
        const int bt = nearest_codeword64<DS>(ct, LLOYD_CT, k, half, cmax, lane, [&](int d) { return mu[d]; },
                                              [&](int v, int d) { return row_of(v)[d]; }, exact, all, walk);
        const int64_t row = row0 + lane;
        if (row < nt) {
            unsigned long long *row_img = img + bt * (DS + 1);
            if (want_sums) {
                float r[DS];
                load_row<DS>(X + row * DS, vec, r);
#pragma unroll
                for (int d = 0; d < DS; ++d)
                    if (__float_as_uint(r[d]) << 1 < 0xFF000000u) // finite
                        atomicAdd(&row_img[d], (unsigned long long)llrint((double)r[d] * f));
            }
            atomicAdd(&row_img[DS], 1ull);
            if (assign) assign[row] = bt;
        }
    }
    if (lane == 0 && compared) atomicAdd(&sh_compared, compared);
    __syncthreads();
    if (tid == 0 && sh_compared) atomicAdd(&turns[LLOYD_COMPARED], sh_compared);
    unsigned long long *out = part + (int64_t)blockIdx.x * k * (DS + 1);
    for (int i = tid; i < k * (DS + 1); i += LLOYD_NT) out[i] = img[i];
}

// One workgroup per centroid: the D sums and the count over all images; with C the centroid moves to
// the mean of its members (one without members stays), with counts the number of members is written.
__global__ __launch_bounds__(256) void k_lloyd_reduce(const unsigned long long *__restrict__ part, int blocks, int k,
                                                      int D, const uint32_t *__restrict__ absmax_bits, int shift,
                                                      float *__restrict__ C, int32_t *__restrict__ counts,
                                                      int64_t most, int *__restrict__ turns)
{
    __shared__ unsigned long long sum[256];
    const int tid = threadIdx.x, c = blockIdx.x;
    if (turns && c == 0 && tid == 0) {
        if (turns[LLOYD_WAIT] > 0) {
            --turns[LLOYD_WAIT];
        } else {
            turns[LLOYD_STEP] = turns[LLOYD_COMPARED] > most ? min(4 * turns[LLOYD_STEP] + 3, 1 << 20) : 0;
            turns[LLOYD_WAIT] = turns[LLOYD_STEP];
        }
        turns[LLOYD_COMPARED] = 0;
    }
    const int E = D + 1, slices = 256 / E;
    const int e = tid % E, sl = tid / E;
    unsigned long long s = 0;
    if (sl < slices)
        for (int b = sl; b < blocks; b += slices) s += part[((int64_t)b * k + c) * E + e];
    sum[tid] = s;
    __syncthreads();
    if (tid < E) {
        for (int i = 1; i < slices; ++i) s += sum[i * E + tid];
        sum[tid] = s; // (only this thread reads its own word before)
    }
    __syncthreads();
    const int n = (int)sum[D];
    if (counts && tid == 0) counts[c] = n;
    if (C && tid < D && n > 0) {
        const double inv = scale_of(*absmax_bits) / ldexp(1.0, shift);
        C[(int64_t)c * D + tid] = (float)((double)(long long)s * inv / (double)n);
    }
}

// Codebooks whose image fits a workgroup's share of LDS (256 centroids of 16 dimensions: 35 KB).  A lane walks all k
// centroids, so an iteration takes that walk's time however few vectors there are; up to 32 768 vectors (64 of 256 compute
// units at work) the contraction of the general path is faster from some k on, which depends on the length of the walk.
// Ten iterations of 3 000 vectors, ms of the general path and of this one: D = 16, k = 300 0.86 and 0.85, 380 0.85 and 1.02,
// 481 0.95 and 1.24; D = 12, k = 330 0.86 and 0.80, 430 0.91 and 1.02, 630 0.99 and 1.44; D = 8, k = 850 1.09 and 1.02, 910 0.97
// and 1.06; D = 6, k = 800 1.08 and 0.98, 950 0.99 and 1.12; D = 4, k = 1 638 1.11 and 1.03.  At 33 000 vectors: D = 16, k = 380
// 1.72 and 1.09, D = 6, k = 950 2.12 and 1.14.
bool lloyd_lanes_supported(int64_t nt, int D, int k)
{
    if (D != 4 && D != 6 && D != 8 && D != 12 && D != 16) return false;
    if ((int64_t)k * (D + 1) * 8 > LLOYD_LDS) return false;
    return nt > 32768 || D == 4 || k <= (D == 16 ? 304 : D == 12 ? 360 : 880);
}

static int lloyd_blocks(int64_t nt)
{
    const int64_t b = (nt + LLOYD_NT - 1) / LLOYD_NT;
    return (int)(b < LLOYD_BLOCKS ? b : LLOYD_BLOCKS);
}

size_t lloyd_lanes_words(int64_t nt, int D, int k) { return (size_t)lloyd_blocks(nt) * k * (D + 1); }

void launch_lloyd_lanes(const float *X, int64_t nt, int D, int k, float *C, const uint32_t *absmax_bits, int shift,
                        bool update, uint64_t *part, int32_t *assign, int32_t *counts, int *turns, hipStream_t st)
{
    const int blocks = lloyd_blocks(nt);
    const int vec = ((uintptr_t)X) % 16 == 0;
    const size_t lds = (size_t)k * (D + 1) * 8;
    auto go = [&](auto kern, auto... more) {
        if (lds > 49152 && // (48 KB of dynamic LDS need no asking)
            hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return; // (the caller asks for the error)
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(LLOYD_NT), lds, st, X, nt, k, (const float *)C, absmax_bits,
                           shift, update ? 1 : 0, vec, (unsigned long long *)part, assign, more...);
    };
    // The products' fixed cost (norms, direct distances of four centroids a vector) against the walk, ten iterations of
    // 262 144 vectors, us: D = 16, k = 256 780 and 1 112; D = 6, k = 256 599 and 1 129; D = 4, k = 256 459 and 470; D = 8, k = 64
    // 390 and 341; D = 12, k = 40 434 and 376.
    const bool cores = k <= 256 && k * D >= 1536;
    switch (D) {
    case 4: go(k_lloyd_lanes<4>); break;
    case 6: cores ? go(k_lloyd_cores<6>, turns) : go(k_lloyd_lanes<6>); break;
    case 8: cores ? go(k_lloyd_cores<8>, turns) : go(k_lloyd_lanes<8>); break;
    case 12: cores ? go(k_lloyd_cores<12>, turns) : go(k_lloyd_lanes<12>); break;
    default: cores ? go(k_lloyd_cores<16>, turns) : go(k_lloyd_lanes<16>); break;
    }
    // From so many comparisons one by one a batch on the walk alone is as fast: an iteration of 262 144 vectors, k = 256, the walk and the
    // products with none of them, us: D = 6 50 and 46, D = 8 54 and 49, D = 12 80 and 56, D = 16 92 and 65.
    const int64_t most = (D < 12 ? 3 : 14) * ((nt + 63) / 64);
    if (update || counts)
        hipLaunchKernelGGL(k_lloyd_reduce, dim3((unsigned)k), dim3(256), 0, st, (const unsigned long long *)part, blocks, k,
                           D, absmax_bits, shift, update ? C : nullptr, counts, most, cores ? turns : nullptr);
}
