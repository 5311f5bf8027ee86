// List scan with K-selection for the shapes the per-wave lists of scan_stream.hip do not serve:
// K > 128 (a re-ranking stage asks for up to 1 024 results) and code lengths other than 8 and 16.
//
// Same split of the distance as there (one table per query, m lookups per point, s_x streamed with the
// code), other organisation:
//  * the points of all visited lists of a (query, split) are laid end to end and handed out 256 to a
//    wave and 2 048 to a workgroup and turn, so that lists of any length fill the lanes;
//  * one candidate buffer of SW_CAP keys per workgroup, unsorted.  When it could overflow in the next
//    turn, a radix selection (512 bins over the range of the keys present, refined inside the bin of
//    the K-th key) drops what cannot be among the K best and lowers the threshold: two or three passes
//    over at most 8 keys per thread.  Sorting happens once, for the K survivors.
//  * the fast sums only shortlist.  Every point whose fast distance is within twice the error bound `slack` of the
//    K-th smallest fast distance stays in the buffer; at the end those (K and a few more) get the distance of the
//    2m-lookup scan (search.hip, k_scan) in the same operations and order, read from the centroids and
//    codewords themselves, and the K smallest (distance, id) of these are the result: the same bits as that
//    scan's.  If more points lie within the bound than the buffer holds (masses of coinciding points), or the
//    bound is not finite, the workgroup leaves its lists to a second launch, which takes that distance for every
//    candidate (a workgroup with nothing to do ends at once): point by point (EXACT) or, where lists are long, with
//    the tables of k_scan (scan_redo_by_list).
//    (The bound goes summand by summand: with (D + m) 2 Z^2, Z the sum of all sizes, clusters of 2 % of the distance of
//    their centre from the mean were already taken for coinciding: 256 queries x 16 lists of 8 000 points, K = 1 000,
//    2.6 ms, and 0.53 so; 1 024 x 2 048 lists of 125 points, m = 64, D = 1 024, K = 1 024: 105 and 35 ms.)
//
// Measured, 1 501 queries x 512 lists of 19 points (14.7M points), m = 8, K = 1 000: 0.314 ms, and 4 us for a
// second launch that finds nothing to do, against 66.7 ms of the 2m-lookup scan, which builds m * 256 table entries per
// 19-point list and sorts its whole buffer of keys at every cut.  Half of it are the 1.5M points taken again, 1.5 KB of centroid and codeword rows each.  (With the exact pass in
// the same kernel 22 to 99 registers were spilled, whatever the code length: 0.387 ms; 1 024 queries x 2 048 lists, m = 64,
// D = 1 024, K = 1 024: the call took 35 ms, 9.1 ms so.)
#include "bounds.h"
#include "common.h"

#define SW_NW (SW_NT / 64)
#define SW_CAP (2 * SW_TURN)          // candidate keys per workgroup
#define SW_BINS SW_NT               // one bin of the selection's histogram per thread
static_assert(SW_CAP - SW_TURN >= VLQ_MAX_K, "the K best and one turn's candidates fit the buffer");

// bytes of LDS of one workgroup: keys, table, query, list ends / shifts / (a, b - a) / places in the descriptors
static size_t scan_wide_lds(int m, int D, int lists)
{
    return (size_t)SW_CAP * 8 + (size_t)m * 1024 + (size_t)((D + 3) & ~3) * 4 + (size_t)((lists + 3) & ~3) * 18;
}

// One sub-space's part of the 2m-lookup distance: A = ||z^p - w||^2, B = <e^p, w> with z = y - c_i, e = s_ij - c_i
// (the operations and their order are those of k_scan's tables)
__device__ __forceinline__ void sw_subspace(const float *__restrict__ y, const float *__restrict__ ci,
                                            const float *__restrict__ sj, const float *__restrict__ w, int ds, float *A,
                                            float *B)
{
    float sa = 0.f, sb = 0.f;
    auto term = [&](float yv, float c, float sv, float wv) {
        const float z = yv - c, e = sv - c;
        sb = fmaf(e, wv, sb);
        const float t = z - wv;
        sa = fmaf(t, t, sa);
    };
    if ((ds & 3) == 0) { // (rows of C and P start on 16 bytes then; y lies in LDS or in the caller's memory)
#pragma unroll 4
        for (int d = 0; d < ds; d += 4) {
            const f32x4 c4 = *(const f32x4 *)(ci + d), s4 = *(const f32x4 *)(sj + d), w4 = *(const f32x4 *)(w + d);
#pragma unroll
            for (int x = 0; x < 4; ++x) term(y[d + x], c4[x], s4[x], w4[x]);
        }
    } else {
        for (int d = 0; d < ds; ++d) term(y[d], ci[d], sj[d], w[d]);
    }
    *A = sa;
    *B = sb;
}

// M: bytes of a code (0: run-time length).  EXACT: the pass over what the fast one has left, by the 2m-lookup distance
// of every candidate; the fast distance, with its bound, only spares those that are beyond the threshold.
template <int M, bool EXACT>
__global__ __launch_bounds__(SW_NT, 4) void k_scan_wide(ScanArgs a, int lists_max)
{
    if (EXACT && !a.redo[blockIdx.x]) return;
    extern __shared__ __align__(16) unsigned char smem[];
    uint64_t *keys = (uint64_t *)smem;              // [SW_CAP] (distance, place in the concatenation), or (distance, id)
    float *T = (float *)(keys + SW_CAP);            // [m * 256]
    float *yv = T + a.m * 256;                      // [D]
    const int lcap = (lists_max + 3) & ~3;
    float2 *lab = (float2 *)(yv + ((a.D + 3) & ~3)); // [lists] a, b - a
    sw_place_t *lend = (sw_place_t *)(lab + lcap);  // [lists] where the list ends in the concatenation
    uint32_t *lsh = (uint32_t *)(lend + lcap);      // [lists] position in the arrays minus place in the concatenation
    uint16_t *lat = (uint16_t *)(lsh + lcap);       // [lists] the list's descriptor
    __shared__ int hist[SW_BINS];
    __shared__ int sh_wsum[SW_NW], sh_wcnt[SW_NW];
    __shared__ uint64_t sh_lo[SW_NW], sh_hi[SW_NW];
    __shared__ float sh_red[3][SW_NW];
    __shared__ int sh_cnt, sh_bin, sh_before, sh_inbin;
    __shared__ uint64_t sh_thr;
    __shared__ int sh_wmax[VLQ_MAX_M]; // largest ||P[p][.]||^2 (bits of a float that is not negative)

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = blockIdx.x / a.nsplit, split = blockIdx.x - q * a.nsplit;
    const int r0 = (int)((int64_t)a.w2 * split / a.nsplit), r1 = (int)((int64_t)a.w2 * (split + 1) / a.nsplit);
    const int K = a.K, D = a.D, m = a.m, ds = D / m;
    const float *yq = a.Q + (int64_t)q * D;
    const uint4 *dq = a.desc + (int64_t)q * a.w2; // {label, 1 or 0 (no list), a, g}

    float yn = 0.f, amax = 0.f, cmax = 0.f;
    for (int d = tid; d < D; d += SW_NT) {
        const float v = yq[d] - a.mu[d];
        yv[d] = v;
        yn = fmaf(v, v, yn);
    }
    if (tid < VLQ_MAX_M) sh_wmax[tid] = 0;
    // the visited lists that hold points, in the order of the descriptors (at most VLQ_MAX_W2 = 4 x SW_NT)
    int nl = 0;
    sw_place_t total = 0;
    for (int s0 = r0; s0 < r1; s0 += SW_NT) {
        const int s = s0 + tid;
        uint4 d = make_uint4(0u, 0u, 0u, 0u);
        if (s < r1) d = dq[s];
        uint32_t beg = 0;
        int len = 0;
        float av = 0.f, bav = 0.f;
        if (d.y) {
            const int64_t b0 = a.off[d.x];
            const float c = a.E[d.x];
            beg = (uint32_t)b0;
            len = (int)(a.off[d.x + 1] - b0);
            av = __uint_as_float(d.z);
            bav = fmaf(-2.f, __uint_as_float(d.w), c);
            amax = fmaxf(amax, av);
            cmax = fmaxf(cmax, c);
        }
        int end = len;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(end, o, 64);
            if (lane >= o) end += t;
        }
        const uint64_t some = __ballot(len > 0);
        __syncthreads(); // (the sums of the round before have been read)
        if (lane == 63) {
            sh_wsum[wave] = end;
            sh_wcnt[wave] = __popcll(some);
        }
        __syncthreads();
        int before = 0, at = 0, all = 0, alln = 0;
#pragma unroll
        for (int w = 0; w < SW_NW; ++w) {
            const int ws = sh_wsum[w], wc = sh_wcnt[w];
            before += w < wave ? ws : 0;
            at += w < wave ? wc : 0;
            all += ws;
            alln += wc;
        }
        if (len > 0) {
            const int slot = nl + at + __popcll(some & ((1ull << lane) - 1ull));
            const sw_place_t e = total + (sw_place_t)(before + end);
            lend[slot] = e;
            lsh[slot] = beg - (e - (sw_place_t)len);
            lab[slot] = make_float2(av, bav);
            lat[slot] = (uint16_t)s;
        }
        nl += alln;
        total += (sw_place_t)all;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        yn += __shfl_xor(yn, o, 64);
        amax = fmaxf(amax, __shfl_xor(amax, o, 64));
        cmax = fmaxf(cmax, __shfl_xor(cmax, o, 64));
    }
    if (lane == 0) {
        sh_red[0][wave] = yn;
        sh_red[1][wave] = amax;
        sh_red[2][wave] = cmax;
    }
    // T[p][t] = 2 <(y - mu)^p, P[p][t]>
    for (int e = tid * 4; e < m * 256; e += SW_NT * 4) {
        f32x4 w2;
        *(f32x4 *)(T + e) = table_entries(a.Pt, yv, ds, e, &w2);
        float wn = fmaxf(fmaxf(w2.x, w2.y), fmaxf(w2.z, w2.w));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) wn = fmaxf(wn, __shfl_xor(wn, o, 64));
        if (lane == 0) atomicMax(&sh_wmax[e >> 8], (int)__float_as_uint(wn)); // (a wave's 256 entries are of one p)
    }
    __syncthreads();
    // how far the fast distance can be from the 2m-lookup one
    float slack;
    {
        float ysum = 0.f, am = 0.f, cm = 0.f, qn = 0.f;
#pragma unroll
        for (int w = 0; w < SW_NW; ++w) {
            ysum += sh_red[0][w];
            am = fmaxf(am, sh_red[1][w]);
            cm = fmaxf(cm, sh_red[2][w]);
        }
        for (int p = 0; p < m; ++p) qn += __uint_as_float((uint32_t)sh_wmax[p]);
        const float L = fmaxf(fabsf(a.lam_zero), fabsf(255.f - a.lam_zero)) * a.lam_step;
        slack = scan_wide_slack(am, ysum, qn, cm, L, D, m);
    }

    // the 2m-lookup distance of point p of the concatenation (list slot j) by one lane
    auto full_distance = [&](sw_place_t p, int j) -> float {
        const uint32_t g = p + lsh[j];
        const uint4 d = dq[lat[j]];
        const int i = (int)d.x / a.n;
        const float *ci = a.C + (int64_t)i * D, *sj = a.C + (int64_t)a.S[d.x] * D;
        const uint8_t *cp = a.codes + (size_t)g * m;
        float sa = 0.f, sb = 0.f;
        for (int s = 0; s < m; ++s) {
            float A, B;
            sw_subspace(yq + s * ds, ci + s * ds, sj + s * ds, a.P + ((int64_t)s * 256 + cp[s]) * ds, ds, &A, &B);
            sa += A;
            sb += B;
        }
        const float l = ((float)a.lam[g] - a.lam_zero) * a.lam_step;
        return fmaf(l, fmaf(l, a.E[d.x], 2.f * (sb - __uint_as_float(d.w))), sa);
    };

    // Keeps the keys up to a cut that is at or above the K-th smallest; the cut becomes the threshold.  Called by all
    // threads, cnt > K keys in the buffer.
    //  final keys (exact): at most `limit` of them stay (limit >= K);
    //  fast distances: the threshold is raised by 2 slack, and what lies below it stays; returns false, with the
    //  buffer untouched, if that is more than one turn leaves room for.
    auto select = [&](int cnt, int limit, bool exact) -> bool {
        uint64_t k8[SW_CAP / SW_NT];
        uint64_t lo = KEY_MAX, hi = 0;
#pragma unroll
        for (int i = 0; i < SW_CAP / SW_NT; ++i) {
            const int at = tid + i * SW_NT;
            k8[i] = at < cnt ? keys[at] : KEY_MAX;
            if (at < cnt) {
                lo = k8[i] < lo ? k8[i] : lo;
                hi = k8[i] > hi ? k8[i] : hi;
            }
        }
        lo = wave_min_u64(lo);
        hi = ~wave_min_u64(~hi);
        if (lane == 0) {
            sh_lo[wave] = lo;
            sh_hi[wave] = hi;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < SW_NW; ++w) {
            lo = sh_lo[w] < lo ? sh_lo[w] : lo;
            hi = sh_hi[w] > hi ? sh_hi[w] : hi;
        }
        int below = 0;
        uint64_t cut;
        for (;;) {
            const uint64_t range = hi - lo;
            int shift = range ? 55 - __clzll((long long)range) : 0; // range >> shift < SW_BINS = 2^9
            shift = shift < 0 ? 0 : shift;
            hist[tid] = 0;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < SW_CAP / SW_NT; ++i)
                if (tid + i * SW_NT < cnt && k8[i] >= lo && k8[i] <= hi) atomicAdd(&hist[(int)((k8[i] - lo) >> shift)], 1);
            __syncthreads();
            const int h0 = hist[tid];
            int inc = h0;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int t = __shfl_up(inc, o, 64);
                if (lane >= o) inc += t;
            }
            if (lane == 63) sh_wsum[wave] = inc;
            __syncthreads();
            int base = below;
#pragma unroll
            for (int w = 0; w < SW_NW; ++w) base += w < wave ? sh_wsum[w] : 0;
            const int c1 = base + inc, c0 = c1 - h0; // keys before the next bin, before this one
            if (c0 < K && c1 >= K) { // exactly one thread holds the bin of the K-th key
                sh_bin = tid;
                sh_before = c0;
                sh_inbin = h0;
            }
            __syncthreads();
            const uint64_t blo = lo + ((uint64_t)sh_bin << shift), bhi = blo + (((uint64_t)1 << shift) - 1);
            if (sh_before + sh_inbin <= limit || shift == 0) {
                cut = bhi;
                break;
            }
            below = sh_before;
            lo = blo;
            hi = bhi < hi ? bhi : hi;
        }
        // more than `limit` only where keys repeat (the caller's ids do): the last bin is then one key many times over
        const bool crowded = exact && sh_before + sh_inbin > limit;
        const int before = sh_before;
        if (!exact) {
            const float far = ord2f((uint32_t)(cut >> 32)) + 2.f * slack;
            cut = far < INFINITY ? make_key(far, 0xFFFFFFFFu) : KEY_MAX - 1;
            int stay = 0;
#pragma unroll
            for (int i = 0; i < SW_CAP / SW_NT; ++i) stay += __popcll(__ballot(tid + i * SW_NT < cnt && k8[i] <= cut));
            __syncthreads(); // (sh_wsum has been read)
            if (lane == 0) sh_wsum[wave] = stay;
            __syncthreads();
            stay = 0;
#pragma unroll
            for (int w = 0; w < SW_NW; ++w) stay += sh_wsum[w];
            if (stay > SW_CAP - SW_TURN) return false; // uniform over the workgroup
        }
        __syncthreads();
        if (tid == 0) {
            sh_cnt = 0;
            sh_thr = cut;
            sh_bin = before;
        }
        __syncthreads();
        if (crowded) {
#pragma unroll
            for (int i = 0; i < SW_CAP / SW_NT; ++i)
                if (tid + i * SW_NT < cnt && k8[i] == cut) {
                    const int pos = atomicAdd(&sh_bin, 1);
                    if (pos < limit) keys[pos] = cut;
                }
        }
#pragma unroll
        for (int i = 0; i < SW_CAP / SW_NT; ++i) {
            const bool stay = tid + i * SW_NT < cnt && (k8[i] < cut || (k8[i] == cut && !crowded));
            const uint64_t mask = __ballot(stay);
            int pos = 0;
            if (mask) {
                if (lane == 0) pos = atomicAdd(&sh_cnt, __popcll(mask));
                pos = __builtin_amdgcn_readfirstlane(pos) + __popcll(mask & ((1ull << lane) - 1ull));
            }
            if (stay) keys[pos] = k8[i];
        }
        __syncthreads();
        if (crowded) {
            if (tid == 0) sh_cnt = limit;
            __syncthreads();
        }
        return true;
    };
    const int room = K + (K >> 2) + 64; // how far below the buffer's size a cut of fast distances is taken

    constexpr int CW = M > 0 ? (M + 3) / 4 : 1;
    constexpr bool exact = EXACT;
    bool redo = !EXACT && !(slack < INFINITY); // uniform over the workgroup
    if (!redo) {
        if (tid == 0) {
            sh_cnt = 0;
            sh_thr = KEY_MAX;
        }
        __syncthreads();
        for (sw_place_t turn = 0; turn < total; turn += SW_TURN) {
            const sw_place_t base = sw_wave_base(turn, wave);
            const bool any = base < total; // uniform over the wave
            uint32_t g[SW_U];
            int jl[SW_U];
            uint32_t cw[SW_U][CW], lb[SW_U];
            float sv[SW_U];
            if (any) {
                // the list of the wave's first point: lists that end at or before it, counted 64 samples at a time
                int j0 = 0;
                for (int step = (nl + 63) >> 6; step >= 1; step = step == 1 ? 0 : (step + 63) >> 6) {
                    const int at = j0 + (lane + 1) * step - 1;
                    j0 += __popcll(__ballot(at < nl && lend[min(at, nl - 1)] <= base)) * step;
                }
#pragma unroll
                for (int u = 0; u < SW_U; ++u) jl[u] = j0;
                const sw_place_t stop = min(base + 64 * SW_U, total) - 1; // last point of the wave
                for (int jb = j0; jb < nl; jb += 64) {
                    const sw_place_t e = lend[min(jb + lane, nl - 1)];
                    const int cross = __popcll(__ballot(jb + lane < nl && e <= stop)); // lists that end inside the run
                    for (int i = 0; i < cross; ++i) {
                        const sw_place_t ei = (sw_place_t)__builtin_amdgcn_readlane((int)e, i);
#pragma unroll
                        for (int u = 0; u < SW_U; ++u) jl[u] += ei <= min(sw_place(base, u, lane), stop);
                    }
                    if (cross < 64) break;
                }
#pragma unroll
                for (int u = 0; u < SW_U; ++u) {
                    g[u] = min(sw_place(base, u, lane), stop) + lsh[jl[u]]; // idle lanes repeat the last point
                    const uint8_t *cp = a.codes + (size_t)g[u] * m;
                    if (M > 0) __builtin_memcpy(cw[u], M % 4 == 0 ? __builtin_assume_aligned(cp, 4) : cp, M);
                    lb[u] = a.lam[g[u]];
                    sv[u] = a.sx[g[u]];
                }
            }
            __syncthreads(); // all candidates of the turn before are in
            const int fill = sh_cnt;
            __syncthreads();
            if (fill > SW_CAP - SW_TURN && !select(fill, exact ? SW_CAP - SW_TURN : room, exact)) {
                redo = true;
                break;
            }
            const uint64_t thr = sh_thr;
            // (fast distances: the threshold has the slack in it)
            const float thr_f = thr >= KEY_MAX - 1 ? INFINITY : ord2f((uint32_t)(thr >> 32)) + (exact ? slack : 0.f);
            if (any) {
#pragma unroll
                for (int u = 0; u < SW_U; ++u) {
                    if (sw_place(base, u, 0) >= total) break; // uniform over the wave
                    const bool live = sw_place(base, u, lane) < total;
                    const float2 ab = lab[jl[u]];
                    const uint8_t *cp = a.codes + (size_t)g[u] * m;
                    float ts = 0.f;
                    if (M > 0) {
#pragma unroll
                        for (int p = 0; p < M; ++p) ts += T[p * 256 + ((cw[u][p >> 2] >> (8 * (p & 3))) & 255u)];
                    } else {
                        for (int p = 0; p < m; ++p) ts += T[p * 256 + cp[p]];
                    }
                    const float l = ((float)lb[u] - a.lam_zero) * a.lam_step;
                    const float lba = l * ab.y;
                    const float dist = (sv[u] - ts) + (lba + ab.x);
                    bool pass = live && !(dist > thr_f); // (a NaN is a candidate, as in the 2m-lookup scan)
                    const sw_place_t p = sw_place(base, u, lane);
                    uint64_t key = make_key(dist, p);
                    if (exact && pass) {
                        key = make_key(full_distance(p, jl[u]), (uint32_t)a.ids[g[u]]);
                        pass = key < thr; // K keys at or below the threshold are in the buffer already
                    }
                    const uint64_t mask = __ballot(pass);
                    if (mask) {
                        int pos = 0;
                        if (lane == 0) pos = atomicAdd(&sh_cnt, __popcll(mask));
                        pos = __builtin_amdgcn_readfirstlane(pos) + __popcll(mask & ((1ull << lane) - 1ull));
                        if (pass) keys[pos] = key;
                    }
                }
            }
        }
        __syncthreads();
    }
    if (!EXACT && !redo && sh_cnt > K) {
        const int n = sh_cnt;
        __syncthreads();
        redo = !select(n, K, false);
    }
    if (!EXACT && tid == 0) a.redo[blockIdx.x] = redo;
    if (redo) return;
    int cnt = sh_cnt;
    __syncthreads();
    if (!EXACT) {
        // the 2m-lookup distance of what is left, a group of lanes per point: lane s of it takes sub-space s
        int L = 1;
        while (L < m) L <<= 1; // m <= 64
        const int per = SW_NT / L, sub = tid & (L - 1);
        for (int d = tid; d < D; d += SW_NT) yv[d] = yq[d]; // (the tables are done with: the query itself from here on)
        __syncthreads();
        // first where everything lies, a thread per point (the round trips of one point follow one another, those
        // of different points overlap); the upper half of the buffer is free
        static_assert(SW_CAP - SW_TURN <= SW_CAP / 2, "what a cut leaves fits half the buffer");
        for (int at = tid; at < cnt; at += SW_NT) {
            const sw_place_t p = (sw_place_t)keys[at];
            int lo = 0, hi = nl - 1; // first list that ends behind p
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (lend[mid] <= p)
                    lo = mid + 1;
                else
                    hi = mid;
            }
            const int label = (int)dq[lat[lo]].x;
            keys[at] = ((uint64_t)(uint32_t)lat[lo] << 32) | (p + lsh[lo]);
            keys[SW_CAP / 2 + at] = ((uint64_t)(uint32_t)a.S[label] << 32) | (uint32_t)(label / a.n);
        }
        __syncthreads();
        for (int c0 = 0; c0 < cnt; c0 += per) {
            const int at = c0 + tid / L;
            const bool live = at < cnt;
            // (idle groups work on point 0 of the index)
            const uint64_t where = live ? keys[at] : 0, rows = live ? keys[SW_CAP / 2 + at] : 0;
            const uint32_t g = (uint32_t)where;
            const uint4 d = dq[where >> 32];
            float A = 0.f, B = 0.f;
            if (sub < m) {
                const int t = a.codes[(size_t)g * m + sub];
                sw_subspace(yv + sub * ds, a.C + (int64_t)(uint32_t)rows * D + sub * ds,
                            a.C + (int64_t)(uint32_t)(rows >> 32) * D + sub * ds,
                            a.P + ((int64_t)sub * 256 + t) * ds, ds, &A, &B);
            }
            const float l = ((float)a.lam[g] - a.lam_zero) * a.lam_step, c = a.E[d.x];
            const uint32_t id = (uint32_t)a.ids[g];
            float sa = 0.f, sb = 0.f;
            for (int s = 0; s < m; ++s) {
                sa += __shfl(A, s, L);
                sb += __shfl(B, s, L);
            }
            const float dist = fmaf(l, fmaf(l, c, 2.f * (sb - __uint_as_float(d.w))), sa);
            if (live && sub == 0) keys[at] = make_key(dist, id);
        }
        __syncthreads();
    }
    if (cnt > K) {
        select(cnt, next_pow2_dev(K), true);
        cnt = sh_cnt;
    }
    const int sz = next_pow2_dev(max(cnt, K));
    for (int i = cnt + tid; i < sz; i += SW_NT) keys[i] = KEY_MAX;
    __syncthreads();
    block_bitonic_sort<SW_NT>(keys, sz, tid);
    if (a.nsplit > 1) {
        uint64_t *dst = a.partial + ((int64_t)q * a.nsplit + split) * K;
        for (int i = tid; i < K; i += SW_NT) dst[i] = keys[i];
    } else {
        for (int i = tid; i < K; i += SW_NT) {
            const uint64_t key = keys[i];
            const bool ok = key != KEY_MAX;
            a.out_dist[(int64_t)q * K + i] = ok ? ord2f((uint32_t)(key >> 32)) : INFINITY;
            a.out_ids[(int64_t)q * K + i] = ok ? (int32_t)(uint32_t)key : -1;
        }
    }
}

bool scan_wide_supported(const ScanArgs &a)
{
    return a.sx != nullptr && a.mu != nullptr && a.desc != nullptr;
}

void launch_scan_wide(const ScanArgs &a, bool exact, hipStream_t st)
{
    if (a.nq <= 0) return;
    const int lists = (a.w2 + a.nsplit - 1) / a.nsplit;
    const size_t lds = scan_wide_lds(a.m, a.D, lists); // at most 136 KB (m = 64, D = 1 024, 2 048 lists)
    auto go = [&](auto kern) {
        if (lds > 49152 && // (48 KB of dynamic LDS beside the static part need no asking)
            hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return; // (the caller asks for the error)
        hipLaunchKernelGGL(kern, dim3((unsigned)(a.nq * a.nsplit)), dim3(SW_NT), lds, st, a, lists);
    };
    if (exact) { // (rare: one instance for all code lengths)
        go(k_scan_wide<0, true>);
        return;
    }
    switch (a.m) {
    case 4: go(k_scan_wide<4, false>); break;
    case 8: go(k_scan_wide<8, false>); break;
    case 10: go(k_scan_wide<10, false>); break;
    case 12: go(k_scan_wide<12, false>); break;
    case 16: go(k_scan_wide<16, false>); break;
    case 20: go(k_scan_wide<20, false>); break;
    case 32: go(k_scan_wide<32, false>); break;
    default: go(k_scan_wide<0, false>); break;
    }
}
