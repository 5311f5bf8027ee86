// Streaming list scan with fused K-selection (Sec. 3.3.2 - 3.3.3): the fast path.
//
// Eq. 15 splits the ADC distance ||y - q1 - q2||^2 (Eq. 14) into
//     ||y - q1||^2  +  ||q2||^2 + 2 <q1, q2>  -  2 <y, q2>
// and Eq. 17 writes the first part with the coarse distances a = ||y - c_i||^2,
// b = ||y - s_ij||^2 and the edge length c:  (1-l) a + l b + (l^2 - l) c.
// Everything that does not depend on the query,
//     s_x = ||q2||^2 + 2 <q1 - mu, q2> + (l^2 - l) c     (term2 + term3/4 + the term7 part),
// is summed once per point when the lists are built and streamed with the code,
// so that a query needs ONE lookup table for the whole scan,
//     T[p][t] = 2 <(y - mu)^p, P[p][t]>                    (term5, 256 D multiply-adds),
// and per point m table reads:
//     dist = s_x + a + l (b - a) - sum_p T[p][t_p].
// mu is one vector fixed per index (the mean of the centroids); it cancels between s_x and T and
// keeps both inner products, and with them the rounding error of the sum, independent of where
// the data lie relative to the origin.
// a and b come from the traversal kernels (term6 / term8 are by-products of the
// region traversal), so the scan itself touches no centroid.
//
// Streams per point: m code bytes, 1 lambda byte, 4 bytes s_x.  Vector ids are
// not streamed: candidates are tracked by their position in the list arrays and
// ids are looked up for the K survivors only (the paper keeps ids off the scan
// path in the same way, Sec. 4).
//
// Work layout: one workgroup of 512 threads (8 waves) per (query, split).  The
// table lives in LDS.  Waves take whole lists from a shared counter; a wave
// issues all loads of up to 8 chunks of 64 points before it consumes the first,
// and enough waves are resident per compute unit to cover the memory latency.
// K-selection: every wave keeps the keys that passed, unordered, in LDS and prunes them alone when their number has
// grown by 128: the cut is found by bisection with ballot counts over keys in registers.  The waves share one
// monotonically decreasing upper bound of the K-th best key; at the end what lies below it (K keys and a few more) is
// ordered once, by counting.  Before, sorted lists were merged in LDS (bitonic networks, 35 stages a merge, a tree of
// merges and a sort of the result): with few points a query that took more of the LDS pipe than the table lookups
// (10 000 queries of 4 900 points, K = 100: 20 500 of 27 000 clocks a workgroup, 9 400 now; the scan 452 -> 360 us), and
// with many it was in the lookups' way (10 000 queries, 1 024 lists of 238 points, m = 16: 8.7 -> 8.3 ms; 512 of 480, m = 8:
// no difference beyond the noise).
#include "common.h"

#define SS_NT 512
#define SS_NW 8
#define SS_CH 8      // chunks of 64 points loaded ahead per wave
#define SS_KP 128    // results at most (K <= 128)
#define SS_WSZ 256   // keys a wave holds
#define SS_NEW 128   // candidates taken up between two prunings
#define SS_LEFT (SS_NW * SS_KP) // keys left at the end at most: K a wave
#define SS_CROWD (SS_NT / 2)    // keys from which on a cut is looked for before they are counted against each other
#define SS_GL 16     // packed form: lists taken at a time
#define SS_PCH 4     // packed form: chunks loaded ahead

typedef __attribute__((address_space(3))) unsigned long long lds_u64;
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

// PACKED: the lists are short (a few tens of points): a wave takes SS_GL lists at a time and lays
// their points end to end over its lanes, so that a chunk of 64 lanes holds several lists; each
// lane finds its list from the running lengths and carries its own a, b - a.
template <int M, bool PACKED>
__global__ __launch_bounds__(SS_NT, 4) void k_scan_stream(ScanArgs a, const uint4 *__restrict__ desc)
{
    // all LDS is static: the table sits at a fixed address, which folds into the lookups' offsets
    __shared__ __align__(16) float T[M * 256];
    __shared__ __align__(16) uint64_t keys[SS_NW * SS_WSZ];
    __shared__ float yv[VLQ_MAX_DIM];
    __shared__ unsigned long long sh_thr;              // upper bound of the K-th smallest key of the workgroup
    __shared__ unsigned long long sh_q[SS_NW];         // every wave's bound with ceil(K/8) of its keys below it
    __shared__ int sh_cnt[2][SS_NW], sh_ties;
    __shared__ uint32_t sh_range[2][SS_NW];
    __shared__ int sh_slot[SS_KP];                     // results that claim a place
    __shared__ uint64_t sh_out[SS_KP];                 // the results in order
    __shared__ int sh_next;                            // next list to hand out

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = blockIdx.x / a.nsplit, split = blockIdx.x - q * a.nsplit;
    const int r0 = (int)((int64_t)a.w2 * split / a.nsplit), r1 = (int)((int64_t)a.w2 * (split + 1) / a.nsplit);
    const int K = a.K, D = a.D, ds = D / M;
    const int KQ = (K + SS_NW - 1) / SS_NW;
    volatile lds_u64 *wk = (volatile lds_u64 *)(keys + wave * SS_WSZ);
    int wcnt = 0, wlimit = SS_NEW; // keys held; how many may be before the next pruning

    for (int d = tid; d < D; d += SS_NT) yv[d] = a.Q[(int64_t)q * D + d] - a.mu[d];
    if (tid == 0) {
        sh_thr = KEY_MAX;
        sh_next = r0;
    }
    if (tid < SS_NW) sh_q[tid] = KEY_MAX;
    if (tid < SS_KP) sh_slot[tid] = 0;
    if (tid == 0) sh_ties = 0;
    __syncthreads();
    // the query's table: T[p][t] = 2 <(y - mu)^p, P[p][t]>
    for (int e = tid * 4; e < M * 256; e += SS_NT * 4) *(f32x4 *)(T + e) = table_entries(a.Pt, yv, ds, e);
    __syncthreads();

    // Pruning of the wave's keys to its K smallest (of equal distances the first positions).  Publishes two
    // upper bounds of the K-th smallest key of the whole workgroup: the wave's own, and the largest of all waves' bounds
    // with ceil(K/8) keys below them (8 * ceil(K/8) >= K keys lie below it).  No order is needed for either, so the keys
    // stay in registers and the bounds are found by bisection with ballot counts.  (Sorting them in LDS cost 35 stages
    // a time; with short scans that kept the LDS pipe busy, not the table lookups.)
    auto prune = [&]() {
        uint64_t bound = sh_thr, k[SS_WSZ / 64];
        uint32_t o[SS_WSZ / 64], lo = 0xFFFFFFFFu, hi = 0xFFFFFFFFu; // hi: the complement of the largest
        int cnt = 0;
#pragma unroll
        for (int j = 0; j < SS_WSZ / 64; ++j) {
            k[j] = lane + 64 * j < wcnt ? wk[lane + 64 * j] : KEY_MAX;
            const bool in = k[j] < bound;
            o[j] = in ? (uint32_t)(k[j] >> 32) : 0xFFFFFFFFu; // (no key has this high word)
            cnt += __popcll(__ballot(in));
            lo = min(lo, o[j]);
            if (in) hi = min(hi, ~o[j]);
        }
        lo = wave_min_u32(lo);
        hi = ~wave_min_u32(hi);
        if (cnt > K) {
            const uint32_t cut = wave_cut(o, lo, hi, K);
            uint64_t own = (uint64_t)cut << 32;
            int below = 0;
#pragma unroll
            for (int j = 0; j < SS_WSZ / 64; ++j) below += __popcll(__ballot(o[j] < cut));
            if (below > K) { // equal distances at the cut
                uint32_t t[SS_WSZ / 64];
                int less = 0;
#pragma unroll
                for (int j = 0; j < SS_WSZ / 64; ++j) {
                    less += __popcll(__ballot(o[j] < cut - 1));
                    t[j] = o[j] == cut - 1 ? (uint32_t)k[j] : 0xFFFFFFFFu;
                }
                own = ((uint64_t)(cut - 1) << 32) | wave_cut(t, 0u, 0xFFFFFFFEu, K - less);
            }
            bound = own < bound ? own : bound;
            hi = min(hi, (uint32_t)(own >> 32));
        }
        wcnt = 0;
#pragma unroll
        for (int j = 0; j < SS_WSZ / 64; ++j) {
            const bool in = k[j] < bound;
            const uint64_t mask = __ballot(in);
            if (in) wk[wcnt + __popcll(mask & ((1ull << lane) - 1ull))] = k[j];
            wcnt += __popcll(mask);
        }
        wlimit = min(wcnt + SS_NEW, SS_WSZ);
        if (cnt >= KQ) {
            const uint32_t q = wave_cut(o, lo, hi, KQ);
            if (lane == 0) sh_q[wave] = (uint64_t)q << 32;
        }
        __builtin_amdgcn_wave_barrier();
        uint64_t all = 0;
#pragma unroll
        for (int w = 0; w < SS_NW; ++w) {
            const uint64_t t = ((volatile lds_u64 *)sh_q)[w];
            all = t > all ? t : all;
        }
        bound = all < bound ? all : bound;
        if (lane == 0 && bound != KEY_MAX) atomicMin(&sh_thr, (unsigned long long)bound);
        __builtin_amdgcn_wave_barrier();
    };

    // The distance a key below the bound has at most.  Bounds go one past the keys they are found from: behind infinite
    // distances that would be the pattern of a NaN, to which no distance compares.
    auto distance_bound = [](uint64_t bound) {
        return bound >= 0xFF80000000000000ull ? INFINITY : ord2f((uint32_t)(bound >> 32));
    };
    uint64_t thr = KEY_MAX;
    float thr_f = INFINITY;
    // one chunk of 64 points: m table reads per point, the distance, and the candidates that pass
    auto score_chunk = [&](const uint32_t (&cw)[M / 4], uint32_t lbv, float sxv, float av, float bav, uint32_t gpos,
                           bool live) __attribute__((always_inline)) {
        float ts = 0.f;
#pragma unroll
        for (int x = 0; x < M / 4; ++x)
#pragma unroll
            for (int bb = 0; bb < 4; ++bb) {
                const uint32_t byte_off = ((cw[x] >> (8 * bb)) & 255u) << 2;
                ts += *(const float *)((const char *)(T + (x * 4 + bb) * 256) + byte_off);
            }
        const float l = ((float)lbv - a.lam_zero) * a.lam_step;
        const float dist = (sxv - ts) + fmaf(l, bav, av);
        // cheap test on the distance alone; the exact (distance, position) key only for the few that pass
        bool pass = live && dist <= thr_f;
        uint64_t mask = __ballot(pass);
        if (mask) {
            const uint64_t key = make_key(dist, gpos);
            pass = pass && key < thr;
            mask = __ballot(pass);
            int np = __popcll(mask);
            if (np && wcnt + np > wlimit) {
                prune();
                thr = sh_thr;
                thr_f = distance_bound(thr);
                pass = pass && key < thr;
                mask = __ballot(pass);
                np = __popcll(mask);
            }
            if (pass) wk[wcnt + __popcll(mask & ((1ull << lane) - 1ull))] = key;
            wcnt += np;
        }
    };
    if (PACKED) {
        // up to SS_GL lists per turn, fewer when the workgroup has few lists, so that all waves get some
        int gl = (r1 - r0) / SS_NW;
        gl = gl < 1 ? 1 : (gl > SS_GL ? SS_GL : gl);
        for (;;) {
            int s = 0;
            if (lane == 0) s = atomicAdd(&sh_next, gl);
            s = __builtin_amdgcn_readfirstlane(s);
            if (s >= r1) break;
            // lane i < gl holds the descriptor of list s + i
            uint4 dsc = make_uint4(0u, 0u, 0u, 0u);
            if (lane < gl && s + lane < r1) dsc = desc[(int64_t)q * a.w2 + s + lane];
            const int len = max((int)dsc.y, 0);
            int end = len; // inclusive prefix sum: where the list ends in the concatenation
#pragma unroll
            for (int o = 1; o < SS_GL; o <<= 1) {
                const int t = __shfl_up(end, o, 64);
                if (lane >= o) end += t;
            }
            const int start = end - len;
            const int total = __builtin_amdgcn_readlane(end, SS_GL - 1);
            if (total <= 0) continue;
            int ends[SS_GL]; // uniform copies
#pragma unroll
            for (int i = 0; i < SS_GL; ++i) ends[i] = __builtin_amdgcn_readlane(end, i);
            thr = sh_thr;
            thr_f = distance_bound(thr);
            for (int base = 0; base < total; base += 64 * SS_PCH) {
                uint32_t cw[SS_PCH][M / 4];
                uint32_t lb[SS_PCH], gp[SS_PCH];
                float sv[SS_PCH], fav[SS_PCH], fbav[SS_PCH];
#pragma unroll
                for (int u = 0; u < SS_PCH; ++u) {
                    if (base + 64 * u < total) { // uniform over the wave
                        const int p = min(base + 64 * u + lane, total - 1); // idle lanes repeat the last point
                        int j = 0; // the list that holds position p: the lists before it end at or before p
#pragma unroll
                        for (int i = 0; i < SS_GL - 1; ++i) j += ends[i] <= p;
                        const uint32_t g = (uint32_t)__shfl((int)dsc.x, j, 64) + (uint32_t)(p - __shfl(start, j, 64));
                        fav[u] = __uint_as_float((uint32_t)__shfl((int)dsc.z, j, 64));
                        fbav[u] = __uint_as_float((uint32_t)__shfl((int)dsc.w, j, 64));
                        gp[u] = g;
                        const uint32_t *cp = (const uint32_t *)(a.codes + (size_t)g * M);
                        if (M == 8) {
                            const u32x2_t c2 = *(const u32x2_t *)cp;
                            cw[u][0] = c2.x;
                            cw[u][1] = c2.y;
                        } else {
                            const u32x4_t c4 = *(const u32x4_t *)cp;
#pragma unroll
                            for (int x = 0; x < M / 4; ++x) cw[u][x] = c4[x];
                        }
                        lb[u] = a.lam[g];
                        sv[u] = a.sx[g];
                    }
                }
#pragma unroll
                for (int u = 0; u < SS_PCH; ++u)
                    if (base + 64 * u < total)
                        score_chunk(cw[u], lb[u], sv[u], fav[u], fbav[u], gp[u], base + 64 * u + lane < total);
            }
        }
    } else {
    for (;;) {
        int s = 0;
        if (lane == 0) s = atomicAdd(&sh_next, 1);
        s = __builtin_amdgcn_readfirstlane(s);
        if (s >= r1) break;
        const uint4 dsc = desc[(int64_t)q * a.w2 + s]; // uniform address: scalar load
        const uint32_t beg = dsc.x;
        const int len = (int)dsc.y;
        const float av = __uint_as_float(dsc.z), bav = __uint_as_float(dsc.w);
        if (len <= 0) continue;
        // range-checked raw buffers over the three streams of this list: reads past the end
        // return zero and are masked out, so the chunk loop needs no address arithmetic
        const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc((void *)(a.codes + (int64_t)beg * M), 0, len * M, 0x00020000);
        const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc((void *)(a.lam + beg), 0, len, 0x00020000);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)(a.sx + beg), 0, len * 4, 0x00020000);
        thr = sh_thr;
        thr_f = distance_bound(thr);
        for (int base = 0; base < len; base += 64 * SS_CH) {
            // ---- all loads of up to SS_CH chunks ----
            uint32_t cw[SS_CH][M / 4];
            uint32_t lb[SS_CH];
            float sv[SS_CH];
#pragma unroll
            for (int u = 0; u < SS_CH; ++u) {
                if (base + 64 * u < len) { // uniform over the wave
                    const int so = base + 64 * u;
                    if (M == 8) {
                        const u32x2_t c2 = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(rc, lane * 8, so * 8, 0));
                        cw[u][0] = c2.x;
                        cw[u][1] = c2.y;
                    } else {
                        const u32x4_t c4 = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rc, lane * 16, so * 16, 0));
#pragma unroll
                        for (int x = 0; x < M / 4; ++x) cw[u][x] = c4[x];
                    }
                    lb[u] = __builtin_amdgcn_raw_buffer_load_b8(rl, lane, so, 0);
                    sv[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4, so * 4, 0));
                }
            }
            // ---- score ----
#pragma unroll
            for (int u = 0; u < SS_CH; ++u)
                if (base + 64 * u < len) {
                    const int within = base + 64 * u + lane;
                    score_chunk(cw[u], lb[u], sv[u], av, bav, beg + (uint32_t)within, within < len);
                }
        }
    }
    }

    // ---- the K smallest of all waves' keys; ids; order by (distance, id) ----
    // What is left below the last bound (K keys and a few more) goes to one array, distances and positions apart; a key's
    // place is the number of smaller distances, counted by one to four lanes a key.
    prune();
    __syncthreads();
    thr = sh_thr;
    uint64_t left[SS_WSZ / 64];
    int mine = 0;
#pragma unroll
    for (int j = 0; j < SS_WSZ / 64; ++j) {
        left[j] = lane + 64 * j < wcnt ? wk[lane + 64 * j] : KEY_MAX;
        mine += __popcll(__ballot(left[j] < thr));
    }
    if (lane == 0) sh_cnt[0][wave] = mine;
    __syncthreads(); // (all keys are in registers)
    uint32_t *od = (uint32_t *)keys;                // [SS_LEFT + 16] ordered distances
    uint32_t *op = od + SS_LEFT + 16;               // [SS_LEFT] positions
    uint32_t *to = (uint32_t *)T, *tp = to + SS_LEFT; // [SS_LEFT] those of equal distance (the table is dead)
    static_assert(M * 256 >= 2 * SS_LEFT, "they take the table's place");
    int at = 0, total = 0;
    auto places = [&](const int (&cnt)[SS_NW]) {
        at = total = 0;
#pragma unroll
        for (int w = 0; w < SS_NW; ++w) {
            const int c = cnt[w];
            at += w < wave ? c : 0;
            total += c;
        }
    };
    places(sh_cnt[0]);
    if (total > SS_CROWD) {
        // Waves of few keys publish no bound, and all keys are left: a cut over the workgroup, until at most SS_CROWD are (a
        // barrier a round; equal distances at the cut stay).  300 queries of 2 500 points, K = 128, the scan: 58 us without, 44
        // with it, 47 with sorted lists.
        uint32_t lo = 0xFFFFFFFFu, hi = 0xFFFFFFFFu; // hi: the complement of the largest
#pragma unroll
        for (int j = 0; j < SS_WSZ / 64; ++j) {
            const uint32_t o = (uint32_t)(left[j] >> 32);
            lo = min(lo, left[j] < thr ? o : 0xFFFFFFFFu);
            hi = min(hi, left[j] < thr ? ~o : 0xFFFFFFFFu);
        }
        lo = wave_min_u32(lo);
        hi = wave_min_u32(hi);
        if (lane == 0) {
            sh_range[0][wave] = lo;
            sh_range[1][wave] = hi;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < SS_NW; ++w) {
            lo = min(lo, sh_range[0][w]);
            hi = min(hi, sh_range[1][w]);
        }
        lo = __builtin_amdgcn_readfirstlane((int)lo);
        hi = __builtin_amdgcn_readfirstlane((int)~hi);
        int turn = 1;
        auto count = [&](uint64_t bound) {
            int c = 0;
#pragma unroll
            for (int j = 0; j < SS_WSZ / 64; ++j) c += __popcll(__ballot(left[j] < bound));
            if (lane == 0) sh_cnt[turn][wave] = c;
            __syncthreads();
            places(sh_cnt[turn]);
            turn ^= 1;
        };
        uint64_t cut = KEY_MAX;
        while (lo < hi) {
            const uint32_t mid = lo + ((hi - lo + 1) >> 1);
            count((uint64_t)mid << 32);
            const int below = __builtin_amdgcn_readfirstlane(total);
            if (below >= K && below <= SS_CROWD) {
                cut = (uint64_t)mid << 32;
                break;
            }
            if (below < K)
                lo = mid;
            else
                hi = mid - 1;
        }
        if (cut == KEY_MAX) { // (fewer than K below lo, K or more up to it)
            cut = ((uint64_t)lo + 1) << 32;
            cut = cut < thr ? cut : thr;
            count(cut);
        }
        thr = cut;
    }
#pragma unroll
    for (int j = 0; j < SS_WSZ / 64; ++j) {
        const bool in = left[j] < thr;
        const uint64_t mask = __ballot(in);
        if (in) {
            const int i = at + __popcll(mask & ((1ull << lane) - 1ull));
            od[i] = (uint32_t)(left[j] >> 32);
            op[i] = (uint32_t)left[j];
        }
        at += __popcll(mask);
    }
    if (tid < 16) od[total + tid] = 0xFFFFFFFFu; // up to a multiple of 16
    __syncthreads();
    const int gs = total <= SS_NT / 4 ? 2 : (total <= SS_NT / 2 ? 1 : 0); // 2^gs lanes a key
    const int per = (total + (4 << gs) - 1) >> (2 + gs), g = tid & ((1 << gs) - 1); // quadruples a lane goes through
    auto over_group = [&](int c) {
        if (gs >= 1) c += __builtin_amdgcn_update_dpp(0, c, 0xB1, 0xF, 0xF, true);
        if (gs == 2) c += __builtin_amdgcn_update_dpp(0, c, 0x4E, 0xF, 0xF, true);
        return c;
    };
    int place[SS_LEFT / SS_NT]; // of the keys tid >> gs, + 512
#pragma unroll
    for (int e = 0; e < SS_LEFT / SS_NT; ++e) {
        place[e] = K;
        if (e * SS_NT >= total) break; // uniform
        const int i = e * SS_NT + (tid >> gs);
        const uint32_t o = od[min(i, total - 1)];
        int c = 0;
#pragma unroll 4
        for (int j = 0; j < per; ++j) {
            const u32x4_t v = *(const u32x4_t *)(od + 4 * (g * per + j));
            c += (v.x < o) + (v.y < o) + (v.z < o) + (v.w < o);
        }
        place[e] = over_group(c);
        if (i < total && g == 0 && place[e] < K) atomicAdd(&sh_slot[place[e]], 1);
    }
    __syncthreads();
    // a place that one key claims is settled; equal distances claim the same one and go on a list
    int tied[SS_LEFT / SS_NT];
    bool any = false;
#pragma unroll
    for (int e = 0; e < SS_LEFT / SS_NT; ++e) {
        tied[e] = -1;
        const int i = e * SS_NT + (tid >> gs);
        if (i < total && g == 0 && place[e] < K) {
            if (sh_slot[place[e]] == 1) {
                sh_out[place[e]] = ((uint64_t)od[i] << 32) | (uint32_t)a.ids[op[i]];
            } else {
                tied[e] = atomicAdd(&sh_ties, 1);
                to[tied[e]] = od[i];
                tp[tied[e]] = op[i];
                any = true;
            }
        }
    }
    if (__syncthreads_or(any)) {
        // the first positions of a distance are taken, and ordered by id
        const int nt = sh_ties;
        if (tid < 4 && nt + tid < SS_LEFT) to[nt + tid] = 0xFFFFFFFFu; // (read four at a time)
        __syncthreads();
        // entries of the list with distance o and x below v (or x == v and an earlier entry than `own`)
        auto before = [&](uint32_t o, uint32_t v, int own) {
            int c = 0;
#pragma unroll 4
            for (int j = 0; j < nt; j += 4) {
                const u32x4_t d = *(const u32x4_t *)(to + j), x = *(const u32x4_t *)(tp + j);
#pragma unroll
                for (int u = 0; u < 4; ++u) c += d[u] == o && (x[u] < v || (x[u] == v && j + u < own));
            }
            return c;
        };
        uint32_t o[SS_LEFT / SS_NT], id[SS_LEFT / SS_NT];
#pragma unroll
        for (int e = 0; e < SS_LEFT / SS_NT; ++e) {
            if (tied[e] < 0) continue;
            const uint32_t p = tp[tied[e]];
            o[e] = to[tied[e]];
            const bool in = place[e] + before(o[e], p, 0) < K;
            id[e] = in ? (uint32_t)a.ids[p] : 0u;
            if (!in) place[e] = K;
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < SS_LEFT / SS_NT; ++e) {
            if (tied[e] < 0) continue;
            tp[tied[e]] = id[e];
            if (place[e] == K) to[tied[e]] = 0xFFFFFFFFu;
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < SS_LEFT / SS_NT; ++e)
            if (tied[e] >= 0 && place[e] < K)
                sh_out[place[e] + before(o[e], id[e], tied[e])] = ((uint64_t)o[e] << 32) | id[e];
        __syncthreads();
    }
    for (int i = tid; i < K; i += SS_NT) {
        const uint64_t key = i < total ? sh_out[i] : KEY_MAX;
        if (a.nsplit > 1) {
            a.partial[((int64_t)q * a.nsplit + split) * K + i] = key;
        } else {
            a.out_dist[(int64_t)q * K + i] = i < total ? ord2f((uint32_t)(key >> 32)) : INFINITY;
            a.out_ids[(int64_t)q * K + i] = i < total ? (int32_t)(uint32_t)key : -1;
        }
    }
}

__global__ void k_transpose_codewords(const float *__restrict__ P, int ds, float *__restrict__ Pt)
{
    const float *p = P + (int64_t)blockIdx.x * 256 * ds;
    for (int d = 0; d < ds; ++d) Pt[((int64_t)blockIdx.x * ds + d) * 256 + threadIdx.x] = p[threadIdx.x * ds + d];
}

void launch_transpose_codewords(const float *P, int m, int ds, float *Pt, hipStream_t st)
{
    hipLaunchKernelGGL(k_transpose_codewords, dim3((unsigned)m), dim3(256), 0, st, P, ds, Pt);
}

// Shapes served by this kernel; the others go to k_scan_wide or k_scan (scan_will_stream).
bool scan_stream_supported(const ScanArgs &a)
{
    return (a.m == 8 || a.m == 16) && a.K <= SS_KP && a.sx != nullptr && a.mu != nullptr && a.desc != nullptr &&
           (((uintptr_t)a.codes) % 16 == 0);
}

void launch_scan_stream(const ScanArgs &a, hipStream_t st)
{
    if (a.nq <= 0) return;
    const dim3 grid((unsigned)(a.nq * a.nsplit));
    const uint4 *desc = (const uint4 *)a.desc;
    if (a.m == 8) {
        if (a.packed)
            hipLaunchKernelGGL((k_scan_stream<8, true>), grid, dim3(SS_NT), 0, st, a, desc);
        else
            hipLaunchKernelGGL((k_scan_stream<8, false>), grid, dim3(SS_NT), 0, st, a, desc);
    } else {
        if (a.packed)
            hipLaunchKernelGGL((k_scan_stream<16, true>), grid, dim3(SS_NT), 0, st, a, desc);
        else
            hipLaunchKernelGGL((k_scan_stream<16, false>), grid, dim3(SS_NT), 0, st, a, desc);
    }
}
