// Inverted lists (Sec. 4): list lengths (as offsets), ids, codes and lambda
// bytes of the k*n sub-regions, list l = cell * n + edge, ascending id inside a
// list.  Built by a counting sort of the staged points.
#include "common.h"

__global__ void k_iota_i32(int32_t *p, int64_t n, int32_t start)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = start + (int32_t)i;
}
void launch_iota_i32(int32_t *p, int64_t n, int32_t start, hipStream_t st)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_iota_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, start);
}

__global__ void k_pack_labels(const int32_t *__restrict__ cell, const int32_t *__restrict__ edge, int n, int k,
                              int32_t *__restrict__ label, int64_t nb, int32_t *__restrict__ bad)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nb) return;
    const int c = cell[i], e = edge[i];
    if (c < 0 || c >= k || e < 0 || e >= n) {
        label[i] = -1;
        atomicOr(bad, 1);
    } else {
        label[i] = c * n + e;
    }
}
void launch_pack_labels(const int32_t *cell, const int32_t *edge, int n, int k, int32_t *label, int64_t nb,
                        int32_t *bad, hipStream_t st)
{
    if (nb <= 0) return;
    hipLaunchKernelGGL(k_pack_labels, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, st, cell, edge, n, k,
                       label, nb, bad);
}

__global__ void k_list_histogram(const int32_t *__restrict__ label, int64_t N, int32_t *__restrict__ cnt)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride) {
        const int l = label[i];
        if (l >= 0) atomicAdd(&cnt[l], 1);
    }
}
void launch_list_histogram(const int32_t *label, int64_t N, int32_t *cnt, hipStream_t st)
{
    if (N <= 0) return;
    int64_t blocks = (N + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_list_histogram, dim3((unsigned)blocks), dim3(256), 0, st, label, N, cnt);
}

// off[i] = sum of cnt[0..i), off[nl] = total; one workgroup walks the array in tiles of 16 384
// (sixteen consecutive counts per thread: few rounds, each with two barriers), carrying the sum.
#define XS_PER 16
__global__ __launch_bounds__(1024) void k_exclusive_scan(const int32_t *__restrict__ cnt, int64_t nl,
                                                         int64_t *__restrict__ off)
{
    __shared__ int64_t wsum[16];
    __shared__ int64_t carry_sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool vec = ((uintptr_t)cnt) % 16 == 0;
    int64_t carry = 0;
    for (int64_t t0 = 0; t0 < nl; t0 += 1024 * XS_PER) {
        const int64_t i0 = t0 + XS_PER * tid;
        int32_t c[XS_PER];
        if (vec && i0 + XS_PER <= nl) {
#pragma unroll
            for (int e = 0; e < XS_PER; e += 4) {
                const int4 v = *(const int4 *)(cnt + i0 + e);
                c[e] = v.x;
                c[e + 1] = v.y;
                c[e + 2] = v.z;
                c[e + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int e = 0; e < XS_PER; ++e) c[e] = i0 + e < nl ? cnt[i0 + e] : 0;
        }
        int64_t mine = 0;
#pragma unroll
        for (int e = 0; e < XS_PER; ++e) mine += c[e];
        int64_t inc = mine; // inclusive scan over the wave
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t v = __shfl_up(inc, o, 64);
            if (lane >= o) inc += v;
        }
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        int64_t before = carry;
        for (int w = 0; w < wave; ++w) before += wsum[w];
        int64_t run = before + inc - mine;
#pragma unroll
        for (int e = 0; e < XS_PER; ++e) {
            if (i0 + e < nl) off[i0 + e] = run;
            run += c[e];
        }
        if (tid == 1023) carry_sh = run;
        __syncthreads();
        carry = carry_sh;
    }
    if (tid == 0) off[nl] = carry;
}
// The same for short arrays (the per-cell pair counts of a search) without the serial walk: a workgroup per
// 4 096 counts first adds up everything before its tile (read again by every later workgroup: a few
// hundred KB from L2 at most), then scans its own tile.
#define XB_TILE 4096
// With chunk > 0, a power of two, the scan of ceil(cnt / chunk) goes to off2 beside it (both are summed in one word, the counts
// in the low 32 bits, the chunk counts above them: for counts that add up to less than 2^31).
__global__ __launch_bounds__(256) void k_exclusive_scan_tiles(const int32_t *__restrict__ cnt, int64_t nl,
                                                              int64_t *__restrict__ off, int chunk,
                                                              int64_t *__restrict__ off2)
{
    __shared__ int64_t wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t t0 = (int64_t)blockIdx.x * XB_TILE;
    // (chunk is a power of two)
    const int csh = chunk > 0 ? 31 - __clz(chunk) : 0;
    auto both = [&](int32_t c) { return (int64_t)c + (chunk > 0 ? (int64_t)((c + chunk - 1) >> csh) << 32 : 0); };
    const int64_t low = chunk > 0 ? (((int64_t)1 << 32) - 1) : ~(int64_t)0;
    int64_t before = 0;
    for (int64_t i = 4 * tid; i < t0; i += XB_TILE) { // t0 is a multiple of the tile: four loads in flight
        int4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = *(const int4 *)(cnt + i + 1024 * u);
#pragma unroll
        for (int u = 0; u < 4; ++u) before += both(v[u].x) + both(v[u].y) + both(v[u].z) + both(v[u].w);
    }
    const int64_t i0 = t0 + XS_PER * tid;
    int32_t c[XS_PER];
#pragma unroll
    for (int e = 0; e < XS_PER; ++e) c[e] = i0 + e < nl ? cnt[i0 + e] : 0;
    int64_t mine = 0;
#pragma unroll
    for (int e = 0; e < XS_PER; ++e) mine += both(c[e]);
    // the sum of `before` over the workgroup, and the scan of `mine`
    int64_t inc = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t v = __shfl_up(inc, o, 64);
        if (lane >= o) inc += v;
        before += __shfl_xor(before, o, 64);
    }
    if (lane == 63) wsum[wave] = inc;
    __shared__ int64_t bsum[4];
    if (lane == 0) bsum[wave] = before;
    __syncthreads();
    int64_t run = bsum[0] + bsum[1] + bsum[2] + bsum[3] + inc - mine;
    for (int w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
    for (int e = 0; e < XS_PER; ++e) {
        if (i0 + e < nl) {
            off[i0 + e] = run & low;
            if (chunk > 0) off2[i0 + e] = run >> 32;
        }
        run += both(c[e]);
    }
    if (i0 <= nl - 1 && nl - 1 < i0 + XS_PER) { // the thread that holds the last count
        off[nl] = run & low;
        if (chunk > 0) off2[nl] = run >> 32;
    }
}

void launch_exclusive_scan(const int32_t *cnt, int64_t nl, int64_t *off, hipStream_t st)
{
    if (nl > 0 && nl <= ((int64_t)1 << 18) && ((uintptr_t)cnt) % 16 == 0)
        hipLaunchKernelGGL(k_exclusive_scan_tiles, dim3((unsigned)((nl + XB_TILE - 1) / XB_TILE)), dim3(256), 0, st, cnt,
                           nl, off, 0, (int64_t *)nullptr);
    else
        hipLaunchKernelGGL(k_exclusive_scan, dim3(1), dim3(1024), 0, st, cnt, nl, off);
}

void launch_exclusive_scan_chunks(const int32_t *cnt, int64_t nl, int64_t *off, int chunk, int64_t *off2, hipStream_t st)
{
    hipLaunchKernelGGL(k_exclusive_scan_tiles, dim3((unsigned)((nl + XB_TILE - 1) / XB_TILE)), dim3(256), 0, st, cnt, nl,
                       off, chunk, off2);
}

__global__ void k_list_scatter(const int32_t *__restrict__ label, const int32_t *__restrict__ st_ids,
                               const uint8_t *__restrict__ st_codes, const uint8_t *__restrict__ st_lam,
                               int64_t N, int m, const int64_t *__restrict__ off,
                               int32_t *__restrict__ cursor, int32_t *__restrict__ ids,
                               uint8_t *__restrict__ codes, uint8_t *__restrict__ lam)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride) {
        const int l = label[i];
        if (l < 0) continue;
        const int64_t pos = off[l] + atomicAdd(&cursor[l], 1);
        ids[pos] = st_ids[i];
        lam[pos] = st_lam[i];
        if ((m & 3) == 0) {
            const uint32_t *s = (const uint32_t *)(st_codes + i * m);
            uint32_t *d = (uint32_t *)(codes + pos * m);
            for (int p = 0; p < m / 4; ++p) d[p] = s[p];
        } else {
            for (int p = 0; p < m; ++p) codes[pos * m + p] = st_codes[i * m + p];
        }
    }
}
void launch_list_scatter(const int32_t *label, const int32_t *st_ids, const uint8_t *st_codes,
                         const uint8_t *st_lam, int64_t N, int m, const int64_t *off, int32_t *cursor,
                         int32_t *ids, uint8_t *codes, uint8_t *lam, hipStream_t st)
{
    if (N <= 0) return;
    int64_t blocks = (N + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_list_scatter, dim3((unsigned)blocks), dim3(256), 0, st, label, st_ids, st_codes, st_lam,
                       N, m, off, cursor, ids, codes, lam);
}

// The scatter places the points of a list in arbitrary order; this pass orders
// every list by id.  One 64-thread workgroup per list sorts lists of up to
// SORT_MAX points in LDS; longer unsorted lists are reported to the host.
#define SORT_MAX 1024

// one list, by a workgroup of 64 threads; keys [SORT_MAX], pay [SORT_MAX (m + 1)] and unsorted in LDS
__device__ __forceinline__ void sort_list(const int64_t *__restrict__ off, int64_t l, int m, int32_t *__restrict__ ids,
                                          uint8_t *__restrict__ codes, uint8_t *__restrict__ lam,
                                          int32_t *__restrict__ long_lists, int32_t *__restrict__ n_long, int max_long,
                                          uint64_t *keys, uint8_t *pay, int *unsorted, int tid)
{
    const int64_t beg = off[l], len = off[l + 1] - beg;
    if (len <= 1) return;
    __syncthreads(); // (the list before has been read)
    if (tid == 0) *unsorted = 0;
    __syncthreads();
    for (int64_t i = tid; i + 1 < len; i += 64)
        if (ids[beg + i] > ids[beg + i + 1]) *unsorted = 1;
    __syncthreads();
    if (!*unsorted) return;
    if (len > SORT_MAX) {
        if (tid == 0) {
            const int p = atomicAdd(n_long, 1);
            if (p < max_long) long_lists[p] = (int32_t)l;
        }
        return;
    }
    const int sz = next_pow2_dev((int)len);
    for (int i = tid; i < sz; i += 64)
        keys[i] = i < len ? (((uint64_t)(uint32_t)ids[beg + i] << 32) | (uint32_t)i) : KEY_MAX;
    for (int64_t i = tid; i < len * m; i += 64) pay[i] = codes[beg * m + i];
    for (int i = tid; i < len; i += 64) pay[len * m + i] = lam[beg + i];
    __syncthreads();
    block_bitonic_sort<64>(keys, sz, tid);
    for (int i = tid; i < len; i += 64) {
        const uint64_t key = keys[i];
        const int src = (int)(uint32_t)key;
        ids[beg + i] = (int32_t)(uint32_t)(key >> 32);
        lam[beg + i] = pay[len * m + src];
        for (int p = 0; p < m; ++p) codes[(beg + i) * m + p] = pay[src * m + p];
    }
}

// A workgroup per list; with `work`, the lists on it (n_work[0] of them, handed out through n_work[1] after the first of each
// workgroup: where there are none, thousands of workgroups would queue for the one address).
__global__ __launch_bounds__(64) void k_list_sort(const int64_t *__restrict__ off, int m, int32_t *__restrict__ ids,
                                                  uint8_t *__restrict__ codes, uint8_t *__restrict__ lam,
                                                  int32_t *__restrict__ long_lists, int32_t *__restrict__ n_long,
                                                  int max_long, const int32_t *__restrict__ work,
                                                  int32_t *__restrict__ n_work)
{
    extern __shared__ unsigned char smem[];
    uint64_t *keys = (uint64_t *)smem;            // [SORT_MAX]
    uint8_t *pay = (uint8_t *)(keys + SORT_MAX);  // [SORT_MAX * (m + 1)]
    __shared__ int unsorted;
    const int tid = threadIdx.x;
    if (!work) {
        sort_list(off, blockIdx.x, m, ids, codes, lam, long_lists, n_long, max_long, keys, pay, &unsorted, tid);
        return;
    }
    const int n = n_work[0];
    for (int i = blockIdx.x; i < n;) {
        sort_list(off, work[i], m, ids, codes, lam, long_lists, n_long, max_long, keys, pay, &unsorted, tid);
        if (tid == 0) i = (int)gridDim.x + atomicAdd(&n_work[1], 1);
        i = __builtin_amdgcn_readfirstlane(i); // (the workgroup is one wave)
    }
}

// Lists of few points: 4 to 64 of them a workgroup, those of up to 16 points sorted by 16 lanes each, those of up to LS_FEW by the wave,
// without keys in LDS or barriers (2 M points in 524 288 lists, a workgroup each: 1.90 -> 0.23 ms); longer ones go on the
// worklist.  (Sorted here as well, one after the other, the lists of a crowded cell, which lie next to each other, kept one
// wave busy: 2 M points in 2 560 of 1 M lists, finalisation 2.0 -> 6.7 ms.)  As few lists a workgroup as give 64 waves a compute unit:
// 64 lists each are one chain of loads behind the other and leave a small index on a few waves (16 384 lists of 4 points, uneven cells:
// 53 us with 16 lists each, 16 with 4).  Finalisation of 65 536 points in those lists, D/m = 6: a workgroup and a wave a list 222 us, 364 with 64
// lists a workgroup and the long lists' terms in a launch of their own, 218 now; even cells 211, 166, 154.
#define LS_SHORT 16 // mean points a list up to which that is done
#define LS_FEW 64
#define LS_WAVES 8192 // waves that run at once: 32 a compute unit
__global__ __launch_bounds__(64) void k_list_sort_few(const int64_t *__restrict__ off, int64_t nl, int per, int m,
                                                      int32_t *__restrict__ ids, uint8_t *__restrict__ codes,
                                                      uint8_t *__restrict__ lam, int32_t *__restrict__ work,
                                                      int32_t *__restrict__ n_work)
{
    extern __shared__ unsigned char smem[]; // [4][16 (m + 1)], or [64 (m + 1)]
    const int tid = threadIdx.x;
    const int64_t l0 = (int64_t)blockIdx.x * per;
    const int64_t mybeg = off[min(l0 + tid, nl)], mylen = tid < per ? off[min(l0 + tid + 1, nl)] - mybeg : 0;
    const uint64_t more = __ballot(mylen > LS_FEW);
    if (more) {
        int at = 0;
        if (tid == 0) at = atomicAdd(&n_work[0], __popcll(more));
        at = __builtin_amdgcn_readfirstlane(at);
        if (mylen > LS_FEW) work[at + __popcll(more & ((1ull << tid) - 1ull))] = (int32_t)(l0 + tid);
    }
    // four lists at a time, a point's place counted over the group
    uint64_t todo = __ballot(mylen > 1 && mylen <= 16);
    while (todo) {
        int src[4]; // (uniform)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            src[u] = todo ? __ffsll((unsigned long long)todo) - 1 : -1;
            todo &= todo - 1;
        }
        const int sub = tid >> 4, l16 = tid & 15;
        const int from = sub == 0 ? src[0] : (sub == 1 ? src[1] : (sub == 2 ? src[2] : src[3]));
        const int llen = __shfl((int)mylen, max(from, 0), 64), len = from >= 0 ? llen : 0;
        const int64_t beg = ((int64_t)__shfl((int)(mybeg >> 32), max(from, 0), 64) << 32) |
                            (uint32_t)__shfl((int)(uint32_t)mybeg, max(from, 0), 64);
        const bool on = l16 < len;
        const uint32_t id = on ? (uint32_t)ids[beg + l16] : 0xFFFFFFFFu;
        const int next = __shfl_down((int)id, 1, 16);
        const uint64_t falls = __ballot(l16 + 1 < len && (int)id > next);
        if (!falls) continue;
        int place = 0;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const uint32_t o = (uint32_t)__shfl((int)id, 16 * sub + j, 64);
            place += o < id || (o == id && j < l16);
        }
        uint8_t *pg = smem + sub * 16 * (m + 1); // the group's codes and lambdas, as they were
        if (on) {
            for (int p = 0; p < m; ++p) pg[l16 * m + p] = codes[(beg + l16) * m + p];
            pg[16 * m + l16] = lam[beg + l16];
        }
        wave_lds_order();
        if (on && place != l16 && ((falls >> (16 * sub)) & 0xFFFFull)) { // (a list that is in order stays)
            ids[beg + place] = (int32_t)id;
            lam[beg + place] = pg[16 * m + l16];
            for (int p = 0; p < m; ++p) codes[(beg + place) * m + p] = pg[l16 * m + p];
        }
        wave_lds_order();
    }
    // one list at a time
    for (uint64_t left = __ballot(mylen > 16 && mylen <= LS_FEW); left; left &= left - 1) {
        const int from = __ffsll((unsigned long long)left) - 1;
        const int64_t beg = off[l0 + from];
        const int len = (int)(off[l0 + from + 1] - beg);
        const bool on = tid < len;
        const uint32_t id = on ? (uint32_t)ids[beg + tid] : 0xFFFFFFFFu;
        const int next = __shfl_down((int)id, 1, 64);
        if (!__ballot(tid + 1 < len && (int)id > next)) continue;
        int place = 0;
        for (int j = 0; j < len; ++j) {
            const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)id, j);
            place += o < id || (o == id && j < tid);
        }
        if (on) {
            for (int p = 0; p < m; ++p) smem[tid * m + p] = codes[(beg + tid) * m + p];
            smem[LS_FEW * m + tid] = lam[beg + tid];
        }
        wave_lds_order();
        if (on) {
            ids[beg + place] = (int32_t)id;
            lam[beg + place] = smem[LS_FEW * m + tid];
            for (int p = 0; p < m; ++p) codes[(beg + place) * m + p] = smem[tid * m + p];
        }
        wave_lds_order();
    }
}

bool lists_are_short(int64_t nl, int64_t N) { return N <= LS_SHORT * nl; }

void launch_list_sort(const int64_t *off, int64_t nl, int m, int32_t *ids, uint8_t *codes, uint8_t *lam,
                      int64_t N, int32_t *long_lists, int32_t *n_long, int max_long, int32_t *work, int32_t *n_work,
                      hipStream_t st)
{
    if (nl <= 0) return;
    const size_t smem = (size_t)SORT_MAX * 8 + (size_t)SORT_MAX * (m + 1);
    (void)hipFuncSetAttribute((const void *)k_list_sort, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (!lists_are_short(nl, N)) {
        hipLaunchKernelGGL(k_list_sort, dim3((unsigned)nl), dim3(64), smem, st, off, m, ids, codes, lam, long_lists, n_long,
                           max_long, (const int32_t *)nullptr, (int32_t *)nullptr);
        return;
    }
    int per = 4; // lists a workgroup
    while (per < 64 && nl > (int64_t)per * 2 * LS_WAVES) per *= 2;
    hipLaunchKernelGGL(k_list_sort_few, dim3((unsigned)((nl + per - 1) / per)), dim3(64), (size_t)LS_FEW * (m + 1), st, off, nl, per,
                       m, ids, codes, lam, work, n_work);
    const int64_t most = N / (LS_FEW + 1); // lists on the worklist; more workgroups than run at once are of no use
    if (most > 0)
        hipLaunchKernelGGL(k_list_sort, dim3((unsigned)(most < 4096 ? most : 4096)), dim3(64), smem, st, off, m, ids, codes, lam,
                           long_lists, n_long, max_long, (const int32_t *)work, n_work);
}

// Second tier: the lists the 64-thread pass reported (more than SORT_MAX points), one
// 256-thread workgroup each, keys and payload in up to 150 KB of LDS.  Lists beyond mid_max
// points are passed on to the third tier.
__global__ __launch_bounds__(256) void k_list_sort_mid(const int64_t *__restrict__ off, int m, int mid_max,
                                                       const int32_t *__restrict__ in_lists, int n_in,
                                                       int32_t *__restrict__ ids, uint8_t *__restrict__ codes,
                                                       uint8_t *__restrict__ lam, int32_t *__restrict__ out_lists,
                                                       int32_t *__restrict__ n_out, int max_out)
{
    extern __shared__ unsigned char smem[];
    uint64_t *keys = (uint64_t *)smem;           // [mid_max]
    uint8_t *pay = (uint8_t *)(keys + mid_max);  // [mid_max * (m + 1)]
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= n_in) return;
    const int64_t l = in_lists[blockIdx.x];
    const int64_t beg = off[l];
    const int64_t len = off[l + 1] - beg;
    if (len > mid_max) {
        if (tid == 0) {
            const int p = atomicAdd(n_out, 1);
            if (p < max_out) out_lists[p] = (int32_t)l;
        }
        return;
    }
    const int sz = next_pow2_dev((int)len);
    for (int i = tid; i < sz; i += 256)
        keys[i] = i < len ? (((uint64_t)(uint32_t)ids[beg + i] << 32) | (uint32_t)i) : KEY_MAX;
    for (int64_t i = tid; i < len * m; i += 256) pay[i] = codes[beg * m + i];
    for (int i = tid; i < len; i += 256) pay[len * m + i] = lam[beg + i];
    __syncthreads();
    block_bitonic_sort<256>(keys, sz, tid);
    for (int i = tid; i < len; i += 256) {
        const uint64_t key = keys[i];
        const int src = (int)(uint32_t)key;
        ids[beg + i] = (int32_t)(uint32_t)(key >> 32);
        lam[beg + i] = pay[len * m + src];
        for (int p = 0; p < m; ++p) codes[(beg + i) * m + p] = pay[src * m + p];
    }
}

int list_sort_mid_max(int m)
{
    // keys (8 B) + payload (m + 1 B) per point within 150 KB, as a power of two, at least 2 * SORT_MAX
    int mm = 8192;
    while (mm > 2 * SORT_MAX && (size_t)mm * (8 + m + 1) > 150 * 1024) mm >>= 1;
    return (size_t)mm * (8 + m + 1) <= 150 * 1024 ? mm : 0;
}

void launch_list_sort_mid(const int64_t *off, int m, const int32_t *in_lists, int n_in, int32_t *ids, uint8_t *codes,
                          uint8_t *lam, int32_t *out_lists, int32_t *n_out, int max_out, hipStream_t st)
{
    const int mm = list_sort_mid_max(m);
    if (n_in <= 0 || mm == 0) return;
    const size_t smem = (size_t)mm * (8 + m + 1);
    (void)hipFuncSetAttribute((const void *)k_list_sort_mid, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    hipLaunchKernelGGL(k_list_sort_mid, dim3((unsigned)n_in), dim3(256), smem, st, off, m, mm, in_lists, n_in, ids,
                       codes, lam, out_lists, n_out, max_out);
}

// A list too long for LDS: bitonic sort of (id, position) keys in global memory
// by a single workgroup, then the payload is permuted through a scratch copy.
__global__ __launch_bounds__(1024) void k_long_list_sort(int64_t beg, int64_t len, int64_t sz, int m,
                                                         int32_t *__restrict__ ids, uint8_t *__restrict__ codes,
                                                         uint8_t *__restrict__ lam, uint64_t *__restrict__ keys,
                                                         uint8_t *__restrict__ pay)
{
    const int tid = threadIdx.x;
    for (int64_t i = tid; i < sz; i += 1024)
        keys[i] = i < len ? (((uint64_t)(uint32_t)ids[beg + i] << 32) | (uint32_t)i) : KEY_MAX;
    for (int64_t i = tid; i < len * m; i += 1024) pay[i] = codes[beg * m + i];
    for (int64_t i = tid; i < len; i += 1024) pay[len * m + i] = lam[beg + i];
    __syncthreads();
    for (int64_t k = 2; k <= sz; k <<= 1)
        for (int64_t j = k >> 1; j > 0; j >>= 1) {
            for (int64_t i = tid; i < (sz >> 1); i += 1024) {
                const int64_t lo = ((i & ~(j - 1)) << 1) | (i & (j - 1)), hi = lo | j;
                const uint64_t x = keys[lo], y = keys[hi];
                if ((x > y) == ((lo & k) == 0)) {
                    keys[lo] = y;
                    keys[hi] = x;
                }
            }
            __syncthreads();
        }
    for (int64_t i = tid; i < len; i += 1024) {
        const uint64_t key = keys[i];
        const int64_t src = (int64_t)(uint32_t)key;
        ids[beg + i] = (int32_t)(uint32_t)(key >> 32);
        lam[beg + i] = pay[len * m + src];
        for (int p = 0; p < m; ++p) codes[(beg + i) * m + p] = pay[src * m + p];
    }
}
void launch_long_list_sort_at(int64_t beg, int64_t len, int m, int32_t *ids, uint8_t *codes, uint8_t *lam,
                              uint64_t *scratch_keys, uint8_t *scratch_payload, hipStream_t st)
{
    int64_t sz = 1;
    while (sz < len) sz <<= 1;
    hipLaunchKernelGGL(k_long_list_sort, dim3(1), dim3(1024), 0, st, beg, len, sz, m, ids, codes, lam, scratch_keys,
                       scratch_payload);
}

// Query-independent part of the ADC distance of every stored point (Eq. 15-17):
//   s_x = ||q2||^2 + 2 <q1 - mu, q2> + (l^2 - l) c,  q1 = c_i + l (s_ij - c_i),  q2 = codewords of x,
// i.e. term2 + 2 (1-l) term3 + 2 l term4 + (l^2 - l) term7 of Eq. 16-17 summed per point, with the
// inner products taken relative to a fixed vector mu (the scan's table is 2 <y - mu, q2>, so mu drops
// out of the distance; what it removes is the part of both inner products that grows with the
// distance of the data from the origin and would cancel between them in fp32).
// Summed in fp64 and rounded once.  LPL lanes a list: the edge length c is formed by them together, then they stride over
// the points, every lane walking the D coordinates of its point (the lanes of a list read the same centroid rows and mean:
// with a list a wave its number is uniform, and the rows come through scalar loads).  Sums in the same order for every LPL: the
// squared edge is added up as 64 lanes do it, a point's terms one after the other.  V: components a load takes; D/m is a multiple
// of it and rows lie on 4 V bytes.
struct StaticArgs {
    const int64_t *off;
    int64_t nl;
    int n, D, m;
    const float *C;
    const int32_t *S;
    const float *P, *mu;
    const uint8_t *codes, *lam;
    double lam_step;
    float lam_zero;
    float *sx;
};
template <int LPL, int V>
__device__ __forceinline__ void list_terms(const StaticArgs &a, int64_t l, int64_t beg, int64_t end, int lane)
{
    typedef float vec __attribute__((ext_vector_type(V)));
    const int D = a.D, m = a.m;
    const float *ci = a.C + (int64_t)(int)(l / a.n) * D;
    const float *sj = a.C + (int64_t)a.S[l] * D;
    double part[64 / LPL]; // of the lanes lane, lane + LPL, .. of 64
#pragma unroll
    for (int u = 0; u < 64 / LPL; ++u) {
        part[u] = 0.0;
        for (int d = lane + LPL * u; d < D; d += 64) {
            const double e = (double)sj[d] - (double)ci[d];
            part[u] = fma(e, e, part[u]);
        }
    }
#pragma unroll
    for (int o = 32 / LPL; o > 0; o >>= 1)
#pragma unroll
        for (int u = 0; u < o; ++u) part[u] += part[u + o];
    double c = part[0];
#pragma unroll
    for (int o = LPL / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    const int ds = D / m;
#pragma unroll 1
    for (int64_t t = beg + lane; t < end; t += LPL) {
        const double lh = ((double)a.lam[t] - (double)a.lam_zero) * a.lam_step;
        double q2n = 0.0, q12 = 0.0;
        for (int p = 0; p < m; ++p) {
            const float *w = a.P + ((int64_t)p * 256 + a.codes[t * m + p]) * ds;
#pragma unroll V
            for (int d = 0; d < ds; d += V) {
                const int g = p * ds + d;
                const vec cv4 = *(const vec *)(ci + g), s4 = *(const vec *)(sj + g), m4 = *(const vec *)(a.mu + g);
                const vec w4 = *(const vec *)(w + d);
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const double cv = (double)cv4[e], wv = (double)w4[e];
                    const double q1 = (cv - (double)m4[e]) + lh * ((double)s4[e] - cv);
                    q2n = fma(wv, wv, q2n);
                    q12 = fma(q1, wv, q12);
                }
            }
        }
        a.sx[t] = (float)(q2n + 2.0 * q12 + (lh * lh - lh) * c);
    }
}

// a wave a list: lists of many points
template <int V>
__global__ __launch_bounds__(256, 4) void k_list_static(StaticArgs a)
{
    const int64_t l = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    if (l >= a.nl) return;
    const int64_t beg = a.off[l], end = a.off[l + 1];
    if (beg < end) list_terms<64, V>(a, l, beg, end, threadIdx.x & 63);
}

// Short lists: 16 lanes each, four a wave (2 M points in 524 288 lists: a wave each left 60 of 64 lanes idle: 3.34 -> 0.90 ms).
// Lists of more than LS_FEW points are on a worklist (n_work[0] of them, handed out through n_work[2] after the first of each
// wave) and get a wave each, of the first `blocks` workgroups: their points would be walked by 16 lanes alone (2 M points in 8 cells
// of 16 384, finalisation 3.1 -> 4.0 ms; half of them in one list 255 -> 382), and behind the short ones, in a launch of their own, the
// longest list would be waited for with the chip idle.
template <int V>
__global__ __launch_bounds__(256, 5) void k_list_static_few(StaticArgs a, const int32_t *__restrict__ work,
                                                            int32_t *__restrict__ n_work, int blocks)
{
    if ((int)blockIdx.x < blocks) {
        const int todo = n_work[0], waves = blocks * 4, lane = threadIdx.x & 63;
        for (int i = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / 64); i < todo;) {
            const int64_t l = work[i];
            list_terms<64, V>(a, l, a.off[l], a.off[l + 1], lane);
            if (lane == 0) i = waves + atomicAdd(&n_work[2], 1);
            i = __builtin_amdgcn_readfirstlane(i);
        }
        return;
    }
    const int64_t l = (int64_t)((int)blockIdx.x - blocks) * 16 + threadIdx.x / 16;
    if (l >= a.nl) return; // (whole groups of 16 lanes)
    const int64_t beg = a.off[l], end = a.off[l + 1];
    if (beg < end && end - beg <= LS_FEW) list_terms<16, V>(a, l, beg, end, threadIdx.x & 15);
}

void launch_list_static(const int64_t *off, int64_t nl, int n, int D, int m, const float *C, const int32_t *S,
                        const float *P, const float *mu, const uint8_t *codes, const uint8_t *lam, double lam_step,
                        float lam_zero, int64_t N, const int32_t *work, int32_t *n_work, float *sx, hipStream_t st)
{
    if (nl <= 0) return;
    const StaticArgs a = {off, nl, n, D, m, C, S, P, mu, codes, lam, lam_step, lam_zero, sx};
    const uintptr_t rows = (uintptr_t)C | (uintptr_t)P | (uintptr_t)mu;
    const int v = (D / m) % 4 == 0 && rows % 16 == 0 ? 4 : ((D / m) % 2 == 0 && rows % 8 == 0 ? 2 : 1);
    auto go = [&](auto kern, auto few) {
        if (!lists_are_short(nl, N) || nl <= LS_WAVES) { // (up to LS_WAVES a wave each is all there is to run at once)
            hipLaunchKernelGGL(kern, dim3((unsigned)((nl + 3) / 4)), dim3(256), 0, st, a);
            return;
        }
        const int64_t most = N / (LS_FEW + 1); // lists on the worklist; eight workgroups per compute unit at most
        const int blocks = (int)(most < 4 * 2048 ? (most + 3) / 4 : 2048);
        hipLaunchKernelGGL(few, dim3((unsigned)(blocks + (nl + 15) / 16)), dim3(256), 0, st, a, work, n_work, blocks);
    };
    switch (v) {
    case 4: go(k_list_static<4>, k_list_static_few<4>); break;
    case 2: go(k_list_static<2>, k_list_static_few<2>); break;
    default: go(k_list_static<1>, k_list_static_few<1>); break;
    }
}
