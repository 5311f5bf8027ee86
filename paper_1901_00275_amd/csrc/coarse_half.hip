// Nearest-centroid shortlist (Eq. 2; Alg. 1) on the fp16 matrix cores: ONE product per pair.
//
// Rows and centroids (minus the index's origin) are rounded once to fp16 with a power-of-two scale per block
// of 128 rows that brings the block's largest magnitude to [2^14, 2^15): 11 significant bits, and 28 binades
// below the largest value before a component is flushed to zero.  How far a row's image is from the row is
// measured when the image is written (residual norm), so the error of a product is bounded by Cauchy-Schwarz
// from what was actually lost: |<a, b> - <a', b'>| <= |a - a'||b| + |a'||b - b'|; integer-valued descriptors lose
// nothing.  A block whose rows differ by more than HALF_GAP binades (a corrupt vector among ordinary ones) gets a scale
// per row, so that no row loses its components to another's size.  Every column inside the band of the row minimum is handed on and re-evaluated as a direct fp32 sum
// of squared differences, so the decision is taken in fp32 exactly, whatever the product's precision.
// (The form before split both operands into two bf16 parts and multiplied two or three pairs of pages: 213 571 x 128
// integer vectors against 65 536 centroids 7.67 ms, 4.19 ms so, 0.86 PFLOP/s; 2^18 x 96 against 16 384: 2.26 and 1.02 ms.)
//
// Image: blocks of 128 rows x steps of 16 indices; a 4 KB page per (block, step) holds 128 rows x 2 chunks of
// 8 values, chunk c of row r at position 2 r + (c ^ ((r >> 2) & 1)): fragment reads are free of bank conflicts.
//
// Product kernel: 256 threads = 4 waves, 128 rows against all column tiles of the split, a 64 x 64 quadrant per wave.
// The A fragments stay in registers for the whole sweep (read straight from the image: A takes no LDS), a whole tile
// of B (D / 16 pages) is copied memory -> LDS without passing registers while the tile before it is multiplied:
// one barrier per tile, and two workgroups per compute unit, so that one's selection overlaps the other's products.
// Per tile a wave has 4 D / 16 MFMAs of 32 clocks (D = 128: 1 024) and 192 vector instructions of 4 clocks: the two
// columns (j = 0, 1) that a lane sees of a row enter the running two smallest as one key, their smaller value.
//
// Crowded rows (more columns inside the band than the shortlist holds, or several of them in one lane's slot) would
// leave the consumer whole slots or splits to compare: 65 536 rows of 512 bytes for one vector.  Where a strip has
// enough of that, the workgroup multiplies its tiles a second time with the band known, takes the exact distance of
// every column inside it and hands on the nearest.  Where even those are too many (a tenth of a tile's pairs: all
// columns alike as far as fp16 sees them), the shortlists stay as they are.
// (2^18 x 128, 16 384 centroids in groups of 16 / 64 with a spread of 0.04 |x|: 63 / 135 ms without, 3.6 / 3.7 ms with
// the second sweep, 6.3 / 8.7 ms with two bf16 parts and no second sweep; 2.2 ms where nothing is crowded.)
#include "common.h"

#include <type_traits>

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

#define HT 128        // rows per block (= VLQ_NN_TILE columns per tile)
#define HPAGE 256     // 16-byte chunks per page
#define HALF_NORMAL 6.103515625e-5f // 2^-14: smaller halves are written as zero
#define NO_COLUMN 3e38f // "norm" of columns past the end: finite, so that index bits can be planted in the key
#define NO_KEY 1e38f    // from here on a key counts as absent
#define PAIR_CAP 2048 // (row, column) pairs of the second sweep that wait for their exact distance
#define PAIR_COL_BITS 25
#define PAIR_BATCH 4  // pairs a group of 16 lanes has under way
// From this many slots in a strip's shortlists on the strip takes the second sweep: a tile of it costs what the exact
// distances of some 40 slots (two columns of every tile each) cost the consumer, one wave after another, and 8 to 64
// measured alike.  A row with all columns in its shortlist is reason enough by itself.
#define SLOTS_MAX 16

size_t half_image_bytes(int64_t rows, int D)
{
    const int64_t blocks = (rows + HT - 1) / HT;
    return 256 + ((size_t)blocks * 4 + 255) / 256 * 256 + (size_t)blocks * HT * 4 + (size_t)blocks * HT * D * 2;
}

// header (256 bytes: [0] largest relative residual of a row, [1] largest residual of the rows whose relative one is
// beyond fp16's rounding), scales, rows' inverse scales, pages
struct HalfImage {
    float *hdr;
    float *scale; // [blocks] a block's values are multiplied by this; 0: every row has its own
    float *rinv;  // [blocks][HT] 1 / scale of the row, of the blocks whose scale is 0
    u32x4 *pages;
    HalfImage(const void *img, int64_t rows)
    {
        char *p = (char *)(uintptr_t)img;
        const int64_t blocks = (rows + HT - 1) / HT;
        hdr = (float *)p;
        scale = (float *)(p + 256);
        rinv = (float *)(p + 256 + ((size_t)blocks * 4 + 255) / 256 * 256);
        pages = (u32x4 *)(rinv + blocks * HT);
    }
};

__global__ void k_half_header(float *hdr)
{
    if (threadIdx.x < 2) hdr[threadIdx.x] = 0.f;
}

__device__ __forceinline__ float pow2f(int ex) { return __uint_as_float((uint32_t)(127 + ex) << 23); }

// One workgroup per block of 128 rows, a thread per (row, chunk of 8 values), SPT times: one pass over X gives the
// block's scale, the pages, and per row the squared norm and the residual's norm.  Bound by memory.
template <int SPT>
__global__ __launch_bounds__(256) void k_half_image(const float *__restrict__ X, int64_t rows,
                                                    const float *__restrict__ mu, float *__restrict__ hdr,
                                                    float *__restrict__ scale, float *__restrict__ rinv,
                                                    u32x4 *__restrict__ pages,
                                                    float *__restrict__ norm2, float *__restrict__ resid)
{
    constexpr int D = SPT * 16, CPR = SPT * 2;
    __shared__ float pn[HT][CPR + 1], pr[HT][CPR + 1];
    __shared__ float wmax[4];
    __shared__ int rex[HT]; // exponents of the rows' scales, where every row has its own
    __shared__ int apart;
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t blk = blockIdx.x;
    float v[SPT][8];
    float mx = 0.f;
#pragma unroll
    for (int j = 0; j < SPT; ++j) {
        const int i = j * 256 + tid, r = i / CPR, ch = i - r * CPR;
        const int64_t row = blk * HT + r;
        f32x4 v0 = {0.f, 0.f, 0.f, 0.f}, v1 = v0;
        if (row < rows) {
            v0 = *(const f32x4 *)(X + row * D + ch * 8) - *(const f32x4 *)(mu + ch * 8);
            v1 = *(const f32x4 *)(X + row * D + ch * 8 + 4) - *(const f32x4 *)(mu + ch * 8 + 4);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[j][e] = e < 4 ? v0[e] : v1[e - 4];
            const float m = fabsf(v[j][e]);
            if (m < INFINITY) mx = fmaxf(mx, m);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if (lane == 0) wmax[tid >> 6] = mx;
    if (tid == 0) apart = 0;
    __syncthreads();
    mx = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
    const int ex = half_exponent(mx);
    const float sb = pow2f(ex);
    if (tid == 0) scale[blk] = sb;
    // pages, norms and residuals at one scale for the block or (own) with a scale per row
    auto write = [&](bool own) {
#pragma unroll
        for (int j = 0; j < SPT; ++j) {
            const int i = j * 256 + tid, r = i / CPR, ch = i - r * CPR;
            const float s = own ? pow2f(rex[r]) : sb;
            half8 h;
            float n2 = 0.f, r2 = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float t = v[j][e] * s;
                _Float16 q = (_Float16)t;
                if (fabsf((float)q) < HALF_NORMAL) q = (_Float16)0.f;
                const float d = t - (float)q;
                n2 = fmaf(t, t, n2);
                r2 = fmaf(d, d, r2);
                h[e] = q;
            }
            pn[r][ch] = n2;
            pr[r][ch] = r2;
            pages[(blk * SPT + (ch >> 1)) * HPAGE + 2 * r + ((ch & 1) ^ ((r >> 2) & 1))] = __builtin_bit_cast(u32x4, h);
        }
        __syncthreads();
        if (tid >= HT) return;
        float n2 = 0.f, r2 = 0.f;
#pragma unroll
        for (int c = 0; c < CPR; ++c) {
            n2 += pn[tid][c];
            r2 += pr[tid][c];
        }
        const float inv = pow2f(own ? -rex[tid] : -ex);
        const float nrm = sqrtf(n2), res = sqrtf(r2) * 1.0001f; // (the rounding of the sums)
        const int64_t row = blk * HT + tid;
        if (row < rows && norm2) norm2[row] = n2 * inv * inv;
        if (row < rows && resid) resid[row] = res * inv;
        if (!own && !hdr && row < rows && nrm < pow2f(14 - HALF_GAP)) apart = 1;
        if (hdr) {
            const bool ok = res < INFINITY && n2 > 0.f; // (a non-finite row's products never count)
            float rel = ok && res <= HALF_REL_MAX * nrm ? res / nrm * 1.0001f : 0.f;
            float big = ok && !(res <= HALF_REL_MAX * nrm) ? res * inv : 0.f;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                rel = fmaxf(rel, __shfl_xor(rel, o, 64));
                big = fmaxf(big, __shfl_xor(big, o, 64));
            }
            if (lane == 0) {
                if (rel > ((volatile float *)hdr)[0]) atomicMax((unsigned *)hdr, __float_as_uint(rel));
                if (big > ((volatile float *)hdr)[1]) atomicMax((unsigned *)hdr + 1, __float_as_uint(big));
            }
        }
    };
    write(false);
    if (hdr) return; // (the columns keep one scale per block: what a column loses is bounded by the header)
    __syncthreads();
    if (!apart) return;
    // a row far below the block's largest: its own size decides (a row of zeros is no reason)
#pragma unroll
    for (int j = 0; j < SPT; ++j) {
        const int i = j * 256 + tid, r = i / CPR, ch = i - r * CPR;
        float cm = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float m = fabsf(v[j][e]);
            if (m < INFINITY) cm = fmaxf(cm, m);
        }
        pn[r][ch] = cm;
    }
    __syncthreads();
    bool own = false;
    if (tid < HT) {
        float rm = 0.f;
        for (int c = 0; c < CPR; ++c) rm = fmaxf(rm, pn[tid][c]);
        rex[tid] = half_exponent(rm);
        rinv[blk * HT + tid] = pow2f(-rex[tid]);
        own = rm > 0.f && rex[tid] > ex + HALF_GAP;
    }
    if (!__syncthreads_or(own)) return;
    if (tid == 0) scale[blk] = 0.f;
    write(true);
}

void launch_half_image(const float *X, int64_t rows, int D, const float *mu, void *img, bool header, float *norm2,
                       float *resid, hipStream_t st)
{
    if (rows <= 0) return;
    const HalfImage h(img, rows);
    const dim3 grid((unsigned)((rows + HT - 1) / HT));
    if (header) hipLaunchKernelGGL(k_half_header, dim3(1), dim3(64), 0, st, h.hdr);
#define HALF_LAUNCH(S)                                                                                         \
    hipLaunchKernelGGL(k_half_image<S>, grid, dim3(256), 0, st, X, rows, mu, header ? h.hdr : nullptr, h.scale, h.rinv, \
                       h.pages, norm2, resid)
    switch (D / 16) {
    case 2: HALF_LAUNCH(2); break;
    case 4: HALF_LAUNCH(4); break;
    case 6: HALF_LAUNCH(6); break;
    default: HALF_LAUNCH(8); break;
    }
#undef HALF_LAUNCH
}

struct HalfArgs {
    const u32x4 *A, *B;
    const float *ascale, *arinv, *bscale, *bhdr;
    int M, N;
    const float *X, *C; // the rows and columns themselves
    bool vec;           // rows of C on 16 bytes
    const float *an, *ares, *bn;
    int nsplit, tiles_per_split;
    uint64_t *cand;
    int idx_bits; // low mantissa bits of a running key that hold the tile
    float band_dist;
};

template <int SPT>
__global__ __launch_bounds__(256, 2) void k_nearest_half(HalfArgs a)
{
    extern __shared__ u32x4 lds[]; // two tiles of B: [2][SPT][HPAGE]; the tail of the kernel reuses the front
    float *rinv = (float *)(lds + 2 * SPT * HPAGE);               // [HT] inverse scales of the rows
    unsigned long long *best = (unsigned long long *)(rinv + HT); // [HT] second sweep: nearest column so far
    uint32_t *pairs = (uint32_t *)(best + HT);                    // [PAIR_CAP] row << PAIR_COL_BITS | column of the split
    __shared__ uint8_t crowded[HT];
    __shared__ int sh_pairs, sh_slots;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
    const int64_t m0 = (int64_t)blockIdx.x * HT;
    const int split = blockIdx.y;
    const int ntiles = (a.N + HT - 1) / HT;
    const int t0 = split * a.tiles_per_split;
    const int t1 = min(ntiles, t0 + a.tiles_per_split);

    // a tile of B into LDS: thread t's chunk of every page goes to place t of that page (a wave's 64 chunks are
    // contiguous on both sides, as the direct copy requires)
    auto copy_tile = [&](int t) {
        const u32x4 *src = a.B + (int64_t)t * SPT * HPAGE + tid;
        u32x4 *dst = lds + ((t - t0) & 1) * SPT * HPAGE + wave * 64;
#pragma unroll
        for (int p = 0; p < SPT; ++p)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + p * HPAGE),
                                             (__attribute__((address_space(3))) void *)(dst + p * HPAGE), 16, 0, 0);
    };
    // fragment of a 32-row block: lane reads row (lane & 31), chunk (lane >> 5)
    const int frow = lane & 31;
    const int fpos = 2 * frow + ((lane >> 5) ^ ((frow >> 2) & 1));
    half8 ah[SPT][2];
    {
        const u32x4 *src = a.A + (int64_t)blockIdx.x * SPT * HPAGE + 2 * wm + fpos;
#pragma unroll
        for (int u = 0; u < SPT; ++u) {
            ah[u][0] = __builtin_bit_cast(half8, src[u * HPAGE]);
            ah[u][1] = __builtin_bit_cast(half8, src[u * HPAGE + 64]);
        }
    }
    // accumulator register r of block i holds row wm + 32 i + 8 (r / 4) + 4 (lane / 32) + r % 4
    auto slot_row = [&](int i, int r) { return wm + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); };
    float b1[2][16], b2[2][16]; // per row slot: smallest and second smallest key
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) b1[i][r] = b2[i][r] = INFINITY;
    const uint32_t keep = ~((1u << a.idx_bits) - 1u);
    const uint32_t aexp = __float_as_uint(a.ascale[blockIdx.x]);
    // column norms and scale of a tile, asked for a tile ahead and before its copies, so that the one wait covers both
    float cbn[2], scn;
    auto fetch_cols = [&](int t) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int64_t col = (int64_t)t * HT + wn + 32 * j + (lane & 31);
            cbn[j] = a.bn[min(col, (int64_t)a.N - 1)];
        }
        scn = a.bscale[t];
    };
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    if (t0 < t1) {
        fetch_cols(t0);
        copy_tile(t0);
    }
    if (aexp == 0u && tid < HT) rinv[tid] = a.arinv[m0 + tid]; // (read behind the first tile's barrier)
    // exact distances of the n pairs that wait, 16 lanes a pair
    auto settle = [&](int n) {
        const int grp = tid >> 4, l16 = tid & 15;
        for (int p0 = 0; p0 < n; p0 += 16 * PAIR_BATCH) { // (the loads of a batch are under way together)
            float d[PAIR_BATCH];
            uint32_t e[PAIR_BATCH];
#pragma unroll
            for (int u = 0; u < PAIR_BATCH; ++u) {
                e[u] = pairs[min(p0 + 16 * u + grp, n - 1)];
                const int64_t row = m0 + (e[u] >> PAIR_COL_BITS), col = (int64_t)t0 * HT + (e[u] & ((1u << PAIR_COL_BITS) - 1u));
                d[u] = sqdist16(a.X + row * (SPT * 16), a.C + col * (SPT * 16), SPT * 16, l16, a.vec);
            }
#pragma unroll
            for (int u = 0; u < PAIR_BATCH; ++u)
                if (p0 + 16 * u + grp < n && l16 == 0)
                    atomicMin(&best[e[u] >> PAIR_COL_BITS],
                              make_key(d[u], (uint32_t)t0 * HT + (e[u] & ((1u << PAIR_COL_BITS) - 1u))));
        }
    };
    // OWN: the rows' scales are read from rinv, not one for the block.  EMIT (second sweep): b1 holds the rows' bands,
    // and what lies inside is collected.  Returns false (to all threads) where a tile finds no room for its pairs.
    auto sweep = [&](auto OWN, auto EMIT) -> bool {
        constexpr bool own = decltype(OWN)::value, emit = decltype(EMIT)::value;
        for (int t = t0; t < t1; ++t) {
            // this tile has arrived (every wave waits for its own copies), and the other half of the ring is free
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (emit) {
                const int n = sh_pairs;
                __syncthreads(); // (read by all before the next tile adds to it)
                if (n > PAIR_CAP) return false;
                if (n > PAIR_CAP / 2) {
                    settle(n);
                    __syncthreads();
                    if (tid == 0) sh_pairs = 0;
                    __syncthreads();
                }
            }
            float cb[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) cb[j] = (int64_t)t * HT + wn + 32 * j + (lane & 31) < a.N ? cbn[j] : NO_COLUMN;
            // -2 / (scale of the rows * scale of the columns): powers of two, 1 / 2^x by its exponent
            const float binv = -2.f * __uint_as_float(0x7F000000u - __float_as_uint(scn));
            const float inv = own ? binv : binv * __uint_as_float(0x7F000000u - aexp);
            if (t + 1 < t1) {
                fetch_cols(t + 1);
                copy_tile(t + 1);
            }
            const u32x4 *bp = lds + ((t - t0) & 1) * SPT * HPAGE + 2 * wn + fpos;
            f32x16 acc[2][2];
#pragma unroll
            for (int u = 0; u < SPT; ++u) {
                half8 bh[2];
                bh[0] = __builtin_bit_cast(half8, bp[u * HPAGE]);
                bh[1] = __builtin_bit_cast(half8, bp[u * HPAGE + 64]);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[u][i], bh[j], u == 0 ? zero16 : acc[i][j], 0, 0, 0);
            }
            const uint32_t tj = (uint32_t)(t - t0);
            if constexpr (emit) {
                uint32_t miss[2] = {0u, 0u};
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float f = inv * rinv[slot_row(i, r)];
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            miss[j] = __builtin_amdgcn_alignbit(
                                miss[j], __float_as_uint(b1[i][r] - fmaf(f, acc[i][j][r], cb[j])), 31);
                    }
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const uint32_t col = tj * HT + wn + 32 * j + (lane & 31);
                    uint32_t hit = (int64_t)t0 * HT + col < a.N ? ~miss[j] : 0u;
                    while (hit) {
                        const int b = __clz(hit); // bit 31 is the first row slot
                        hit &= ~(0x80000000u >> b);
                        const int rl = slot_row(b >> 4, b & 15);
                        if (!crowded[rl]) continue; // (the products of a row with a NaN have any sign)
                        const int at = atomicAdd(&sh_pairs, 1);
                        if (at < PAIR_CAP) pairs[at] = ((uint32_t)rl << PAIR_COL_BITS) | col;
                    }
                }
                continue;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float f = own ? inv * rinv[slot_row(i, r)] : inv;
                    const float e = fminf(fmaf(f, acc[i][0][r], cb[0]), fmaf(f, acc[i][1][r], cb[1]));
                    const float key = __uint_as_float((__float_as_uint(e) & keep) | tj);
                    b2[i][r] = __builtin_amdgcn_fmed3f(b1[i][r], b2[i][r], key);
                    b1[i][r] = fminf(b1[i][r], key);
                }
        }
        return true;
    };
    if (aexp != 0u)
        sweep(std::false_type{}, std::false_type{});
    else
        sweep(std::true_type{}, std::false_type{});

    // ---- row minimum over the workgroup, then every kept key inside the band of it ----
    __syncthreads(); // the tiles are dead from here on
    unsigned *rowmin = (unsigned *)lds;                                // [HT]
    int *rowcnt = (int *)(rowmin + HT);                                // [HT]
    unsigned long long *rowcand = (unsigned long long *)(rowcnt + HT); // [HT][VLQ_NN_CANDS]
    if (tid == 0) sh_slots = 0;
    if (tid < HT) {
        rowmin[tid] = 0xFFFFFFFFu;
        rowcnt[tid] = 0;
#pragma unroll
        for (int s = 0; s < VLQ_NN_CANDS; ++s) rowcand[tid * VLQ_NN_CANDS + s] = KEY_MAX;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (b1[i][r] < NO_KEY) atomicMin(&rowmin[slot_row(i, r)], f2ord(b1[i][r]));
    __syncthreads();
    const float rho = a.bhdr[0], big = a.bhdr[1];
    // where the band of row rl (one with a minimum) ends
    auto band_end = [&](int rl) {
        const float ra = a.an[m0 + rl];
        const float emin = __uint_as_float(__float_as_uint(ord2f(rowmin[rl])) & keep);
        const float dmin = fmaxf(emin + ra, 0.f);
        return emin + nn_half_band(ra, a.ares[m0 + rl], rho, big, dmin, a.band_dist, SPT * 16);
    };
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int rl = slot_row(i, r);
            if (rowmin[rl] == 0xFFFFFFFFu || m0 + rl >= a.M) continue;
            const float ra = a.an[m0 + rl], band = band_end(rl);
            const float e = __uint_as_float(__float_as_uint(b1[i][r]) & keep);
            if (!(b1[i][r] < NO_KEY) || !(e <= band)) continue;
            // the key stands for both columns of its tile; a second one inside the band may have pushed out a
            // third, so the slot's columns are handed on instead
            const bool more = b2[i][r] < NO_KEY && __uint_as_float(__float_as_uint(b2[i][r]) & keep) <= band;
            const uint32_t col = (uint32_t)(t0 + (int)(__float_as_uint(b1[i][r]) & ~keep)) * HT + wn + (lane & 31);
            const uint32_t entry = more ? VLQ_NN_SLOT | (uint32_t)((wn >> 6) * 32 + (lane & 31)) : col;
            const int pos = atomicAdd(&rowcnt[rl], 1);
            if (pos < VLQ_NN_CANDS)
                rowcand[rl * VLQ_NN_CANDS + pos] = ((uint64_t)__float_as_uint(fmaxf(e + ra, 0.f) + 0.f) << 32) | entry;
        }
    __syncthreads();
    uint64_t *dst = nullptr;
    uint64_t near = 0; // high word of the split's smallest key
    int slots = 0;
    if (tid < HT && m0 + tid < a.M) {
        dst = a.cand + ((m0 + tid) * a.nsplit + split) * VLQ_NN_CANDS;
        const bool all = rowcnt[tid] > VLQ_NN_CANDS; // more than there is room for: the split's columns
        const float emin = __uint_as_float(__float_as_uint(ord2f(rowmin[tid])) & keep);
        near = (uint64_t)__float_as_uint(fmaxf(emin + a.an[m0 + tid], 0.f) + 0.f) << 32;
        slots = all ? SLOTS_MAX : 0;
#pragma unroll
        for (int s = 0; s < VLQ_NN_CANDS; ++s) {
            const uint64_t key = rowcand[tid * VLQ_NN_CANDS + s];
            if (!all && key != KEY_MAX && ((uint32_t)key & VLQ_NN_SLOT)) ++slots;
            dst[s] = all ? (s == 0 ? near | VLQ_NN_ALL : KEY_MAX) : key;
        }
        if (slots) atomicAdd(&sh_slots, slots);
    }
    __syncthreads();
    if (sh_slots < SLOTS_MAX || a.tiles_per_split > (1 << (PAIR_COL_BITS - 7))) return;

    // ---- second sweep, for the strip's rows with slots or all columns in their shortlists ----
    if (tid < HT) {
        rowcnt[tid] = slots; // (read by all threads below, before the tiles overwrite it)
        best[tid] = KEY_MAX;
        rinv[tid] = aexp != 0u ? __uint_as_float(0x7F000000u - aexp) : a.arinv[m0 + tid];
    }
    if (tid == 0) sh_pairs = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int rl = slot_row(i, r);
            b1[i][r] = rowcnt[rl] ? band_end(rl) : -INFINITY;
        }
    __syncthreads();
    if (tid < HT) crowded[tid] = slots != 0;
    fetch_cols(t0);
    copy_tile(t0);
    if (!sweep(std::true_type{}, std::true_type{})) return;
    __syncthreads();
    if (sh_pairs > PAIR_CAP) return;
    settle(sh_pairs);
    __syncthreads();
    if (slots && best[tid] != KEY_MAX) { // the nearest, at the distance the split's smallest key has
        dst[0] = near | (uint32_t)best[tid];
#pragma unroll
        for (int s = 1; s < VLQ_NN_CANDS; ++s) dst[s] = KEY_MAX;
    }
}

int launch_nearest_half(const void *Aimg, int M, const void *Bimg, int N, int D, const float *X, const float *C,
                        const float *an, const float *ares, const float *bn, uint64_t *cand, int nsplit, float *band_dist,
                        const float **bhdr, hipStream_t st)
{
    const HalfImage A(Aimg, M), B(Bimg, N);
    HalfArgs a = {};
    a.A = A.pages;
    a.ascale = A.scale;
    a.arinv = A.rinv;
    a.B = B.pages;
    a.bscale = B.scale;
    a.bhdr = B.hdr;
    a.M = M;
    a.N = N;
    a.X = X;
    a.C = C;
    a.vec = ((uintptr_t)C) % 16 == 0;
    a.an = an;
    a.ares = ares;
    a.bn = bn;
    a.cand = cand;
    a.nsplit = nsplit;
    const int ntiles = (N + HT - 1) / HT;
    a.tiles_per_split = (ntiles + nsplit - 1) / nsplit;
    a.idx_bits = half_idx_bits(a.tiles_per_split);
    a.band_dist = half_band_dist(a.idx_bits);
    *band_dist = a.band_dist;
    *bhdr = B.hdr;
    if (M <= 0 || N <= 0) return 0;
    // the ring of tiles (the tail of the kernel takes HT * (8 + 8 * VLQ_NN_CANDS) bytes of it), the rows' scales, and
    // the nearest columns and the pairs of the second sweep: 73.5 KB at most, so that two workgroups share the LDS
    const size_t bytes = (size_t)2 * (D / 16) * HPAGE * 16 + HT * (4 + 8) + PAIR_CAP * 4;
    const dim3 grid((unsigned)((M + HT - 1) / HT), (unsigned)nsplit);
    auto go = [&](auto kern) -> int {
        if (bytes > 49152) { // (48 KB of dynamic LDS need no asking)
            hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
            if (e != hipSuccess) return (int)e;
        }
        hipLaunchKernelGGL(kern, grid, dim3(256), bytes, st, a);
        return 0;
    };
    switch (D / 16) {
    case 2: return go(k_nearest_half<2>);
    case 4: return go(k_nearest_half<4>);
    case 6: return go(k_nearest_half<6>);
    case 8: return go(k_nearest_half<8>);
    }
    return (int)hipErrorInvalidValue;
}
