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
//
// Image: blocks of 128 rows x steps of 32 indices; an 8 KB page per (block, step) holds 8 groups of 16 rows, of each
// the 64 chunks of 8 values in the order of the lanes that read them: chunk c of row r at position 16 c + r % 16.
//
// Product kernel: 512 threads = 8 waves, one workgroup per compute unit.  A strip of 256 rows against all column tiles of
// the split; waves 0-3 (group 0) take the first 128 rows, waves 4-7 (group 1) the others, a 64 x 64 quadrant per wave, so
// that every SIMD holds a wave of each group and a tile of B serves both.  The A fragments stay in registers for the whole
// sweep; tiles of B (D / 32 pages) go memory -> LDS without passing registers, into a ring of HRING tiles, HSTEP of them
// between two barriers.
//
// What bounds it is the issue of instructions: per tile a wave has 2 D 16x16x32 MFMAs / 4 of 16 clocks (D = 128: 1 024),
// beside which a SIMD issues two vector instructions to an MFMA at most (measured: 2.3), and the clock, which falls to
// 1.9 GHz under the load (random operands from registers alone: 1.88 PFLOP/s; 1.69 with the 32x32x16 form, which this
// kernel had before).  Hence:
//  - group 1 runs half a step behind, one group's selection beside the other's products, and the products have priority;
//  - 115 vector instructions a tile instead of 288: the four columns (j = 0 .. 3) that a lane sees of a row enter the
//    running three smallest as one key, their smallest value; the products are added to the column's norm (in their own
//    units) instead of the norm to them; and nothing is quieted (see `select`);
//  - a tile's copies are asked for between the products, one or two at a time: asked for together behind the barrier they
//    kept the waves waiting for the queue for 1 070 clocks a tile, as long as the tile's MFMAs.
// k = 65 536, D = 128: 213 571 rows 4.08 -> 2.96 ms (836 strips, a fifth of the last round idle), 2^18 rows 3.11 ms =
// 1.41 PFLOP/s; before, with 128-row workgroups, two columns and the two smallest keys a lane: 0.88 PFLOP/s.
// k = 16 384, D = 96, 2^18 rows: 1.02 -> 0.70 ms.
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
#define HPAGE 512     // 16-byte chunks per page
#define HNT 512       // threads of the product kernel
#define HR 256        // rows of its strip: two blocks
#define HCOLS (HT + 64) // floats of a tile's norms and scale
#define HRING 4       // tiles of columns in LDS
#define HSTEP 2       // of which so many are multiplied between two barriers, while the others arrive
static_assert(HRING == 2 * HSTEP, "the tiles to come take the place of those before");
#define HALF_NORMAL 6.103515625e-5f // 2^-14: smaller halves are written as zero
#define NO_COLUMN 3e38f // "norm" of columns past the end: finite, so that index bits can be planted in the key
#define NO_KEY 1e38f    // from here on a key counts as absent
#define PAIR_CAP 2048 // (row, column) pairs of the second sweep that wait for their exact distance
#define PAIR_COL_BITS 24
#define PAIR_BATCH 4  // pairs a group of 16 lanes has under way
// From this many slots in a strip's shortlists on the strip takes the second sweep: a tile of it costs what the exact
// distances of some 40 slots (four columns of every tile each, for 256 rows) cost the consumer, one wave after another,
// and 8 to 64 measured alike.  A row with all columns in its shortlist is reason enough by itself.
#define SLOTS_MAX 16

size_t half_image_bytes(int64_t rows, int D)
{
    const int64_t blocks = (rows + HT - 1) / HT;
    return 256 + ((size_t)blocks * 4 + 255) / 256 * 256 + (size_t)blocks * HT * 4 + (size_t)blocks * HT * D * 2;
}

// header (256 bytes: [0] largest relative residual of a row, [1] largest residual of the rows whose relative one is
// beyond fp16's rounding, [2] smallest scale), scales, rows' inverse scales, pages
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
    if (threadIdx.x < 3) hdr[threadIdx.x] = threadIdx.x < 2 ? 0.f : INFINITY;
}

__device__ __forceinline__ float pow2f(int ex) { return __uint_as_float((uint32_t)(127 + ex) << 23); }

// One workgroup per block of 128 rows, a thread per (row, chunk of 8 values), SPT times: one pass over X gives the
// block's scale, the pages, and per row the squared norm and the residual's norm.  Bound by memory.
template <int KS>
__global__ __launch_bounds__(256) void k_half_image(const float *__restrict__ X, int64_t rows,
                                                    const float *__restrict__ mu, float *__restrict__ hdr,
                                                    float *__restrict__ scale, float *__restrict__ rinv,
                                                    u32x4 *__restrict__ pages,
                                                    float *__restrict__ norm2, float *__restrict__ resid)
{
    constexpr int D = KS * 32, CPR = D / 8, SPT = KS * 2;
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
    if (tid == 0) {
        scale[blk] = sb;
        if (hdr && sb < ((volatile float *)hdr)[2]) atomicMin((unsigned *)hdr + 2, __float_as_uint(sb));
    }
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
                if (fabsf((float)q) < HALF_NORMAL || (hdr && !(fabsf((float)q) < INFINITY))) q = (_Float16)0.f;
                const float d = t - (float)q;
                n2 = fmaf(t, t, n2);
                r2 = fmaf(d, d, r2);
                h[e] = q;
            }
            pn[r][ch] = n2;
            pr[r][ch] = r2;
            pages[(blk * KS + (ch >> 2)) * HPAGE + (r >> 4) * 64 + (ch & 3) * 16 + (r & 15)] = __builtin_bit_cast(u32x4, h);
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
            // (the products of a row whose norm overflows or is no number never count, whatever the image lost of it)
            const bool ok = res < INFINITY && n2 > 0.f && n2 * inv * inv < INFINITY;
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
    switch (D / 32) {
    case 1: HALF_LAUNCH(1); break;
    case 2: HALF_LAUNCH(2); break;
    case 3: HALF_LAUNCH(3); break;
    default: HALF_LAUNCH(4); break;
    }
#undef HALF_LAUNCH
}

// front of the product kernel's LDS: the ring of tiles, later the rows' minima, counts and shortlists
__host__ __device__ constexpr size_t half_front_bytes(int KS)
{
    const size_t ring = (size_t)HRING * KS * HPAGE * 16, tail = HR * (8 + 8 * VLQ_NN_CANDS);
    return ring > tail ? ring : tail;
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

template <int KS>
__global__ __launch_bounds__(HNT, 2) void k_nearest_half(HalfArgs a)
{
    extern __shared__ u32x4 lds[]; // a ring of tiles of B: [HRING][KS][HPAGE]; the tail of the kernel reuses the front
    float *cnorm = (float *)((char *)lds + half_front_bytes(KS)); // [2 HRING][HCOLS] norms of the tiles' columns, then their scale
    float *rinv = cnorm + 2 * HRING * HCOLS;                       // [HR] inverse scales of the rows
    unsigned long long *best = (unsigned long long *)(rinv + HR); // [HR] second sweep: nearest column so far
    uint32_t *pairs = (uint32_t *)(best + HR);                    // [PAIR_CAP] row << PAIR_COL_BITS | column of the split
    __shared__ uint8_t crowded[HR];
    __shared__ int sh_pairs, sh_slots;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = wave >> 2; // waves 0-3 take the strip's first 128 rows, 4-7 the others
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
    const int64_t m0 = (int64_t)blockIdx.x * HR;
    const int64_t blk = (int64_t)blockIdx.x * 2 + group;
    const bool has_rows = blk * HT < a.M; // (the last strip may have one block of rows)
    const int split = blockIdx.y;
    const int ntiles = (a.N + HT - 1) / HT;
    const int t0 = split * a.tiles_per_split;
    const int t1 = min(ntiles, t0 + a.tiles_per_split);

    // page u of tile t (columns past the split: of its last tile) into LDS: a wave's 64 chunks are contiguous on both
    // sides, as the direct copy requires
    auto copy_page = [&](int t, int u) {
        const u32x4 *src = a.B + ((int64_t)min(t, t1 - 1) * KS + u) * HPAGE;
        u32x4 *dst = lds + (((t - t0) & (HRING - 1)) * KS + u) * HPAGE + wave * 64;
        const __amdgpu_buffer_rsrc_t page = __builtin_amdgcn_make_buffer_rsrc((void *)src, 0, HPAGE * 16, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(page, (__attribute__((address_space(3))) void *)dst, 16, tid * 16, 0, 0, 0);
    };
    // the norms of its columns, the four of a lane (wn + 16 j + lane % 16) side by side (past the last: zero, not looked
    // at), and its scale
    const int norm_off = wave < 2 ? (wave * 64 + 16 * (lane & 3) + (lane >> 2)) * 4 : 0;
    auto copy_norms = [&](int t) {
        if (wave >= 3) return;
        t = min(t, t1 - 1);
        float *cn = cnorm + ((t - t0) & (2 * HRING - 1)) * HCOLS + wave * 64;
        const float *src = wave < 2 ? a.bn + (int64_t)t * HT : a.bscale + t;
        const int bytes = wave < 2 ? min(a.N - t * HT, HT) * 4 : 4;
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)src, 0, bytes, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)cn, 4, norm_off, 0, 0, 0);
    };
    // fragment of 16 rows: lane reads row (lane & 15), chunk (lane >> 4)
    half8 ah[KS][4];
    {
        const u32x4 *src = a.A + (has_rows ? blk : 0) * KS * HPAGE + 4 * (wm & 64) + lane;
#pragma unroll
        for (int u = 0; u < KS; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                u32x4 w = src[u * HPAGE + 64 * i] ^ 0x80008000u;
                asm("" : "+v"(w)); // (negated once, here)
                ah[u][i] = __builtin_bit_cast(half8, w);
            }
    }
    // accumulator register r of block (i, j) holds row wm + 16 i + 4 (lane / 16) + r, column wn + 16 j + lane % 16
    auto slot_row = [&](int i, int r) { return wm + 16 * i + 4 * (lane >> 4) + r; };
    const int slot_col = wn + (lane & 15);
    float b1[4][4], b2[4][4], b3[4][4]; // per row slot: the three smallest keys
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) b1[i][r] = b2[i][r] = b3[i][r] = INFINITY;
    const uint32_t keep = ~((1u << a.idx_bits) - 1u);
    // One scale for the block's rows, and not so far above the columns' that their norms would leave fp32 in it: then the
    // sums of the products start from the norm (see `select`).  Otherwise (own) the rows' scales are looked up.
    const float as = has_rows ? a.ascale[blk] : 1.f;
    const bool own = as == 0.f || !(as <= 0x1p80f * a.bhdr[2]);
    const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};

    auto copy_first = [&]() {
#pragma unroll
        for (int i = 0; i < HSTEP; ++i) {
            copy_norms(t0 + i);
#pragma unroll
            for (int u = 0; u < KS; ++u) copy_page(t0 + i, u);
        }
    };
    copy_first();
    if (own && (tid & (HNT / 2 - 1)) < HT) // (read behind the first tile's barrier)
        rinv[group * HT + (tid & (HT - 1))] = as == 0.f ? a.arinv[blk * HT + (tid & (HT - 1))] : 1.f / as;
    // exact distances of the n pairs that wait, 16 lanes a pair
    auto settle = [&](int n) {
        const int grp = tid >> 4, l16 = tid & 15;
        for (int p0 = 0; p0 < n; p0 += HNT / 16 * PAIR_BATCH) { // (the loads of a batch are under way together)
            float d[PAIR_BATCH];
            uint32_t e[PAIR_BATCH];
#pragma unroll
            for (int u = 0; u < PAIR_BATCH; ++u) {
                e[u] = pairs[min(p0 + HNT / 16 * u + grp, n - 1)];
                const int64_t row = m0 + (e[u] >> PAIR_COL_BITS), col = (int64_t)t0 * HT + (e[u] & ((1u << PAIR_COL_BITS) - 1u));
                d[u] = sqdist16(a.X + row * (KS * 32), a.C + col * (KS * 32), KS * 32, l16, a.vec);
            }
#pragma unroll
            for (int u = 0; u < PAIR_BATCH; ++u)
                if (p0 + HNT / 16 * u + grp < n && l16 == 0)
                    atomicMin(&best[e[u] >> PAIR_COL_BITS],
                              make_key(d[u], (uint32_t)t0 * HT + (e[u] & ((1u << PAIR_COL_BITS) - 1u))));
        }
    };
    // Waits for the tiles t .. t + HSTEP - 1 (every wave for its own copies); the next ones are asked for by `multiply`.
    auto next_tiles = [&](int t) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads(); // (the other half of the ring is free from here on)
#pragma unroll
        for (int i = 0; i < HSTEP; ++i) copy_norms(t + HSTEP + i);
    };
    // scale of tile t's columns, norms of the lane's
    auto column_scale = [&](int t) { return cnorm[((t - t0) & (2 * HRING - 1)) * HCOLS + HT]; };
    auto column_norms = [&](int t, float f, float absent) {
        f32x4 cb = *(const f32x4 *)(cnorm + ((t - t0) & (2 * HRING - 1)) * HCOLS + wn + 4 * (lane & 15)) * f;
#pragma unroll
        for (int j = 0; j < 4; ++j) cb[j] = fminf(cb[j], absent); // (a column with a non-finite norm is none; its image is zero)
        if ((int64_t)(t + 1) * HT > a.N)                          // (the last tile)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((int64_t)t * HT + slot_col + 16 * j >= a.N) cb[j] = absent;
        return cb;
    };
    f32x4 acc[4][4];
    half8 bh[2][4]; // fragments of the columns, read a step ahead
    auto read_columns = [&](int t, int u) {
        const u32x4 *bp = lds + (((t - t0) & (HRING - 1)) * KS + u) * HPAGE + 4 * wn + lane;
#pragma unroll
        for (int j = 0; j < 4; ++j) bh[u & 1][j] = __builtin_bit_cast(half8, bp[64 * j]);
        asm volatile("" ::: "memory"); // (the reads stay here, they are not moved down to their use)
        __builtin_amdgcn_sched_barrier(0);
    };
    // The products of tile t, whose first fragments have been asked for.  COPY: between them the pages of the next
    // HSTEP tiles are asked for, a few at a time (a wave that issues all its copies at once waits for the queue).
    auto multiply = [&](auto OWN, auto COPY, int t) {
        __builtin_amdgcn_s_setprio(1); // (the products go first, the other group's selection takes the slots between them)
        f32x4 c0[4] = {zero4, zero4, zero4, zero4};
        if (!decltype(OWN)::value) {
            const float f = 0.5f * as * column_scale(t); // (a power of two)
            const f32x4 cb = column_norms(t, f, fminf(NO_COLUMN * f, NO_COLUMN));
#pragma unroll
            for (int j = 0; j < 4; ++j) c0[j] = f32x4{cb[j], cb[j], cb[j], cb[j]};
        }
#pragma unroll
        for (int u = 0; u < KS; ++u) {
            if (u + 1 < KS) read_columns(t, u + 1);
            if (decltype(COPY)::value)
#pragma unroll
                for (int i = 0; i < HSTEP; ++i) copy_page(t + HSTEP + i, u);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[u][i], bh[u & 1][j], u == 0 ? c0[j] : acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
    };
    // The products of tile t enter the running three smallest.  A holds the negated rows: what the products leave is
    // ||b||^2 - 2 <a, b> in units of 2 / (scale of the rows * scale of the columns), the norm being what they are added to
    // (OWN: without the norm, in units of 2 / scale of the columns).  The units are powers of two: 1 / 2^x by its exponent.
    // (fminf on b1 would make the compiler quiet both operands first, an instruction each; see the mode set around the sweep.)
    auto select = [&](auto OWN, int t) {
        const float binv = 2.f * __uint_as_float(0x7F000000u - __float_as_uint(column_scale(t)));
        const float inv = decltype(OWN)::value ? binv : binv * __uint_as_float(0x7F000000u - __float_as_uint(as));
        f32x4 cb = zero4;
        if (decltype(OWN)::value) cb = column_norms(t, 1.f, NO_COLUMN);
        uint32_t tj = (uint32_t)(t - t0);
        asm("" : "+v"(tj)); // (in a vector register: one scalar operand an instruction)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float e;
                if (decltype(OWN)::value) {
                    const float f = inv * rinv[slot_row(i, r)];
                    e = fminf(fminf(fminf(fmaf(f, acc[i][0][r], cb[0]), fmaf(f, acc[i][1][r], cb[1])),
                                    fmaf(f, acc[i][2][r], cb[2])), fmaf(f, acc[i][3][r], cb[3]));
                } else {
                    e = inv * __builtin_elementwise_minimum(__builtin_elementwise_minimum(__builtin_elementwise_minimum(
                                  acc[i][0][r], acc[i][1][r]), acc[i][2][r]), acc[i][3][r]);
                }
                const float key = __uint_as_float((__float_as_uint(e) & keep) | tj);
                b3[i][r] = __builtin_amdgcn_fmed3f(b2[i][r], b3[i][r], key);
                b2[i][r] = __builtin_amdgcn_fmed3f(b1[i][r], b2[i][r], key);
                asm("v_min_f32 %0, %0, %1" : "+v"(b1[i][r]) : "v"(key));
            }
    };
    // OWN: the rows' scales are read from rinv, not one for the block.
    auto sweep = [&](auto OWN) {
        for (int t = t0; t < t1; t += HSTEP) {
            next_tiles(t);
#pragma unroll
            for (int i = 0; i < HSTEP; ++i) {
                if (t + i >= t1) break;
                if (group == 1 || i == 0) read_columns(t + i, 0);
                __builtin_amdgcn_sched_barrier(0);
                // the second group is half a step behind: the selection of the tile before, then this tile's products
                if (group == 1 && t + i > t0) select(OWN, t + i - 1);
                __builtin_amdgcn_sched_barrier(0);
                if (i == 0)
                    multiply(OWN, std::true_type{}, t);
                else
                    multiply(OWN, std::false_type{}, t + i);
                __builtin_amdgcn_sched_barrier(0);
                if (group == 0) {
                    if (i + 1 < HSTEP && t + i + 1 < t1) read_columns(t + i + 1, 0);
                    select(OWN, t + i);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (group == 1 && t0 < t1) select(OWN, t1 - 1);
    };
    // Second sweep: b1 holds the rows' bands, and what lies inside is collected.  Returns false (to all threads) where
    // a tile finds no room for its pairs.
    auto sweep_pairs = [&]() -> bool {
        for (int t = t0; t < t1; ++t) {
            if ((t - t0) % HSTEP == 0)
                next_tiles(t);
            else
                __syncthreads();
            const int n = sh_pairs;
            __syncthreads(); // (read by all before the next tile adds to it)
            if (n > PAIR_CAP) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // (no copy outlives the workgroup)
                return false;
            }
            if (n > PAIR_CAP / 2) {
                settle(n);
                __syncthreads();
                if (tid == 0) sh_pairs = 0;
                __syncthreads();
            }
            read_columns(t, 0);
            if ((t - t0) % HSTEP == 0)
                multiply(std::true_type{}, std::true_type{}, t);
            else
                multiply(std::true_type{}, std::false_type{}, t);
            const float inv = 2.f * __uint_as_float(0x7F000000u - __float_as_uint(column_scale(t)));
            const f32x4 cb = column_norms(t, 1.f, NO_COLUMN);
            uint32_t miss[2] = {0u, 0u}; // of columns j = 0, 1 and j = 2, 3: 16 row slots each
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float f = inv * rinv[slot_row(i, r)];
                        miss[j >> 1] = __builtin_amdgcn_alignbit(
                            miss[j >> 1], __float_as_uint(b1[i][r] - fmaf(f, acc[i][j][r], cb[j])), 31);
                    }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t hit = ~miss[h];
                while (hit) {
                    const int b = __clz(hit); // bit 31 is the first row slot of the first column
                    hit &= ~(0x80000000u >> b);
                    const uint32_t col = (uint32_t)(t - t0) * HT + slot_col + 32 * h + (b & 16);
                    const int rl = slot_row((b >> 2) & 3, b & 3);
                    // (the products of a row with a NaN have any sign)
                    if ((int64_t)t0 * HT + col >= a.N || !crowded[rl]) continue;
                    const int at = atomicAdd(&sh_pairs, 1);
                    if (at < PAIR_CAP) pairs[at] = ((uint32_t)rl << PAIR_COL_BITS) | col;
                }
            }
        }
        return true;
    };
    // Keys of infinite products with a tile planted in them are signalling NaNs: with the IEEE bit of the mode cleared
    // v_min_f32 passes over them instead of handing a NaN on.
    __builtin_amdgcn_s_setreg(0 << 11 | 9 << 6 | 1, 0);
    if (own)
        sweep(std::true_type{});
    else
        sweep(std::false_type{});
    __builtin_amdgcn_s_setreg(0 << 11 | 9 << 6 | 1, 1);

    // ---- row minimum over the workgroup, then every kept key inside the band of it ----
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // (the last copies too)
    __syncthreads();                                  // the tiles are dead from here on
    unsigned *rowmin = (unsigned *)lds;                                // [HR]
    int *rowcnt = (int *)(rowmin + HR);                                // [HR]
    unsigned long long *rowcand = (unsigned long long *)(rowcnt + HR); // [HR][VLQ_NN_CANDS]
    if (tid == 0) sh_slots = 0;
    if (tid < HR) {
        rowmin[tid] = 0xFFFFFFFFu;
        rowcnt[tid] = 0;
#pragma unroll
        for (int s = 0; s < VLQ_NN_CANDS; ++s) rowcand[tid * VLQ_NN_CANDS + s] = KEY_MAX;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (b1[i][r] < NO_KEY) atomicMin(&rowmin[slot_row(i, r)], f2ord(b1[i][r]));
    __syncthreads();
    const float rho = a.bhdr[0], big = a.bhdr[1];
    // where the band of row rl (one with a minimum) ends
    auto band_end = [&](int rl) {
        const float ra = a.an[m0 + rl];
        const float emin = __uint_as_float(__float_as_uint(ord2f(rowmin[rl])) & keep);
        const float dmin = fmaxf(emin + ra, 0.f);
        return emin + nn_half_band(ra, a.ares[m0 + rl], rho, big, dmin, a.band_dist, KS * 32);
    };
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rl = slot_row(i, r);
            if (rowmin[rl] == 0xFFFFFFFFu || m0 + rl >= a.M) continue;
            const float ra = a.an[m0 + rl], band = band_end(rl);
            // A key stands for the lane's four columns of its tile; where a third one lies inside the band a fourth may
            // have been pushed out, so the slot's columns are handed on instead.
            auto in_band = [&](float key) { return key < NO_KEY && __uint_as_float(__float_as_uint(key) & keep) <= band; };
            auto hand_on = [&](float key, bool slot) {
                const float e = __uint_as_float(__float_as_uint(key) & keep);
                const uint32_t entry = slot ? VLQ_NN_SLOT | (uint32_t)((wn >> 6) * 16 + (lane & 15))
                                            : (uint32_t)(t0 + (int)(__float_as_uint(key) & ~keep)) * HT + slot_col;
                const int pos = atomicAdd(&rowcnt[rl], 1);
                if (pos < VLQ_NN_CANDS)
                    rowcand[rl * VLQ_NN_CANDS + pos] = ((uint64_t)__float_as_uint(fmaxf(e + ra, 0.f) + 0.f) << 32) | entry;
            };
            if (!in_band(b1[i][r])) continue;
            const bool slot = in_band(b3[i][r]);
            hand_on(b1[i][r], slot);
            if (!slot && in_band(b2[i][r])) hand_on(b2[i][r], false);
        }
    __syncthreads();
    uint64_t *dst = nullptr;
    uint64_t near = 0; // high word of the split's smallest key
    int slots = 0;
    if (tid < HR && m0 + tid < a.M) {
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
    if (tid < HR) {
        rowcnt[tid] = slots; // (read by all threads below, before the tiles overwrite it)
        best[tid] = KEY_MAX;
        const int64_t b = (int64_t)blockIdx.x * 2 + tid / HT; // (rows past the last block: not looked at)
        const float s = b * HT < a.M ? a.ascale[b] : 1.f;
        rinv[tid] = s != 0.f ? 1.f / s : a.arinv[m0 + tid];
    }
    if (tid == 0) sh_pairs = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rl = slot_row(i, r);
            b1[i][r] = rowcnt[rl] ? band_end(rl) : -INFINITY;
        }
    __syncthreads();
    if (tid < HR) crowded[tid] = slots != 0;
    copy_first();
    if (!sweep_pairs()) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
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
    // the ring of tiles (or the tail of the kernel in its place), the columns' norms, the rows' scales, and the nearest
    // columns and the pairs of the second sweep: 148.5 KB at most
    const size_t bytes = half_front_bytes(D / 32) + 2 * HRING * HCOLS * 4 + HR * (4 + 8) + PAIR_CAP * 4;
    const dim3 grid((unsigned)((M + HR - 1) / HR), (unsigned)nsplit);
    auto go = [&](auto kern) -> int {
        if (bytes > 49152) { // (48 KB of dynamic LDS need no asking)
            hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
            if (e != hipSuccess) return (int)e;
        }
        hipLaunchKernelGGL(kern, grid, dim3(HNT), bytes, st, a);
        return 0;
    };
    switch (D / 32) {
    case 1: return go(k_nearest_half<1>);
    case 2: return go(k_nearest_half<2>);
    case 3: return go(k_nearest_half<3>);
    case 4: return go(k_nearest_half<4>);
    }
    return (int)hipErrorInvalidValue;
}
