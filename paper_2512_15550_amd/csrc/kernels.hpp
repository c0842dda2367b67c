// gfx950 kernels of the CTkvr path.
//
// Decode step (Algorithm 2 lines 1-9), four to eight launches:
//   centroid_cos  lines 1-2   cosine to every centroid, max over the GQA group
//   recall_gather lines 3-4a  top-C' centroids; their lists OR-ed into a bitmap
//   recall_score  lines 4b-5a the bitmap as an ascending id list plus each id's physical
//                             KV row; z = (q . k) * scale for the G heads, running max
//   denom         line 5b     softmax denominators, integer fixed point
//   keyhist       line 5c     max over the group of log-softmax as a ranking key,
//                             and a histogram of the keys
//   classify      line 6a     chip-wide pass over the keys: sure picks as a bitmap, the
//                             deciding bucket as a list
//   rerank_select line 6b     top-rho' ids
//   sparse_attn   lines 7-9   softmax(z_sel) . V_sel, one block per slice of the
//                             head dimension (no cross-block reduction)
//   (keyclass = keyhist and classify, select_attn = the last two in one launch, tail = all from denom on, for small batches)
// The exact index build (Algorithm 1 lines 2-4) takes the same formula with "the recalled set" = all s keys and the centroid in the
// role of the query: exact_score -> exact_list, beyond 515072 tokens score -> denom -> keyhist -> rerank_select.
#pragma once
#include "arith.hpp"
#include "common.hpp"

namespace ctkvr {

// Words and sums of a unit that blocks of the whole chip update by atomics: a cache line to a unit, because atomics on one
// line are served one after the other (units of a step side by side: 32K, eight units 34.9 -> 34.4 us a step, with the
// centroid update 41.5 -> 40.7, 4K 22.9 -> 22.7; the list cursors: 128K x 4 124.2 -> 123.6, sixteen of 8K to 64K 146.8 -> 145.7).
constexpr int kMaxStride = 32;   // maxima and list cursors, 4 bytes
constexpr int kSumStride = 16;   // denominators, 8 bytes

// A "unit" is what one selection is made for: in a decode step a (sequence, KV
// head) pair; in the build a (sequence, KV head, centroid) triple.
struct Units {
    int g, G, h;
    int build;               // 0: unit = b*g + kv            1: unit = unit0 + local = (b*g + kv)*c_max + j
    int unit0, c_max;
    const int32_t *n_cent;   // [batch] centroids per sequence
};

__device__ __forceinline__ bool decode_unit(const Units &u, int local, int &b, int &kv, int &j)
{
    if (!u.build) {
        b = local / u.g;
        kv = local - b * u.g;
        j = 0;
        return true;
    }
    int id = u.unit0 + local;
    int bk = id / u.c_max;
    j = id - bk * u.c_max;
    b = bk / u.g;
    kv = bk - b * u.g;
    return j < u.n_cent[b];
}

// Block -> (unit, block of the unit) for grids (blocks per unit, units).  Workgroups go to the 8 XCDs round-robin by
// linear id, every XCD has an L2 of its own, and what a kernel wrote is still in its XCD's L2 when the next kernel
// runs (a dependent load of such a line: 88 ns on the XCD that wrote it, 220 ns on another).  With by_xcd (the host
// sets it when the units are a multiple of 8) the blocks of unit u are those with linear id congruent u modulo the
// number of units: all on XCD u mod 8, in every kernel of a decode step, so that a unit's intermediate results are read
// where they were written.
__device__ __forceinline__ void unit_block_of(const int by_xcd, int &ul, int &bx)
{
    if (by_xcd) {
        const int lin = (int)(blockIdx.y * gridDim.x + blockIdx.x);
        ul = lin % (int)gridDim.y;
        bx = lin / (int)gridDim.y;
    } else {
        ul = (int)blockIdx.y;
        bx = (int)blockIdx.x;
    }
}

// ------------------------------------------------------------------------------
// small utilities
// ------------------------------------------------------------------------------
__global__ void fill_u32_kernel(uint32_t *p, uint32_t v, size_t n)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ranges of words cleared by one launch: grid (any, ranges)
struct ZeroRanges {
    static constexpr int kMax = 8;
    uint32_t *p[kMax];
    size_t words[kMax];
    int n;
};
__device__ __forceinline__ void zero_range(const ZeroRanges &z)
{
    uint32_t *p = z.p[blockIdx.y];
    const size_t n = z.words[blockIdx.y], step = (size_t)gridDim.x * blockDim.x, n4 = n / 4;
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;   // every range starts on a 256-byte boundary
    for (size_t i = i0; i < n4; i += step) reinterpret_cast<uint4 *>(p)[i] = make_uint4(0u, 0u, 0u, 0u);
    for (size_t i = 4 * n4 + i0; i < n; i += step) p[i] = 0u;
}
__global__ void zero_ranges_kernel(ZeroRanges z) { zero_range(z); }

// integers that travel as a kernel argument
struct IntPack {
    static constexpr int kMax = 512;
    int32_t v[kMax];
};
__global__ void put_ints_kernel(int32_t *dst, int n, IntPack pack)
{
    for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = pack.v[i];
}

// both in one launch: grid (any, z.n + 1); the pack holds rows.n integers for each of the destinations (null: not wanted), one after the other
struct IntRows {
    static constexpr int kMax = 3;
    int32_t *dst[kMax];
    int n;
};
__global__ void set_up_kernel(ZeroRanges z, IntRows rows, IntPack pack)
{
    if ((int)blockIdx.y < z.n) {
        zero_range(z);
        return;
    }
    if (blockIdx.x) return;
    for (int r = 0; r < IntRows::kMax; ++r)
        if (rows.dst[r])
            for (int i = threadIdx.x; i < rows.n; i += blockDim.x) rows.dst[r][i] = pack.v[r * rows.n + i];
}

// The lowest flat index of a list entry that is not a key id of its sequence goes to *bad (~0: none).  grid (c_max, units)
__global__ void check_lists_kernel(const int32_t *lists, const int32_t *ctx_lens, const int32_t *n_cent, int g, int c_max, int rho,
                                   unsigned long long *bad)
{
    const int j = blockIdx.x, ul = blockIdx.y, b = ul / g;
    if (j >= n_cent[b]) return;
    const int s = ctx_lens[b];
    const size_t row = ((size_t)ul * c_max + j) * rho;
    for (int r = threadIdx.x; r < rho; r += blockDim.x)
        if ((uint32_t)lists[row + r] >= (uint32_t)s) atomicMin(bad, (unsigned long long)(row + r));
}

// three ranges cleared by one launch: grid ceil((n0 + n1 + n2) / blockDim.x)
__global__ void zero3_u32_kernel(uint32_t *p0, size_t n0, uint32_t *p1, size_t n1, uint32_t *p2, size_t n2)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n0) {
        p0[i] = 0u;
    } else if (i < n0 + n1) {
        p1[i - n0] = 0u;
    } else if (i < n0 + n1 + n2) {
        p2[i - n0 - n1] = 0u;
    }
}

// Algorithm 1 line 1: centroid j of sequence b, head hd = prompt query at position s_b - C_b + j, and its inverse norm.
// q_prefill rows [first_row_b + j][h][128] -> centroids [b][h][c_max][128]; the norms of rows beyond n_cent are 0, the rows
// themselves are left alone (zeros).  A row is 16 bytes a lane of 16, or twice that (an element a thread and the norms in a launch of
// their own: 2048 centroids of 32 heads, bf16, 20.4 + 4.5 us).  grid (ceil(c_max / 16), h, batch), 256 threads
template <typename T>
__global__ __launch_bounds__(256) void copy_centroids_kernel(const T *q_prefill, const int32_t *first_row /*[batch]*/,
                                                             const int32_t *n_cent, int h, int c_max, T *centroids, float *inv_norm)
{
    const int j = blockIdx.x * 16 + (threadIdx.x >> 4), lane16 = threadIdx.x & 15, hd = blockIdx.y, b = blockIdx.z;
    const int C = n_cent[b];
    const size_t row = ((size_t)b * h + hd) * c_max + j;
    Chunk<T> c;   // (the caller's rows start on any element)
    __builtin_memcpy(&c, q_prefill + ((size_t)(first_row[b] + min(j, C - 1)) * h + hd) * kD + 8 * lane16, sizeof c);
    float x[8];
    unpack(c, x);
    const float n2 = group16_sum(lane_partial(x, x));
    if (j < C) __builtin_memcpy(__builtin_assume_aligned(centroids + row * kD + 8 * lane16, 16), &c, sizeof c);
    if (j < c_max && lane16 == 0) inv_norm[row] = j < C ? inv_norm_from_sq(n2) : 0.0f;
}

// inverse norms of n rows of 128
template <typename T> __global__ __launch_bounds__(256) void inv_norm_kernel(const T *rows, size_t n, float *out)
{
    size_t r = (size_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    int lane16 = threadIdx.x & 15;
    size_t rr = r < n ? r : n - 1;
    float x[8];
    unpack(load_chunk(rows + rr * kD, lane16), x);
    float n2 = group16_sum(lane_partial(x, x));
    if (r < n && lane16 == 0) out[r] = inv_norm_from_sq(n2);
}

// ------------------------------------------------------------------------------
// Algorithm 2 lines 1-2: Cos_kv[b][kv][j] = max over the group of cos(q_h, c_{h,j})
// grid (ceil(c_max/16), batch*g), 256 threads: one centroid per 16-lane group, its
// G head rows loaded together.  Block x == 0 also clears the step's accumulators.
// ------------------------------------------------------------------------------
struct CosArgs {
    const void *q;            // [batch][h][128]
    const void *centroids;    // [batch][h][c_max][128]
    const float *inv_norm_c;  // [batch][h][c_max]
    const int32_t *n_cent;
    float *cos;               // [batch*g][c_max]
    uint32_t *m_key;          // [batch*g][kMaxStride]  cleared here
    unsigned long long *S;    // [batch*g][kSumStride]  cleared here
    unsigned long long *xs;   // [batch*g][n_xs] the tail kernel's exchange slots, cleared here (n_xs <= 64; 0: none)
    int n_xs;
    int g, h, c_max;
    int by_xcd;               // blocks -> (unit, block of the unit) by unit_block_of
};

template <typename T, int G> __global__ __launch_bounds__(256) void centroid_cos_kernel(CosArgs a)
{
    int ul, bx;
    unit_block_of(a.by_xcd, ul, bx);
    const int b = ul / a.g, kv = ul - b * a.g;
    const int C = a.n_cent[b];
    const int tid = threadIdx.x, lane16 = tid & 15, grp = tid >> 4;
    if (bx == 0 && tid < G) {
        a.m_key[ul * kMaxStride + tid] = 0u;
        a.S[ul * kSumStride + tid] = 0ull;
    }
    if (bx == 0 && tid < a.n_xs) a.xs[ul * a.n_xs + tid] = 0ull;
    CTKVR_STAMP(0);
    const int tile0 = bx * 16;
    if (tile0 >= C) return;
    const int j = tile0 + grp;
    const int jj = j < C ? j : C - 1;
    const T *qb = (const T *)a.q + ((size_t)b * a.h + kv * G) * kD;
    const T *cb = (const T *)a.centroids;
    Chunk<T> cq[G], cc[G];
    float inc[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) {
        size_t row = ((size_t)b * a.h + kv * G + hh) * a.c_max + jj;
        cc[hh] = load_chunk(cb + row * kD, lane16);
        cq[hh] = load_chunk(qb + (size_t)hh * kD, lane16);
        inc[hh] = a.inv_norm_c[row];
    }
    float best = -__builtin_huge_valf();
#pragma unroll
    for (int hh = 0; hh < G; ++hh) {
        float q[8], cx[8];
        unpack(cq[hh], q);
        unpack(cc[hh], cx);
        float inv_q = inv_norm_from_sq(group16_sum(lane_partial(q, q)));
        float dot = group16_sum(lane_partial(q, cx));
        float cs = (dot * inc[hh]) * inv_q;
        best = fmaxf(best, cs);
    }
    if (j < C && lane16 == 0) a.cos[(size_t)ul * a.c_max + j] = best;
    CTKVR_STAMP(1);
}

// ------------------------------------------------------------------------------
// Algorithm 2 lines 3-4, first part, each (sequence, KV head) spread over several
// blocks so that no single CU has to pull all the probed lists (the bitmap becomes the
// ascending id list in recall_score_kernel).
//
// recall_gather: every block of a unit finds the same top-C' centroids (keys in
// registers, C <= 256*KPT), takes every gridDim.x-th probed list, ORs its ids into a bitmap in shared memory and then
// ORs the non-empty words into the unit's bitmap in global memory (integer ORs: any
// order gives the same bitmap).  grid (blocks per unit, batch*g), 256 threads; dynamic shared
// memory: kSelLds + n_probe + bitmap words.
// ------------------------------------------------------------------------------
struct GatherArgs {
    const float *cos;         // [batch*g][c_max]
    const int32_t *lists;     // [batch*g][c_max][rho]
    const int32_t *n_cent, *ctx_lens;
    int32_t *probe;           // [batch*g][n_probe]
    int32_t *out_probe;       // optional copy for the caller
    uint32_t *gbits;          // [batch*g][bitmap_words], all zero between steps
    int g, c_max, rho, n_probe, bitmap_words;
    int by_xcd;               // blocks -> (unit, block of the unit) by unit_block_of
};

template <int KPT> __global__ __launch_bounds__(256) void recall_gather_kernel(GatherArgs a)
{
    extern __shared__ uint32_t smem[];
    uint32_t *s_sel = smem;
    int32_t *s_probe = (int32_t *)(smem + kSelLds);
    uint32_t *s_bits = smem + kSelLds + a.n_probe;
    int ul, bx;
    unit_block_of(a.by_xcd, ul, bx);
    const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
    const int b = ul / a.g;
    const int C = a.n_cent[b], s = a.ctx_lens[b];
    const float *cosv = a.cos + (size_t)ul * a.c_max;
    const int W = (s + 31) >> 5;
    CTKVR_STAMP(8);
    CTKVR_STAMP_BLK(0);
    for (int w = tid; w < W; w += 256) s_bits[w] = 0u;
    auto keep = [&](int pos, int j) {
        s_probe[pos] = j;
        if (bx == 0) {
            a.probe[(size_t)ul * a.n_probe + pos] = j;
            if (a.out_probe) a.out_probe[(size_t)ul * a.n_probe + pos] = j;
        }
    };
    // line 3
    // (more than 64 probes: bisection by the block, of thousands of centroids 11-bit radix rounds)
    auto cos_key = [&](int j) { return ordered_key(cosv[j]); };
    if (a.n_probe <= 64)
        split_topk<256, KPT>(cos_key, a.c_max, C, a.n_probe, keep, s_sel);   // (every row of a.cos has c_max entries)
    else if constexpr (KPT > 8)
        block_select_topk<256, KPT>(cos_key, C, a.n_probe, keep, s_sel);
    else
        block_bisect_topk<256, KPT>(cos_key, C, a.n_probe, keep, s_sel);
    __syncthreads();
    CTKVR_STAMP(9);
    // line 4: this block's share of the probed lists, one list per wave at a time
    const int32_t *lb = a.lists + (size_t)ul * a.c_max * a.rho;
    // Two lists per round and wave, all of a round's loads requested before the first id is used.
    const int pstride = gridDim.x * 4;
    auto mark = [&](int t) { atomicOr(&s_bits[t >> 5], 1u << (t & 31)); };
    for (int p = bx + gridDim.x * wv; p < a.n_probe; p += 2 * pstride) {
        const bool two = p + pstride < a.n_probe;
        const int32_t *l0 = lb + (size_t)s_probe[p] * a.rho;
        const int32_t *l1 = lb + (size_t)s_probe[two ? p + pstride : p] * a.rho;
        if ((a.rho & 3) == 0) {
            const int4 *s0 = reinterpret_cast<const int4 *>(l0), *s1 = reinterpret_cast<const int4 *>(l1);
            const int rho4 = a.rho >> 2;
            for (int r0 = 0; r0 < rho4; r0 += 64 * 8) {
                // (entries beyond the list's end re-read its last one and are not marked: a load under
                // a per-lane condition is waited for before the next is requested)
                int4 t0[8], t1[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) t0[u] = s0[min(r0 + u * 64 + ln, rho4 - 1)];
                if (two) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) t1[u] = s1[min(r0 + u * 64 + ln, rho4 - 1)];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int r = r0 + u * 64 + ln;
                    if (r < rho4) {
                        mark(t0[u].x); mark(t0[u].y); mark(t0[u].z); mark(t0[u].w);
                        if (two) { mark(t1[u].x); mark(t1[u].y); mark(t1[u].z); mark(t1[u].w); }
                    }
                }
            }
        } else {   // list rows not 16-byte aligned: the same rounds with 4-byte loads
            for (int r0 = 0; r0 < a.rho; r0 += 64 * 8) {
                int32_t t0[8], t1[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) t0[u] = l0[min(r0 + u * 64 + ln, a.rho - 1)];
                if (two) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) t1[u] = l1[min(r0 + u * 64 + ln, a.rho - 1)];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (r0 + u * 64 + ln < a.rho) {
                        mark(t0[u]);
                        if (two) mark(t1[u]);
                    }
                }
            }
        }
    }
    __syncthreads();
    CTKVR_STAMP(10);
    uint32_t *gb = a.gbits + (size_t)ul * a.bitmap_words;
    for (int w = tid; w < W; w += 256) {
        uint32_t v = s_bits[w];
        if (v) atomicOr(&gb[w], v);
    }
    CTKVR_STAMP_BLK(1);
}

// ------------------------------------------------------------------------------
// Algorithm 2 line 5 / Algorithm 1 line 2, first half: z[h][i] = (q_h . k_i) * scale
// for the G heads of the group, plus the running maximum per head.  A block walks
// tiles of 16*R ids (R rows per 16-lane group, all R loads issued before the first
// use) with stride gridDim.x.  grid (nbx, units), 256 threads.
// ------------------------------------------------------------------------------
struct ScoreArgs {
    Units u;
    const void *q;            // decode: [batch][h][128] (qrows = 1); build: centroids [batch][h][c_max][128] (qrows = c_max)
    int qrows;
    Paged k;
    const int32_t *ctx_lens;
    const uint32_t *crow;     // [units][l_stride] physical rows of the recalled ids, or nullptr = all ids 0..s-1
    const int32_t *ncand;     // [units] (with crow)
    int l_stride;
    float *z;                 // [units][l_stride][G]
    uint32_t *m_key;          // [units][kMaxStride] ordered-key running max per head (atomicMax)
    uint32_t *ghist;          // decode only: [units][kBuckets] key histogram, cleared here for keyhist
    float scale;
};

template <typename T, int G, int R> __global__ __launch_bounds__(256) void score_kernel(ScoreArgs a)
{
    constexpr int TILE = 16 * R;
    int b, kv, j;
    const int ul = blockIdx.y;
    if (!decode_unit(a.u, ul, b, kv, j)) return;
    const int tid = threadIdx.x, lane16 = tid & 15, grp = tid >> 4;
    // decode: the first tile's row ids are requested together with L, not after it (slots beyond
    // L hold stale words; they are never used as rows, see the clamp below)
    uint32_t pre = 0;
    if (a.crow && tid < TILE) pre = a.crow[(size_t)ul * a.l_stride + min((int)blockIdx.x * TILE + tid, a.l_stride - 1)];
    const int L = a.crow ? a.ncand[ul] : a.ctx_lens[b];
    if (a.ghist)
        for (int w = blockIdx.x * 256 + threadIdx.x; w < kBuckets; w += gridDim.x * 256) a.ghist[(size_t)ul * kBuckets + w] = 0u;
    if ((int)blockIdx.x * TILE >= L) return;
    __shared__ uint32_t s_row[TILE];
    __shared__ uint32_t s_max[G];
    CTKVR_STAMP(20);
    if (tid < G) s_max[tid] = 0u;
    float q[G][8];
    const T *qb = (const T *)a.q + (((size_t)b * a.u.h + kv * G) * a.qrows + j) * kD;
#pragma unroll
    for (int hh = 0; hh < G; ++hh) unpack(load_chunk(qb + (size_t)hh * a.qrows * kD, lane16), q[hh]);
    const T *K = (const T *)a.k.pages;
    float *zb = a.z + (size_t)ul * a.l_stride * G;
    // lane l of a 16-lane group keeps head (l mod G): its score, and that head's running maximum
    float mxl = -__builtin_huge_valf();
    const int myh = lane16 & (G - 1);
    for (int tile0 = blockIdx.x * TILE; tile0 < L; tile0 += gridDim.x * TILE) {
        __syncthreads();   // previous tile's rows are consumed
        if (tid < TILE) {
            int i = min(tile0 + tid, L - 1);
            if (a.crow)
                s_row[tid] = (tile0 == (int)blockIdx.x * TILE) ? pre : a.crow[(size_t)ul * a.l_stride + i];
            else
                s_row[tid] = row_of(a.k.block_table, a.k.max_pages, a.k.page_shift, a.u.g, b, kv, i);
        }
        __syncthreads();
        const int last = L - 1 - tile0;   // slots of the tile beyond it repeat the last valid row
        CTKVR_STAMP(21);
        Chunk<T> ck[R];
#pragma unroll
        for (int r = 0; r < R; ++r) ck[r] = load_chunk(K + (size_t)s_row[min(r * 16 + grp, last)] * kD, lane16);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float kx[8];
            unpack(ck[r], kx);
            float mine = 0.0f;
#pragma unroll
            for (int hh = 0; hh < G; ++hh) {
                float tot = group16_sum(lane_partial(q[hh], kx));
                if (hh == 0 || myh == hh) mine = tot;
            }
            mine = mine * a.scale;
            const int i = tile0 + r * 16 + grp;
            if (i < L) {
                mxl = __builtin_amdgcn_fmed3f(mxl, mine, __builtin_huge_valf());   // max of two non-NaN values
                if (lane16 < G) zb[(size_t)i * G + lane16] = mine;
            }
        }
    }
    {
        float v = mxl;
        v = __builtin_amdgcn_fmed3f(v, __shfl_xor(v, 16), __builtin_huge_valf());
        v = __builtin_amdgcn_fmed3f(v, __shfl_xor(v, 32), __builtin_huge_valf());
        if (lane_id() < G) atomicMax(&s_max[lane_id()], ordered_key(v));
    }
    __syncthreads();
    if (tid < G) atomicMax(&a.m_key[ul * kMaxStride + tid], s_max[tid]);
    CTKVR_STAMP(22);
}

// ------------------------------------------------------------------------------
// Algorithm 2 lines 10-11: attention over the resident window -- the first n_init keys and the
// keys from s - n_local to the current end of the cache (the tokens decoded since the index was
// built join the local window) -- and its merge with the sparse attention.
// window_attn_kernel: block x of a unit takes every kWinSplit-th run of 64 window rows and leaves
// a partial result relative to its own maximum: m[G], l[G] = sum of exp(z - m), o[G][128] = sum of
// exp(z - m) v.  Online softmax over runs of 64 rows (one row per 16-lane group and pass, four
// passes).  It depends on q, K and V only: as a launch of its own it is the first of a step (grid (kWinSplit,
// units), 256 threads); the step of one launch per stage runs the same blocks as kWinSplit extra blocks per
// unit of recall_score_kernel's launch instead, where they cost no launch and run beside the scoring blocks.
// ------------------------------------------------------------------------------

struct WindowArgs {
    Units u;
    const void *q;            // [batch][h][128]
    Paged k;
    const void *v_pages;
    const int32_t *ctx_lens;  // [batch] s: the prefix the index was built on
    const int32_t *cur_lens;  // optional [batch]: tokens in the cache now (>= s)
    int n_init, n_local;
    int by_xcd;               // blocks -> (unit, block of the unit) by unit_block_of
    float scale;
    float *win;               // [units][kWinSplit][G][2 + 128]
};

// One block's share: bx of kWinSplit, unit ul; 256 threads.
template <typename T, int G> __device__ __forceinline__ void window_attn_block(const WindowArgs &a, const int bx, const int ul)
{
    __shared__ float s_z[64][G];
    __shared__ float s_part[4][G][kD];
    __shared__ float s_ml[G];
    const int b = ul / a.u.g, kv = ul - b * a.u.g;
    const int tid = threadIdx.x, lane16 = tid & 15, grp = tid >> 4;
    const int s = a.ctx_lens[b];
    int cur = a.cur_lens ? a.cur_lens[b] : s;
    cur = max(s, min(cur, a.k.max_pages << a.k.page_shift));
    const int ni = min(a.n_init, s), nl = min(a.n_local, s - ni);
    const int n_w = ni + nl + (cur - s);
    auto id_of = [&](int r) { return r < ni ? r : s - nl + (r - ni); };
    float q[G][8];
    const T *qb = (const T *)a.q + ((size_t)b * a.u.h + kv * G) * kD;
#pragma unroll
    for (int hh = 0; hh < G; ++hh) unpack(load_chunk(qb + (size_t)hh * kD, lane16), q[hh]);
    const T *K = (const T *)a.k.pages;
    const T *V = (const T *)a.v_pages;
    float m_run[G], l_run[G], acc[G][8];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) {
        m_run[hh] = -__builtin_huge_valf();
        l_run[hh] = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[hh][e] = 0.0f;
    }
    for (int r0 = bx * 64; r0 < n_w; r0 += kWinSplit * 64) {
        const int nr = min(64, n_w - r0);
        uint32_t row[4];
        Chunk<T> ck[4], cv[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int r = min(p * 16 + grp, nr - 1);
            row[p] = row_of(a.k.block_table, a.k.max_pages, a.k.page_shift, a.u.g, b, kv, id_of(r0 + r));
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            ck[p] = load_chunk(K + (size_t)row[p] * kD, lane16);
            cv[p] = load_chunk(V + (size_t)row[p] * kD, lane16);
        }
        __syncthreads();   // the previous run's s_z and s_ml have been read
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            float kx[8];
            unpack(ck[p], kx);
#pragma unroll
            for (int hh = 0; hh < G; ++hh) {
                float tot = group16_sum(lane_partial(q[hh], kx)) * a.scale;
                if (lane16 == hh) s_z[p * 16 + grp][hh] = tot;
            }
        }
        __syncthreads();
        if (tid < 64) {   // the run's maximum per head (one row per lane of the first wave)
#pragma unroll
            for (int hh = 0; hh < G; ++hh) {
                float mx = tid < nr ? s_z[tid][hh] : -__builtin_huge_valf();
#pragma unroll
                for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
                if (tid == 0) s_ml[hh] = mx;
            }
        }
        __syncthreads();
        float corr[G];
#pragma unroll
        for (int hh = 0; hh < G; ++hh) {
            const float m_new = fmaxf(m_run[hh], s_ml[hh]);   // the same in every thread
            corr[hh] = __expf(m_run[hh] - m_new);          // exp(-inf) = 0 on the first run
            m_run[hh] = m_new;
            l_run[hh] *= corr[hh];
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[hh][e] *= corr[hh];
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int r = p * 16 + grp;
            if (r < nr) {
                float vx[8];
                unpack(cv[p], vx);
#pragma unroll
                for (int hh = 0; hh < G; ++hh) {
                    const float pr = __expf(s_z[r][hh] - m_run[hh]);
                    if (lane16 == 0) l_run[hh] += pr;   // lane 0 of each group carries the group's share of l
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[hh][e] = __fmaf_rn(pr, vx[e], acc[hh][e]);
                }
            }
        }
    }
    // the 16 groups hold partial sums over their rows, all relative to the same running maximum:
    // first the four groups of a wave (lanes l, l+16, l+32, l+48), then the four waves
#pragma unroll
    for (int hh = 0; hh < G; ++hh) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float v = acc[hh][e];
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);
            acc[hh][e] = v;
        }
        float l = l_run[hh];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        l_run[hh] = l;
    }
    __syncthreads();
    const int wv = tid >> 6;
    if ((tid & 63) < 16) {
#pragma unroll
        for (int hh = 0; hh < G; ++hh) {
#pragma unroll
            for (int e = 0; e < 8; ++e) s_part[wv][hh][lane16 * 8 + e] = acc[hh][e];
        }
        if (lane16 == 0) {
#pragma unroll
            for (int hh = 0; hh < G; ++hh) s_z[wv][hh] = l_run[hh];
        }
    }
    __syncthreads();
    float *dst = a.win + ((size_t)ul * kWinSplit + bx) * G * (2 + kD);
    for (int i = tid; i < G * kD; i += 256) {
        const int hh = i >> 7, e = i & 127;
        dst[hh * (2 + kD) + 2 + e] = (s_part[0][hh][e] + s_part[1][hh][e]) + (s_part[2][hh][e] + s_part[3][hh][e]);
    }
    if (tid < G) {
        dst[tid * (2 + kD)] = m_run[tid];
        dst[tid * (2 + kD) + 1] = (s_z[0][tid] + s_z[1][tid]) + (s_z[2][tid] + s_z[3][tid]);
    }
}

template <typename T, int G> __global__ __launch_bounds__(256) void window_attn_kernel(WindowArgs a)
{
    int ul, bx;
    unit_block_of(a.by_xcd, ul, bx);
    window_attn_block<T, G>(a, bx, ul);
}

// ------------------------------------------------------------------------------
// Algorithm 2 lines 4-5 in one launch (decode).  A unit's bitmap of recalled ids is split over the
// unit's blocks; a block turns its part into ascending ids 64 words at a time (one byte per thread,
// positions by a block scan), writes them and their physical rows to their ranks of the recalled
// list, and scores the rows like score_kernel: z[rank][G], running maximum per head.
// Two ways to split, chosen by the host:
//   by id range -- block x owns words [x wpb, (x + 1) wpb), wpb <= 64, and counts the ids in the words
//     before its own (coalesced 4-byte loads, no scan).  The cheapest prologue; recalled keys cluster,
//     so some blocks get several times the rows of others, which does not matter while every CU has
//     many blocks' worth of rows to stream.
//   by rank -- block x takes ranks [x q, (x + 1) q), q = ceil(L / blocks): every block counts the whole
//     bitmap (a contiguous stretch of words per thread, one block scan), which gives L, and the threads
//     whose stretches hold the block's ranks leave their words with the ids before each in shared memory.  Every block
//     then has the same number of rows: for small batches, where a block's rows are one or two round trips to memory and the
//     slowest block is the launch.
// Either way all that the prologue reads -- words, the block-table entries of the block's pages, the queries -- is
// requested at once, one round trip before the rows (under load a dependent trip takes 2-4 us); ids and rows are written
// behind the scoring, off that chain.
// The block that sees the unit's last word (by id) or block 0 (by rank) also writes L.
// grid (nbx [+ kWinSplit], units), 256 threads; by id nbx >= W_max / 64, by rank nbx >= l_stride / kRecallCap.  Dynamic shared
// memory: RecallLds.
// ------------------------------------------------------------------------------
constexpr int kRecallWpb = 64;     // by id range: at most 2048 ids per block
constexpr int kRecallCap = 2048;   // ids per block at most
// Rows in flight per 16-lane group.  By id range in bf16 eight: four blocks a CU with groups up to four.  By rank in bf16 twelve, which take
// the 125 to 170 rows of a block of the 32K step in one trip, not two (step 33.9 -> 32.9 us with two blocks a CU; sixteen: the same).  In fp32
// four: eight are 169 to 220 registers, with groups of two and more two blocks a CU, where the grid often has three and more, and no faster
// where it has two (by rank, 24 units of 16K, groups of two 42.2 -> 36.5 us a step, of four 47.2 -> 41.3; eight units of 32K, groups of four 34.6 -> 34.1;
// by id range, sixteen sequences of 8K to 32K on eight KV heads, groups of four, the launch 115.7 -> 109.9, on four, of eight 68.8 -> 65.3).
template <typename T> constexpr int kRankRows = sizeof(T) == 2 ? 12 : 4;
template <typename T> constexpr int kRangeRows = sizeof(T) == 2 ? 8 : 4;
// In bf16 by rank (recall_score_kernel's SHORT) four too where a block has 64 ids at most, or a CU more than two blocks: the loop's
// requests have no branches, and twelve where a block has rows for two or four cost their issue and their answers, and 98 to 163
// registers, i.e. four or three blocks a CU (in a launch with a resident window its blocks' registers set that).  Steps: sixteen units of 4K, groups of four 23.16 -> 23.05 us; 40 of 8K 36.0 -> 33.5, 128 of 4K 49.7
// -> 43.8, 32 of 16K, groups of eight 48.2 -> 45.0.
constexpr int kShortRows = 4;
constexpr int kRecallWords = 4096; // by rank: bitmap words (contexts up to 128K) that the prologue takes in one trip

// words of shared memory: ids and rows of the block, block-table entries, by rank the bitmap and the ids before each word
struct RecallLds {
    int pages, words;
    __host__ __device__ int total() const { return 2 * kRecallCap + pages + 2 * words; }
};

struct RecallScoreArgs {
    Units u;
    const void *q;            // [batch][h][128]
    Paged k;
    const int32_t *ctx_lens;
    const uint32_t *gbits;    // [units][bitmap_words]
    int bitmap_words, l_stride;
    int32_t *cand;            // [units][l_stride] recalled ids, ascending
    uint32_t *crow;           // [units][l_stride] their physical rows
    int32_t *ncand;           // [units] L
    int32_t *out_ncand;       // optional copy for the caller
    float *z;                 // [units][l_stride][G]
    uint32_t *m_key;          // [units][kMaxStride] ordered-key running max per head (atomicMax)
    uint4 *clear;             // optional: [units][clear_n] words that the launches behind expect to find zero, cleared here
    int clear_n;
    float scale;
    int by_xcd;               // blocks -> (unit, block of the unit) by unit_block_of
    RecallLds lds;            // by rank: words = 0 where the bitmap is read again instead, pages = 0 where the pages do not fit
    int nbx;                  // blocks per unit that score; with WIN blocks nbx .. nbx + kWinSplit - 1 take the resident window
    WindowArgs win;
};

// RANK: how the bitmap is split over a unit's blocks.  STREAM: the keys of all sequences exceed what the memory-side cache holds, and are
// loaded non-temporal.  SHORT: by rank, with kShortRows
template <typename T, int G, bool WIN, bool RANK, bool STREAM, bool SHORT = false>
__global__ __launch_bounds__(256) void recall_score_kernel(RecallScoreArgs a)
{
    constexpr int R = SHORT ? kShortRows : RANK ? kRankRows<T> : kRangeRows<T>, TILE = 16 * R;
    extern __shared__ __align__(16) uint32_t smem[];
    uint32_t *s_ids = smem, *s_rows = smem + kRecallCap;     // ids of this block's ranks, their rows
    int32_t *s_page = (int32_t *)(smem + 2 * kRecallCap);    // block-table entries
    uint32_t *s_word = (uint32_t *)s_page + a.lds.pages, *s_before = s_word + a.lds.words;
    __shared__ uint32_t s_tmp[8];
    __shared__ uint32_t s_edge[3];                // first word, ids before it, last word
    __shared__ uint32_t s_max[G];
    int ul, bx;
    unit_block_of(a.by_xcd, ul, bx);
    if constexpr (WIN) {
        if (bx >= a.nbx) {   // Algorithm 2 lines 10-11 beside lines 4-5
            window_attn_block<T, G>(a.win, bx - a.nbx, ul);
            return;
        }
    }
    const int b = ul / a.u.g, kv = ul - b * a.u.g;
    const int tid = threadIdx.x, lane16 = tid & 15, grp = tid >> 4;
    const int ln = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    CTKVR_STAMP_BLK(6);
    const uint32_t *gb = a.gbits + (size_t)ul * a.bitmap_words;
    const int32_t *bt_row = a.k.block_table + (size_t)b * a.k.max_pages;
    const int pmask = (1 << a.k.page_shift) - 1;
    if (tid < G) s_max[tid] = 0u;
    // The ids of byte `part` of word w, the first of them at rank rk: those of ranks [r0, r1) with their rows into shared
    // memory.  page_of(p): the block-table entry of page p
    auto expand = [&](uint32_t word, int w, int part, uint32_t rk, uint32_t r0, uint32_t r1, auto page_of) __attribute__((always_inline)) {
        uint32_t m = (word >> (part << 3)) & 0xffu;
        if (!m) return;
        const int id0 = (w << 5) + (part << 3);
        int page = a.k.page_shift >= 3 ? page_of(id0 >> a.k.page_shift) : 0;   // one page holds all eight
        do {
            const int t = id0 + __ffs((int)m) - 1;
            m &= m - 1u;
            if (rk >= r0 && rk < r1) {
                if (a.k.page_shift < 3) page = page_of(t >> a.k.page_shift);
                s_ids[rk - r0] = (uint32_t)t;
                s_rows[rk - r0] = (uint32_t)((page * a.u.g + kv) << a.k.page_shift) + (uint32_t)(t & pmask);
            }
            ++rk;
        } while (m);
    };
    auto clear = [&]() {
        for (int w = bx * 256 + tid; w < a.clear_n; w += a.nbx * 256) a.clear[(size_t)ul * a.clear_n + w] = make_uint4(0u, 0u, 0u, 0u);
    };
    uint32_t r0, r1;   // the block's ranks
    if (RANK && a.lds.words) {
        // thread t counts words [t wpt, (t + 1) wpt), wpt a multiple of four, and keeps them (those from the sequence's end up to
        // the row's are zero)
        constexpr int NV = kRecallWords / 1024, NP = kRecallWords / 256;
        const int wpt = a.lds.words >> 8, w0 = tid * wpt;
        uint4 v[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if (4 * i < wpt) v[i] = *reinterpret_cast<const uint4 *>(gb + min(w0 + 4 * i, a.bitmap_words - 4));   // uniform
        int32_t pg[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i)
            if (i * 256 < a.lds.pages) pg[i] = bt_row[min(i * 256 + tid, a.k.max_pages - 1)];   // uniform
        clear();
        uint32_t cnt = 0;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (4 * i >= wpt || w0 + 4 * i >= a.bitmap_words) v[i] = make_uint4(0u, 0u, 0u, 0u);
            cnt += (uint32_t)(__popc(v[i].x) + __popc(v[i].y) + __popc(v[i].z) + __popc(v[i].w));
        }
        uint32_t L;
        const uint32_t pre = block_excl_scan<256>(cnt, s_tmp, &L);   // barriers inside
        if (bx == 0 && tid == 0) {
            a.ncand[ul] = (int32_t)L;
            if (a.out_ncand) a.out_ncand[ul] = (int32_t)L;
        }
        const uint32_t qn = (L + (uint32_t)a.nbx - 1) / (uint32_t)a.nbx;
        r0 = bx * qn;
        if (r0 >= L) return;
        r1 = min(L, r0 + qn);
        // the threads that hold ranks of the block leave their words and the ids before each (also those without ids between two
        // with some: pre lies strictly between r0 and r1 there)
        if (pre < r1 && pre + cnt > r0) {
            uint32_t p = pre;
#pragma unroll
            for (int i = 0; i < NV; ++i)
                if (4 * i < wpt) {   // uniform
                    const uint32_t p1 = p + (uint32_t)__popc(v[i].x), p2 = p1 + (uint32_t)__popc(v[i].y), p3 = p2 + (uint32_t)__popc(v[i].z);
                    *reinterpret_cast<uint4 *>(s_word + w0 + 4 * i) = v[i];
                    *reinterpret_cast<uint4 *>(s_before + w0 + 4 * i) = make_uint4(p, p1, p2, p3);
                    p = p3 + (uint32_t)__popc(v[i].w);
                }
            if (pre <= r0) s_edge[0] = (uint32_t)w0;
            if (pre + cnt >= r1) s_edge[2] = (uint32_t)(w0 + wpt);
        }
#pragma unroll
        for (int i = 0; i < NP; ++i)
            if (i * 256 < a.lds.pages) s_page[i * 256 + tid] = pg[i];
        __syncthreads();
        CTKVR_STAMP_BLK(7);
        const int wb = (int)s_edge[2], part = tid & 3;
        for (int w = (int)s_edge[0] + (tid >> 2); w < wb; w += 64) {
            const uint32_t word = s_word[w], rk = s_before[w] + (uint32_t)__popc(word & ((1u << (part << 3)) - 1u));
            if (a.lds.pages)
                expand(word, w, part, rk, r0, r1, [&](int p) { return s_page[p]; });
            else
                expand(word, w, part, rk, r0, r1, [&](int p) { return bt_row[p]; });
        }
    } else if (RANK) {
        // longer contexts: two passes over the words, the second over those between the block's first and last rank
        const int wpt = ((((a.bitmap_words + 255) >> 8) + 3) >> 2) << 2;
        const int w0 = tid * wpt, w1 = min(w0 + wpt, a.bitmap_words);
        clear();
        uint32_t cnt = 0;
#pragma unroll 4
        for (int w = w0; w < w1; w += 4) {
            const uint4 x = *reinterpret_cast<const uint4 *>(gb + w);
            cnt += (uint32_t)(__popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w));
        }
        uint32_t L;
        const uint32_t pre = block_excl_scan<256>(cnt, s_tmp, &L);   // barriers inside
        if (bx == 0 && tid == 0) {
            a.ncand[ul] = (int32_t)L;
            if (a.out_ncand) a.out_ncand[ul] = (int32_t)L;
        }
        const uint32_t qn = (L + (uint32_t)a.nbx - 1) / (uint32_t)a.nbx;
        r0 = bx * qn;
        if (r0 >= L) return;
        r1 = min(L, r0 + qn);
        // the threads whose stretches hold ranks r0 and r1 - 1 walk their words to the one that holds it
        if (cnt && pre <= r0 && r0 < pre + cnt) {
            uint32_t p = pre;
            for (int w = w0; w < w1; ++w) {
                const uint32_t c = (uint32_t)__popc(gb[w]);
                if (r0 < p + c) {
                    s_edge[0] = (uint32_t)w;
                    s_edge[1] = p;
                    break;
                }
                p += c;
            }
        }
        if (cnt && pre < r1 && r1 <= pre + cnt) {
            uint32_t p = pre;
            for (int w = w0; w < w1; ++w) {
                p += (uint32_t)__popc(gb[w]);
                if (r1 <= p) {
                    s_edge[2] = (uint32_t)w;
                    break;
                }
            }
        }
        __syncthreads();
        const int wa = (int)s_edge[0], wb = (int)s_edge[2], part = tid & 3;
        uint32_t rank0 = s_edge[1];   // ids before the pass's first word
        for (int wp = wa; wp <= wb; wp += 64) {
            const int w = wp + (tid >> 2);
            const uint32_t word = w <= wb ? gb[w] : 0u;
            uint32_t n_pass;
            const uint32_t rk = rank0 + block_excl_scan<256>((uint32_t)__popc((word >> (part << 3)) & 0xffu), s_tmp, &n_pass);
            expand(word, w, part, rk, r0, r1, [&](int p) { return bt_row[p]; });
            rank0 += n_pass;
        }
    } else {
        // the unit's own words split evenly over the blocks of its row (a short sequence of a ragged
        // batch still uses all of them)
        const int W = (a.ctx_lens[b] + 31) >> 5;
        const int wpb = min(kRecallWpb, (W + a.nbx - 1) / a.nbx);
        const int w_beg = bx * wpb, w_end = min(W, w_beg + wpb);
        clear();
        if (w_beg >= W) return;
        const int mine = w_beg + (tid >> 2), part = tid & 3;
        uint32_t word = gb[min(mine, W - 1)];
        const int page0 = (w_beg << 5) >> a.k.page_shift;
        const int npages = min((((w_end << 5) - 1) >> a.k.page_shift) - page0 + 1, a.k.max_pages - page0);
        const bool lds_pages = npages <= a.lds.pages;
        int32_t pg = 0;
        if (lds_pages) pg = bt_row[page0 + min(tid, npages - 1)];
        uint32_t before = 0;
        for (int w8 = 0; w8 < w_beg; w8 += 8 * 256) {   // eight words a thread requested together
            uint32_t x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = gb[min(w8 + u * 256 + tid, w_beg - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) before += w8 + u * 256 + tid < w_beg ? (uint32_t)__popc(x[u]) : 0u;
        }
        if (mine >= w_end) word = 0u;
        // one barrier for the ids before the block's words and the scan over its own
        const uint32_t c = (uint32_t)__popc((word >> (part << 3)) & 0xffu), inc = wave_incl_scan(c);
        before = wave_sum_uniform(before);
        if (ln == 63) {
            s_tmp[wv] = inc;
            s_tmp[4 + wv] = before;
        }
        if (lds_pages && tid < npages) s_page[tid] = pg;
        __syncthreads();
        r0 = s_tmp[4] + s_tmp[5] + s_tmp[6] + s_tmp[7];
        const uint32_t t0 = s_tmp[0], t1 = s_tmp[1], t2 = s_tmp[2], t3 = s_tmp[3];
        r1 = r0 + t0 + t1 + t2 + t3;
        CTKVR_STAMP_BLK(7);
        if (w_end == W && tid == 0) {
            a.ncand[ul] = (int32_t)r1;
            if (a.out_ncand) a.out_ncand[ul] = (int32_t)r1;
        }
        if (r1 == r0) return;
        const uint32_t rk = r0 + (wv > 0 ? t0 : 0u) + (wv > 1 ? t1 : 0u) + (wv > 2 ? t2 : 0u) + inc - c;
        if (lds_pages)
            expand(word, mine, part, rk, r0, r1, [&](int p) { return s_page[p - page0]; });
        else
            expand(word, mine, part, rk, r0, r1, [&](int p) { return bt_row[p]; });
    }
    const uint32_t n_blk = r1 - r0, base = r0;
    __syncthreads();
    CTKVR_STAMP_BLK(2);
    const T *K = (const T *)a.k.pages;
    float *zb = a.z + ((size_t)ul * a.l_stride + base) * G;
    // the queries are requested with the first rows (cached, they arrive well before the rows do)
    float q[G][8];
    const T *qb = (const T *)a.q + ((size_t)b * a.u.h + kv * G) * kD;
#pragma unroll
    for (int hh = 0; hh < G; ++hh) unpack(load_chunk(qb + (size_t)hh * kD, lane16), q[hh]);
    // a lane keeps the score of one head, and that head's running maximum
    float mxl = -__builtin_huge_valf();
    const int myh = head_of_lane<G>(lane16);
    constexpr int SUB = G == 8 ? 2 : 4;      // lanes of a head that stand for a round of rows each when scores are written
    const int sub = lane16 & (SUB - 1);
    static_assert(R % SUB == 0, "rounds are written SUB at a time");
    const int last = (int)n_blk - 1;
    Chunk<T> ck[R];
    // (beyond the block's rows its own last one, whose line is at hand: row 0 of the pool for all blocks cost fp32 0.4 to 1.6 % of a step, 128K x 4
    // 0.2 to 0.3)
    auto row_at = [&](int i) __attribute__((always_inline)) { return s_rows[min(i, last)]; };
    auto request = [&](int r, uint32_t row) __attribute__((always_inline)) {
        const T *p = K + (size_t)row * kD;
        ck[r] = STREAM ? load_chunk_nt(p, lane16) : load_chunk(p, lane16);
    };
    auto score = [&](const float(&kx)[8]) __attribute__((always_inline)) {
        float part[G];
#pragma unroll
        for (int hh = 0; hh < G; ++hh) part[hh] = lane_partial(q[hh], kx);
        return group16_sums<G>(part, lane16) * a.scale;
    };
    auto keep = [&](float z) __attribute__((always_inline)) { asm("v_max_f32 %0, %0, %1" : "+v"(mxl) : "v"(z)); };
    {
        uint32_t row[R];
#pragma unroll
        for (int r = 0; r < R; ++r) row[r] = row_at(r * 16 + grp);
#pragma unroll
        for (int r = 0; r < R; ++r) request(r, row[r]);
    }
    // Each round of rows is requested again for the next tile as soon as it is unpacked, so that a wave always has all its R rounds but
    // one in flight; requested a tile at a time, and rounds without rows left out by branches, the first round was waited for
    // together with most others.  (No branch between these requests either: what may not have been requested is waited for as well.)
    // With that and 60 vector instructions a round where there were 80: steps of 128K x 4 111.8 -> 104.8 us, sixteen of 8K to 64K
    // 122.3 -> 114.5, 32K 31.9 -> 31.2.
    float *zl = zb + (size_t)(sub * 16 + grp) * G + myh;
    int t0 = 0;
#pragma unroll 1
    for (; t0 + TILE < (int)n_blk; t0 += TILE) {
        uint32_t row[R];
#pragma unroll
        for (int r = 0; r < R; ++r) row[r] = row_at(t0 + TILE + r * 16 + grp);
#pragma unroll
        for (int r0 = 0; r0 < R; r0 += SUB) {
            float zw = 0.0f;
#pragma unroll
            for (int r = r0; r < r0 + SUB; ++r) {
                float kx[8];
                unpack(ck[r], kx);
                request(r, row[r]);
                __builtin_amdgcn_sched_barrier(0);   // (moved together, the rounds would all be waited for first)
                const float z = score(kx);
                keep(z);
                zw = r == r0 || sub == r - r0 ? z : zw;
                __builtin_amdgcn_sched_barrier(0);
            }
            zl[(size_t)(t0 + r0 * 16) * G] = zw;
        }
    }
#pragma unroll
    for (int r0 = 0; r0 < R; r0 += SUB) {
        if (t0 + r0 * 16 > last) break;   // uniform
        float zw = 0.0f;
#pragma unroll
        for (int r = r0; r < r0 + SUB; ++r) {
            if (t0 + r * 16 > last) break;   // uniform
            float kx[8];
            unpack(ck[r], kx);
            const float z = score(kx);
            keep(t0 + r * 16 + grp <= last ? z : -__builtin_huge_valf());
            zw = r == r0 || sub == r - r0 ? z : zw;
        }
        if (t0 + (r0 + sub) * 16 + grp <= last) zl[(size_t)(t0 + r0 * 16) * G] = zw;
    }
    {
        float v = mxl;
        v = __builtin_amdgcn_fmed3f(v, __shfl_xor(v, 16), __builtin_huge_valf());
        v = __builtin_amdgcn_fmed3f(v, __shfl_xor(v, 32), __builtin_huge_valf());
        if (ln < 16 && (G == 1 ? lane16 == 0 : G == 2 ? (lane16 & 11) == 0 : sub == 0)) atomicMax(&s_max[myh], ordered_key(v));
    }
    int32_t *cd = a.cand + (size_t)ul * a.l_stride + base;
    uint32_t *rw = a.crow + (size_t)ul * a.l_stride + base;
    for (uint32_t i = tid; i < n_blk; i += 256) {
        cd[i] = (int32_t)s_ids[i];
        rw[i] = s_rows[i];
    }
    __syncthreads();
    if (tid < G) atomicMax(&a.m_key[ul * kMaxStride + tid], s_max[tid]);
    CTKVR_STAMP_BLK(3);
}

// ------------------------------------------------------------------------------
// Algorithm 1 line 2 on the matrix cores (bf16 only): the same z = (c_{h,j} . k_t) *
// scale as score_kernel in build mode, but the 128-term dot is a chain of eight
// v_mfma_f32_32x32x16_bf16.  A block owns 8/G sub-tiles of 32 centroids of one
// (sequence, KV head) for all G heads: eight (head, sub-tile) items, their A fragments resident in
// registers, four to a wave, and walks a range of keys 64 at a time, one wave of each item on either
// half (B fragments are 16-byte pieces of the paged key rows, staged through shared memory).
// A wave has all heads of its centroids, so a ranking key is finished in its registers and the block meets only for
// the key rows; one fragment read feeds four matrix instructions.  (Two items per wave and the head pairs
// meeting in shared memory, 128K x 8 KV heads x 2048 centroids, half of the heads per launch: candidate pass 1.69 ms,
// 0.65 PFLOP/s, now 1.11 ms, 0.99 PFLOP/s; statistics 1.16 -> 1.11 ms, bound by the exponentials.)
// grid (t_splits, tiles), MfmaShape::NT threads.
// The scores differ from the fixed arithmetic in the accumulation order inside the MFMA and
// the softmax denominators in how they are summed; on inputs whose dot products are exact in
// fp32 only the latter is left.
// ------------------------------------------------------------------------------
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

constexpr int kVmcnt0 = 0x0f70;   // s_waitcnt: all vector memory, nothing else

struct MfmaScoreArgs {
    int g, G, h, c_max;
    int bk0;                   // first (sequence, KV head) pair of this chunk
    int tiles_per_bk;          // ceil(c_max / (32 * 8/G))
    int t_splits;
    const int32_t *n_cent, *ctx_lens;
    const bf16_t *centroids;   // [batch][h][c_max][128]
    Paged k;
    int l_stride;              // s_max
    float2 *part;              // [chunk units][G][t_splits] (maximum of z log2(e), sum of 2^(z log2(e) - maximum)) over a block's keys
    float *off;                // [chunk units][G] -(m + log S) over all keys (mfma_merge_kernel)
    uint32_t *kbuf;            // KEY: [chunk units][l_stride] ranking keys; SAMPLE: [chunk units][sample_stride]
    int n_init, n_local;       // keys of the resident window get the lowest ranking key
    float scale;
    int step_stride;           // SAMPLE: every step_stride-th step of 32 keys is taken (1 in the other passes)
    int sample_stride;         // SAMPLE: keys per unit in kbuf
    const uint32_t *tau;       // PICK: [chunk units] keys at or above it are candidates
    uint2 *cand;               // PICK: [chunk units][t_splits][seg_cap] (key, id): block x of a tile fills segment x of its units
    uint32_t *seg_cnt;         // PICK: [chunk units][t_splits] candidates of the segment (may exceed seg_cap: the excess is not stored)
    int seg_cap;
};

// The scores are never stored: the contraction is repeated in two passes over the same tiles, each
// with its own epilogue -- MFMA_STAT: per (centroid, head) the running maximum m of the scores and the
// running sum of exp(z - m), rescaled whenever the maximum moves, in fp32 with the hardware
// exponential (this route's lists are compared with the fixed arithmetic inside an error band anyway,
// and the band has room for a denominator that is a few 1e-5 off); one (m, sum) pair per block, merged
// in block order by mfma_merge_kernel.  MFMA_KEY: ranking keys max_h ((z - m_h) - log S_h), written as
// ordered uint32 (4 bytes per (centroid, key) instead of 4 G bytes of scores read twice).
// Writing, and twice re-reading, a key for every (centroid, key) pair is most of that route's time, and only
// rho of a unit's s keys are wanted.  MFMA_SAMPLE computes the keys of every step_stride-th step only (a
// systematic sample of the positions) into a small buffer, from which a threshold tau per unit is taken
// (a sample rank chosen so that about 2 rho keys of the unit lie at or above it); MFMA_PICK then computes all
// keys again and keeps the (key, id) pairs at or above tau -- a few thousand per unit -- from which the rho
// largest are selected exactly.  Should a unit end with fewer than rho candidates, or more than fit, its
// (sequence, KV head) pair is redone by the KEY route: the result never depends on the sample.
enum { MFMA_STAT = 0, MFMA_KEY = 2, MFMA_SAMPLE = 3, MFMA_PICK = 4 };

// A wave's share of a block: ITEMS (head, 32-centroid sub-tile) pairs with their fragments resident, against one of
// the two 32-key halves of a step.  The key passes give a wave all heads of its sub-tiles, so a ranking key is
// complete in the wave's own registers; with eight heads that is 256 registers of fragments, one wave per SIMD.
template <int G, int MODE> struct MfmaShape {
    static constexpr int CT = 32 * (8 / G);                            // centroids of a block
    static constexpr int ITEMS = MODE != MFMA_STAT && G == 8 ? 8 : 4;
    static constexpr int WC = 8 / ITEMS;                               // waves side by side over the items
    static constexpr int NT = 2 * WC * 64;
    static constexpr int kWaves = ITEMS == 8 ? 1 : 2;                  // per SIMD
};

template <int G, int MODE>
__global__ __launch_bounds__((MfmaShape<G, MODE>::NT), (MfmaShape<G, MODE>::kWaves)) void mfma_score_kernel(MfmaScoreArgs a)
{
    using S = MfmaShape<G, MODE>;
    constexpr int CT = S::CT, ITEMS = S::ITEMS, NT = S::NT;
    constexpr bool KEYS = MODE != MFMA_STAT;       // the passes that form ranking keys
    constexpr int SUB = ITEMS >= G ? ITEMS / G : 1;   // sub-tiles of a wave (key passes: each with all G heads)
    // PICK: the tile's thresholds and how many candidates this block has found for each of its centroids.  A block
    // owns a segment of every unit's candidate list, so positions are handed out by shared-memory counters: no
    // atomic on device memory (on this part those are served beyond the XCD's cache, a round trip each).
    __shared__ uint32_t s_cnt[MODE == MFMA_PICK ? CT : 1];
    // key passes: 32 x 32 ranking keys of a wave on their way out, [centroid][key]; a wave's own, so no barrier.  A
    // lane's four consecutive keys are one 16-byte access, 36-word rows spread them over the banks.
    constexpr int ZS = 36;
    __shared__ __align__(16) float s_z[KEYS ? (NT / 64) * 32 * ZS : 4];
    __shared__ float2 s_stat[KEYS ? 1 : S::WC * ITEMS * 32];
    constexpr int ROWB = 272;   // bytes per staged key row (256 + padding: fragment reads spread over the banks)
    __shared__ __align__(16) unsigned char s_k[2][64 * ROWB];
    const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
    const int col = ln & 31, half = ln >> 5;
    const int wc = wv >> 1, sub = wv & 1;          // the wave's items, its half of a step's keys
    const int bkl = blockIdx.y / a.tiles_per_bk, jt = blockIdx.y - bkl * a.tiles_per_bk;
    const int bk = a.bk0 + bkl;
    const int b = bk / a.g, kv = bk - b * a.g;
    const int C = a.n_cent[b], s = a.ctx_lens[b];
    const int j0 = jt * CT;
    if (j0 >= C) return;
    const int tper = (((s + a.t_splits - 1) / a.t_splits) + 31) & ~31;
    // a step is two groups of 32 keys, ST apart.  SAMPLE: the groups taken are those that start at a multiple of ST; a
    // block starts at the first one in its range
    const int ST = MODE == MFMA_SAMPLE ? 32 * a.step_stride : 32;
    const int tbeg = MODE == MFMA_SAMPLE ? ((int)(blockIdx.x * tper) + ST - 1) / ST * ST : (int)(blockIdx.x * tper);
    const int tend = min(s, (int)(blockIdx.x * tper) + tper);
    if (tbeg >= tend) return;
    if constexpr (MODE == MFMA_PICK) {
        for (int c = tid; c < CT; c += NT) s_cnt[c] = 0u;
    }
    // The matrix instruction is issued with the keys as its row operand and the centroids as its
    // column operand: a lane then holds ONE centroid (column `col` of its sub-tile) against 16
    // keys (rows 8 (r / 4) + 4 half + r % 4), and that centroid's statistics are single registers.
    // Item q of the wave: head q % G of sub-tile wc * SUB + q / G (G = 8 with four items: head 4 wc + q of the one).
    auto head_of = [&](int q) { return ITEMS >= G ? q % G : wc * ITEMS + q; };
    auto tile_of = [&](int q) { return ITEMS >= G ? wc * SUB + q / G : 0; };
    bf16x8_t cfrag[ITEMS][8];              // the centroid fragments, resident
    float mx[ITEMS];                       // STAT: running maximum (base two)
    float lsv[ITEMS];                      // STAT: running sum of 2^(z log2(e) - mx)
    float off[ITEMS];                      // key passes: -(m + log S), so that a key is one fused multiply-add per score
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        const int j = min(j0 + tile_of(q) * 32 + col, C - 1);   // columns beyond C repeat centroid C-1 and are dropped at the end
        const bf16_t *row = a.centroids + (((size_t)b * a.h + kv * G + head_of(q)) * a.c_max + j) * kD;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) cfrag[q][ks] = *reinterpret_cast<const bf16x8_t *>(row + ks * 16 + 8 * half);
        mx[q] = -__builtin_huge_valf();
        lsv[q] = off[q] = 0.0f;
        if constexpr (KEYS) off[q] = a.off[((size_t)bkl * a.c_max + j) * G + head_of(q)];
    }
    float tau[SUB];
    uint2 *seg[SUB];   // PICK: the block's segment of the lane's centroid
    if constexpr (MODE == MFMA_PICK) {
#pragma unroll
        for (int m = 0; m < SUB; ++m) {
            const size_t unit = (size_t)bkl * a.c_max + min(j0 + tile_of(m * G) * 32 + col, C - 1);
            const uint32_t tk = a.tau[unit];
            // 0: no threshold, every key is a candidate.  A column beyond C keeps nothing
            tau[m] = tk ? ordered_value(tk) : -__builtin_huge_valf();
            seg[m] = a.cand + (unit * a.t_splits + blockIdx.x) * a.seg_cap;
        }
    }
    const float sc2 = a.scale * 1.44269504088896341f;   // scores in base two (statistics pass)
    // The 64 key rows of a step (16 KB) go through shared memory once for all waves, in two
    // buffers; a step's rows are requested one step ahead (a step is 2048 cycles of matrix work per SIMD with two
    // waves on it) and their block-table entries two.  Rows beyond the sequence are clamped to its last key.
    const bf16_t *K = (const bf16_t *)a.k.pages;
    constexpr int TPR = NT / 64, NU = 16 / TPR;   // threads per row, 16-byte pieces per thread
    const int srow = tid / TPR, spart = tid % TPR;
    const int skey = (srow >> 5) * ST + (srow & 31);
    const int32_t *bt_row = a.k.block_table + (size_t)b * a.k.max_pages;
    auto page_at = [&](int t0) { return bt_row[min(t0 + skey, s - 1) >> a.k.page_shift]; };
    auto row_from = [&](int page, int t0) {
        return (uint32_t)((page * a.g + kv) << a.k.page_shift) + (uint32_t)(min(t0 + skey, s - 1) & ((1 << a.k.page_shift) - 1));
    };
    auto piece_of = [&](uint32_t row, int u) { return (reinterpret_cast<const uint4 *>(K + (size_t)row * kD) + spart)[u * TPR]; };
    auto put = [&](const uint4 &x, int u, int buf) {
        *reinterpret_cast<uint4 *>(&s_k[buf][srow * ROWB + (u * TPR + spart) * 16]) = x;
    };
    // the wave's 32 ranking keys of a sub-tile's 32 centroids, keys tb .. tb + 31
    float *const zw = &s_z[KEYS ? wv * (32 * ZS) : 0];
    auto keys_out = [&](const bool tail, int tb, int m, const float (&best)[16]) __attribute__((always_inline)) {
        const int jt0 = j0 + tile_of(m * G) * 32;
        if constexpr (MODE == MFMA_PICK) {
            // Few keys pass (a few per cent): a lane's verdicts as a mask, one counter bump for all of them, then as
            // many rounds as the fullest lane has candidates (about three); the keys are picked out of shared memory
            // because registers have no run-time index.  Compared as floats: the same verdict as on the ordered images
            // except that -0 passes a threshold of +0, i.e. at most a candidate too many.
            uint32_t msk = 0;
            const bool inner = !tail && tb >= a.n_init && tb + 32 <= s - a.n_local && jt0 + 32 <= C;
            if (inner) {   // the whole group lies inside the block's range and outside the window, every centroid is real
#pragma unroll
                for (int r = 0; r < 16; ++r) msk |= (uint32_t)(best[r] >= tau[m]) << r;
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int t = tb + 8 * (r >> 2) + 4 * half + (r & 3);
                    const bool in = t < tend && t >= a.n_init && t < s - a.n_local && (jt0 + col) < C;
                    msk |= (uint32_t)(in && best[r] >= tau[m]) << r;
                }
            }
            float *const mine = zw + col * ZS + 4 * half;
#pragma unroll
            for (int rq = 0; rq < 4; ++rq)
                *reinterpret_cast<float4 *>(mine + 8 * rq) = make_float4(best[4 * rq], best[4 * rq + 1], best[4 * rq + 2], best[4 * rq + 3]);
            if (msk) {
                uint32_t at = atomicAdd(&s_cnt[tile_of(m * G) * 32 + col], (uint32_t)__popc(msk));
                do {
                    const int r = __ffs(msk) - 1, k = 2 * (r & 12) + (r & 3);
                    msk &= msk - 1u;
                    if (at < (uint32_t)a.seg_cap) seg[m][at] = make_uint2(ordered_key(mine[k]), (uint32_t)(tb + 4 * half + k));
                    ++at;
                } while (msk);
            }
        } else {
            // through the wave's shared memory so that eight lanes store 128 contiguous bytes of a unit's keys, 16 each
            // where the key rows allow it (whole group in range, row length a multiple of four)
            float *const mine = zw + col * ZS + 4 * half;
#pragma unroll
            for (int rq = 0; rq < 4; ++rq)
                *reinterpret_cast<float4 *>(mine + 8 * rq) = make_float4(best[4 * rq], best[4 * rq + 1], best[4 * rq + 2], best[4 * rq + 3]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const bool wide = !tail && ((MODE == MFMA_SAMPLE ? a.sample_stride : a.l_stride) & 3) == 0;
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int n4 = (ln & 7) * 4, jl = it * 8 + (ln >> 3);
                const float4 v = *reinterpret_cast<const float4 *>(&zw[jl * ZS + n4]);
                const int t = tb + n4;
                uint32_t ok[4] = {ordered_key(v.x), ordered_key(v.y), ordered_key(v.z), ordered_key(v.w)};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if ((t + e) < a.n_init || (t + e) >= s - a.n_local) ok[e] = 0x007fffffu;   // the image of -inf
                if (jt0 + jl < C && tb < tend) {
                    const size_t unit = (size_t)bkl * a.c_max + jt0 + jl;
                    uint32_t *dst = MODE == MFMA_SAMPLE ? a.kbuf + unit * a.sample_stride + (tb / ST) * 32 + n4
                                                        : a.kbuf + unit * a.l_stride + t;
                    if (wide) {
                        // plain stores: the keys of a 20K build (200 MB) then wait for their reader in the memory-side cache (480 ->
                        // 461 us against non-temporal ones); where they do not fit (0.64 GB) there is no difference
                        *reinterpret_cast<uint4 *>(dst) = make_uint4(ok[0], ok[1], ok[2], ok[3]);
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if ((t + e) < tend) dst[e] = ok[e];
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();   // read before the next sub-tile's keys overwrite it (a wave's accesses are served in order)
        }
    };
    // tail: a step whose keys may reach beyond the block's range (a literal at every call).  Such
    // keys are real keys of the sequence, repeated: harmless for a maximum, left out of a sum,
    // not written as ranking keys.
    auto compute = [&](const bool tail, int buf, int tb) __attribute__((always_inline)) {
        const unsigned char *kr = &s_k[buf][(sub * 32 + col) * ROWB + half * 16];
        // four items at a time: independent back-to-back matrix instructions
        float best[16];
#pragma unroll
        for (int q0 = 0; q0 < ITEMS; q0 += 4) {
            f32x16_t acc[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[q][r] = 0.0f;
            bf16x8_t kf[2];
            kf[0] = *reinterpret_cast<const bf16x8_t *>(kr);
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                if (ks < 7) kf[(ks + 1) & 1] = *reinterpret_cast<const bf16x8_t *>(kr + (ks + 1) * 32);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks & 1], cfrag[q0 + q][ks], acc[q], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);   // the next fragment is requested before these products, not behind them
            }
            if constexpr (MODE == MFMA_STAT) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    // the step's maximum first (repeated keys of a tail are real keys: harmless), then its sixteen
                    // terms relative to the new running maximum, summed as a tree, and the old sum rescaled
                    // (in base two: the scores' maximum as fl(max acc * sc2), monotone since sc2 > 0, and each term
                    // 2^(acc * sc2 - m) with one fused multiply-add and the hardware's base-two exponential)
                    float am = acc[q][0];
#pragma unroll
                    for (int r = 1; r < 16; r += 2) am = fmaxf(fmaxf(acc[q][r], r + 1 < 16 ? acc[q][r + 1] : acc[q][r]), am);
                    const float m = fmaxf(mx[q], am * sc2);
                    float e[16];
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        e[r] = __builtin_amdgcn_exp2f(__fmaf_rn(acc[q][r], sc2, -m));
                        if (tail) e[r] = (tb + 8 * (r >> 2) + 4 * half + (r & 3)) < tend ? e[r] : 0.0f;
                    }
#pragma unroll
                    for (int w = 8; w >= 1; w >>= 1)
#pragma unroll
                        for (int r = 0; r < w; ++r) e[r] += e[r + w];
                    lsv[q] = __fmaf_rn(lsv[q], __builtin_amdgcn_exp2f(mx[q] - m), e[0]);   // first step: 0 * 2^(-inf) = 0
                    mx[q] = m;
                }
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float v = __fmaf_rn(acc[q][r], a.scale, off[q0 + q]);
                        best[r] = (q0 + q) % G == 0 ? v : fmaxf(best[r], v);
                    }
                    if ((q0 + q) % G == G - 1) keys_out(tail, tb, (q0 + q) / G, best);
                }
            }
        }
    };
    int pg = page_at(tbeg + 2 * ST);
    {
        const uint32_t row = row_from(page_at(tbeg), tbeg);
#pragma unroll
        for (int u = 0; u < NU; ++u) put(piece_of(row, u), u, 0);
    }
    __syncthreads();
    auto step = [&](const bool tail, int buf, int t0) __attribute__((always_inline)) {
        uint4 st[NU];   // used in this body only: an array that other helpers index would be kept in private memory
        const uint32_t row = row_from(pg, t0 + 2 * ST);
#pragma unroll
        for (int u = 0; u < NU; ++u) st[u] = piece_of(row, u);
        pg = page_at(t0 + 4 * ST);
        compute(tail, buf, t0 + sub * ST);
#pragma unroll
        for (int u = 0; u < NU; ++u) put(st[u], u, buf ^ 1);
        __syncthreads();
    };
    int t0 = tbeg, buf = 0;
    for (; t0 + ST + 32 <= tend; t0 += 2 * ST, buf ^= 1) step(false, buf, t0);
    if (t0 < tend) step(true, buf, t0);
    if constexpr (MODE == MFMA_PICK) {   // the last step ended with a barrier
        for (int c = tid; c < CT; c += NT)
            if (j0 + c < C) a.seg_cnt[((size_t)bkl * a.c_max + j0 + c) * a.t_splits + blockIdx.x] = s_cnt[c];
    }
    if constexpr (KEYS) return;
    // the two halves of a wave, then the two waves of an item, hold different keys of the same (centroid, head):
    // merged, one pair per block
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        const float m_o = __shfl_xor(mx[q], 32), l_o = __shfl_xor(lsv[q], 32);
        const float m = fmaxf(mx[q], m_o);
        lsv[q] = lsv[q] * __builtin_amdgcn_exp2f(mx[q] - m) + l_o * __builtin_amdgcn_exp2f(m_o - m);
        mx[q] = m;
        if (sub == 1 && half == 0) s_stat[(wc * ITEMS + q) * 32 + col] = make_float2(m, lsv[q]);
    }
    __syncthreads();
    if (sub == 0 && half == 0) {
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            const int j = j0 + tile_of(q) * 32 + col;
            const float2 o = s_stat[(wc * ITEMS + q) * 32 + col];
            const float m = fmaxf(mx[q], o.x);
            const float l = lsv[q] * __builtin_amdgcn_exp2f(mx[q] - m) + o.y * __builtin_amdgcn_exp2f(o.x - m);
            if (j < C) a.part[(((size_t)bkl * a.c_max + j) * G + head_of(q)) * a.t_splits + blockIdx.x] = make_float2(m, l);
        }
    }
}

// -(m + log S) of every (centroid, head) of a chunk from the blocks' pairs of the statistics pass, in block order.  (Made by every
// block of the two passes behind it, before its first product, it was most of their time where a tile has many blocks:
// 50K tokens, 700 centroids, 24 blocks a tile: sample pass 157 -> 49 us, candidate pass 312 -> 214,
// all keys 400 -> 304; 128K, 2048 centroids, 8 blocks a tile: 160 -> 118, 1241 -> 1180, 1774 -> 1733; this kernel 7 to 9.)
// grid ceil(chunk units * G / 256), 256 threads
__global__ __launch_bounds__(256) void mfma_merge_kernel(MfmaScoreArgs a, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int u = i / a.G, bkl = u / a.c_max, b = (a.bk0 + bkl) / a.g, s = a.ctx_lens[b];
    if (u - bkl * a.c_max >= a.n_cent[b]) return;
    const int tper = (((s + a.t_splits - 1) / a.t_splits) + 31) & ~31, nx = min(a.t_splits, (s + tper - 1) / tper);
    const float2 *pp = a.part + (size_t)i * a.t_splits;
    float m = -__builtin_huge_valf();
#pragma unroll 8
    for (int x = 0; x < nx; ++x) m = fmaxf(m, pp[x].x);
    float sum = 0.0f;
#pragma unroll 8
    for (int x = 0; x < nx; ++x) sum += pp[x].y * __builtin_amdgcn_exp2f(pp[x].x - m);
    a.off[i] = -(m * 0.693147180559945309f + logf(sum));   // the pairs hold base-two maxima
}

// ------------------------------------------------------------------------------
// self-check: to_fixed40(exp_series(x)) against exp_fixed40_parts(x) on the fp32 values whose bit
// patterns are first .. first + n - 1; counts the inputs on which they differ.
// ------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void exp_selftest_kernel(uint32_t first, uint32_t n, unsigned long long *bad)
{
    uint32_t mine = 0;
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) {
        const float x = __uint_as_float(first + i);
        uint32_t hi, lo;
        exp_fixed40_parts(x, hi, lo);
        mine += (to_fixed40(exp_series(x)) != (((uint64_t)hi << 24) + lo)) ? 1u : 0u;
    }
    if (mine) atomicAdd(bad, (unsigned long long)mine);
}

// ------------------------------------------------------------------------------
// softmax denominators: S[h] += sum_i floor(exp(z[h][i] - m[h]) * 2^40), integer
// adds, hence the same value in any order.  grid (nbx, units), 256 threads, each
// block walks chunks of 1024 ids with stride gridDim.x.
// ------------------------------------------------------------------------------
struct DenomArgs {
    Units u;
    const int32_t *ctx_lens, *ncand;   // ncand == nullptr => L = ctx_len
    int l_stride;
    const float *z;
    const uint32_t *m_key;
    unsigned long long *S;
    uint32_t *gbits;          // decode only: the recall bitmap, cleared here for the next step
    int bitmap_words;
    int by_xcd;               // blocks -> (unit, block of the unit) by unit_block_of
    uint32_t *gcur;           // optional: [units][kMaxStride] list cursors of keyclass_kernel, cleared here
};

template <int G> __global__ __launch_bounds__(256) void denom_kernel(DenomArgs a)
{
    int b, kv, j;
    int ul, bx;
    unit_block_of(a.by_xcd, ul, bx);
    if (!decode_unit(a.u, ul, b, kv, j)) return;
    // everything the block needs to know is requested at once (the maxima before L decides whether
    // the block has work: one round trip instead of three)
    uint32_t mk[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) mk[hh] = a.m_key[ul * kMaxStride + hh];
    const int s_len = a.ctx_lens[b];
    const int L = a.ncand ? a.ncand[ul] : s_len;
    if (a.gcur && bx == 0 && threadIdx.x == 0) a.gcur[ul * kMaxStride] = 0u;
    if (a.gbits) {
        const int W = (s_len + 31) >> 5;
        for (int w = bx * 256 + threadIdx.x; w < W; w += gridDim.x * 256) a.gbits[(size_t)ul * a.bitmap_words + w] = 0u;
    }
    if (bx * 1024 >= L) return;
    const int tid = threadIdx.x;
    __shared__ unsigned long long s_acc[4][G];
    float m[G];
    unsigned long long acc[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) {
        m[hh] = ordered_value(mk[hh]);
        acc[hh] = 0ull;
    }
    const float *zb = a.z + (size_t)ul * a.l_stride * G;
    for (int c0 = bx * 1024; c0 < L; c0 += gridDim.x * 1024) {
        // four terms per head as 32-bit partial sums (hi < 2^17, lo < 2^24 each), then one 64-bit add
        uint32_t shi[G], slo[G];
#pragma unroll
        for (int hh = 0; hh < G; ++hh) shi[hh] = slo[hh] = 0u;
        // the four loads first (ids beyond L read entry L-1 and are left out below): taken one at a
        // time, each would be waited for before the next is requested
        float zv[4][G];
#pragma unroll
        for (int q = 0; q < 4; ++q) load_z<G>(zb, min(c0 + q * 256 + tid, L - 1), zv[q]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool ok = (c0 + q * 256 + tid) < L;
#pragma unroll
            for (int hh = 0; hh < G; ++hh) {
                uint32_t hi, lo;
                exp_fixed40_parts(zv[q][hh] - m[hh], hi, lo);
                shi[hh] += ok ? hi : 0u;
                slo[hh] += ok ? lo : 0u;
            }
        }
#pragma unroll
        for (int hh = 0; hh < G; ++hh) acc[hh] += ((unsigned long long)shi[hh] << 24) + slo[hh];
    }
#pragma unroll
    for (int hh = 0; hh < G; ++hh) {
        unsigned long long v = acc[hh];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
        if (lane_id() == 0) s_acc[tid >> 6][hh] = v;
    }
    __syncthreads();
    if (tid < G) atomicAdd(&a.S[ul * kSumStride + tid], s_acc[0][tid] + s_acc[1][tid] + s_acc[2][tid] + s_acc[3][tid]);
}

// ------------------------------------------------------------------------------
// ranking keys, chip-wide: key_i = max_h ((z[h][i] - m[h]) - log S[h]) as an ordered
// uint32 into kbuf, and the unit's histogram of key_bucket() (shared-memory
// histogram per block, non-empty buckets added to the global one: integer adds).
// grid (nbx, units), 1024 threads, chunks of 4096 ids with stride gridDim.x.
// ------------------------------------------------------------------------------
struct KeyArgs {
    Units u;
    const int32_t *ctx_lens, *ncand;   // ncand == nullptr => L = ctx_len
    int l_stride;
    const float *z;     // nullptr: kbuf holds the keys already, only their histogram is taken
    const uint32_t *m_key;
    const unsigned long long *S;
    uint32_t *kbuf;     // [units][l_stride]
    uint32_t *ghist;    // [units][kBuckets], zero on entry
    uint32_t *gcur;     // decode only: [units][kMaxStride] list cursors of classify_kernel, cleared here
    int n_init, n_local;   // build only: ids below n_init or from L - n_local on are never listed
    int by_xcd;              // blocks -> (unit, block of the unit) by unit_block_of
};

template <int G> __global__ __launch_bounds__(1024) void keyhist_kernel(KeyArgs a)
{
    int b, kv, j;
    int ul, bx;
    unit_block_of(a.by_xcd, ul, bx);
    if (!decode_unit(a.u, ul, b, kv, j)) return;
    const int tid = threadIdx.x;
    // the unit's statistics are requested together with L, before L decides whether the block has work
    uint32_t mk[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) mk[hh] = a.z ? a.m_key[ul * kMaxStride + hh] : 0u;
    const unsigned long long S_mine = (a.z && tid < G) ? a.S[ul * kSumStride + tid] : 1ull;
    const int L = a.ncand ? a.ncand[ul] : a.ctx_lens[b];
    if (a.gcur && bx == 0 && threadIdx.x == 0) a.gcur[ul * kMaxStride] = 0u;
    if (bx * 4096 >= L) return;
    __shared__ uint32_t s_h[kBuckets];
    __shared__ float s_ls[G];
    for (int w = tid; w < kBuckets; w += 1024) s_h[w] = 0u;
    if (tid < G) s_ls[tid] = a.z ? (float)log_fixed40(S_mine) : 0.0f;
    float m[G], ls[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) m[hh] = a.z ? ordered_value(mk[hh]) : 0.0f;
    __syncthreads();
#pragma unroll
    for (int hh = 0; hh < G; ++hh) ls[hh] = s_ls[hh];
    const float *zb = a.z + (size_t)ul * a.l_stride * G;
    uint32_t *kb = a.kbuf + (size_t)ul * a.l_stride;
    if (!a.z) {   // the keys are there already (matrix-core build): histogram only, four keys per load
        const bool wide = (reinterpret_cast<uintptr_t>(kb) & 15u) == 0;
        // The last bucket takes every key below the histogram's range, often most of them: its
        // count is taken per wave with a ballot (64 lanes adding to one word would be served
        // one after the other); the other buckets are added to directly.
        auto count4 = [&](const uint32_t(&k4)[4], int i) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool valid = i + e < L;
                const uint32_t bk = key_bucket(k4[e]);
                const bool tail = valid && bk == (uint32_t)(kBuckets - 1);
                const uint64_t mt = __ballot(tail);
                if (valid && !tail) atomicAdd(&s_h[bk], 1u);
                if (mt && lane_id() == 0) atomicAdd(&s_h[kBuckets - 1], (uint32_t)__popcll(mt));
            }
        };
        // four chunks of 4096 keys per trip; when all four lie wholly below L their loads are plain
        // and go out together
        const int stride = gridDim.x * 4096;
        for (int c0 = bx * 4096; c0 < L; c0 += 4 * stride) {
            if (wide && c0 + 3 * stride + 4096 <= L) {
                uint4 v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = *reinterpret_cast<const uint4 *>(kb + c0 + q * stride + 4 * tid);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t k4[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
                    count4(k4, c0 + q * stride + 4 * tid);
                }
            } else {
                for (int q = 0; q < 4; ++q) {
                    const int cq = c0 + q * stride;
                    if (cq >= L) break;   // uniform
                    const int i = cq + 4 * tid;
                    uint32_t k4[4] = {0u, 0u, 0u, 0u};
                    if (wide && i + 3 < L) {
                        const uint4 v = *reinterpret_cast<const uint4 *>(kb + i);
                        k4[0] = v.x; k4[1] = v.y; k4[2] = v.z; k4[3] = v.w;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (i + e < L) k4[e] = kb[i + e];
                    }
                    count4(k4, i);
                }
            }
        }
    }
    for (int c0 = bx * 4096; a.z && c0 < L; c0 += gridDim.x * 4096) {
        // the four loads first (ids beyond L read entry L-1 and are dropped): see denom_kernel
        float zv[4][G];
#pragma unroll
        for (int q = 0; q < 4; ++q) load_z<G>(zb, min(c0 + q * 1024 + tid, L - 1), zv[q]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = c0 + q * 1024 + tid;
            const bool valid = i < L;
            float best = -__builtin_huge_valf();
#pragma unroll
            for (int hh = 0; hh < G; ++hh) best = fmaxf(best, (zv[q][hh] - m[hh]) - ls[hh]);
            uint32_t ok = ordered_key(best);
            // keys of the resident window rank below every other key (the image of -inf)
            if (i < a.n_init || i >= L - a.n_local) ok = 0x007fffffu;
            if (valid) kb[i] = ok;
            const uint32_t bk = key_bucket(ok);
            const bool tail = valid && bk == (uint32_t)(kBuckets - 1);   // counted per wave, as above
            const uint64_t mt = __ballot(tail);
            if (valid && !tail) atomicAdd(&s_h[bk], 1u);
            if (mt && lane_id() == 0) atomicAdd(&s_h[kBuckets - 1], (uint32_t)__popcll(mt));
        }
    }
    __syncthreads();
    uint32_t *gh = a.ghist + (size_t)ul * kBuckets;
    for (int w = tid; w < kBuckets; w += 1024) {
        uint32_t v = s_h[w];
        if (v) atomicAdd(&gh[w], v);
    }
}

// ------------------------------------------------------------------------------
// Algorithm 2 line 6, the pass over the ranking keys, spread over the chip (decode).  Every block
// scans its unit's key histogram for the bucket that holds the top_k-th key, then walks its share
// of the ids in groups of 64: ids in higher buckets go into a bitmap (one ballot per group, plain
// stores), the (key, id) pairs of the deciding bucket are appended to the unit's list (one
// cursor bump per wave; the order of the list is arbitrary and nothing depends on it).
// Units with top_k >= L, or with more than kListCap keys in the deciding bucket, are left to the
// select kernel.  grid (nbx, units), 256 threads; keyhist_kernel has cleared the cursors.
// ------------------------------------------------------------------------------
struct ClassifyArgs {
    Units u;
    const int32_t *ctx_lens, *ncand;
    int l_stride, top_k;
    const uint32_t *kbuf;    // [units][l_stride]
    const uint32_t *ghist;   // [units][kBuckets]
    int bits_stride;         // bitmap words per unit
    uint32_t *gbm;           // [units][bits_stride] ids above the deciding bucket
    uint2 *glist;            // [units][kListCap] (key, id) of the deciding bucket
    uint32_t *gcur;          // [units][kMaxStride] list cursor (first word), zero on entry
    uint32_t *ginfo;         // [units][4] deciding bucket, keys wanted from it, its population, unused
    int by_xcd;              // blocks -> (unit, block of the unit) by unit_block_of
};

__global__ __launch_bounds__(256) void classify_kernel(ClassifyArgs a)
{
    int b, kv, j;
    int ul, bx;
    unit_block_of(a.by_xcd, ul, bx);
    if (!decode_unit(a.u, ul, b, kv, j)) return;
    const int L = a.ncand ? a.ncand[ul] : a.ctx_lens[b];
    if (a.top_k >= L) return;
    __shared__ uint32_t s_scan[8];
    __shared__ uint32_t s_res[3];
    const int tid = threadIdx.x, ln = lane_id();
    const int nw64 = (L + 63) >> 6;
    const int wg = bx * 4 + (tid >> 6), nwg = gridDim.x * 4;
    const uint32_t *kb = a.kbuf + (size_t)ul * a.l_stride;
    constexpr int UNR = 4;
    // this wave's first groups of keys are requested before the histogram is looked at
    uint32_t kk[UNR];
#pragma unroll
    for (int q = 0; q < UNR; ++q) {
        int i = (wg + q * nwg) * 64 + ln;
        kk[q] = (i < L) ? kb[i] : 0u;
    }
    // thread t owns buckets BPT*t .. BPT*t + BPT-1, in descending key order
    constexpr int BPT = kBuckets / 256;
    static_assert(BPT % 4 == 0, "bucket counts are read as uint4");
    uint32_t c[BPT];
    {
        const uint4 *gh = reinterpret_cast<const uint4 *>(a.ghist + (size_t)ul * kBuckets) + (BPT / 4) * tid;
#pragma unroll
        for (int q = 0; q < BPT / 4; ++q) {
            uint4 v = gh[q];
            c[4 * q] = v.x; c[4 * q + 1] = v.y; c[4 * q + 2] = v.z; c[4 * q + 3] = v.w;
        }
    }
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < BPT; ++q) mine += c[q];
    uint32_t tot;
    uint32_t before = block_excl_scan<256>(mine, s_scan, &tot);
#pragma unroll
    for (int q = 0; q < BPT; ++q) {
        if (before < (uint32_t)a.top_k && (uint32_t)a.top_k <= before + c[q]) {
            s_res[0] = (uint32_t)(BPT * tid + q);
            s_res[1] = (uint32_t)a.top_k - before;
            s_res[2] = c[q];
        }
        before += c[q];
    }
    __syncthreads();
    const uint32_t bkt = s_res[0], nb = s_res[2];
    if (bx == 0 && tid == 0)
        *reinterpret_cast<uint4 *>(a.ginfo + 4 * (size_t)ul) = make_uint4(bkt, s_res[1], nb, 0u);
    if (nb > (uint32_t)kListCap) return;
    uint32_t *bm = a.gbm + (size_t)ul * a.bits_stride;
    uint2 *lst = a.glist + (size_t)ul * kListCap;
    const uint64_t below = (1ull << ln) - 1ull;
    for (int g0 = wg; g0 < nw64; g0 += UNR * nwg) {
        if (g0 != wg) {
#pragma unroll
            for (int q = 0; q < UNR; ++q) {
                int i = (g0 + q * nwg) * 64 + ln;
                kk[q] = (i < L) ? kb[i] : 0u;
            }
        }
#pragma unroll
        for (int q = 0; q < UNR; ++q) {
            const int gq = g0 + q * nwg;
            if (gq < nw64) {
                const int i = gq * 64 + ln;
                const bool valid = i < L;
                const uint32_t bk = key_bucket(kk[q]);
                const bool inb = valid && bk == bkt;
                const uint64_t above = __ballot(valid && bk < bkt);
                const uint64_t listed = __ballot(inb);
                if (ln == 0) *reinterpret_cast<uint2 *>(bm + 2 * gq) = make_uint2((uint32_t)above, (uint32_t)(above >> 32));
                if (listed) {
                    uint32_t at0 = 0;
                    if (ln == 0) at0 = atomicAdd(&a.gcur[ul * kMaxStride], (uint32_t)__popcll(listed));
                    at0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)at0);
                    if (inb) lst[at0 + (uint32_t)__popcll(listed & below)] = make_uint2(kk[q], (uint32_t)i);
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------
// keyhist_kernel and classify_kernel as ONE launch, for small batches (decode).  The histogram of a unit's
// keys is needed whole before any key can be classified; here every block of the unit takes it itself, over
// ALL the unit's ids (the same few thousand scores read by each of its blocks, from the cache; the histogram
// stays in shared memory), finds the deciding bucket, and then writes and classifies the keys of its own share
// as classify_kernel does.  One launch and one round trip fewer, for work that is repeated per block: only
// where that work is small (the host's choice).  grid (nbx, units), 1024 threads; denom_kernel has cleared the
// list cursors.  No 2048-bucket histogram is left in global memory.
// ------------------------------------------------------------------------------
struct KeyClassArgs {
    Units u;
    const int32_t *ctx_lens, *ncand;
    int l_stride, top_k;
    const float *z;
    const uint32_t *m_key;
    const unsigned long long *S;
    uint32_t *kbuf;          // [units][l_stride]
    int bits_stride;
    uint32_t *gbm;           // [units][bits_stride]
    uint2 *glist;            // [units][kListCap]
    uint32_t *gcur;          // [units][kMaxStride], zero on entry
    uint32_t *ginfo;         // [units][4]
    int by_xcd;              // blocks -> (unit, block of the unit) by unit_block_of
};

template <int G> __global__ __launch_bounds__(1024) void keyclass_kernel(KeyClassArgs a)
{
    int b, kv, j;
    int ul, bx;
    unit_block_of(a.by_xcd, ul, bx);
    if (!decode_unit(a.u, ul, b, kv, j)) return;
    const int tid = threadIdx.x, wv = tid >> 6, ln = lane_id();
    uint32_t mk[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) mk[hh] = a.m_key[ul * kMaxStride + hh];
    const unsigned long long S_mine = tid < G ? a.S[ul * kSumStride + tid] : 1ull;
    const int L = a.ncand ? a.ncand[ul] : a.ctx_lens[b];
    __shared__ uint32_t s_h[kBuckets];
    __shared__ float s_ls[G];
    __shared__ uint32_t s_scan[1024 / 64 + 2];
    __shared__ uint32_t s_res[3];
    for (int w = tid; w < kBuckets; w += 1024) s_h[w] = 0u;
    if (tid < G) s_ls[tid] = (float)log_fixed40(S_mine);
    if (tid == 0) s_res[2] = 0xffffffffu;
    float m[G], ls[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) m[hh] = ordered_value(mk[hh]);
    __syncthreads();
#pragma unroll
    for (int hh = 0; hh < G; ++hh) ls[hh] = s_ls[hh];
    const float *zb = a.z + (size_t)ul * a.l_stride * G;
    auto key_of = [&](const float(&zv)[G]) __attribute__((always_inline)) {
        float best = -__builtin_huge_valf();
#pragma unroll
        for (int hh = 0; hh < G; ++hh) best = fmaxf(best, (zv[hh] - m[hh]) - ls[hh]);
        return ordered_key(best);
    };
    const bool rank = a.top_k < L;   // otherwise every recalled key is kept and nothing needs classifying
    // pass 1: the histogram of ALL the unit's keys (the last bucket, which takes every key below the range, counted
    // per wave with a ballot)
    for (int c0 = 0; rank && c0 < L; c0 += 4096) {
        float zv[4][G];
#pragma unroll
        for (int q = 0; q < 4; ++q) load_z<G>(zb, min(c0 + q * 1024 + tid, L - 1), zv[q]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool valid = c0 + q * 1024 + tid < L;
            const uint32_t bk = key_bucket(key_of(zv[q]));
            const bool tail = valid && bk == (uint32_t)(kBuckets - 1);
            const uint64_t mt = __ballot(tail);
            if (valid && !tail) atomicAdd(&s_h[bk], 1u);
            if (mt && ln == 0) atomicAdd(&s_h[kBuckets - 1], (uint32_t)__popcll(mt));
        }
    }
    __syncthreads();
    uint32_t bkt = 0, nb = 0xffffffffu;
    if (rank) {
        // thread t owns buckets 2t, 2t+1, in descending key order
        constexpr int BPT = kBuckets / 1024;
        uint32_t c[BPT], mine = 0;
#pragma unroll
        for (int q = 0; q < BPT; ++q) {
            c[q] = s_h[BPT * tid + q];
            mine += c[q];
        }
        uint32_t tot;
        uint32_t before = block_excl_scan<1024>(mine, s_scan, &tot);
#pragma unroll
        for (int q = 0; q < BPT; ++q) {
            if (before < (uint32_t)a.top_k && (uint32_t)a.top_k <= before + c[q]) {
                s_res[0] = (uint32_t)(BPT * tid + q);
                s_res[1] = (uint32_t)a.top_k - before;
                s_res[2] = c[q];
            }
            before += c[q];
        }
        __syncthreads();
        bkt = s_res[0];
        nb = s_res[2];
        if (bx == 0 && tid == 0) *reinterpret_cast<uint4 *>(a.ginfo + 4 * (size_t)ul) = make_uint4(bkt, s_res[1], nb, 0u);
    }
    const bool classify = rank && nb <= (uint32_t)kListCap;
    // pass 2: this block's share of the ids in groups of 64: keys written, and classified against the deciding bucket
    uint32_t *kb = a.kbuf + (size_t)ul * a.l_stride;
    uint32_t *bm = a.gbm + (size_t)ul * a.bits_stride;
    uint2 *lst = a.glist + (size_t)ul * kListCap;
    const uint64_t below = (1ull << ln) - 1ull;
    const int nw64 = (L + 63) >> 6;
    for (int g0 = bx * 16 + wv; g0 < nw64; g0 += gridDim.x * 16) {
        const int i = g0 * 64 + ln;
        const bool valid = i < L;
        float zv[G];
        load_z<G>(zb, min(i, L - 1), zv);
        const uint32_t ok = key_of(zv);
        if (valid) kb[i] = ok;
        if (classify) {
            const uint32_t bk = key_bucket(ok);
            const bool inb = valid && bk == bkt;
            const uint64_t above = __ballot(valid && bk < bkt);
            const uint64_t listed = __ballot(inb);
            if (ln == 0) *reinterpret_cast<uint2 *>(bm + 2 * g0) = make_uint2((uint32_t)above, (uint32_t)(above >> 32));
            if (listed) {
                uint32_t at0 = 0;
                if (ln == 0) at0 = atomicAdd(&a.gcur[ul * kMaxStride], (uint32_t)__popcll(listed));
                at0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)at0);
                if (inb) lst[at0 + (uint32_t)__popcll(listed & below)] = make_uint2(ok, (uint32_t)i);
            }
        }
    }
}

// ------------------------------------------------------------------------------
// Algorithm 2 line 6 / Algorithm 1 line 4.  One block of 1024 threads per unit: the
// top-k ids by ranking key (kbuf), ascending, helped by the key histogram.
//   decode: sel[unit][pos] = cand[i], srow[unit][pos] = crow[i],
//           zsel[unit][pos][G] = z[i][G], nsel[unit]
//   build : lists[(b*g+kv)*c_max + j][pos] = i
// Dynamic shared memory: kSelLds + 2*kListCap + bits_words + top_k words (the last: positions of
// the picked ids, decode only).
// ------------------------------------------------------------------------------
struct SelectArgs {
    Units u;
    const int32_t *ctx_lens, *ncand, *cand;
    const uint32_t *crow;
    int l_stride, top_k;
    int bits_words;          // shared-memory words set aside for the two id bitmaps (0: none)
    const float *z;
    const uint32_t *m_key;
    const uint32_t *kbuf;    // [units][l_stride] ranking keys (keyhist_kernel)
    const uint32_t *ghist;   // [units][kBuckets] their histogram
    const uint32_t *gbm;     // decode: classify_kernel's outputs (nullptr: the block makes the pass itself)
    const uint2 *glist;
    const uint32_t *ginfo;
    int bits_stride;
    int32_t *sel;       // decode [units][top_k] ; build: lists base
    uint32_t *srow;     // decode [units][top_k]
    float *zsel;        // decode [units][top_k][G]
    int32_t *nsel;      // decode [units]
    int32_t *out_sel;   // optional copy for the caller
    int ids_only;       // decode: write sel and nsel only (the dynamic centroid update's second ranking)
};

// writes the decode outputs of one unit from the positions picked into s_idx[0..n)
template <int G>
__device__ __forceinline__ void select_gather(const SelectArgs &a, int ul, int n, const float *zb, const int32_t *s_idx)
{
    const int tid = threadIdx.x;
    const int32_t *cb = a.cand + (size_t)ul * a.l_stride;
    int32_t *dst = a.sel + (size_t)ul * a.top_k;
    if (a.ids_only) {
        for (int pos = tid; pos < a.top_k; pos += 1024) dst[pos] = pos < n ? cb[s_idx[pos]] : -1;
        if (tid == 0) a.nsel[ul] = n;
        return;
    }
    const uint32_t *rb = a.crow + (size_t)ul * a.l_stride;
    uint32_t *dstr = a.srow + (size_t)ul * a.top_k;
    int32_t *dst2 = a.out_sel ? a.out_sel + (size_t)ul * a.top_k : nullptr;
    float *zd = a.zsel + (size_t)ul * a.top_k * G;
#pragma unroll 2
    for (int pos = tid; pos < a.top_k; pos += 1024) {
        if (pos < n) {
            int i = s_idx[pos];
            int t = cb[i];
            uint32_t r = rb[i];
            float zv[G];
            load_z<G>(zb, i, zv);
            dst[pos] = t;
            dstr[pos] = r;
            if (dst2) dst2[pos] = t;
            store_z<G>(zd, pos, zv);
        } else {
            dst[pos] = -1;
            if (dst2) dst2[pos] = -1;
        }
    }
    if (tid == 0) a.nsel[ul] = n;
}

template <int KPT, typename KeyFn, typename EmitFn>
__device__ __forceinline__ int select_generic(KeyFn key, int L, int k, EmitFn emit, uint32_t *s_sel)
{
    return block_select_topk<1024, KPT>(key, L, k, emit, s_sel);
}

// Shared-memory words of the selection: radix scratch, the deciding bucket's list, the two id
// bitmaps, then the positions of the picks (decode).
__device__ __forceinline__ int select_smem_words(int bits_words, int top_k) { return kSelLds + 2 * kListCap + bits_words + top_k; }

// The selection of one unit: positions (decode: into s_idx, ascending; build: ids straight into
// the list) of the top_k ranking keys among L.  Returns their number.  Every thread of the
// 1024-thread block takes part.
template <int G> __device__ __forceinline__ int select_unit(const SelectArgs &a, int ul, int L, uint32_t *smem)
{
    uint32_t *s_sel = smem;                          // kSelLds
    uint32_t *s_list = smem + kSelLds;               // 2 * kListCap
    uint32_t *s_bits = s_list + 2 * kListCap;        // a.bits_words (two bitmaps over the ids)
    int32_t *s_idx = (int32_t *)(s_bits + a.bits_words);   // top_k (decode)
    const uint32_t *kb = a.kbuf + (size_t)ul * a.l_stride;
    auto key = [&](int i) { return kb[i]; };
    int32_t *lst = a.u.build ? a.sel + (size_t)(a.u.unit0 + ul) * a.top_k : nullptr;
    auto emit = [&](int pos, int i) {
        if (lst)
            lst[pos] = i;
        else
            s_idx[pos] = i;
    };
    int n = -1;
    if (a.top_k >= L) {
        for (int i = threadIdx.x; i < L; i += 1024) emit(i, i);
        n = L;
    } else if (4 * ((L + 63) >> 6) <= a.bits_words) {
        if (a.ginfo) {
            const uint4 info = *reinterpret_cast<const uint4 *>(a.ginfo + 4 * (size_t)ul);
            if (info.z <= (uint32_t)kListCap)
                n = block_select_classified<1024>(L, a.top_k, info.y, info.z, a.gbm + (size_t)ul * a.bits_stride,
                                                  a.glist + (size_t)ul * kListCap, emit, s_sel, s_bits, s_list);
        } else {
            n = block_select_hist<1024>(kb, L, a.top_k, emit, s_sel, s_bits, s_list, a.ghist + (size_t)ul * kBuckets);
        }
    }
    if (n < 0) {   // crowded deciding bucket (or no room for the bitmaps): the histogram-free route
        if (L <= 1024 * 8)
            n = select_generic<8>(key, L, a.top_k, emit, s_sel);
        else if (L <= 1024 * 32)
            n = select_generic<32>(key, L, a.top_k, emit, s_sel);
        else
            n = select_generic<0>(key, L, a.top_k, emit, s_sel);
    }
    return n;
}

template <int G> __global__ __launch_bounds__(1024) void rerank_select_kernel(SelectArgs a)
{
    extern __shared__ __align__(16) uint32_t smem[];
    int b, kv, j;
    const int ul = blockIdx.x;
    if (!decode_unit(a.u, ul, b, kv, j)) return;
    const int L = a.cand ? a.ncand[ul] : a.ctx_lens[b];
    CTKVR_STAMP(28);
    CTKVR_STAMP_BLK(2);
    const int n = select_unit<G>(a, ul, L, smem);
    if (!a.u.build) {
        __syncthreads();
        select_gather<G>(a, ul, n, a.z + (size_t)ul * a.l_stride * G,
                         (const int32_t *)(smem + kSelLds + 2 * kListCap + a.bits_words));
    }
    CTKVR_STAMP(31);
    CTKVR_STAMP_BLK(3);
}

// ------------------------------------------------------------------------------
// Matrix-core list build, candidate route (Algorithm 1 line 4 on a few thousand candidates per unit
// instead of all s keys).
// sample_threshold_kernel: tau[unit] = the lower end of the histogram bucket (1/32 wide) that holds the r-th largest of the
// unit's sampled keys, or that key itself where the bucket is below the histogram's range or so crowded that the candidates might not
// fit (slot i of the sample row is key id (i / 32) * 32 * step_stride + i % 32; slots of ids beyond s or inside the resident window
// do not count), with r = 2 ceil(rho / step_stride) + 16.  With n of its samples at or above tau, about n step_stride of the unit's
// keys are: 2 rho + 16 step_stride at the key itself, more at a bucket's end, which is taken as long as n + 3.5 sqrt(n) steps are
// within cand_cap (the count of the sample spreads by sqrt(n)).  Where even the samples equal to the key are twice what fits
// (equal keys), tau = +inf and the unit has no candidates: it is handed back whatever is collected (storing and
// counting every key first, a build of 65536 tokens and 1024 centroids, 8 KV heads: 9.16 ms, now 8.05).  Fewer samples than r: tau = 0, every key is a candidate.
// (The key itself for every unit, by radix rounds: 159 us for 8192 units of 8192 samples, 83 by the histogram.)  Bound by the latencies of a
// unit's phases, which many small blocks on a CU hide better than few of 1024 threads: 512 threads of sixteen samples 83 -> 58 us (256 of
// 32: 59.5), up to 2048 samples 256 of eight, 4860 units 38 -> 12.6.
// cand_select_kernel: the rho largest of the unit's candidates (key, id), gathered from the segments the
// blocks of the PICK pass filled, ties to the lowest id, written to the unit's list in ascending id order.
// A unit with fewer than rho candidates, more than cand_cap, or a segment that ran over, raises the flag of its (sequence, KV head)
// pair instead (the caller then redoes the pair by the route that keeps every key).
// Both: grid = chunk units, NT threads of KPT slots.  cand_select holds the candidates in registers (through shared memory, 75 KB a
// block at rho = 2048, two blocks of 1024 threads shared a CU: 270 us for 8192 units, now 184): sixteen a thread, 256 threads where cand_cap
// allows it (4860 units of 4096 at most 59 -> 54 us, a build of three of 9K..30K 806 -> 784), 512 beyond (256 of 32 a thread: 266); dynamic shared memory 2112 + kCandTies +
// ceil(s_max / 32) words (one bitmap over the ids; the candidates that tie with the rho-th key, normally one, are
// sorted out in a short list: more than kCandTies of them also raise the flag); cand_cap <= kCandCap.
// ------------------------------------------------------------------------------
constexpr int kCandCap = 8192;
constexpr int kSampleCap = 8192;   // sampled keys per unit at most

struct CandArgs {
    Units u;
    const int32_t *ctx_lens;
    int rho, step_stride, sample_stride, cand_cap;
    int n_init, n_local;
    const uint32_t *ksamp;    // [chunk units][sample_stride]
    uint32_t *tau;            // [chunk units]
    const uint2 *cand;        // [chunk units][t_splits][seg_cap]
    uint32_t *seg_cnt;        // [chunk units][t_splits], zeroed by sample_threshold_kernel for the segments no block writes
    int t_splits, seg_cap;
    int32_t *lists;           // [all units][rho]
    uint32_t *fail;           // [chunk's (sequence, KV head) pairs], zeroed by sample_threshold_kernel
};

template <int NT, int KPT> __global__ __launch_bounds__(NT) void sample_threshold_kernel(CandArgs a)
{
    static_assert(NT >= 64, "a segment's counter per thread");
    constexpr int BPT = kBuckets / NT;   // buckets per thread
    __shared__ uint32_t s_hist[2048 + 64];
    __shared__ uint32_t s_cnt, s_res[2];
    int b, kv, j;
    const int ul = blockIdx.x, tid = threadIdx.x;
    if (tid < a.t_splits) a.seg_cnt[(size_t)ul * a.t_splits + tid] = 0u;   // for the candidate pass
    if (tid == 0 && ul % a.u.c_max == 0) a.fail[ul / a.u.c_max] = 0u;
    if (!decode_unit(a.u, ul, b, kv, j)) return;
#pragma unroll
    for (int q = 0; q < BPT; ++q) s_hist[q * NT + tid] = 0u;
    const int s = a.ctx_lens[b];
    const int ST = 32 * a.step_stride;
    const int n = ((s + ST - 1) / ST) * 32;   // sample slots of this unit (the last step's may reach beyond s)
    const uint32_t *ks = a.ksamp + (size_t)ul * a.sample_stride;
    if (tid == 0) s_cnt = 0u;
    uint32_t kreg[KPT];
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
        const int i = q * NT + tid;
        const int t = (i >> 5) * ST + (i & 31);
        const bool valid = i < n && t < s - a.n_local && t >= a.n_init;
        kreg[q] = ks[min(i, n - 1)];
        if (!valid) kreg[q] = 0u;   // below the image of every real key
        mine += valid;
    }
    __syncthreads();
    mine = wave_sum_uniform(mine);
    if ((tid & 63) == 0 && mine) atomicAdd(&s_cnt, mine);
    __syncthreads();
    const uint32_t n_valid = s_cnt;
    const uint32_t r = 2u * (uint32_t)((a.rho + a.step_stride - 1) / a.step_stride) + 16u;
    if (r > n_valid) {   // uniform
        if (tid == 0) a.tau[ul] = 0u;
        return;
    }
    // the bucket of the r-th largest (the last bucket, everything below the range, is not counted)
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
        const uint32_t bk = key_bucket(kreg[q]);
        if (kreg[q] && bk < (uint32_t)(kBuckets - 1)) atomicAdd(&s_hist[bk], 1u);
    }
    __syncthreads();
    {
        uint32_t c[BPT], sum = 0;   // in descending key order
#pragma unroll
        for (int q = 0; q < BPT; ++q) {
            c[q] = s_hist[BPT * tid + q];
            sum += c[q];
        }
        uint32_t tot;
        uint32_t before = block_excl_scan<NT>(sum, s_hist + 2048 + 4, &tot);
#pragma unroll
        for (int q = 0; q < BPT; ++q) {
            if (before < r && r <= before + c[q]) {
                s_res[0] = (uint32_t)(BPT * tid + q);
                s_res[1] = before + c[q];   // samples at or above the bucket's lower end
            }
            before += c[q];
        }
        if (tid == 0) s_cnt = 0u;
        __syncthreads();
        const float n_at = (float)s_res[1];
        if (r <= tot && (n_at + 3.5f * sqrtf(n_at)) * (float)a.step_stride <= (float)a.cand_cap) {   // uniform
            if (tid == 0) a.tau[ul] = ordered_key(-(float)(s_res[0] + 1u) / 32.0f);
            return;
        }
    }
    auto for_slots = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < KPT; ++q) f(q * NT + tid, kreg[q] != 0u, kreg[q]);
    };
    uint32_t T, need_eq;
    block_kth_largest<NT>(for_slots, r, s_hist, T, need_eq);
    uint32_t n_at = 0;
#pragma unroll
    for (int q = 0; q < KPT; ++q) n_at += kreg[q] >= T ? 1u : 0u;
    n_at = wave_sum_uniform(n_at);
    if ((tid & 63) == 0 && n_at) atomicAdd(&s_cnt, n_at);
    __syncthreads();
    if (tid == 0) a.tau[ul] = s_cnt * (uint32_t)a.step_stride > 2u * (uint32_t)a.cand_cap ? 0xff800000u : T;
}

constexpr int kCandTies = 256;   // candidates equal to the rho-th key that cand_select_kernel sorts out itself

template <int NT, int KPT> __global__ __launch_bounds__(NT, 8) void cand_select_kernel(CandArgs a)
{
    extern __shared__ __align__(16) uint32_t smem[];
    int b, kv, j;
    const int ul = blockIdx.x, tid = threadIdx.x, ln = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (!decode_unit(a.u, ul, b, kv, j)) return;
    const int s = a.ctx_lens[b];
    // the unit's candidates, segment after segment: lane x of every wave has segment x's count (t_splits <= 64) and its place
    const uint32_t c_x = ln < a.t_splits ? a.seg_cnt[(size_t)ul * a.t_splits + ln] : 0u;
    const uint32_t end_x = wave_incl_scan(c_x);
    const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)end_x, 63);
    if (__ballot(c_x > (uint32_t)a.seg_cap) || n < (uint32_t)a.rho || n > (uint32_t)a.cand_cap) {   // uniform
        if (tid == 0) atomicOr(&a.fail[ul / a.u.c_max], 1u);
        return;
    }
    uint32_t *s_hist = smem;                                   // 2048 + 64
    uint32_t *s_ties = smem + 2112;                            // ids of the candidates equal to the rho-th key
    uint32_t *s_bm = s_ties + kCandTies;                       // one bitmap over the ids
    const int nw = (s + 31) >> 5;
    uint32_t *s_x = s_hist + 2048 + 56;                        // [1]: tie cursor (free once the threshold is known)
    // wave w takes every eighth run of 64 of them, from its segment or the two or more it lies in
    const uint2 *src = a.cand + (size_t)ul * a.t_splits * a.seg_cap;
    uint32_t key[KPT], id[KPT];
    int x = 0;   // segment of the run's first candidate
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
        const uint32_t base = (uint32_t)(q * (NT / 64) + wv) * 64u, e = base + (uint32_t)ln;
        key[q] = 0u;   // below every candidate (their images are >= 1)
        id[q] = 0u;
        if (base < n) {   // uniform
            while ((uint32_t)__builtin_amdgcn_readlane((int)end_x, x) <= base) ++x;
            size_t at = 0;
            for (int y = x;; ++y) {
                const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)end_x, y), beg = end - (uint32_t)__builtin_amdgcn_readlane((int)c_x, y);
                if (e >= beg && e < end) at = (size_t)y * a.seg_cap + (e - beg);
                if (end >= min(base + 64u, n)) break;
            }
            const uint2 en = src[at];
            key[q] = e < n ? en.x : 0u;
            id[q] = en.y;
        }
    }
    for (int w = tid; w < nw; w += NT) s_bm[w] = 0u;
    auto for_slots = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < KPT; ++q) {
            if ((uint32_t)(q * (NT / 64) + wv) * 64u >= n) break;   // uniform
            f(q * NT + tid, key[q] != 0u, key[q]);
        }
    };
    // T = the rho-th largest key, need_eq = how many of the candidates equal to T belong to the rho largest
    uint32_t T, need_eq;
    block_kth_largest<NT>(for_slots, (uint32_t)a.rho, s_hist, T, need_eq);
    __syncthreads();
    if (tid == 0) s_x[1] = 0u;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
        if (key[q] > T) atomicOr(&s_bm[id[q] >> 5], 1u << (id[q] & 31u));
        if (key[q] == T) {
            const uint32_t at = atomicAdd(&s_x[1], 1u);
            if (at < (uint32_t)kCandTies) s_ties[at] = id[q];
        }
    }
    __syncthreads();
    const uint32_t n_eq = s_x[1];
    if (n_eq > (uint32_t)kCandTies) {   // uniform: more exact ties at the threshold than are sorted out here
        if (tid == 0) atomicOr(&a.fail[ul / a.u.c_max], 1u);
        return;
    }
    // the need_eq lowest ids among the ties join the bitmap
    if ((uint32_t)tid < n_eq) {
        const uint32_t mine = s_ties[tid];
        uint32_t lower = 0;
        for (uint32_t e = 0; e < n_eq; ++e) lower += s_ties[e] < mine;
        if (lower < need_eq) atomicOr(&s_bm[mine >> 5], 1u << (mine & 31u));
    }
    __syncthreads();
    // thread t owns words [t wpt, (t + 1) wpt) of the bitmap: count, scan, emit in ascending id order
    uint32_t *s_scan = s_hist + 2048 + 4;
    const int wpt = (nw + NT - 1) / NT;
    const int w0 = min(nw, tid * wpt), w1 = min(nw, w0 + wpt);
    uint32_t cnt = 0;
    for (int w = w0; w < w1; ++w) cnt += (uint32_t)__popc(s_bm[w]);
    uint32_t tot;
    uint32_t pos = block_excl_scan<NT>(cnt, s_scan, &tot);
    int32_t *lst = a.lists + (size_t)(a.u.unit0 + ul) * a.rho;
    for (int w = w0; w < w1; ++w) {
        uint32_t m = s_bm[w];
        while (m) {
            const int bpos = __ffs((int)m) - 1;
            m &= m - 1u;
            lst[pos++] = w * 32 + bpos;
        }
    }
}

// ------------------------------------------------------------------------------
// Algorithm 2 lines 7-9: o_h = softmax(z_sel[h]) . V_sel.  grid SL*batch*g, 1024
// threads, SL = 4 or 8 slices: block x owns head dimensions (128/SL) x .. of all G heads of its
// (sequence, KV head), so no partial result crosses a block.  16/SL lanes share a
// row (8 dimensions each; lanes 64 SL/16 apart in a wave), 64 SL rows per pass.  Dynamic shared memory:
// top_k*G floats (softmax weights of the two-pass fallback).
// ------------------------------------------------------------------------------
struct AttnArgs {
    const void *v_pages;
    int g, h, top_k;
    const uint32_t *srow;
    const int32_t *nsel;
    const float *zsel;
    float *out;  // [batch*h][128]
    float *out_lse;
    const float *win;   // optional: window_attn_kernel's partial results, [units][kWinSplit][G][2 + 128]
    const uint32_t *m_key;   // [units][kMaxStride] ordered-key maxima of the logits over all recalled keys
};


// out element `dim` of head hh of a unit: the sparse part (v = sum of exp(z - m_s) * value, l_s = sum of
// exp(z - m_s); l_s = 0 for an empty part) merged with the window's partial results, if there are any.
template <int G>
__device__ __forceinline__ float merge_window(const float *win, int ul, int hh, int dim, float v, float m_s, float l_s, float &lse)
{
    // all partial results are requested at once (no load depends on another)
    float mx[kWinSplit], lx[kWinSplit], ox[kWinSplit];
#pragma unroll
    for (int x = 0; x < kWinSplit; ++x) {
        mx[x] = -__builtin_huge_valf();
        lx[x] = 0.0f;
        ox[x] = 0.0f;
    }
    if (win) {
        const float *wp = win + (size_t)ul * kWinSplit * G * (2 + kD) + hh * (2 + kD);
#pragma unroll
        for (int x = 0; x < kWinSplit; ++x) {
            mx[x] = wp[x * G * (2 + kD)];
            lx[x] = wp[x * G * (2 + kD) + 1];
            ox[x] = wp[x * G * (2 + kD) + 2 + dim];
        }
    }
    float M = l_s > 0.0f ? m_s : -__builtin_huge_valf();
#pragma unroll
    for (int x = 0; x < kWinSplit; ++x)
        if (lx[x] > 0.0f) M = fmaxf(M, mx[x]);
    if (M == -__builtin_huge_valf()) {   // nothing to attend over at all: defined output
        lse = -__builtin_huge_valf();
        return 0.0f;
    }
    float num = 0.0f, den = 0.0f;
    if (l_s > 0.0f) {
        const float w = __expf(m_s - M);
        num = v * w;
        den = l_s * w;
    }
#pragma unroll
    for (int x = 0; x < kWinSplit; ++x)
        if (lx[x] > 0.0f) {
            const float w = __expf(mx[x] - M);
            num += ox[x] * w;
            den += lx[x] * w;
        }
    lse = M + __logf(den);
    return num / den;
}

// Block id -> (unit, slice).  A slice is 128 / SL head dimensions of all G heads, SL = 4 or 8 (8 while every
// block still has a CU of its own: each block then moves half the bytes and weighs half the rows; beyond that the
// launch is oversubscribed and 4 is faster).  Workgroups go to the 8 XCDs round-robin by linear id; the slices of a
// unit read the same 128-byte lines, so they get ids that are congruent modulo 8: one XCD, one L2.
template <int SL> __device__ __forceinline__ void attn_block_of(int &ul, int &slice)
{
    const int lin = blockIdx.x, nu = gridDim.x / SL;
    if ((nu & 7) == 0) {
        const int xcd = lin & 7, k = lin >> 3;
        ul = (k / SL) * 8 + xcd;
        slice = k % SL;
    } else {
        ul = lin / SL;
        slice = lin % SL;
    }
}

// The attention of one (unit, slice), NT threads.  row_of(t) = physical row of the t-th selected key (valid for
// every t < top_k), z_of(t, zv) = its G logits, nsel_of() = how many keys were selected; nsel_of is
// asked only after the first value rows have been requested.  s_p: top_k*G floats of shared memory (z_of may read from it).
template <typename T, int G, int SL, int NU, int NT, typename RowFn, typename ZFn, typename NFn>
__device__ __forceinline__ void attend_unit(const AttnArgs &a, int ul, int slice, float *s_p, RowFn row_of, ZFn z_of, NFn nsel_of)
{
    constexpr int NW = NT / 64;
    constexpr int kSliceDims = kD / SL;            // head dimensions per block
    constexpr int kSliceLanes = kSliceDims / 8;    // lanes that share a value row (8 dimensions each)
    constexpr int kSliceRows = 64 / kSliceLanes;   // rows per wave and pass
    static_assert(kSliceRows % 16 == 0, "the sum over a wave's rows starts with a butterfly inside each 16-lane row");
    // A wave's 64 lanes are kSliceLanes parts of kSliceRows rows: lane l works on row (l mod kSliceRows) of the
    // pass and on the 8 values (l / kSliceRows) of the slice.  Every 16-lane row of a wave thus belongs to one part; the two rows of
    // a part (eight slices) are summed pairwise, each keeping half of the values.  A wave is one producer of partial sums per part.
    constexpr int PASS = NW * kSliceRows, kProd = NW;   // rows per pass of the block; NU passes in flight
    constexpr bool kPairs = kSliceRows == 32;
    static_assert(kPairs || kSliceRows == 16, "one or two rows of 16 lanes per part");
    __shared__ float s_red[kProd][G];
    __shared__ float s_m[G];
    __shared__ uint32_t s_big[NW];
    __shared__ float s_o[kProd][G][kSliceDims];
    const int b = ul / a.g, kv = ul - b * a.g;
    const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
    const int quad = ln / kSliceRows, rin = wv * kSliceRows + (ln % kSliceRows);
    CTKVR_STAMP(44);
    CTKVR_STAMP_BLK(4);
    const T *V = (const T *)a.v_pages + slice * kSliceDims + quad * 8;
    // The first NU * PASS value rows are requested before anything else (rows beyond nsel are valid
    // stale ones whose products get weight 0).
    // The row numbers first, then the rows: taken in turn, each row number would be
    // waited for together with the row requested just before it.
    Chunk<T> cv[NU];
    uint32_t vrow[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) vrow[u] = row_of(min(u * PASS + rin, a.top_k - 1));
#pragma unroll
    for (int u = 0; u < NU; ++u) cv[u] = load_chunk(V + (size_t)vrow[u] * kD, 0);
    // those keys' logits travel with their value rows
    float zq[NU][G];
#pragma unroll
    for (int u = 0; u < NU; ++u) z_of(min(u * PASS + rin, a.top_k - 1), zq[u]);
    const int nsel = nsel_of();
    if (nsel == 0) {   // nothing recalled: the window alone, or zeros
        if (tid < G * kSliceDims) {
            int hh = tid / kSliceDims, e = tid % kSliceDims;
            float lse;
            const float o = merge_window<G>(a.win, ul, hh, slice * kSliceDims + e, 0.0f, -__builtin_huge_valf(), 0.0f, lse);
            a.out[((size_t)b * a.h + kv * G + hh) * kD + slice * kSliceDims + e] = o;
            if (slice == 0 && e == 0 && a.out_lse) a.out_lse[(size_t)b * a.h + kv * G + hh] = lse;
        }
        return;
    }
    // One pass: weights relative to the unit's maxima over ALL its recalled keys, known since the scoring
    // (every selected logit is at most that maximum), so that no statistics of the selected keys have to be
    // gathered before their value rows can be used.  Lane groups that share a key row compute the same
    // weights; the lanes of a wave's first row carry them into the denominators.
    float acc[G][8], lsum[G], mref[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) {
        mref[hh] = ordered_value(a.m_key[ul * kMaxStride + hh]);
        lsum[hh] = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[hh][e] = 0.0f;
    }
    if (tid < G) s_m[tid] = ordered_value(a.m_key[ul * kMaxStride + tid]);
    for (int r0 = 0; r0 < nsel; r0 += NU * PASS) {
        if (r0 > 0) {
#pragma unroll
            for (int u = 0; u < NU; ++u) vrow[u] = row_of(min(r0 + u * PASS + rin, a.top_k - 1));
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                cv[u] = load_chunk(V + (size_t)vrow[u] * kD, 0);
                z_of(min(r0 + u * PASS + rin, a.top_k - 1), zq[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int t = r0 + u * PASS + rin;
            if (t < nsel) {
                float vx[8];
                unpack(cv[u], vx);
#pragma unroll
                for (int hh = 0; hh < G; ++hh) {
                    const float pw = __expf(zq[u][hh] - mref[hh]);
                    lsum[hh] += pw;
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[hh][e] = __fmaf_rn(pw, vx[e], acc[hh][e]);
                }
            }
        }
    }
    CTKVR_STAMP(48);
    // Sums over the lanes of a part: two values at a time across its two 16-lane rows (then the even row has the first
    // of them and the odd row the second), then inside a row (a DPP butterfly); one barrier for denominators and outputs together.
    auto hand_over = [&]() __attribute__((always_inline)) {
        if constexpr (kPairs) {
            const int odd = (ln >> 4) & 1;
            float o[G][4];
#pragma unroll
            for (int hh = 0; hh < G; ++hh)
#pragma unroll
                for (int e = 0; e < 4; ++e) o[hh][e] = group16_sum(row_pair_sum(acc[hh][e], acc[hh][e + 4]));
            float l[(G + 1) / 2];
#pragma unroll
            for (int j = 0; j < (G + 1) / 2; ++j) l[j] = group16_sum(row_pair_sum(lsum[2 * j], lsum[G > 1 ? 2 * j + 1 : 0]));
            if ((ln & 15) == 0) {
#pragma unroll
                for (int hh = 0; hh < G; ++hh)
#pragma unroll
                    for (int e = 0; e < 4; ++e) s_o[wv][hh][quad * 8 + odd * 4 + e] = o[hh][e];
                if (quad == 0) {
#pragma unroll
                    for (int j = 0; j < (G + 1) / 2; ++j) s_red[wv][G > 1 ? 2 * j + odd : 0] = l[j];   // (G = 1: both rows write the sum)
                }
            }
        } else {
#pragma unroll
            for (int hh = 0; hh < G; ++hh)
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[hh][e] = group16_sum(acc[hh][e]);
#pragma unroll
            for (int hh = 0; hh < G; ++hh) lsum[hh] = group16_sum(lsum[hh]);
            if ((ln & 15) == 0) {
#pragma unroll
                for (int hh = 0; hh < G; ++hh)
#pragma unroll
                    for (int e = 0; e < 8; ++e) s_o[wv][hh][quad * 8 + e] = acc[hh][e];
                if (quad == 0) {
#pragma unroll
                    for (int hh = 0; hh < G; ++hh) s_red[wv][hh] = lsum[hh];
                }
            }
        }
    };
    {
        uint32_t big = 0;   // heads of which this wave has seen a weight that is not vanishing
#pragma unroll
        for (int hh = 0; hh < G; ++hh) big |= (uint32_t)(__ballot(lsum[hh] >= 1e-30f) != 0ull) << hh;
        if (ln == 0) s_big[wv] = big;
    }
    hand_over();
    __syncthreads();
    CTKVR_STAMP(45);
    uint32_t big = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) big |= s_big[w];
    if (big != (1u << G) - 1u) {   // uniform: a head whose selected logits all lie far below its maximum
        // two passes instead: the selected keys' own maxima first, then weights relative to them
        __syncthreads();
        float mx[G];
#pragma unroll
        for (int hh = 0; hh < G; ++hh) mx[hh] = -__builtin_huge_valf();
        for (int t = tid; t < nsel; t += NT) {
            float zv[G];
            z_of(t, zv);
#pragma unroll
            for (int hh = 0; hh < G; ++hh) {
                s_p[t * G + hh] = zv[hh];
                mx[hh] = fmaxf(mx[hh], zv[hh]);
            }
        }
#pragma unroll
        for (int hh = 0; hh < G; ++hh) {
            float v = mx[hh];
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
            if (ln == 0) s_red[wv][hh] = v;
        }
        __syncthreads();
        if (tid < G) {
            float v = s_red[0][tid];
#pragma unroll
            for (int w = 1; w < NW; ++w) v = fmaxf(v, s_red[w][tid]);
            s_m[tid] = v;
        }
        __syncthreads();
#pragma unroll
        for (int hh = 0; hh < G; ++hh) {
            mx[hh] = s_m[hh];
            lsum[hh] = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[hh][e] = 0.0f;
        }
        // weighted sum of the value rows
        for (int r0 = 0; r0 < nsel; r0 += NU * PASS) {
#pragma unroll
            for (int u = 0; u < NU; ++u) vrow[u] = row_of(min(r0 + u * PASS + rin, a.top_k - 1));
#pragma unroll
            for (int u = 0; u < NU; ++u) cv[u] = load_chunk(V + (size_t)vrow[u] * kD, 0);
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                int t = r0 + u * PASS + rin;
                if (t < nsel) {
                    float vx[8], zv[G];
                    unpack(cv[u], vx);
                    load_z<G>(s_p, t, zv);
#pragma unroll
                    for (int hh = 0; hh < G; ++hh) {
                        const float pw = __expf(zv[hh] - mx[hh]);
                        lsum[hh] += pw;
#pragma unroll
                        for (int e = 0; e < 8; ++e) acc[hh][e] = __fmaf_rn(pw, vx[e], acc[hh][e]);
                    }
                }
            }
        }
        __syncthreads();
        hand_over();
        __syncthreads();
    }
    CTKVR_STAMP(46);
    // then over the block's waves, in order
    if (tid < G * kSliceDims) {
        int hh = tid / kSliceDims, e = tid % kSliceDims;
        float v = 0.0f, l = 0.0f;
#pragma unroll
        for (int w = 0; w < kProd; ++w) {
            v += s_o[w][hh][e];
            l += s_red[w][hh];
        }
        float lse;
        const float o = merge_window<G>(a.win, ul, hh, slice * kSliceDims + e, v, s_m[hh], l, lse);
        a.out[((size_t)b * a.h + kv * G + hh) * kD + slice * kSliceDims + e] = o;
        if (slice == 0 && e == 0 && a.out_lse) a.out_lse[(size_t)b * a.h + kv * G + hh] = lse;
    }
    CTKVR_STAMP(47);
    CTKVR_STAMP_BLK(5);
}

template <typename T, int G, int SL> __global__ __launch_bounds__(1024) void sparse_attn_kernel(AttnArgs a)
{
    extern __shared__ __align__(16) float s_p[];   // [top_k][G]
    int ul, slice;
    attn_block_of<SL>(ul, slice);
    const uint32_t *rb = a.srow + (size_t)ul * a.top_k;
    const float *zb = a.zsel + (size_t)ul * a.top_k * G;
    attend_unit<T, G, SL, (G == 8 ? 2 : 4), 1024>(a, ul, slice, s_p, [&](int t) { return rb[t]; }, [&](int t, float(&zv)[G]) { load_z<G>(zb, t, zv); },
                      [&]() { return a.nsel[ul]; });
}

// ------------------------------------------------------------------------------
// Algorithm 2 lines 6-9 in one launch, for batches small enough that every block has a CU of its
// own: each of the SL slice blocks of a unit makes the unit's selection itself (the same work
// several times over, on as many CUs, instead of a second launch and a round trip of the picks through
// global memory) and then attends over the picks straight from the recalled ids' rows and logits.
// Slice 0 also writes the selected ids and their number.  grid SL*batch*g, 1024 threads; dynamic
// shared memory: the selection's words, then top_k*G floats.
// ------------------------------------------------------------------------------
template <typename T, int G, int SL> __global__ __launch_bounds__(1024) void select_attn_kernel(SelectArgs sa, AttnArgs a)
{
    extern __shared__ __align__(16) uint32_t smem[];
    int ul, slice;
    attn_block_of<SL>(ul, slice);
    const int L = sa.ncand[ul];
    CTKVR_STAMP(28);
    const int n = select_unit<G>(sa, ul, L, smem);
    __syncthreads();
    const int32_t *s_idx = (const int32_t *)(smem + kSelLds + 2 * kListCap + sa.bits_words);
    float *s_p = reinterpret_cast<float *>(smem + select_smem_words(sa.bits_words, sa.top_k));
    const int32_t *cb = sa.cand + (size_t)ul * sa.l_stride;
    const uint32_t *rb = sa.crow + (size_t)ul * sa.l_stride;
    const float *zb = sa.z + (size_t)ul * sa.l_stride * G;
    CTKVR_STAMP(31);
    if (slice == 0) {
        int32_t *dst = sa.sel + (size_t)ul * sa.top_k;
        int32_t *dst2 = sa.out_sel ? sa.out_sel + (size_t)ul * sa.top_k : nullptr;
        for (int pos = threadIdx.x; pos < sa.top_k; pos += 1024) {
            const int t = pos < n ? cb[s_idx[pos]] : -1;
            dst[pos] = t;
            if (dst2) dst2[pos] = t;
        }
        if (threadIdx.x == 0) sa.nsel[ul] = n;
    }
    // positions beyond n repeat the last pick; when nothing was recalled every position reads slot 0 of
    // the row table and then names row 0 of the pool (selects, not a branch: the four row numbers of a
    // pass are then requested together)
    attend_unit<T, G, SL, (G == 8 ? 2 : 4), 1024>(a, ul, slice, s_p,
                      [&](int t) {
                          const uint32_t r = rb[n > 0 ? s_idx[min(t, n - 1)] : 0];
                          return n > 0 ? r : 0u;
                      },
                      [&](int t, float(&zv)[G]) { load_z<G>(zb, n > 0 ? s_idx[min(t, n - 1)] : 0, zv); }, [&]() { return n; });
}

// ------------------------------------------------------------------------------
// The top_k largest of L ranking keys, n_real > top_k of them above -inf (ties: lowest positions), by one block of NT threads: the keys of positions
// (q NT/64 + wave) 64 + lane sit in kreg[q] of their thread (-inf beyond L and where a key is out of the running), those beyond KPT NT come from for_far (f(group of
// 64 positions, key) for the groups of the calling wave).  Histogram over key buckets in shared memory, the deciding
// bucket, a bitmap of the positions above it, that bucket's own keys ranked against each other, and the picks in
// ascending order: either (PLACE, all keys in registers) place(q, group, rank) for the lane's own key in kreg[q], and the function
// returns true, or emit(rank, position) by any thread, and it returns false.  Placing walks all groups of a wave, some twenty
// instructions each: for callers that need the lane's registers.  s_hist: kSelLds words whose first kBuckets are zero; s_list: 2 kListCap;
// s_bits: 4 ceil(L / 64); s_res: 4, s_res[3] zero.  The caller places a barrier before and after.
// key(position) = the key's ordered image, for a crowded deciding bucket (all keys are then walked again).
// ------------------------------------------------------------------------------
template <int NT, int KPT, bool PLACE, typename FarFn, typename PlaceFn, typename EmitFn, typename KeyFn>
__device__ __forceinline__ bool select_keys(const float (&kreg)[KPT], const int L, const int n_real, const int top_k, FarFn for_far,
                                            PlaceFn place, EmitFn emit, KeyFn key, uint32_t *s_hist, uint32_t *s_list, uint32_t *s_bits, uint32_t *s_res)
{
    constexpr int NW = NT / 64;
    static_assert(KPT <= 64, "the picks' ranks: a round of groups per lane");
    const int tid = threadIdx.x, ln = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // key_bucket(ordered_key(x)), from the key as a float
    auto bucket_of = [&](float x) __attribute__((always_inline)) {
        return (uint32_t)__builtin_amdgcn_fmed3f(x * -32.0f, 0.0f, (float)(kBuckets - 1));
    };
    // the last bucket (everything below the histogram's range, often most keys) is not counted: L minus the others
    const float floor_k = -(float)(kBuckets - 1) / 32.0f;
    // (no branch: lanes that do not count add to a word of their own)
    auto count = [&](int, float kk) __attribute__((always_inline)) {
        uint32_t *bin = &s_hist[bucket_of(kk)];
        bin = kk > floor_k ? bin : s_list + tid;
        atomicAdd(bin, 1u);
    };
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
        if (q % 4 == 0 && (q * NW + wv) * 64 >= L) break;
        count(q, kreg[q]);
    }
    for_far(count);
    CTKVR_STAMP(67);
    __syncthreads();
    uint32_t *s_scan = s_hist + 2048 + 4;
    {
        constexpr int BPT = kBuckets / NT;   // buckets per thread, in descending key order
        uint32_t c[BPT], mine = 0;
#pragma unroll
        for (int q = 0; q < BPT; ++q) {
            c[q] = s_hist[BPT * tid + q];
            mine += c[q];
        }
        uint32_t tot;
        uint32_t before = block_excl_scan<NT>(mine, s_scan, &tot);
        const uint32_t want = (uint32_t)top_k;
        if (want > tot) {   // (uniform) the last bucket decides
            if (tid == 0) {
                s_res[0] = (uint32_t)(kBuckets - 1);
                s_res[1] = want - tot;
                s_res[2] = (uint32_t)n_real - tot;
            }
        } else
#pragma unroll
        for (int q = 0; q < BPT; ++q) {
            if (before < want && want <= before + c[q]) {
                s_res[0] = (uint32_t)(BPT * tid + q);
                s_res[1] = want - before;
                s_res[2] = c[q];
            }
            before += c[q];
        }
    }
    __syncthreads();
    const uint32_t bkt = s_res[0], rem = s_res[1], nb = s_res[2];
    CTKVR_STAMP(68);
    // the deciding bucket as an interval of keys: x > hi is above it, lo < x <= hi in it (exact: x * 32 is)
    const float hi_k = bkt == 0u ? __builtin_huge_valf() : -(float)bkt / 32.0f;
    const float lo_k = bkt == (uint32_t)(kBuckets - 1) ? -__builtin_huge_valf() : -(float)(bkt + 1u) / 32.0f;
    if (nb <= (uint32_t)kListCap) {
        const int nw32 = 2 * ((L + 63) >> 6);
        uint32_t *s_gt = s_bits, *s_eq = s_bits + nw32;
        uint2 *l_ent = reinterpret_cast<uint2 *>(s_list);
        const bool few = nb <= (uint32_t)NT / 2;   // ranked by all-pairs comparison: ids decide between equal keys
        uint32_t *s_rank = s_hist;     // (everyone has read the histogram)
        if (tid < NT / 2) s_rank[tid] = 0u;
        auto list = [&](uint64_t listed, uint32_t at, float kk, int i) __attribute__((always_inline)) {
            const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(listed >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)listed, at));
            if (__builtin_amdgcn_inverse_ballot_w64(listed)) l_ent[pos] = make_uint2(ordered_key(kk), (uint32_t)i);
        };
        // the wave's verdicts first, then one cursor bump for all its entries of the deciding bucket
        uint64_t mine_gt = 0;   // lane q: the verdicts of group q
        uint32_t n_in = 0;
#pragma unroll
        for (int q = 0; q < KPT; ++q) {
            if (q % 4 == 0 && (q * NW + wv) * 64 >= L) break;
            const uint64_t above = __ballot(kreg[q] > hi_k);
            n_in += (uint32_t)__popcll(__ballot(kreg[q] > lo_k) & ~above);
            mine_gt = ln == q ? above : mine_gt;
        }
        if (ln < KPT && (ln * NW + wv) * 64 < L)
            *reinterpret_cast<uint2 *>(s_gt + 2 * (ln * NW + wv)) = make_uint2((uint32_t)mine_gt, (uint32_t)(mine_gt >> 32));
        if (n_in) {
            uint32_t at0 = 0;
            if (ln == 0) at0 = atomicAdd(&s_res[3], n_in);
            at0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)at0);
#pragma unroll
            for (int q = 0; q < KPT; ++q) {
                if (q % 4 == 0 && (q * NW + wv) * 64 >= L) break;
                const uint64_t in = __ballot(kreg[q] > lo_k) & ~__ballot(kreg[q] > hi_k);
                if (in) {
                    list(in, at0, kreg[q], (q * NW + wv) * 64 + ln);
                    at0 += (uint32_t)__popcll(in);
                }
            }
        }
        for_far([&](int gq, float kk) __attribute__((always_inline)) {
            const uint64_t above = __ballot(kk > hi_k);
            const uint64_t listed = __ballot(kk > lo_k) & ~above;
            if (ln == 0) *reinterpret_cast<uint2 *>(s_gt + 2 * gq) = make_uint2((uint32_t)above, (uint32_t)(above >> 32));
            if (listed) {
                uint32_t at1 = 0;
                if (ln == 0) at1 = atomicAdd(&s_res[3], (uint32_t)__popcll(listed));
                list(listed, (uint32_t)__builtin_amdgcn_readfirstlane((int)at1), kk, gq * 64 + ln);
            }
        });
        if (!few)
            for (int w = tid; w < nw32; w += NT) s_eq[w] = 0u;
        __syncthreads();
        CTKVR_STAMP(69);
        if (few) {
            uint32_t cap = 64;
            while (cap < nb) cap <<= 1;
            const uint32_t parts = (uint32_t)NT / cap, e = (uint32_t)tid & (cap - 1u), part = (uint32_t)tid / cap;
            if (e < nb) {
                const uint2 me = l_ent[e];
                uint32_t rank = 0;
                for (uint32_t f = part; f < nb; f += parts) {
                    const uint2 o = l_ent[f];
                    rank += (o.x > me.x) || (o.x == me.x && o.y < me.y);
                }
                atomicAdd(&s_rank[e], rank);
            }
            __syncthreads();
            if ((uint32_t)tid < nb && s_rank[tid] < rem) {
                const uint32_t id = l_ent[tid].y;
                atomicOr(&s_gt[id >> 5], 1u << (id & 31u));
            }
            __syncthreads();
            CTKVR_STAMP(70);
            if (PLACE && L <= KPT * NT) {   // uniform
                // every wave counts the whole bitmap (lane q: the NW groups of round q), scans it by itself, and places its
                // own groups' picks
                uint32_t all = 0, before = 0;
#pragma unroll
                for (int j = 0; j < NW; j += 2) {
                    const int gq = ln * NW + j;
                    uint4 w4 = make_uint4(0u, 0u, 0u, 0u);
                    if (ln < KPT && 2 * gq < nw32) w4 = *reinterpret_cast<const uint4 *>(s_gt + 2 * gq);
                    const uint32_t c0 = (uint32_t)(__popc(w4.x) + __popc(w4.y));
                    const uint32_t c1 = 2 * gq + 2 < nw32 ? (uint32_t)(__popc(w4.z) + __popc(w4.w)) : 0u;
                    all += c0 + c1;
                    before += (j < wv ? c0 : 0u) + (j + 1 < wv ? c1 : 0u);
                }
                const uint32_t first = wave_incl_scan(all) - all + before;
                uint2 mine = make_uint2(0u, 0u);
                if (ln < KPT && 2 * (ln * NW + wv) < nw32) mine = *reinterpret_cast<const uint2 *>(s_gt + 2 * (ln * NW + wv));
#pragma unroll
                for (int q = 0; q < KPT; ++q) {
                    const int gq = q * NW + wv;
                    if (q % 4 == 0 && gq * 64 >= L) break;
                    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)mine.x, q);
                    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)mine.y, q);
                    const uint32_t base = (uint32_t)__builtin_amdgcn_readlane((int)first, q);
                    const uint32_t pos = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, base));
                    if (__builtin_amdgcn_inverse_ballot_w64(((uint64_t)hi << 32) | lo)) place(q, gq, pos);
                }
                return true;
            } else if (2 * nw32 >= NT) {
                // thread t owns the words [t wpt, (t + 1) wpt) of the bitmap: count, scan, emit in ascending order
                const int wpt = (nw32 + NT - 1) / NT, w0 = min(nw32, tid * wpt), w1 = min(nw32, w0 + wpt);
                uint32_t cnt = 0;
                for (int w = w0; w < w1; ++w) cnt += (uint32_t)__popc(s_gt[w]);
                uint32_t tot;
                uint32_t pos = block_excl_scan<NT>(cnt, s_scan, &tot);
                for (int w = w0; w < w1; ++w) {
                    uint32_t mm = s_gt[w];
                    while (mm) {
                        const int bit = __ffs((int)mm) - 1;
                        mm &= mm - 1u;
                        emit((int)pos++, w * 32 + bit);
                    }
                }
            } else {
                // the same by bytes, where there are few words
                const unsigned char *bytes = reinterpret_cast<const unsigned char *>(s_gt);
                const int nbyte = nw32 * 4, bpt = (nbyte + NT - 1) / NT;
                const int b0 = min(nbyte, tid * bpt), b1 = min(nbyte, b0 + bpt);
                uint32_t cnt = 0;
                for (int w = b0; w < b1; ++w) cnt += (uint32_t)__popc((uint32_t)bytes[w]);
                uint32_t tot;
                uint32_t pos = block_excl_scan<NT>(cnt, s_scan, &tot);
                for (int w = b0; w < b1; ++w) {
                    uint32_t mm = bytes[w];
                    while (mm) {
                        const int bit = __ffs((int)mm) - 1;
                        mm &= mm - 1u;
                        emit((int)pos++, w * 8 + bit);
                    }
                }
            }
        } else {
            block_resolve_emit<NT>(nb, rem, L, s_hist, s_gt, s_eq, l_ent, emit);
        }
    } else {   // a crowded deciding bucket (equal keys, or keys below the histogram's range)
        block_select_topk<NT, 0>(key, L, top_k, emit, s_hist);
    }
    return false;
}

// ------------------------------------------------------------------------------
// Exact list build (Algorithm 1 lines 2-4 in the fixed arithmetic of the decode path) on the fp32 matrix cores.  A
// v_mfma_f32_32x32x2f32 adds its two products to the accumulator one after the other, each as a fused multiply-add with
// one rounding (probes/mfma_chain_probe.hip compares 2 M results of normal, bf16, wide-range and subnormal values with fmaf: no
// bit differs), so the fixed dot product -- sixteen chains of eight fused multiply-adds, combined as a balanced tree -- is
// sixteen groups of four such instructions, each group from zero, and fifteen vector adds.
// exact_score_kernel: z[unit][head][key] = (c . k) scale for a chunk of tiles of CT = 32 (8 / G) centroids of one
// (sequence, KV head), all its G heads and all s keys, and the block's maximum of each unit and head, for exact_list_kernel to merge
// (as atomics, with few lists the blocks of all keys met on a few lines: 4096 tokens, 64 centroids, two KV heads 39.2 -> 20.6 us,
// 8192 tokens, 128 centroids, one 71 -> 22; large builds the same).  Eight waves, each with one item of 32
// centroids of one head, whose fragments stay in 64 registers (a lane needs every other element: the instruction's two
// k's sit in the two halves of a wave); the keys go by 32 at a time through shared memory as fp32, even and odd elements of
// each group of eight apart so that a fragment is one 16-byte read.  Bound by the matrix pipe (64 instructions of 64 clocks
// per 32 x 32 scores against about 1.2 k clocks of vector work; fp32 peak 157 TFLOP/s): at 32K tokens, C = 512,
// 32/8 heads 1.45 ms (four chunks of 361 us, 95 TFLOP/s) where the scalar form (score_kernel) took 4.7; at 128K 104 TFLOP/s with the
// matrix pipe busy for 65 % of the cycles, vector instructions issuing for another 20 %, waves waiting for 24 %.
// grid (t_splits, tiles of the chunk), 512 threads
// ------------------------------------------------------------------------------
struct ExactScoreArgs {
    int g, h, c_max;
    int tile0, tiles_per_bk;   // first tile of the chunk; tiles per (sequence, KV head)
    int t_splits;
    const int32_t *n_cent, *ctx_lens;
    const void *centroids;     // [batch][h][c_max][128]
    Paged k;
    int z_stride;              // floats per (unit, head) row: a multiple of 4, >= s_max
    float *z;                  // [chunk units = tiles * CT][G][z_stride]
    uint32_t *m_part;          // [chunk units][t_splits][G] ordered keys of the blocks' maxima
    float scale;
};

template <typename T, int G> __global__ __launch_bounds__(512) void exact_score_kernel(ExactScoreArgs a)
{
    constexpr int CT = 32 * (8 / G), ROWW = 132;   // floats per staged key row (128 + 4: rows spread over the banks)
    __shared__ __align__(16) float s_k[2][64 * ROWW];   // two steps of 32 keys per buffer and barrier
    const int tid = threadIdx.x, ln = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = ln & 31, half = ln >> 5;
    const int tile = a.tile0 + (int)blockIdx.y, bk = tile / a.tiles_per_bk, jt = tile - bk * a.tiles_per_bk;
    const int b = bk / a.g, kv = bk - b * a.g;
    const int C = a.n_cent[b], s = a.ctx_lens[b];
    const int j0 = jt * CT;
    if (j0 >= C) return;
    const int tper = (((s + a.t_splits - 1) / a.t_splits) + 31) & ~31;
    const int tbeg = (int)blockIdx.x * tper, tend = min(s, tbeg + tper);
    if (tbeg >= tend) return;
    const int mt = wv / G, hh = wv - mt * G;   // this wave's item
    float cf[64];                              // elements 8 l + 2 i + half of centroid j0 + 32 mt + col at [4 l + i]
    {
        const int j = min(j0 + mt * 32 + col, C - 1);   // rows beyond C repeat centroid C-1; nothing reads their units
        const T *row = (const T *)a.centroids + (((size_t)b * a.h + kv * G + hh) * a.c_max + j) * kD;
#pragma unroll
        for (int l = 0; l < 16; ++l) {
            float x[8];
            unpack(load_chunk(row, l), x);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                asm volatile("" : "+v"(x[2 * i]), "+v"(x[2 * i + 1]));   // (a select of two registers, not an indexed load)
                cf[4 * l + i] = half ? x[2 * i + 1] : x[2 * i];
            }
        }
    }
    const T *K = (const T *)a.k.pages;
    const int srow = tid >> 4, lane16 = tid & 15;
    const int32_t *bt_row = a.k.block_table + (size_t)b * a.k.max_pages;
    auto page_at = [&](int t0) { return bt_row[min(t0 + srow, s - 1) >> a.k.page_shift]; };
    auto fetch = [&](int page, int t0) {
        const uint32_t row = (uint32_t)((page * a.g + kv) << a.k.page_shift) + (uint32_t)(min(t0 + srow, s - 1) & ((1 << a.k.page_shift) - 1));
        return load_chunk(K + (size_t)row * kD, lane16);
    };
    auto put = [&](const Chunk<T> &c, int buf, int sub) __attribute__((always_inline)) {
        float x[8];
        unpack(c, x);
        float4 *dst = reinterpret_cast<float4 *>(&s_k[buf][(sub * 32 + srow) * ROWW + lane16 * 8]);
        dst[0] = make_float4(x[0], x[2], x[4], x[6]);
        dst[1] = make_float4(x[1], x[3], x[5], x[7]);
    };
    float mx[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) mx[r] = -__builtin_huge_valf();
    // The centroids are the rows of the instruction and the keys its columns: result register r holds centroid row
    // 8 (r / 4) + 4 half + r % 4 of the item against key `col` of the step, and a store writes two whole 128-byte lines (with
    // the roles exchanged a lane stores 16 bytes, but 32 to a line, and the stores took longer than the matrix work).
    const size_t unit0 = (size_t)blockIdx.y * CT + mt * 32;
    const size_t rstep = (size_t)G * a.z_stride;
    char *zb = reinterpret_cast<char *>(a.z + (unit0 * G + hh) * a.z_stride);   // wave-uniform
    const uint32_t lane_off = ((uint32_t)(4 * half * rstep) + col) * 4u;
    // A step's results leave the registers during the next step, a row per chain (all of them at the end of a step, before a
    // barrier, left the matrix pipe half idle).
    f32x16_t pz;
#pragma unroll
    for (int r = 0; r < 16; ++r) pz[r] = -__builtin_huge_valf();
    int pt = tend;   // the step they belong to (none yet)
    auto row_out = [&](int r, bool whole, uint32_t off) __attribute__((always_inline)) {
        const float z = pz[r] * a.scale;
        mx[r] = fmaxf(mx[r], z);   // (a tail's repeated keys are real ones: harmless for a maximum)
        float *dst = reinterpret_cast<float *>(zb + (8 * (r >> 2) + (r & 3)) * rstep * 4 + off);
        if (whole || pt + col < tend) *dst = z;
    };
    auto step = [&](const float *kr, int t0, bool have_prev) __attribute__((always_inline)) {   // have_prev: and it is a whole step
        const uint32_t off = lane_off + (uint32_t)pt * 4u;
        // the tree over the sixteen partials
        f32x16_t lv[4], p;
        float4 kn = *reinterpret_cast<const float4 *>(kr);
#pragma unroll
        for (int l = 0; l < 16; ++l) {
            const float4 kx = kn;
            if (l < 15) kn = *reinterpret_cast<const float4 *>(kr + (l + 1) * 8);
            p = f32x16_t{};
            p = __builtin_amdgcn_mfma_f32_32x32x2f32(cf[4 * l + 0], kx.x, p, 0, 0, 0);
            p = __builtin_amdgcn_mfma_f32_32x32x2f32(cf[4 * l + 1], kx.y, p, 0, 0, 0);
            p = __builtin_amdgcn_mfma_f32_32x32x2f32(cf[4 * l + 2], kx.z, p, 0, 0, 0);
            p = __builtin_amdgcn_mfma_f32_32x32x2f32(cf[4 * l + 3], kx.w, p, 0, 0, 0);
            if (have_prev) row_out(l, true, off);
            if (l & 1) p = lv[0] + p;
            if ((l & 3) == 3) p = lv[1] + p;
            if ((l & 7) == 7) p = lv[2] + p;
            if (l == 15) p = lv[3] + p;
            // (left to itself the compiler starts all the chains before the first add, and spills: the sum is pinned here)
            asm volatile("" : "+v"(p));
            __builtin_amdgcn_sched_barrier(0);
            if (!(l & 1)) lv[0] = p;
            else if ((l & 3) == 1) lv[1] = p;
            else if ((l & 7) == 3) lv[2] = p;
            else if (l == 7) lv[3] = p;
        }
        pz = p;
        pt = t0;
    };
    int pg0 = page_at(tbeg + 64), pg1 = page_at(tbeg + 96);
    Chunk<T> st0 = fetch(page_at(tbeg), tbeg), st1 = fetch(page_at(tbeg + 32), tbeg + 32);
    put(st0, 0, 0);
    put(st1, 0, 1);
    __syncthreads();
    int buf = 0;
    auto pair = [&](int t0, bool have_prev) __attribute__((always_inline)) {
        const float *kr = &s_k[buf][col * ROWW + half * 4];
        st0 = fetch(pg0, t0 + 64);   // the next pair of steps (clamped rows beyond the sequence)
        st1 = fetch(pg1, t0 + 96);
        pg0 = page_at(t0 + 128);
        pg1 = page_at(t0 + 160);
        step(kr, t0, have_prev);
        put(st0, buf ^ 1, 0);
        put(st1, buf ^ 1, 1);
        if (t0 + 32 < tend) step(kr + 32 * ROWW, t0 + 32, true);   // uniform
        __syncthreads();
        buf ^= 1;
    };
    pair(tbeg, false);
    for (int t0 = tbeg + 64; t0 < tend; t0 += 64) pair(t0, true);
#pragma unroll
    for (int r = 0; r < 16; ++r) row_out(r, false, lane_off + (uint32_t)pt * 4u);
    // the maxima over the wave's 32 keys of a row: DPP inside rows of 16 lanes, then the two rows of a half; lane r of a half
    // stores row r's
    uint32_t own = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        float v = mx[r];
        v = fmaxf(v, dpp_f<0xB1>(v));
        v = fmaxf(v, dpp_f<0x4E>(v));
        v = fmaxf(v, dpp_f<0x141>(v));
        v = fmaxf(v, dpp_f<0x140>(v));
        v = fmaxf(v, __shfl_xor(v, 16));
        own = col == r ? ordered_key(v) : own;
    }
    if (col < 16) a.m_part[((unit0 + 4 * half + 8 * (col >> 2) + (col & 3)) * a.t_splits + blockIdx.x) * G + hh] = own;
}

// exact_list_kernel: the list of one unit of the chunk per block: denominators of its G heads over all s scores, ranking
// keys max_h ((z - m_h) - log S_h), the rho largest (select_keys; keys of up to KPT NT positions in registers, the
// scores of positions beyond that are read again).  The scores are read twice, the second time mostly from the memory-side
// cache; nothing is written but the list.  Bound by the vector instructions of the exponentials (about 16 us a list of 32K and a
// CU) and by the latencies of a block's phases, which other blocks on the CU hide: 512 threads up to 16384 positions (two
// blocks at 108 registers a thread; with 1024 threads one, and 6000 / 10000 / 16384 positions took 70 / 124 / 226 us where
// this takes 38 / 87 / 177 for 1024 / 1536 / 2048 lists), beyond that 1024 threads, one block at 102 to 116 registers, or (PAIR)
// held to 64, two blocks in spite of some 40 spilled (four heads: 197 -> 176 us for 1024 lists of 32768).  The rule is at the launch.
// The heads' maxima are kept in scalar registers: as vector registers they made a block of eight heads and 131072 positions take 411 us,
// now 341.
// grid (chunk units), NT threads; dynamic shared memory: kSelLds + 2 kListCap + 4 ceil(s_max / 64) words
struct ExactListArgs {
    int g, c_max, tile0, tiles_per_bk, ct;   // ct: centroids per tile
    const int32_t *n_cent, *ctx_lens;
    int z_stride, rho, n_init, n_local;
    const float *z;
    int t_splits;                            // of exact_score_kernel
    const uint32_t *m_part;
    int32_t *lists;                          // [all units][c_max][rho]
};

template <int G, int NT, int KPT, bool PAIR = false> __global__ __launch_bounds__(NT, (PAIR ? 8 : 1)) void exact_list_kernel(ExactListArgs a)
{
    extern __shared__ __align__(16) uint32_t smem[];
    constexpr int NW = NT / 64;
    __shared__ unsigned long long s_acc[NW][G];
    __shared__ float s_ls[G];
    __shared__ uint32_t s_res[4];
    uint32_t *s_hist = smem, *s_list = smem + kSelLds, *s_bits = s_list + 2 * kListCap;
    const int ul = blockIdx.x, tid = threadIdx.x, ln = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile = a.tile0 + ul / a.ct, bk = tile / a.tiles_per_bk, j = (tile - bk * a.tiles_per_bk) * a.ct + ul % a.ct;
    const int b = bk / a.g;
    if (j >= a.n_cent[b]) return;
    const int s = a.ctx_lens[b];
    const float *zb = a.z + (size_t)ul * G * a.z_stride;
    // the maxima over the scoring blocks that had keys, in every wave
    float m[G];
    {
        const int tper = (((s + a.t_splits - 1) / a.t_splits) + 31) & ~31, nx = min(a.t_splits, (s + tper - 1) / tper);
        const uint32_t *pp = a.m_part + (size_t)ul * a.t_splits * G;
        uint32_t mk[G];
#pragma unroll
        for (int hh = 0; hh < G; ++hh) mk[hh] = 0u;
        for (int x = ln; x < nx; x += 64) {
#pragma unroll
            for (int hh = 0; hh < G; ++hh) mk[hh] = max(mk[hh], pp[x * G + hh]);
        }
#pragma unroll
        for (int hh = 0; hh < G; ++hh) {
            const float v = ordered_value(wave_fold_uniform(mk[hh], [](uint32_t x, uint32_t y) { return max(x, y); }));
            m[hh] = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(v)));
        }
    }
    for (int w = tid; w < kBuckets / 4; w += NT) reinterpret_cast<uint4 *>(s_hist)[w] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0) s_res[3] = 0u;
    // denominators: four keys per load, two loads in flight per head (terms beyond s count as none)
#pragma unroll
    for (int hh = 0; hh < G; ++hh) {
        const float4 *row = reinterpret_cast<const float4 *>(zb + (size_t)hh * a.z_stride);
        const int n4 = (s + 3) >> 2;
        unsigned long long acc = 0;
        constexpr int UN = 4;
        for (int i0 = tid; i0 - ln < n4; i0 += UN * NT) {
            float4 v[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) v[u] = row[min(i0 + u * NT, n4 - 1)];
            uint32_t shi = 0, slo = 0;   // 16 terms: hi <= 2^16 and lo < 2^24 each
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int i = 4 * (i0 + u * NT);
                const float x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint32_t hi, lo;
                    exp_fixed40_parts(i + e < s ? x[e] - m[hh] : -40.0f, hi, lo);
                    shi += hi;
                    slo += lo;
                }
            }
            acc += ((unsigned long long)shi << 24) + slo;
        }
        // a wave's sum in three 24-bit pieces: 64 lanes of each fit 32 bits
        const uint32_t p0 = wave_sum_last((uint32_t)acc & 0xffffffu), p1 = wave_sum_last((uint32_t)(acc >> 24) & 0xffffffu),
                       p2 = wave_sum_last((uint32_t)(acc >> 48));
        if (ln == 63) s_acc[wv][hh] = (unsigned long long)p0 + ((unsigned long long)p1 << 24) + ((unsigned long long)p2 << 48);
    }
    __syncthreads();
    if (tid < G) {
        unsigned long long v = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += s_acc[w][tid];
        s_ls[tid] = (float)log_fixed40(v);
    }
    __syncthreads();
    float ls[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) ls[hh] = s_ls[hh];
    auto key_at = [&](int i) __attribute__((always_inline)) {   // i < s_max
        float best = (zb[i] - m[0]) - ls[0];
#pragma unroll
        for (int hh = 1; hh < G; ++hh) best = fmaxf(best, (zb[(size_t)hh * a.z_stride + i] - m[hh]) - ls[hh]);
        return fmaxf(best, -3.0e38f);
    };
    auto listed = [&](int i) { return i < s - a.n_local && i >= a.n_init; };   // keys of the resident window enter no list
    float kreg[KPT];
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
        const int i = q * NT + tid;
        const float x = key_at(min(i, s - 1));
        kreg[q] = listed(i) ? x : -__builtin_huge_valf();
    }
    int32_t *dst = a.lists + ((size_t)bk * a.c_max + j) * a.rho;
    const int n_real = s - a.n_local - a.n_init;
    if (a.rho >= n_real) {   // every key outside the window
        for (int i = tid; i < a.rho; i += NT) dst[i] = a.n_init + i;
        return;
    }
    select_keys<NT, KPT, false>(
        kreg, s, n_real, a.rho,
        [&](auto f) __attribute__((always_inline)) {
            for (int gq = KPT * NW + wv; gq * 64 < s; gq += NW) {
                const int i = gq * 64 + ln;
                const float x = key_at(min(i, s - 1));
                f(gq, listed(i) ? x : -__builtin_huge_valf());
            }
        },
        [&](int, int gq, uint32_t pos) __attribute__((always_inline)) { dst[pos] = gq * 64 + ln; },
        [&](int pos, int i) __attribute__((always_inline)) { dst[pos] = i; },
        [&](int i) { return listed(i) ? ordered_key(key_at(i)) : 0x007fffffu; }, s_hist, s_list, s_bits, s_res);
}

// key_list_kernel: the list of one unit of the chunk per block, from its s ranking keys (the matrix-core build's every-key
// route): the same selection, keys of up to KPT NT positions read once into registers.  A histogram launch and a
// selection launch, each reading all keys and meeting in memory, took 0.41 + 0.40 ms for the 160 M keys of 9720 lists;
// this 0.47 ms, bound by the latencies of a list's phases: two blocks of 512 threads per CU hide them better than one of
// 1024 (0.61 ms).  Beyond 32768 positions, where keys are read again, 1024 threads are 5 % faster.
// grid (chunk units), NT threads, dynamic shared memory as above.
struct KeyListArgs {
    int g, c_max, unit0;
    const int32_t *n_cent, *ctx_lens;
    int l_stride, rho, n_init, n_local;
    const uint32_t *kbuf;                    // [chunk units][l_stride], the window's keys the image of -inf
    int32_t *lists;                          // [all units][rho]
};

template <int NT, int KPT> __global__ __launch_bounds__(NT, 4) void key_list_kernel(KeyListArgs a)
{
    extern __shared__ __align__(16) uint32_t smem[];
    constexpr int NW = NT / 64;
    __shared__ uint32_t s_res[4];
    uint32_t *s_hist = smem, *s_list = smem + kSelLds, *s_bits = s_list + 2 * kListCap;
    const int ul = blockIdx.x, tid = threadIdx.x, ln = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int unit = a.unit0 + ul, bk = unit / a.c_max, b = bk / a.g;
    if (unit - bk * a.c_max >= a.n_cent[b]) return;
    const int s = a.ctx_lens[b];
    const uint32_t *kb = a.kbuf + (size_t)ul * a.l_stride;
    int32_t *dst = a.lists + (size_t)unit * a.rho;
    const int n_real = s - a.n_local - a.n_init;
    if (a.rho >= n_real) {   // every key outside the window
        for (int i = tid; i < a.rho; i += NT) dst[i] = a.n_init + i;
        return;
    }
    auto key_at = [&](int i) __attribute__((always_inline)) {   // above -inf exactly outside the window
        const float x = fmaxf(ordered_value(kb[min(i, s - 1)]), -3.0e38f);
        return i < s - a.n_local && i >= a.n_init ? x : -__builtin_huge_valf();
    };
    float kreg[KPT];
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
        if (q % 4 == 0 && (q * NW + wv) * 64 >= s) break;   // rounds that select_keys does not look at either
        kreg[q] = key_at(q * NT + tid);
    }
    for (int w = tid; w < kBuckets / 4; w += NT) reinterpret_cast<uint4 *>(s_hist)[w] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0) s_res[3] = 0u;
    __syncthreads();
    select_keys<NT, KPT, false>(
        kreg, s, n_real, a.rho,
        [&](auto f) __attribute__((always_inline)) {
            for (int gq = KPT * NW + wv; gq * 64 < s; gq += NW) f(gq, key_at(gq * 64 + ln));
        },
        [&](int, int gq, uint32_t pos) __attribute__((always_inline)) { dst[pos] = gq * 64 + ln; },
        [&](int pos, int i) __attribute__((always_inline)) { dst[pos] = i; },
        [&](int i) { return ordered_key(key_at(i)); }, s_hist, s_list, s_bits, s_res);
}

// ------------------------------------------------------------------------------
// Algorithm 2 lines 5b-9 in ONE launch, for small batches: denominators, ranking, selection and attention.  Three
// launches (denom, keyclass, select_attn) spent 24 us on it at 32K tokens / 8 KV heads, of which about 9 are the gaps, ramps
// and drains of the launches and most of the rest round trips of intermediate results through memory.  SL blocks per unit,
// each of 512 threads and with a CU of its own (every instruction that all waves of a block execute costs it issue slots: eight
// waves, not sixteen); block x of a unit
//   1. sums the denominators of its share of the unit's recalled keys (every SL-th group of 64) and leaves them in its
//      exchange slots: one 64-bit word per head, the sum and a valid bit in one atomic store, so that no fence is needed;
//      the first wave then reads the slots of all SL blocks until they are valid -- the only thing that crosses blocks,
//      about 0.7 us against 3 us for a launch.  The wait is bounded (kTailSpins reads): a block that gives up takes the sums of
//      ALL keys itself, the same integers, so that no result and no progress depends on the other blocks being resident;
//   2. forms the ranking keys of ALL the unit's recalled keys (their scores and rows were requested before the exchange; up to
//      16 per thread stay in registers, later ones are read again, eight rounds requested together: one after the other a unit's
//      65536 cost 11 us more), their histogram, the deciding bucket, the bitmap of the picks and their positions, all in shared
//      memory -- the same work in every block instead of a hand-over;
//   3. attends over the picks, for its 128 / SL head dimensions.
// grid SL*batch*g; dynamic shared memory: tail_smem_words.  Same integers as the separate kernels.
// ------------------------------------------------------------------------------
constexpr int kTailSpins = 256;    // reads of the slots before a block gives up (each about 0.5 us)
constexpr int kTailKeys = 8192;    // recalled keys whose scores, rows and ranking keys a block keeps in registers
constexpr int kTailThreads = 512;

struct TailArgs {
    const int32_t *ctx_lens, *ncand, *cand;
    const uint32_t *crow;
    int l_stride, top_k, bits_words;
    const float *z;
    const uint32_t *m_key;
    unsigned long long *xs;     // [units][SL][G], zero on entry
    int spins;                  // reads of the slots before a block gives up (kTailSpins)
    uint32_t *gbits;            // the recall bitmap, cleared here for the next step
    int bitmap_words;
    uint32_t *kbuf;             // optional: [units][l_stride] the ranking keys (for the dynamic centroid update)
    int32_t *sel, *nsel, *out_sel;
    AttnArgs at;
};

__host__ __device__ __forceinline__ size_t tail_smem_words(int bits_words, int top_k, int G)
{
    return (size_t)kSelLds + 2 * kListCap + bits_words + 2 * (size_t)((top_k + 3) & ~3) + (size_t)top_k * G;
}

template <typename T, int G, int SL> __global__ __launch_bounds__(kTailThreads) void tail_kernel(TailArgs a)
{
    extern __shared__ __align__(16) uint32_t smem[];
    constexpr int NT = kTailThreads, NW = NT / 64, KPT = kTailKeys / NT;
    __shared__ unsigned long long s_acc[NW][G];
    __shared__ float s_ls[G];
    __shared__ uint32_t s_res[4];      // deciding bucket, keys wanted from it, its population, list cursor
    __shared__ uint32_t s_ok;
    const int kpad = (a.top_k + 3) & ~3;
    uint32_t *s_hist = smem;                               // kSelLds
    uint32_t *s_list = smem + kSelLds;                     // 2 * kListCap
    uint32_t *s_bits = s_list + 2 * kListCap;              // bits_words: two bitmaps over the recalled ids
    uint2 *s_pick = (uint2 *)(s_bits + a.bits_words);      // top_k: (position among the recalled keys, row) of the picks, ascending
    float *s_p = (float *)(s_pick + kpad);                 // top_k * G: their scores
    int ul, slice;
    attn_block_of<SL>(ul, slice);
    const int tid = threadIdx.x, ln = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float *zb = a.z + (size_t)ul * a.l_stride * G;
    const uint32_t *rb = a.crow + (size_t)ul * a.l_stride;
    CTKVR_STAMP(60);
    // requested at once, before L is known (slots beyond L hold stale values that are never used)
    constexpr int PRE = 2;                        // rounds of this block's share of the denominators
    constexpr int NF = G == 8 ? 4 : 8;            // rounds of later keys, which are not kept, requested together
    const int i0 = (wv * SL + slice) * 64 + ln;   // the share: every SL-th group of 64
    float zo[PRE][G], zr[KPT][G];
#pragma unroll
    for (int q = 0; q < PRE; ++q) load_z<G>(zb, min(i0 + q * SL * NT, a.l_stride - 1), zo[q]);
    const int L = a.ncand[ul];
    float m[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) m[hh] = ordered_value(a.m_key[ul * kMaxStride + hh]);
    // The unit's keys, as far as they are kept, and their rows: requested by the first wave now, by the others once their
    // denominators are handed over -- a wave's requests are issued in order, 32 of them from eight waves take the CU's one
    // address path 1.5 us, and the exchange waits for the slowest
    uint32_t rr[KPT];
    auto request_keys = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < KPT; ++q)
            if (q * NT + wv * 64 < L) {   // uniform
                load_z<G>(zb, min(q * NT + tid, a.l_stride - 1), zr[q]);
                rr[q] = rb[min(q * NT + tid, a.l_stride - 1)];
            }
    };
    if (wv == 0) request_keys();
    for (int w = tid; w < kBuckets / 4; w += NT) reinterpret_cast<uint4 *>(s_hist)[w] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0) s_res[3] = 0u;
    {
        const int W = (a.ctx_lens[ul / a.at.g] + 31) >> 5;
        for (int w = slice * NT + tid; w < W; w += SL * NT) a.gbits[(size_t)ul * a.bitmap_words + w] = 0u;
    }
    CTKVR_STAMP(61);
    // --- denominators ---------------------------------------------------------------------------------
    // sums of the terms i = first, first + step, ... (the first PRE of them in zv) as one 64-bit word per wave and head
    auto sum_terms = [&](const int first, const int step, float(&zv)[PRE][G]) __attribute__((always_inline)) {
        uint32_t shi[G], slo[G];
#pragma unroll
        for (int hh = 0; hh < G; ++hh) shi[hh] = slo[hh] = 0u;
        auto add = [&](const bool ok, const float(&x)[G]) __attribute__((always_inline)) {
#pragma unroll
            for (int hh = 0; hh < G; ++hh) {
                uint32_t hi, lo;
                exp_fixed40_parts(x[hh] - m[hh], hi, lo);
                lo = slo[hh] + (ok ? lo : 0u);             // < 2^25
                shi[hh] += (ok ? hi : 0u) + (lo >> 24);
                slo[hh] = lo & 0xffffffu;
            }
        };
#pragma unroll
        for (int q = 0; q < PRE; ++q)
            if (first - ln + q * step < L) add(first + q * step < L, zv[q]);   // wave-uniform
        for (int i = first + PRE * step; i - ln < L; i += NF * step) {
            float zf[NF][G];
#pragma unroll
            for (int u = 0; u < NF; ++u) load_z<G>(zb, min(i + u * step, L - 1), zf[u]);
#pragma unroll
            for (int u = 0; u < NF; ++u)
                if (i - ln + u * step < L) add(i + u * step < L, zf[u]);
        }
        // hi <= 2^16 per term; at most 2^9 terms per lane where the block takes its share only (contexts up to 2^20), so that
        // a wave's sum fits 32 bits; the sum of all terms by one block is put together from halves
#pragma unroll
        for (int hh = 0; hh < G; ++hh) {
            const uint32_t l = wave_sum_last(slo[hh]);
            if (step == NT) {
                const uint32_t h0 = wave_sum_last(shi[hh] & 0xffffu), h1 = wave_sum_last(shi[hh] >> 16);
                if (ln == 63) s_acc[wv][hh] = ((unsigned long long)h1 << 40) + ((unsigned long long)h0 << 24) + l;
            } else {
                const uint32_t h = wave_sum_last(shi[hh]);
                if (ln == 63) s_acc[wv][hh] = ((unsigned long long)h << 24) + l;
            }
        }
    };
    sum_terms(i0, SL * NT, zo);
    CTKVR_STAMP(62);
    __syncthreads();
    if (wv) request_keys();
    if (wv == 0) {
        constexpr unsigned long long kValid = 1ull << 63;   // a sum is below 2^20 * 2^40
        unsigned long long *xs = a.xs + (size_t)ul * SL * G;
        if (ln < G) {
            unsigned long long v = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) v += s_acc[w][ln];
            __hip_atomic_store(&xs[slice * G + ln], v | kValid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        unsigned long long v = kValid;
        bool all = false;
        for (int it = 0; it < a.spins && !all; ++it) {
            if (ln < SL * G) v = __hip_atomic_load(&xs[ln], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            all = __all((v & kValid) != 0ull);
        }
        CTKVR_STAMP(63);
        v &= ~kValid;
#pragma unroll
        for (int o = G; o < SL * G; o <<= 1) v += __shfl_xor(v, o);
        if (ln < G) s_ls[ln] = (float)log_fixed40(v);
        if (ln == 0) s_ok = all ? 1u : 0u;
    }
    __syncthreads();
    CTKVR_STAMP(64);
    if (!s_ok) {   // (uniform) a sibling is late: all terms here
        float zv[PRE][G];
#pragma unroll
        for (int q = 0; q < PRE; ++q) load_z<G>(zb, min(q * NT + tid, a.l_stride - 1), zv[q]);
        sum_terms(tid, NT, zv);
        __syncthreads();
        if (tid < G) {
            unsigned long long v = 0;
            for (int w = 0; w < NW; ++w) v += s_acc[w][tid];
            s_ls[tid] = (float)log_fixed40(v);
        }
        __syncthreads();
    }
    float ls[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) ls[hh] = s_ls[hh];
    // --- ranking keys, histogram, deciding bucket -----------------------------------------------------------
    auto key_of = [&](const float(&zv)[G]) __attribute__((always_inline)) {
        float best = (zv[0] - m[0]) - ls[0];
#pragma unroll
        for (int hh = 1; hh < G; ++hh) best = fmaxf(best, (zv[hh] - m[hh]) - ls[hh]);
        return fmaxf(best, -3.0e38f);   // (above the -inf of the slots beyond L)
    };
    float kreg[KPT];
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
        kreg[q] = key_of(zr[q]);
        if (q * NT + tid >= L) kreg[q] = -__builtin_huge_valf();
    }
    // f(group of 64 ids, key) for the groups of this wave beyond the first kTailKeys ids, whose keys are formed again
    auto for_far = [&](auto f) __attribute__((always_inline)) {
        for (int g0 = KPT * NW + wv; g0 * 64 < L; g0 += NF * NW) {
            float zv[NF][G];
#pragma unroll
            for (int u = 0; u < NF; ++u) load_z<G>(zb, min((g0 + u * NW) * 64 + ln, L - 1), zv[u]);
#pragma unroll
            for (int u = 0; u < NF; ++u) {
                const int gq = g0 + u * NW;
                if (gq * 64 >= L) break;
                const float kk = key_of(zv[u]);
                f(gq, gq * 64 + ln < L ? kk : -__builtin_huge_valf());
            }
        }
    };
    CTKVR_STAMP(65);
    if (a.kbuf) {
        uint32_t *kb = a.kbuf + (size_t)ul * a.l_stride;
        auto put = [&](int gq, float kk) __attribute__((always_inline)) {
            if (gq % SL == slice && gq * 64 + ln < L) kb[gq * 64 + ln] = ordered_key(kk);
        };
#pragma unroll
        for (int q = 0; q < KPT; ++q) put(q * NW + wv, kreg[q]);
        static_assert(KPT * NW % SL == 0, "the block's share of the later groups");
        for (int gq = KPT * NW + wv * SL + slice; gq * 64 < L; gq += NW * SL) {   // its share only: a walk of all cost 4 us more at 28000 keys
            float zv[G];
            load_z<G>(zb, min(gq * 64 + ln, L - 1), zv);
            put(gq, key_of(zv));
        }
    }
    CTKVR_STAMP(66);
    int n = L;
    if (a.top_k >= L) {   // every recalled key is kept
        for (int i = tid; i < L; i += NT) {
            float zv[G];
            load_z<G>(zb, i, zv);
            s_pick[i] = make_uint2((uint32_t)i, rb[i]);
            store_z<G>(s_p, i, zv);
        }
        __syncthreads();
    } else {
        n = a.top_k;
        const bool placed = select_keys<NT, KPT, true>(
            kreg, L, L, a.top_k, for_far,
            [&](int q, int gq, uint32_t pos) __attribute__((always_inline)) {
                s_pick[pos] = make_uint2((uint32_t)(gq * 64 + ln), rr[q]);
                store_z<G>(s_p, (int)pos, zr[q]);
            },
            [&](int pos, int i) __attribute__((always_inline)) { s_pick[pos].x = (uint32_t)i; },
            [&](int i) {
                float zv[G];
                load_z<G>(zb, i, zv);
                return ordered_key(key_of(zv));
            },
            s_hist, s_list, s_bits, s_res);
        __syncthreads();
        if (!placed) {   // uniform
            for (int pos = tid; pos < n; pos += NT) {
                const int i = (int)s_pick[pos].x;
                float zv[G];
                load_z<G>(zb, i, zv);
                s_pick[pos].y = rb[i];
                store_z<G>(s_p, pos, zv);
            }
            __syncthreads();
        }
    }
    // --- the picks: their ids (a share per block), then the attention over them --------------------------------
    const int per = (a.top_k + SL - 1) / SL, p0 = slice * per, p1 = min(a.top_k, p0 + per);
    const int32_t *cb = a.cand + (size_t)ul * a.l_stride;
    auto put_ids = [&](int pos, int t) __attribute__((always_inline)) {
        a.sel[(size_t)ul * a.top_k + pos] = t;
        if (a.out_sel) a.out_sel[(size_t)ul * a.top_k + pos] = t;
    };
    int my_id = -1;   // requested ahead of the value rows, stored after them
    if (p0 + tid < p1 && p0 + tid < n) my_id = cb[s_pick[p0 + tid].x];
    CTKVR_STAMP(72);
    // positions beyond n repeat the last pick; when nothing was recalled they name row 0 of the pool
    attend_unit<T, G, SL, 4, NT>(a.at, ul, slice, s_p,
                          [&](int t) {
                              const uint32_t r = s_pick[max(min(t, n - 1), 0)].y;
                              return n > 0 ? r : 0u;
                          },
                          [&](int t, float(&zv)[G]) { load_z<G>(s_p, max(min(t, n - 1), 0), zv); }, [&]() { return n; });
    if (p0 + tid < p1) put_ids(p0 + tid, my_id);
    for (int pos = p0 + NT + tid; pos < p1; pos += NT) put_ids(pos, pos < n ? cb[s_pick[pos].x] : -1);
    if (slice == 0 && tid == 0) a.nsel[ul] = n;
}

// ------------------------------------------------------------------------------
// Algorithm 2 lines 5b-9 in ONE launch with a unit's recalled keys SHARED OUT over its blocks: denominators, ranking, selection and
// attention, where denom, keyhist, classify, selection and attention as launches of their own took 35 us (128K x 4) and 43 us
// (sixteen of 8K to 64K), of which the passes over memory are the smaller part: each begins with a ramp and a chain of loads and
// ends with a drain.  This one takes 25 and 27 us, bound by its chain: 2.8 us to the scores, 2.0 for the exponentials (vector issue), 1.6, 2
// and 2.8 for the words of the others, 2.5 for the picks, 3 for their value rows, 2 to 4 for weighing them.  Block x of a unit's nb takes every
// step for its own share, a contiguous stretch of the recalled keys (whose scores and ranking keys stay in its registers), and what must be
// known of the others crosses over in 64-bit words that are zero before the launch and carry their own validity, written and read by single
// atomics, so that no fence is needed:
//   1. the share's denominator sums (a word per head);
//   2. the share's histograms of ranking keys (four buckets a word; one, two or three of them): every block then knows the unit's deciding bucket,
//      and from the others' histograms how many picks and how many of that bucket's keys come before its own;
//   3. the deciding bucket's keys (key and position).  The value rows of the share's sure picks and of its keys of that bucket are
//      requested before the others' are waited for;
//   4. the share's weighted sums of value rows, relative to the unit's maxima over all recalled keys: added up in block order,
//      128 G / nb elements by each block.
// Every wait is bounded (kTailSpins reads).  A block that gives up takes the denominators of all keys itself, or later goes on alone: it
// selects among all the unit's keys, attends over all picks and writes its part of the results, so that no progress
// depends on the other blocks being resident.  It does the same where the bucket is crowded (more than kShareList keys, in the finest
// histogram or below -318), and where
// some head's picks all lie so far below its maximum that their weights vanish (weights relative to the picks' own maxima then).
// The integers never depend on who gave up, and neither do the denominators; a block that goes on alone sums the weighted rows in another
// order, so that the outputs' last bits may differ between two calls, and within a head, where a wait expired in one.
// grid nb*batch*g, nb a power of two, kTailThreads threads; dynamic shared memory: share_smem_words.  Same integers as the separate kernels.
// ------------------------------------------------------------------------------
constexpr int kShareList = 512;    // keys of the deciding bucket that are ranked against each other at most
// ... where a finer histogram is to be had: more are counted again.  A histogram more is 2 us, ranking 128 keys 0.4, 256 2 and 512 8 (a key and its
// position compared one after the other instead of as one word: 8 and 30).  Scores of little spread, 32 units of 4096 recalled keys,
// 1024 picks: 75.2 us a step (every bucket up to 512 keys ranked), now 41.9; 128 units of 8192 keys 139 -> 102 (separate launches 46.1 and 114)
constexpr int kShareRank = 128;
constexpr int kShareBlocks = 8;    // blocks per unit at most
constexpr int kShareBuckets = 256; // buckets of a histogram: 1/4 wide in the log domain, 1 wide below them, 1/256 of either inside one
constexpr uint32_t kShareFar = 63; // the buckets of 1 begin at -63, of which what lies above the quarters' end (-63.75) is empty
constexpr int kShareLevels = 3;    // histograms at most
constexpr int kShareCut = 8191;    // a share's count in the exchange is cut there; top_k is at most that, so that a bucket with
                                   // such a count is the deciding one, or comes after it, with or without the cut
constexpr int kSharePicks = 128;   // picks that a wave attends over at a time

struct ShareArgs {
    const int32_t *ctx_lens, *ncand, *cand;
    const uint32_t *crow;
    int l_stride, top_k;
    int nb;                     // blocks per unit
    const float *z;
    const uint32_t *m_key;
    unsigned long long *xs;     // [units][share_words]: the exchange, zero on entry
    uint32_t spins;             // reads before a block gives up (kTailSpins), halved, a byte for each of the four waits
    uint32_t late_spins;        // the same for block late_block (tests)
    int late_block;
    uint32_t *gbits;            // the recall bitmap, cleared here for the next step
    int bitmap_words;
    uint32_t *kbuf;             // [units][l_stride] the ranking keys, written where a block goes on alone
    uint32_t *alone;            // [units][top_k] the picks' positions, likewise
    int keep_keys;              // kbuf is always written (for the dynamic centroid update)
    int32_t *sel, *nsel, *out_sel;
    AttnArgs at;
};

// 64-bit words of a unit's exchange: sums, histograms, the bucket's keys, weighted sums of value rows, sums of weights
__host__ __device__ __forceinline__ size_t share_words(int nb, int G)
{
    return nb > 1 ? (size_t)nb * (G + kShareLevels * (kShareBuckets / 4) + 64 * G + G) + kShareList : 0;
}
// words of shared memory that the histograms, the bucket's keys and later the waves' partial results take
__host__ __device__ __forceinline__ int share_front_words(int G)
{
    const int sel = kSelLds + 2 * kShareList, out = kTailThreads / 64 * G * kD;
    return ((sel > out ? sel : out) + 3) & ~3;
}
// share: groups of 64 keys in the largest share
__host__ __device__ __forceinline__ size_t share_smem_words(int share, int G)
{
    return share_front_words(G) + (size_t)(kTailThreads / 64) * kSharePicks * (2 + G) + 2 * (size_t)share;
}

// a key of the deciding bucket and its position as one word that is never zero: of two, the larger comes first in the ranking
__device__ __forceinline__ unsigned long long share_entry(float key, int pos)
{
    return (unsigned long long)ordered_key(key) << 32 | ~(uint32_t)pos;
}

// two values summed over the halves of a wave, lane by lane: the lower half gets the sum of a, the upper that of b
__device__ __forceinline__ float half_pair_sum(float a, float b)
{
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

template <typename T, int G> __global__ __launch_bounds__(kTailThreads) void share_tail_kernel(ShareArgs a)
{
    extern __shared__ __align__(16) uint32_t smem[];
    constexpr int NT = kTailThreads, NW = NT / 64;
    constexpr int KPT = G == 8 ? 8 : 16;           // groups of 64 keys that a wave keeps in registers
    constexpr int NF = 4;                          // groups of later keys requested together
    constexpr int NU = sizeof(T) == 2 ? 16 : 8;    // value rows in flight per 16-lane group
    constexpr int W = G * 64;                      // pairs of output elements of a unit
    constexpr int NH = kShareBuckets / 4;          // words of a histogram in the exchange
    static_assert(NH == 64 && kShareList <= NT && NW * kShareBuckets <= 2048, "a word of a histogram per lane, a key of the list per thread");
    __shared__ unsigned long long s_acc[NW][G];
    __shared__ float s_ls[G], s_m[G], s_l[NW][G];
    __shared__ uint32_t s_res[5];          // deciding bucket, keys wanted from it, its population, those in earlier shares, some wave gave up
    __shared__ uint32_t s_before, s_cur;   // picks of earlier shares; cursor of the share's part of the bucket's list
    __shared__ uint32_t s_cnt[NW];         // picks of each wave
    uint32_t *s_hist = smem;                                    // a histogram per wave
    unsigned long long *s_ent = reinterpret_cast<unsigned long long *>(smem + kSelLds);   // kShareList: share_entry of the deciding bucket
    float *s_o = reinterpret_cast<float *>(smem);               // [NW][G][128], once those two are done with
    const int tid = threadIdx.x, ln = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the wave's picks: row, position (with a mark on the sure ones), scores and then weights
    uint32_t *w_row = smem + share_front_words(G) + wv * kSharePicks, *w_pos = w_row + NW * kSharePicks;
    float *w_z = reinterpret_cast<float *>(smem + share_front_words(G) + 2 * NW * kSharePicks) + wv * kSharePicks * G;
    uint32_t *s_bits = smem + share_front_words(G) + NW * kSharePicks * (2 + G);   // the share's picks from the deciding bucket
    const int nb = a.nb;
    int ul, x;
    {
        const int lin = blockIdx.x, nu = gridDim.x / nb;
        if ((nu & 7) == 0) {   // a unit's blocks on one XCD
            ul = (lin >> 3) / nb * 8 + (lin & 7);
            x = (lin >> 3) % nb;
        } else {
            ul = lin / nb;
            x = lin % nb;
        }
    }
    const float *zb = a.z + (size_t)ul * a.l_stride * G;
    const uint32_t *rb = a.crow + (size_t)ul * a.l_stride;
    const int32_t *cb = a.cand + (size_t)ul * a.l_stride;
    unsigned long long *xsum = a.xs + (size_t)ul * share_words(nb, G), *xhist = xsum + nb * G, *xlist = xhist + kShareLevels * nb * NH;
    unsigned long long *xout = xlist + kShareList, *xl = xout + nb * W;
    constexpr unsigned long long kValid = 1ull << 63;
    auto put = [](unsigned long long *p, unsigned long long v) __attribute__((always_inline)) {
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto get = [](const unsigned long long *p) __attribute__((always_inline)) {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    const uint32_t spins = x == a.late_block ? a.late_spins : a.spins;   // (one register: with a test at each wait 128K x 4 took 1 us more)
    auto reads = [&](int wait) __attribute__((always_inline)) { return (int)(spins >> (8 * wait) & 0xffu) * 2; };
    auto rank_in = [](uint64_t mask, uint32_t base) __attribute__((always_inline)) {   // base + lanes of the mask below this one
        return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, base));
    };
    CTKVR_STAMP(60);
    const int L = a.ncand[ul];
    float m[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) m[hh] = ordered_value(a.m_key[ul * kMaxStride + hh]);
    // the share, in groups of 64 keys, and this wave's stretch of it
    const int ng = (L + 63) >> 6, gpb = (ng + nb - 1) / nb, gpw = (gpb + NW - 1) / NW;
    const int g0 = min(ng, x * gpb), g1 = min(ng, g0 + gpb);
    const int wg0 = min(g1, g0 + wv * gpw), nwg = min(g1, wg0 + gpw) - wg0;
    const int end = min(L, (wg0 + nwg) * 64);
    auto key_at = [&](int q) __attribute__((always_inline)) { return (wg0 + q) * 64 + ln; };
    float zr[KPT][G];   // scores, less the unit's maxima
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
        if (q % 2 == 0 && q >= nwg) break;   // uniform, here and below: the wave's groups two by two, its last one perhaps without keys
        load_z<G>(zb, min(key_at(q), L - 1), zr[q]);
    }
    reinterpret_cast<uint4 *>(s_hist)[tid] = make_uint4(0u, 0u, 0u, 0u);
    for (int w = tid; w < 2 * gpb; w += NT) s_bits[w] = 0u;
    if (tid == 0) {
        s_res[4] = 0u;
        s_before = 0u;
        s_cur = 0u;
    }
    if (tid < G) s_m[tid] = ordered_value(a.m_key[ul * kMaxStride + tid]);
    {
        const int nwd = (a.ctx_lens[ul / a.at.g] + 31) >> 5;
        for (int w = x * NT + tid; w < nwd; w += nb * NT) a.gbits[(size_t)ul * a.bitmap_words + w] = 0u;
    }
    CTKVR_STAMP(61);
    // --- 1. denominators ----------------------------------------------------------------------------------
    // (positions from `to` on: -inf, whose term is zero and whose key ranks last)
    auto less_max = [&](float(&v)[G], const int i, const int to) __attribute__((always_inline)) {
#pragma unroll
        for (int hh = 0; hh < G; ++hh) v[hh] = i < to ? v[hh] - m[hh] : -__builtin_huge_valf();
    };
    // sums of the terms of n groups from `first` by the calling wave (KEPT: the first KPT of them in registers), as one 64-bit word
    // per head
    auto sum_terms = [&](auto kept, const int first, const int n) __attribute__((always_inline)) {
        uint32_t shi[G], slo[G];
#pragma unroll
        for (int hh = 0; hh < G; ++hh) shi[hh] = slo[hh] = 0u;
        auto add = [&](const float(&v)[G]) __attribute__((always_inline)) {
#pragma unroll
            for (int hh = 0; hh < G; ++hh) {
                uint32_t hi, lo;
                exp_fixed40_parts(v[hh], hi, lo);
                shi[hh] += hi;
                slo[hh] += lo;
            }
        };
        auto carry = [&]() __attribute__((always_inline)) {   // lo < 2^24 a term: at least every 255 terms
#pragma unroll
            for (int hh = 0; hh < G; ++hh) {
                shi[hh] += slo[hh] >> 24;
                slo[hh] &= 0xffffffu;
            }
        };
        constexpr bool KEPT = decltype(kept)::value;
        if constexpr (KEPT) {
#pragma unroll
            for (int q = 0; q < KPT; ++q) {
                if (q % 2 == 0 && q >= nwg) break;
                less_max(zr[q], key_at(q), end);
                add(zr[q]);
            }
            carry();
        }
#pragma unroll 1
        for (int q = KEPT ? KPT : 0; q < n; q += NF) {
            float zf[NF][G];
#pragma unroll
            for (int u = 0; u < NF; ++u) load_z<G>(zb, min((first + q + u) * 64 + ln, L - 1), zf[u]);
#pragma unroll
            for (int u = 0; u < NF; ++u) {
                if (q + u >= n) break;
                less_max(zf[u], (first + q + u) * 64 + ln, L);
                add(zf[u]);
            }
            carry();
        }
        // hi <= 2^16 a term, so that a lane's sum fits 32 bits; a wave's does too up to 2^9 terms a lane, and is put together from halves beyond
#pragma unroll
        for (int hh = 0; hh < G; ++hh) {
            const uint32_t l = wave_sum_last(slo[hh]);
            unsigned long long h;
            if (n > 500)   // uniform
                h = ((unsigned long long)wave_sum_last(shi[hh] >> 16) << 16) + wave_sum_last(shi[hh] & 0xffffu);
            else
                h = wave_sum_last(shi[hh]);
            if (ln == 63) s_acc[wv][hh] = (h << 24) + l;
        }
    };
    sum_terms(std::true_type{}, wg0, nwg);
    CTKVR_STAMP(62);
    __syncthreads();
    uint32_t rr[KPT];   // the rows, requested while the others' sums are waited for
    auto request_rows = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < KPT; ++q) {
            if (q % 2 == 0 && q >= nwg) break;
            rr[q] = rb[min(key_at(q), L - 1)];
        }
    };
    if (wv) request_rows();
    if (wv == 0) {
        unsigned long long v = 0;
        if (ln < G) {
#pragma unroll
            for (int w = 0; w < NW; ++w) v += s_acc[w][ln];
        }
        bool all = true;
        if (nb > 1) {
            if (ln < G) put(&xsum[x * G + ln], v | kValid);   // (a sum is below 2^20 * 2^40)
            all = false;
            v = kValid;
            for (int it = 0; it < reads(0) && !all; ++it) {
                if (ln < nb * G) v = get(&xsum[ln]);
                all = __all((v & kValid) != 0ull);
            }
            v &= ~kValid;
#pragma unroll
            for (int o = G; o < 64; o <<= 1) v += __shfl_xor(v, o);
        }
        request_rows();
        if (ln < G) s_ls[ln] = (float)log_fixed40(v);
        if (ln == 0) s_res[0] = all ? 1u : 0u;
    }
    __syncthreads();
    CTKVR_STAMP(63);
    if (!s_res[0]) {   // (uniform) a sibling is late: all terms here
        const int per = (ng + NW - 1) / NW, f = min(ng, wv * per);
        sum_terms(std::false_type{}, f, min(ng, f + per) - f);
        __syncthreads();
        if (tid < G) {
            unsigned long long v = 0;
            for (int w = 0; w < NW; ++w) v += s_acc[w][tid];
            s_ls[tid] = (float)log_fixed40(v);
        }
        __syncthreads();
    }
    float ls[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) ls[hh] = s_ls[hh];
    // --- 2. ranking keys, their histogram, the deciding bucket ------------------------------------------------
    auto key_of = [&](const float(&v)[G]) __attribute__((always_inline)) {
        float best = v[0] - ls[0];
#pragma unroll
        for (int hh = 1; hh < G; ++hh) best = fmaxf(best, v[hh] - ls[hh]);
        return fmaxf(best, -3.0e38f);   // (above the -inf of the slots beyond L)
    };
    float kreg[KPT];
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
        if (q % 2 == 0 && q >= nwg) break;
        kreg[q] = key_at(q) < end ? key_of(zr[q]) : -__builtin_huge_valf();
    }
    // NF groups of the stretch from `q` on, beyond those in registers: their scores less the maxima
    auto load_far = [&](int q, float(&zf)[NF][G]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NF; ++u) load_z<G>(zb, min(key_at(q + u), L - 1), zf[u]);
#pragma unroll
        for (int u = 0; u < NF; ++u) less_max(zf[u], key_at(q + u), end);
    };
    auto far_key = [&](int q, const float(&v)[G]) __attribute__((always_inline)) { return key_at(q) < end ? key_of(v) : -__builtin_huge_valf(); };
    // f(group of the stretch, key) for the wave's groups
    auto for_keys = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < KPT; ++q) {
            if (q % 2 == 0 && q >= nwg) break;
            f(q, kreg[q]);
        }
#pragma unroll 1
        for (int q = KPT; q < nwg; q += NF) {
            float zf[NF][G];
            load_far(q, zf);
#pragma unroll
            for (int u = 0; u < NF; ++u) {
                if (q + u >= nwg) break;
                f(q + u, far_key(q + u, zf[u]));
            }
        }
    };
    if (a.keep_keys) {
        uint32_t *kb = a.kbuf + (size_t)ul * a.l_stride;
        for_keys([&](int q, float kk) __attribute__((always_inline)) {
            if (key_at(q) < end) kb[key_at(q)] = ordered_key(kk);
        });
    }
    const bool every = a.top_k >= L;   // every recalled key is kept
    bool alone = false;
    // x > hi_k is a sure pick, lo_k < x <= hi_k is in the deciding bucket (exact: the bounds are multiples of 1/1024 above -65, or of
    // 1/256 above -319)
    float hi_k = every ? -__builtin_huge_valf() : __builtin_huge_valf(), lo_k = -__builtin_huge_valf();
    // keys wanted from the deciding bucket, its population, those in earlier shares (at first of all keys)
    uint32_t rem = (uint32_t)a.top_k, n_bkt = (uint32_t)L, e0 = (uint32_t)min(L, g0 * 64);
    // 256 buckets a quarter wide; where more than kShareRank keys share the deciding one, 256 inside it (fine).  The last bucket is all
    // below, and where it decides, 256 buckets of 1 follow first: keys spread with the queries' norms, and a large budget's last
    // one lies beyond -63.75 in earnest (8 units of one head, 33000 keys and 4096 picks 64.2 us a step, going alone there 83.2, separate
    // launches 66.7; of two heads, 89000 keys and 2048 picks 105, 237 and 168)
    float scale = -4.0f, width = -0.25f, upto = hi_k;   // width: 1 / scale, exactly
    uint32_t first = 0;     // number of the first bucket, from zero on downwards
    bool fine = false;
#pragma unroll 1
    for (int level = 0; level < kShareLevels && !every; ++level) {
        // a histogram per wave.  Not counted: the last bucket (what the others leave); when fine, what is not in the deciding one
        uint32_t *hist = s_hist + wv * kShareBuckets, *spare = reinterpret_cast<uint32_t *>(s_ent) + tid;
        const float over = fine ? lo_k : (float)(first + kShareBuckets - 1) * width;
        for_keys([&](int, float kk) __attribute__((always_inline)) {
            uint32_t *bin = hist + ((uint32_t)fmaxf(kk * scale, 0.0f) - first);
            bin = kk > over && kk <= upto ? bin : spare;
            atomicAdd(bin, 1u);
        });
        __syncthreads();
        CTKVR_STAMP(64);
        if (wv == 0) {
            // lane l has the buckets 4 l .. 4 l + 3, in descending key order, 16 bits each in two words
            uint4 c = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const uint4 t = reinterpret_cast<const uint4 *>(s_hist + w * kShareBuckets)[ln];
                c.x += t.x;
                c.y += t.y;
                c.z += t.z;
                c.w += t.w;
            }
            constexpr uint32_t kCut = (uint32_t)kShareCut;
            uint32_t t_lo = min(c.x, kCut) | min(c.y, kCut) << 16, t_hi = min(c.z, kCut) | min(c.w, kCut) << 16;   // the unit's
            uint32_t b_lo = 0u, b_hi = 0u;                                                                         // earlier shares'
            bool all = true;
            if (nb > 1) {
                unsigned long long *xh = xhist + level * nb * NH, hw[kShareBlocks];
                put(&xh[x * NH + ln], kValid | ((unsigned long long)t_hi << 32) | t_lo);
                all = false;
                for (int it = 0; it < reads(1) && !all; ++it) {
                    unsigned long long v = kValid;
#pragma unroll
                    for (int y = 0; y < kShareBlocks; ++y)
                        if (y < nb) hw[y] = get(&xh[y * NH + ln]);   // uniform
#pragma unroll
                    for (int y = 0; y < kShareBlocks; ++y)
                        if (y < nb) v &= hw[y];
                    all = __all((v & kValid) != 0ull);
                }
                t_lo = t_hi = 0u;   // (and stay so where a block did not answer: nothing of the levels counts then)
#pragma unroll
                for (int y = 0; y < kShareBlocks; ++y)
                    if (all && y < nb) {
                        const uint32_t lo = (uint32_t)hw[y], hi = (uint32_t)(hw[y] >> 32) & 0x7fffffffu;
                        b_lo += y < x ? lo : 0u;
                        b_hi += y < x ? hi : 0u;
                        t_lo += lo;
                        t_hi += hi;
                    }
            }
            CTKVR_STAMP(65);
            auto nth = [](uint32_t lo, uint32_t hi, uint32_t j) __attribute__((always_inline)) {
                return ((j & 2u ? hi : lo) >> ((j & 1u) * 16)) & 0xffffu;
            };
            auto sum4 = [](uint32_t lo, uint32_t hi) __attribute__((always_inline)) {
                return (lo & 0xffffu) + (lo >> 16) + (hi & 0xffffu) + (hi >> 16);
            };
            const uint32_t mine = sum4(t_lo, t_hi), inc = wave_incl_scan(mine), tot = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
            uint32_t above;   // picks of earlier shares
            if (!all || rem > tot) {   // a block did not answer, or the last bucket decides
                above = wave_sum_last(sum4(b_lo, b_hi));
                if (ln == 63) {
                    s_res[0] = (uint32_t)(kShareBuckets - 1);
                    s_res[1] = rem - tot;
                    s_res[2] = all ? n_bkt - tot : ~0u;
                    s_res[3] = e0 - above;
                }
            } else {
                const uint64_t has = __ballot(inc >= rem);   // the first of these lanes has the bucket
                const int src = __ffsll((long long)has) - 1;
                uint32_t at = inc - mine, j = 0;
#pragma unroll
                for (uint32_t i = 0; i < 3; ++i)
                    if (j == i && at + nth(t_lo, t_hi, i) < rem) {
                        at += nth(t_lo, t_hi, i);
                        j = i + 1;
                    }
                if (ln == src) {
                    s_res[0] = 4u * (uint32_t)src + j;
                    s_res[1] = rem - at;
                    s_res[2] = nth(t_lo, t_hi, j);
                    s_res[3] = nth(b_lo, b_hi, j);
                }
                above = ln < src ? sum4(b_lo, b_hi) : 0u;
                if (ln == src)
#pragma unroll
                    for (uint32_t i = 0; i < 3; ++i) above += i < j ? nth(b_lo, b_hi, i) : 0u;
                above = wave_sum_last(above);
            }
            if (ln == 63) s_before += above;
        }
        __syncthreads();
        const uint32_t bkt = s_res[0];
        rem = s_res[1];
        n_bkt = s_res[2];
        e0 = s_res[3];
        alone = n_bkt > (uint32_t)kShareList;   // (or ~0: a block did not answer)
        const bool below = !fine && bkt == (uint32_t)(kShareBuckets - 1);
        hi_k = first + bkt ? fminf(upto, (float)(first + bkt) * width) : upto;
        lo_k = below ? -__builtin_huge_valf() : (float)(first + bkt + 1u) * width;
        if (n_bkt <= (uint32_t)kShareRank || n_bkt == ~0u || fine || (below && level)) break;   // uniform
        fine = !below;
        scale = fine ? scale * (float)kShareBuckets : -1.0f;
        width = fine ? width / (float)kShareBuckets : -1.0f;
        first = fine ? (uint32_t)(lo_k * scale) - kShareBuckets : kShareFar;
        upto = hi_k;
        reinterpret_cast<uint4 *>(hist)[ln] = make_uint4(0u, 0u, 0u, 0u);
    }
    CTKVR_STAMP(66);
    // --- 3. the share's keys of the deciding bucket, for all; its picks, sure ones and those, ascending, for the wave -----------
    const int lane16 = ln & 15, row4 = ln >> 4;
    const T *V = (const T *)a.at.v_pages;
    Chunk<T> cv[NU];
    int n_l = 0, qn = 0;   // picks at hand; the wave's next group
    int my_id[kSharePicks / 64];
    // (lanes of the wave read in w_row, w_pos and w_z what others wrote: a wave's accesses to shared memory are served in order, and this
    // keeps the compiler to it)
    auto handed = []() __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // the wave's picks from group qn on, as many groups as fit: the first time from the registers, later from memory
    auto append = [&](int q, float kk, const float(&v)[G], auto row) __attribute__((always_inline)) {
        const uint64_t all = __ballot(kk > lo_k);
        const int n = __popcll(all);
        if (n_l + n > kSharePicks) return;   // uniform
        if (kk > lo_k) {
            const uint32_t p = rank_in(all, (uint32_t)n_l);
            w_row[p] = row();
            w_pos[p] = (uint32_t)key_at(q) | (kk > hi_k ? 0x80000000u : 0u);
            store_z<G>(w_z, (int)p, v);
        }
        n_l += n;
        qn = q + 1;
    };
    auto fill_again = [&]() __attribute__((always_inline)) {
        handed();
        n_l = 0;
#pragma unroll 1
        for (int q = qn; q < nwg && qn == q; q += NF) {
            float zf[NF][G];
            load_far(q, zf);
#pragma unroll
            for (int u = 0; u < NF; ++u)
                if (qn == q + u && q + u < nwg) append(q + u, far_key(q + u, zf[u]), zf[u], [&]() { return rb[min(key_at(q + u), L - 1)]; });
        }
    };
    auto request = [&](int r0) __attribute__((always_inline)) {   // value rows of the picks from r0 on
        uint32_t row[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (u % 4 == 0 && r0 + u * 4 >= n_l) break;   // uniform
            row[u] = w_row[min(r0 + u * 4 + row4, n_l - 1)];
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (u % 4 == 0 && r0 + u * 4 >= n_l) break;
            cv[u] = load_chunk(V + (size_t)row[u] * kD, lane16);
        }
    };
    auto begin = [&]() __attribute__((always_inline)) {   // ids and value rows requested, scores to weights
        if (n_l == 0) return;   // uniform
        handed();
#pragma unroll
        for (int i = 0; i < kSharePicks / 64; ++i) my_id[i] = cb[w_pos[min(i * 64 + ln, n_l - 1)] & 0x7fffffffu];
        request(0);
#pragma unroll
        for (int i = 0; i < kSharePicks / 64; ++i)
            if (i * 64 + ln < n_l) {
                float w[G];
                load_z<G>(w_z, i * 64 + ln, w);
#pragma unroll
                for (int hh = 0; hh < G; ++hh) w[hh] = __expf(w[hh]);
                store_z<G>(w_z, i * 64 + ln, w);
            }
        handed();
    };
    if (!alone) {
        uint32_t n_gt = 0;
        for_keys([&](int q, float kk) __attribute__((always_inline)) {
            const uint64_t gt = __ballot(kk > hi_k), in = __ballot(kk > lo_k) & ~gt;
            n_gt += (uint32_t)__popcll(gt);
            if (in) {   // uniform
                uint32_t e = 0;
                if (ln == 0) e = atomicAdd(&s_cur, (uint32_t)__popcll(in));
                e = rank_in(in, e0 + (uint32_t)__builtin_amdgcn_readfirstlane((int)e));
                if (__builtin_amdgcn_inverse_ballot_w64(in)) {
                    if (nb > 1)
                        put(&xlist[e], share_entry(kk, key_at(q)));
                    else
                        s_ent[e] = share_entry(kk, key_at(q));
                }
            }
        });
        if (ln == 0) s_cnt[wv] = n_gt;
        s_hist[tid] = 0u;   // the ranks of the bucket's keys (everyone has read the histograms)
#pragma unroll
        for (int q = 0; q < KPT; ++q) {
            if (q % 2 == 0 && q >= nwg) break;
            if (q == qn) append(q, kreg[q], zr[q], [&]() { return rr[q]; });   // uniform
        }
        begin();
        CTKVR_STAMP(67);
        if (!every) {
            // which of the bucket's keys are picks: ranked against each other, ids decide between equal keys.  (Zeros, below every entry,
            // to the next power of two.)
            uint32_t cap = 64;
            while (cap < n_bkt) cap <<= 1;
            if (nb > 1) {
                unsigned long long v = 1ull;
                bool all = false;
                for (int it = 0; it < reads(2) && !all; ++it) {
                    if (tid < (int)n_bkt) v = get(&xlist[tid]);
                    all = __all(v != 0ull);
                }
                if (!all) s_res[4] = 1u;
                if (tid < (int)n_bkt) s_ent[tid] = v;
            }
            if (tid >= (int)n_bkt && tid < (int)cap) s_ent[tid] = 0ull;
            __syncthreads();
            CTKVR_STAMP(68);
            const uint32_t parts = (uint32_t)NT / cap, e = (uint32_t)tid & (cap - 1u), part = (uint32_t)tid / cap;
            if (e < n_bkt) {
                const unsigned long long me = s_ent[e];
                uint32_t rank = 0;
                for (uint32_t f = part; f < n_bkt; f += 4 * parts) {   // (f + 3 parts < cap, a multiple of 4 parts)
                    unsigned long long o[4];
#pragma unroll
                    for (uint32_t i = 0; i < 4; ++i) o[i] = s_ent[f + i * parts];
#pragma unroll
                    for (uint32_t i = 0; i < 4; ++i) rank += o[i] > me ? 1u : 0u;
                }
                atomicAdd(&s_hist[e], rank);
            }
            __syncthreads();
            if (tid < (int)n_bkt && s_hist[tid] < rem) {
                const int pos = (int)~(uint32_t)s_ent[tid], rel = pos - g0 * 64;
                if (rel < 0) {
                    atomicAdd(&s_before, 1u);
                } else if (pos < g1 * 64) {
                    atomicOr(&s_bits[rel >> 5], 1u << (rel & 31));
                    atomicAdd(&s_cnt[(rel >> 6) / gpw], 1u);
                }
            }
        }
        __syncthreads();
        alone = s_res[4] != 0u;
    }
    CTKVR_STAMP(69);
    // --- 4. attention over them, or over all the unit's picks where a block goes on alone --------------------------
    const int n = min(L, a.top_k);
    const int per_w = W / nb, word = x * per_w + tid;   // the block's part of the output, a pair of elements a thread
    float2 o = make_float2(0.0f, 0.0f);
    float l_o = 0.0f;
    float acc[G][8], lsum[G];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int hh = 0; hh < G; ++hh) {
            lsum[hh] = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[hh][e] = 0.0f;
        }
    };
    auto add_row = [&](const Chunk<T> &c, const float(&w)[G]) __attribute__((always_inline)) {
        float vx[8];
        unpack(c, vx);
#pragma unroll
        for (int hh = 0; hh < G; ++hh)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[hh][e] = __fmaf_rn(w[hh], vx[e], acc[hh][e]);
    };
    // over the wave's four rows of lanes (each is left with two of the eight values; the weights: over all lanes); then, block_pair and block_l, over the waves
    auto hand_over = [&]() __attribute__((always_inline)) {
        const int e = (ln >> 4 & 1) * 4 + (ln >> 5) * 2;
#pragma unroll
        for (int hh = 0; hh < G; ++hh) {
            float h4[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) h4[j] = row_pair_sum(acc[hh][j], acc[hh][j + 4]);
            *reinterpret_cast<float2 *>(s_o + (wv * G + hh) * kD + lane16 * 8 + e) =
                make_float2(half_pair_sum(h4[0], h4[2]), half_pair_sum(h4[1], h4[3]));
            float l = group16_sum(lsum[hh]);
            l = row_pair_sum(l, l);
            l = half_pair_sum(l, l);
            if (ln == 0) s_l[wv][hh] = l;
        }
        __syncthreads();
    };
    auto block_pair = [&](int w) __attribute__((always_inline)) {   // pair w of the block's sums
        float2 v = make_float2(0.0f, 0.0f);
#pragma unroll
        for (int p = 0; p < NW; ++p) {
            const float2 t = *reinterpret_cast<const float2 *>(s_o + p * G * kD + 2 * w);
            v.x += t.x;
            v.y += t.y;
        }
        return v;
    };
    auto block_l = [&](int hh) __attribute__((always_inline)) {
        float v = 0.0f;
#pragma unroll
        for (int p = 0; p < NW; ++p) v += s_l[p][hh];
        return v;
    };
    if (!alone) {   // uniform
        clear();
        uint32_t rank = every ? (uint32_t)min(L, g0 * 64) : s_before;   // picks before the wave's
#pragma unroll
        for (int w = 0; w < NW; ++w) rank += w < wv ? s_cnt[w] : 0u;
        for (;;) {
            // a pick a lane: those of the deciding bucket that are none lose their place, the others' ids are written
#pragma unroll
            for (int i = 0; i < kSharePicks / 64; ++i) {
                const int p = i * 64 + ln;
                if (i * 64 >= n_l) break;   // uniform
                bool ok = false;
                if (p < n_l) {
                    const uint32_t pos = w_pos[p], rel = (pos & 0x7fffffffu) - (uint32_t)(g0 * 64);
                    ok = (int32_t)(pos | s_bits[rel >> 5] << (31u - (rel & 31u))) < 0;   // (a sure pick's bit is not set, nor looked at)
                    w_pos[p] = ok;
                }
                const uint64_t mask = __ballot(ok);
                if (ok) {
                    float w[G];
                    load_z<G>(w_z, p, w);
#pragma unroll
                    for (int hh = 0; hh < G; ++hh) lsum[hh] += w[hh];
                    const uint32_t r = rank_in(mask, rank);
                    a.sel[(size_t)ul * a.top_k + r] = my_id[i];
                    if (a.out_sel) a.out_sel[(size_t)ul * a.top_k + r] = my_id[i];
                }
                rank += (uint32_t)__popcll(mask);
            }
            handed();
#pragma unroll 1
            for (int r0 = 0; r0 < n_l; r0 += NU * 4) {
                if (r0) request(r0);
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    if (u % 4 == 0 && r0 + u * 4 >= n_l) break;   // uniform
                    const int p = min(r0 + u * 4 + row4, n_l - 1);
                    const bool ok = r0 + u * 4 + row4 < n_l && w_pos[p] != 0u;
                    float w[G];
                    load_z<G>(w_z, p, w);
                    if (ok) add_row(cv[u], w);
                }
            }
            if (qn >= nwg) break;   // uniform
            fill_again();
            begin();
        }
        CTKVR_STAMP(70);
        hand_over();
        if (nb == 1) {   // uniform
            if (tid < per_w) {
                o = block_pair(word);
                l_o = block_l(word >> 6);
            }
        } else {
            if (tid < W) {
                const float2 v = block_pair(tid);
                const unsigned long long w = ((unsigned long long)__float_as_uint(v.y) << 32) | __float_as_uint(v.x);
                put(&xout[x * W + tid], w ? w : 0x80000000u);   // (a zero that counts as written is -0)
            }
            if (tid < G) put(&xl[x * G + tid], (1ull << 32) | __float_as_uint(block_l(tid)));
            if (tid < per_w) {
                unsigned long long w[kShareBlocks], lw[kShareBlocks];
                bool all = false;
                for (int it = 0; it < reads(3) && !all; ++it) {
                    all = true;
#pragma unroll
                    for (int y = 0; y < kShareBlocks; ++y)
                        if (y < nb) {
                            w[y] = get(&xout[y * W + word]);
                            lw[y] = get(&xl[y * G + (word >> 6)]);
                        }
#pragma unroll
                    for (int y = 0; y < kShareBlocks; ++y)
                        if (y < nb) all = all && w[y] != 0ull && lw[y] != 0ull;
                }
                if (all) {
#pragma unroll
                    for (int y = 0; y < kShareBlocks; ++y)
                        if (y < nb) {
                            o.x += __uint_as_float((uint32_t)w[y]);
                            o.y += __uint_as_float((uint32_t)(w[y] >> 32));
                            l_o += __uint_as_float((uint32_t)lw[y]);
                        }
                }
            }
        }
        CTKVR_STAMP(72);
        // a head whose picks' weights all vanish beside its maximum (or a block that did not answer, and l_o = 0)
        alone = __syncthreads_or(tid < per_w && L > 0 && !(l_o >= 1e-30f));
    }
    if (alone) {   // uniform
        clear();
        // all the unit's keys to memory (whoever else does so writes the same), the selection from there, the picks' maxima, then
        // four rows a wave at a time
        __syncthreads();
        uint32_t *kb = a.kbuf + (size_t)ul * a.l_stride, *pk = a.alone + (size_t)ul * a.top_k;
#pragma unroll 1
        for (int i = tid; i < L; i += NT) {
            float v[G];
            load_z<G>(zb, i, v);
            less_max(v, i, L);
            kb[i] = ordered_key(key_of(v));
        }
        __threadfence_block();
        __syncthreads();
        block_select_topk<NT, 0>([kb](int i) { return kb[i]; }, L, a.top_k, [pk](int pos, int i) { pk[pos] = (uint32_t)i; }, s_hist);
        __threadfence_block();
        __syncthreads();
        const int per = (a.top_k + nb - 1) / nb;
        float mx[G];
#pragma unroll
        for (int hh = 0; hh < G; ++hh) mx[hh] = -__builtin_huge_valf();
#pragma unroll 1
        for (int p = tid; p < n; p += NT) {
            float v[G];
            load_z<G>(zb, (int)pk[p], v);
#pragma unroll
            for (int hh = 0; hh < G; ++hh) mx[hh] = fmaxf(mx[hh], v[hh]);
            if (p >= x * per && p < (x + 1) * per) {
                const int id = cb[pk[p]];
                a.sel[(size_t)ul * a.top_k + p] = id;
                if (a.out_sel) a.out_sel[(size_t)ul * a.top_k + p] = id;
            }
        }
#pragma unroll
        for (int hh = 0; hh < G; ++hh) {
            float v = mx[hh];
#pragma unroll
            for (int s = 32; s >= 1; s >>= 1) v = fmaxf(v, __shfl_xor(v, s));
            if (ln == 0) s_l[wv][hh] = v;
        }
        __syncthreads();
        if (tid < G) {
            float v = s_l[0][tid];
#pragma unroll
            for (int w = 1; w < NW; ++w) v = fmaxf(v, s_l[w][tid]);
            s_m[tid] = v;
        }
        __syncthreads();
#pragma unroll 1
        for (int p = wv * 4 + row4; p < n; p += NW * 4) {
            const int i = (int)pk[p];
            float v[G];
            load_z<G>(zb, i, v);
            const Chunk<T> c = load_chunk(V + (size_t)rb[i] * kD, lane16);
#pragma unroll
            for (int hh = 0; hh < G; ++hh) {
                v[hh] = __expf(v[hh] - s_m[hh]);
                if (lane16 == 0) lsum[hh] += v[hh];
            }
            add_row(c, v);
        }
        hand_over();
        if (tid < per_w) {
            o = block_pair(word);
            l_o = block_l(word >> 6);
        }
    }
    if (tid < per_w) {
        const int hh = word >> 6, dim = 2 * (word & 63), b = ul / a.at.g, head = b * a.at.h + (ul - b * a.at.g) * G + hh;
        const float mh = s_m[hh];
        float lse;
        float2 r;
        r.x = merge_window<G>(a.at.win, ul, hh, dim, o.x, mh, l_o, lse);
        r.y = merge_window<G>(a.at.win, ul, hh, dim + 1, o.y, mh, l_o, lse);
        *reinterpret_cast<float2 *>(a.at.out + (size_t)head * kD + dim) = r;
        if (dim == 0 && a.at.out_lse) a.at.out_lse[head] = lse;
    }
    CTKVR_STAMP(47);
    if (x == 0) {
        for (int p = n + tid; p < a.top_k; p += NT) {
            a.sel[(size_t)ul * a.top_k + p] = -1;
            if (a.out_sel) a.out_sel[(size_t)ul * a.top_k + p] = -1;
        }
        if (tid == 0) a.nsel[ul] = n;
    }
}

// ------------------------------------------------------------------------------
// Algorithm 2 line 12 (dynamic centroid update): the step's query becomes the centroid of the
// FIFO slot (updates so far mod C: the oldest mapping goes first) for the G heads of the group,
// with its inverse norm, and the slot's list becomes src[unit][0..rho): the top-rho ids by rerank
// score, ascending (should fewer have been recalled, the last one is repeated; none: no update).
// grid batch*g, 256 threads; the block that ends last counts the update.
// ------------------------------------------------------------------------------
struct DcuArgs {
    int g, h, G, c_max, rho, src_stride;
    const int32_t *n_cent;
    uint32_t *count;          // [2]: updates so far; blocks of this update that are done (zero between updates)
    const void *q;            // [batch][h][128]
    const int32_t *src;       // [units][src_stride]
    const int32_t *nsrc;      // [units]
    void *centroids;          // [batch][h][c_max][128]
    float *inv_norm_c;        // [batch][h][c_max]
    int32_t *lists;           // [units][c_max][rho]
};

__device__ __forceinline__ void store_chunk(float *row, int lane16, const Chunk<float> &c)
{
    float4 *p = reinterpret_cast<float4 *>(row + 8 * lane16);
    p[0] = c.a;
    p[1] = c.b;
}
__device__ __forceinline__ void store_chunk(bf16_t *row, int lane16, const Chunk<bf16_t> &c)
{
    *reinterpret_cast<uint4 *>(row + 8 * lane16) = c.w;
}

// The slot's list from the step's ranking keys and the slot's centroids, one unit per block (NT threads): emit_list(dst) writes
// the list; the rest as described above.
template <typename T, int NT, typename ListFn>
__device__ __forceinline__ void dcu_write_unit(const DcuArgs &a, const int n, ListFn emit_list)
{
    const int ul = blockIdx.x, b = ul / a.g, kv = ul - b * a.g, tid = threadIdx.x;
    const int slot = (int)(a.count[0] % (uint32_t)a.n_cent[b]);
    if (n > 0) {
        emit_list(a.lists + ((size_t)ul * a.c_max + slot) * a.rho);
        if (tid < 16 * a.G) {
            const int hh = tid >> 4, lane16 = tid & 15;
            const size_t head = (size_t)b * a.h + kv * a.G + hh;
            Chunk<T> c = load_chunk((const T *)a.q + head * kD, lane16);
            store_chunk((T *)a.centroids + (head * a.c_max + slot) * kD, lane16, c);
            float x[8];
            unpack(c, x);
            const float n2 = group16_sum(lane_partial(x, x));
            if (lane16 == 0) a.inv_norm_c[head * a.c_max + slot] = inv_norm_from_sq(n2);
        }
    }
    // The update is counted by the block that ends last: every block has read the count before it reports done.
    __syncthreads();
    if (tid == 0 && atomicAdd(&a.count[1], 1u) == gridDim.x - 1) {
        atomicExch(&a.count[1], 0u);
        atomicAdd(&a.count[0], 1u);
    }
}

// rho = rho': the list is the step's selection.  grid batch*g, 256 threads
template <typename T> __global__ __launch_bounds__(256) void dcu_write_kernel(DcuArgs a)
{
    const int ul = blockIdx.x, tid = threadIdx.x;
    const int n = min(a.nsrc[ul], a.rho);
    dcu_write_unit<T, 256>(a, n, [&](int32_t *dst) {
        const int32_t *src = a.src + (size_t)ul * a.src_stride;
        for (int r = tid; r < a.rho; r += 256) dst[r] = src[min(r, n - 1)];
    });
}

// Another budget: the step's ranking keys selected once more and written in the same launch (histogram, classification,
// selection, write and the fills they need took 21 us of a 65 us step with update; this takes 8 up to the 8192 keys it keeps).  One
// block per unit, which reads later keys again, twice, at the 20 GB/s of its CU: the host takes it up to kDcuStride.  grid batch*g, kTailThreads; dynamic shared memory: kSelLds + 2 kListCap + bits_words words
constexpr int kDcuStride = 49152;

struct DcuSelectArgs {
    DcuArgs d;
    const int32_t *ncand, *cand;   // [units], [units][l_stride]
    const uint32_t *kbuf;          // [units][l_stride] ordered images of the ranking keys
    int l_stride;
};

template <typename T> __global__ __launch_bounds__(kTailThreads) void dcu_select_kernel(DcuSelectArgs a)
{
    extern __shared__ __align__(16) uint32_t smem[];
    constexpr int NT = kTailThreads, NW = NT / 64, KPT = kTailKeys / NT;
    __shared__ uint32_t s_res[4];
    uint32_t *s_hist = smem, *s_list = smem + kSelLds, *s_bits = s_list + 2 * kListCap;
    const int ul = blockIdx.x, tid = threadIdx.x, ln = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t *kb = a.kbuf + (size_t)ul * a.l_stride;
    const int32_t *cb = a.cand + (size_t)ul * a.l_stride;
    uint32_t kk[KPT];
    int32_t id[KPT];
#pragma unroll
    for (int q = 0; q < KPT; ++q) kk[q] = kb[min(q * NT + tid, a.l_stride - 1)];   // before L is known; stale beyond it
#pragma unroll
    for (int q = 0; q < KPT; ++q) id[q] = cb[min(q * NT + tid, a.l_stride - 1)];
    const int L = a.ncand[ul];
    for (int w = tid; w < kBuckets / 4; w += NT) reinterpret_cast<uint4 *>(s_hist)[w] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0) s_res[3] = 0u;
    float kreg[KPT];
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
        const float x = fmaxf(ordered_value(kk[q]), -3.0e38f);   // (above the -inf of the slots beyond L)
        kreg[q] = q * NT + tid < L ? x : -__builtin_huge_valf();
    }
    __syncthreads();
    dcu_write_unit<T, NT>(a.d, L, [&](int32_t *dst) {
        if (a.d.rho >= L) {   // every recalled key, the last one repeated should there be fewer than rho
            for (int r = tid; r < a.d.rho; r += NT) dst[r] = cb[min(r, L - 1)];
            return;
        }
        select_keys<NT, KPT, true>(
            kreg, L, L, a.d.rho,
            [&](auto f) __attribute__((always_inline)) {
                constexpr int NF = 8;   // rounds requested together
                for (int g0 = KPT * NW + wv; g0 * 64 < L; g0 += NF * NW) {
                    uint32_t x[NF];
#pragma unroll
                    for (int u = 0; u < NF; ++u) x[u] = kb[min((g0 + u * NW) * 64 + ln, L - 1)];
#pragma unroll
                    for (int u = 0; u < NF; ++u) {
                        const int gq = g0 + u * NW;
                        if (gq * 64 >= L) break;
                        f(gq, gq * 64 + ln < L ? fmaxf(ordered_value(x[u]), -3.0e38f) : -__builtin_huge_valf());
                    }
                }
            },
            [&](int q, int, uint32_t pos) __attribute__((always_inline)) { dst[pos] = id[q]; },
            [&](int pos, int i) __attribute__((always_inline)) { dst[pos] = cb[i]; },
            [&](int i) { return kb[i]; }, s_hist, s_list, s_bits, s_res);
    });
}

}  // namespace ctkvr
