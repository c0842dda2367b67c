// k-means centroid mode of the index build (replaces Algorithm 1 line 1 only; the
// paper itself takes the last C prompt queries).  Per (sequence, KV head) the s
// prompt positions are clustered; a point is the concatenation of the G query-head
// vectors of the group at one position (G*128 numbers, contiguous in q_prefill).
// Lloyd iteration = half-norms -> assignment on the matrix cores -> counting sort of the positions by
// centre (ranks inside stretches of positions, offsets, scatter) -> blocks per centre, one for
// every 256 members, sum them in fixed point and the last writes the new centre.  The centres live in the index's centroid table
// [b][h][c_max][128] all along: head hh of centre c is one 128-element row.
#pragma once
#include "kernels.hpp"

namespace ctkvr {

struct KmeansArgs {
    int g, h, c_max, s_max;
    const int32_t *n_cent, *ctx_lens;
    const int32_t *first_row;      // [batch] row of position 0 of each sequence in q_prefill
    const bf16_t *q;               // [rows][h][128]
    bf16_t *centroids;             // [batch][h][c_max][128]
    const int32_t *init_pos;       // [batch][g][c_max]
    float *half_norm;              // [batch*g][c_max]
    int32_t *assign;               // [batch*g][s_max]
    uint32_t *counts;              // [batch*g][n_stretch][c_max] members per centre in a stretch; then those in the stretches before it
    int stretch, n_stretch;        // positions of a stretch, ceil(s_max / stretch)
    uint32_t *start;               // [batch*g][c_max] first slot of each centre in `order`
    uint32_t *rank;                // [batch*g][s_max] which member of its centre a position is in its stretch, in arrival order
    int32_t *order;                // [batch*g][s_max] positions grouped by centre
    // centres of more than kPartRows members: the blocks that sum their further parts, and where the parts meet
    uint2 *part;                   // [batch*g][ext_max] (centre, part) of the blocks behind the first c_max
    uint32_t *n_part;              // [batch*g] how many of them there are
    uint32_t *slot;                // [batch*g][c_max] first of the centre's entries in `part`; its accumulator
    unsigned long long *sums;      // [batch*g][ext_max][G*128], all zero between iterations
    uint32_t *done;                // [batch*g][ext_max] parts of the slot's centre that are in `sums`; zero likewise
    int ext_max;                   // s_max / kPartRows + 1
};
constexpr uint32_t kPartRows = 256;
constexpr int kStretches = 32;   // of a sequence, of at least 1024 positions each

// centres start as the prompt queries at init_pos; grid (c_max, h, batch), 128 threads
__global__ void kmeans_init_kernel(KmeansArgs a, int G)
{
    const int j = blockIdx.x, hd = blockIdx.y, b = blockIdx.z;
    if (j >= a.n_cent[b]) return;
    const int kv = hd / G;
    int pos = a.init_pos[((size_t)b * a.g + kv) * a.c_max + j];
    pos = max(0, min(pos, a.ctx_lens[b] - 1));
    const bf16_t *src = a.q + ((size_t)(a.first_row[b] + pos) * a.h + hd) * kD;
    a.centroids[(((size_t)b * a.h + hd) * a.c_max + j) * kD + threadIdx.x] = src[threadIdx.x];
}

// half_norm[c] = |mu_c|^2 / 2 (heads summed in order); grid (ceil(c_max/16), batch*g), 256 threads
template <int G> __global__ __launch_bounds__(256) void kmeans_halfnorm_kernel(KmeansArgs a)
{
    const int ul = blockIdx.y, b = ul / a.g, kv = ul - b * a.g;
    const int C = a.n_cent[b];
    const int lane16 = threadIdx.x & 15, grp = threadIdx.x >> 4;
    const int c = blockIdx.x * 16 + grp;
    if (blockIdx.x * 16 >= C) return;
    const int cc = c < C ? c : C - 1;
    float n2 = 0.0f;
#pragma unroll
    for (int hh = 0; hh < G; ++hh) {
        float x[8];
        unpack(load_chunk(a.centroids + (((size_t)b * a.h + kv * G + hh) * a.c_max + cc) * kD, lane16), x);
        n2 = n2 + group16_sum(lane_partial(x, x));
    }
    if (c < C && lane16 == 0) a.half_norm[(size_t)ul * a.c_max + c] = 0.5f * n2;
}

// assignment: argmax_c (x . mu_c - |mu_c|^2/2), ties to the lowest c.  A = 32 centres x 16 dims,
// B = 16 dims x 32 points per v_mfma_f32_32x32x16_bf16.  What bounds it is shared memory as much as the
// matrix pipe: a 16-byte fragment read per lane takes 8 cycles of the CU's LDS, a matrix instruction 32 of one
// of its four SIMDs, so with one read per instruction both are full at once.  Hence a wave holds the whole
// points of PT = 2 column tiles in registers (256 of them at G = 4: one wave per SIMD, 512 registers) and every
// centre fragment read feeds two instructions.  The centres go by in tiles of 32 CTN, whole (all G heads),
// through two shared-memory buffers, the next tile loaded straight into shared memory while this one is multiplied, one barrier
// per tile.  With a
// single wave per SIMD nothing else hides the vector work, so the accumulators are two sets: the argmax of a
// row tile runs between the matrix instructions of the next.  128K points x 2048 centres x 8 heads of G = 4: 1.57 to
// 1.68 ms, 1.31 to 1.40 PFLOP/s (tiles through registers 1.86, also with 32 points a wave and two waves per SIMD 1.95 ms).
// With G = 8 (a point takes 256 registers) a wave has one column tile and the centre tiles are half as high.
// The accumulators start from -|mu_c|^2/2, so the result tile
// is the score itself.
// grid (ceil(s_max / (128 PT)), batch*g), 256 threads, dynamic shared memory AssignShape<G>::kLds.
template <int G> struct AssignShape {
    static constexpr int KS = 8 * G;             // k-steps of 16 dims
    static constexpr int PT = G <= 4 ? 2 : 1;    // column tiles (32 points each) of a wave
    static constexpr int CTN = G <= 4 ? 2 : 1;   // row tiles (32 centres each) of a step
    static constexpr int NC = 32 * CTN;
    static constexpr int kTile = NC * G * kD * 2;   // bytes of a centre tile
    static constexpr int kLds = 2 * (kTile + NC * 4);
    static constexpr int kPoints = 4 * PT * 32;     // points of a block
};

template <int G> __global__ __launch_bounds__(256, G <= 2 ? 2 : 1) void kmeans_assign_kernel(KmeansArgs a)
{
    using S = AssignShape<G>;
    constexpr int KS = S::KS, PT = S::PT, CTN = S::CTN, NC = S::NC;
    constexpr int AHEAD = 4;   // centre fragments in registers: requested three k-steps before their use
    extern __shared__ __align__(16) unsigned char s_dyn[];   // two centre tiles, then their half-norms
    float *const s_hn = reinterpret_cast<float *>(s_dyn + 2 * S::kTile);
    const int ul = blockIdx.y, b = ul / a.g, kv = ul - b * a.g;
    const int C = a.n_cent[b], s = a.ctx_lens[b];
    if ((int)blockIdx.x * S::kPoints >= s) return;
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), ln = tid & 63, col = ln & 31, half = ln >> 5;
    const int p0 = blockIdx.x * S::kPoints + wv * (PT * 32);
    bf16x8_t bfrag[PT][KS];
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) {
        const int t = min(p0 + pt * 32 + col, s - 1);
        const bf16_t *xrow = a.q + ((size_t)(a.first_row[b] + t) * a.h + kv * G) * kD + 8 * half;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) bfrag[pt][kk] = *reinterpret_cast<const bf16x8_t *>(xrow + kk * 16);
    }
    // Staging: a tile is 2 G lines of 128 bytes of NC rows, line after line; 16-byte piece p of a line of row r lies at
    // p ^ swz(r), so that a fragment read (one piece of 32 rows) spreads over the banks.  Loaded straight into shared memory, eight
    // rows of a line (1 KB, whole lines) an instruction, wave w the row groups w, w + 4, ..; all of a tile's loads are requested in
    // the first quarter of a step and waited for at its end.  (Through registers -- 16 loads, 16 writes and 64 registers a
    // thread and tile, in a wave that is alone on its SIMD -- the loop took 100 us per block where the products alone take 77.)
    constexpr int RG = NC / 32, NLD = RG * 2 * G, STEPS = CTN * KS, QUARTER = STEPS / 4;   // row groups, loads of a wave
    const bf16_t *cbase = a.centroids + ((size_t)b * a.h + kv * G) * a.c_max * kD;
    const float *hnrow = a.half_norm + (size_t)ul * a.c_max;
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char *)s_dyn);
    auto request = [&](int p, int c0, int buf) __attribute__((always_inline)) {   // load p: row group p % RG, line p / RG
        const int rg = wv + 4 * (p % RG), line = p / RG;
        const int c = min(c0 + rg * 8 + (ln >> 3), C - 1);   // rows beyond C repeat the last centre; their accumulators start from -inf
        const uint32_t piece = (uint32_t)((ln & 7) ^ (ln >> 3) ^ (rg & 1));
        const char *from = reinterpret_cast<const char *>(cbase + (size_t)(line >> 1) * a.c_max * kD) + (line & 1) * 128;
        load_to_lds(lds0 + buf * S::kTile + line * (NC * 128) + rg * 1024, from, (uint32_t)c * (kD * 2) + piece * 16);
    };
    auto hn_at = [&](int c0) {
        const int c = c0 + (tid & (NC - 1));
        const float v = -hnrow[min(c, C - 1)];
        return c < C ? v : -__builtin_huge_valf();
    };
    float best[PT];
    int bi[PT];
    f32x16_t acc_a[PT], acc_b[PT];
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) {
        best[pt] = -__builtin_huge_valf();
        bi[pt] = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_a[pt][r] = acc_b[pt][r] = -__builtin_huge_valf();
    }
    // scores of a finished row tile against the best so far; `loc` is the row inside it
    constexpr int E = PT * 16;
    float was[PT];
    int loc[PT];
    auto argmax_begin = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) {
            was[pt] = best[pt];
            loc[pt] = 0;
        }
    };
    auto argmax_part = [&](const f32x16_t (&acc)[PT], int e_lo, int e_hi) __attribute__((always_inline)) {
#pragma unroll
        for (int e = e_lo; e < e_hi; ++e) {
            const int pt = e % PT, r = e / PT;
            const float v = acc[pt][r];
            loc[pt] = v > best[pt] ? 8 * (r >> 2) + (r & 3) : loc[pt];
            best[pt] = v > best[pt] ? v : best[pt];
            asm volatile("" : "+v"(loc[pt]));   // or the selects are gathered behind the last product, where nothing hides them
        }
    };
    auto argmax_end = [&](int c) __attribute__((always_inline)) {   // c: first row of the finished tile
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) bi[pt] = best[pt] > was[pt] ? c + loc[pt] + 4 * half : bi[pt];
    };
    // one row tile: its products into cur, the scores of the one before (prev) compared on the way
    auto row_tile = [&](f32x16_t (&cur)[PT], const f32x16_t (&prev)[PT], int ct, int buf, int c0) __attribute__((always_inline)) {
        // fragment kk: 8 elements of row ct * 32 + col: piece 2 (kk % 4) + half of line kk / 4
        const uint32_t mine = (uint32_t)(col * 128 + ((half ^ (col & 7) ^ ((col >> 3) & 1)) * 16));
        uint32_t at4[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) at4[x] = (mine ^ (x * 32)) + buf * S::kTile;
        auto frag = [&](int kk) __attribute__((always_inline)) {
            return *reinterpret_cast<const bf16x8_t *>(s_dyn + at4[kk & 3] + (kk >> 2) * (NC * 128) + ct * 4096);
        };
        f32x16_t hn;
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
            const float4 v = *reinterpret_cast<const float4 *>(&s_hn[buf * NC + ct * 32 + 8 * rq + 4 * half]);
            hn[4 * rq + 0] = v.x;
            hn[4 * rq + 1] = v.y;
            hn[4 * rq + 2] = v.z;
            hn[4 * rq + 3] = v.w;
        }
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) cur[pt] = hn;
        argmax_begin();
        bf16x8_t af[AHEAD];
#pragma unroll
        for (int kk = 0; kk < AHEAD - 1; ++kk) af[kk] = frag(kk);
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            const int at = ct * KS + kk;   // of STEPS
            if (at < QUARTER) {
#pragma unroll
                for (int p = at * NLD / QUARTER; p < (at + 1) * NLD / QUARTER; ++p) request(p, c0 + NC, buf ^ 1);
            }
            if (kk + AHEAD - 1 < KS)
                af[(kk + AHEAD - 1) % AHEAD] = frag(kk + AHEAD - 1);
#pragma unroll
            for (int pt = 0; pt < PT; ++pt)
                cur[pt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[kk % AHEAD], bfrag[pt][kk], cur[pt], 0, 0, 0);
            argmax_part(prev, kk * E / KS, (kk + 1) * E / KS);
            __builtin_amdgcn_sched_barrier(0);   // the order written here is the schedule
        }
        argmax_end(c0 + ct * 32 - 32);
    };
    // a tile, its row tiles into x and y in turn.  The next tile goes into the other buffer (past
    // the end: the last centre again, never used).
    auto step = [&](f32x16_t (&x)[PT], f32x16_t (&y)[PT], int buf, int c0) __attribute__((always_inline)) {
        const float hn_next = hn_at(c0 + NC);
        row_tile(x, y, 0, buf, c0);
        if constexpr (CTN == 2) row_tile(y, x, 1, buf, c0);
        s_hn[(buf ^ 1) * NC + (tid & (NC - 1))] = hn_next;   // the four waves write the same values
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };
#pragma unroll
    for (int p = 0; p < NLD; ++p) request(p, 0, 0);
    s_hn[tid & (NC - 1)] = hn_at(0);
    __builtin_amdgcn_s_waitcnt(kVmcnt0);   // (the builtin: the compiler then knows that the points are there, and puts no waits into the loop)
    __syncthreads();
    int buf = 0, c0 = 0;
    if constexpr (CTN == 2) {
        for (; c0 < C; c0 += NC, buf ^= 1) step(acc_a, acc_b, buf, c0);
        argmax_begin();
        argmax_part(acc_b, 0, E);
    } else {
        for (; c0 < C; c0 += 2 * NC) {   // an odd last tile: the second step of its pair multiplies rows that start from -inf
            step(acc_a, acc_b, 0, c0);
            step(acc_b, acc_a, 1, c0 + NC);
        }
        argmax_begin();
        argmax_part(acc_b, 0, E);
    }
    argmax_end(c0 - 32);
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) {
        const float ob = __shfl_xor(best[pt], 32);
        const int oi = __shfl_xor(bi[pt], 32);
        if (ob > best[pt] || (ob == best[pt] && oi < bi[pt])) bi[pt] = oi;
        const int t = p0 + pt * 32 + col;
        if (half == 0 && t < s) a.assign[(size_t)ul * a.s_max + t] = bi[pt];
    }
}

// Members of every centre in a stretch of positions, and which of them each position is, by counters in shared memory.
// (One returning atomic per position on counters in memory, at the end of the assignment, cost every block of it
// 4-20 us, where nothing else runs on its CU.)  grid (n_stretch, batch*g), 1024 threads, dynamic shared memory c_max words
__global__ __launch_bounds__(1024) void kmeans_rank_kernel(KmeansArgs a)
{
    extern __shared__ __align__(16) uint32_t s_cnt[];
    const int ul = blockIdx.y, b = ul / a.g, tid = threadIdx.x;
    const int C = a.n_cent[b], s = a.ctx_lens[b];
    for (int j = tid; j < C; j += 1024) s_cnt[j] = 0u;
    __syncthreads();
    const int t0 = (int)blockIdx.x * a.stretch, t1 = min(s, t0 + a.stretch);
    const int32_t *as = a.assign + (size_t)ul * a.s_max;
    uint32_t *rk = a.rank + (size_t)ul * a.s_max;
    for (int t = t0 + tid; t - tid < t1; t += 4 * 1024) {   // four positions a thread requested together
        int c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = as[min(t + u * 1024, s - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (t + u * 1024 < t1) rk[t + u * 1024] = atomicAdd(&s_cnt[c[u]], 1u);
    }
    __syncthreads();
    uint32_t *cnt = a.counts + ((size_t)ul * a.n_stretch + blockIdx.x) * a.c_max;
    for (int j = tid; j < C; j += 1024) cnt[j] = s_cnt[j];
}

// start[c] = number of positions assigned to centres below c; counts become the members in the stretches before each; the blocks of
// the update behind the first c_max get the further parts of the large centres.
// grid batch*g, 1024 threads (C <= 8192: eight centres per thread), dynamic shared memory c_max words
__global__ __launch_bounds__(1024) void kmeans_offsets_kernel(KmeansArgs a)
{
    extern __shared__ __align__(16) uint32_t s_cnt[];
    __shared__ uint32_t s_tmp[32];
    const int ul = blockIdx.x, b = ul / a.g;
    const int C = a.n_cent[b], tid = threadIdx.x;
    for (int j = tid; j < C; j += 1024) {
        uint32_t *col = a.counts + (size_t)ul * a.n_stretch * a.c_max + j, x[kStretches], sum = 0;
#pragma unroll
        for (int u = 0; u < kStretches; ++u) x[u] = col[(size_t)min(u, a.n_stretch - 1) * a.c_max];
#pragma unroll
        for (int u = 0; u < kStretches; ++u)
            if (u < a.n_stretch) {   // uniform
                col[(size_t)u * a.c_max] = sum;
                sum += x[u];
            }
        s_cnt[j] = sum;
    }
    __syncthreads();
    uint32_t c[8], mine = 0, parts = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        int j = tid * 8 + q;
        c[q] = j < C ? s_cnt[j] : 0u;
        mine += c[q];
        parts += c[q] ? (c[q] - 1u) / kPartRows : 0u;
    }
    uint32_t tot, n_ext;
    uint32_t before = block_excl_scan<1024>(mine, s_tmp, &tot);
    uint32_t at = block_excl_scan<1024>(parts, s_tmp, &n_ext);   // at most s / kPartRows
    if (tid == 0) a.n_part[ul] = n_ext;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        int j = tid * 8 + q;
        if (j < C) {
            a.start[(size_t)ul * a.c_max + j] = before;
            a.slot[(size_t)ul * a.c_max + j] = at;
            for (uint32_t p = 1; (p * kPartRows) < c[q]; ++p) a.part[(size_t)ul * a.ext_max + at++] = make_uint2((uint32_t)j, p);
        }
        before += c[q];
    }
}

// order[start[assign[t]] + members in the stretches before + rank[t]] = t.  The order inside a centre's range is whatever the
// counters gave: the sums taken over it are integer sums.  grid (ceil(s_max/256), batch*g), 256 threads
__global__ __launch_bounds__(256) void kmeans_scatter_kernel(KmeansArgs a)
{
    const int ul = blockIdx.y, b = ul / a.g;
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= a.ctx_lens[b]) return;
    const int c = a.assign[(size_t)ul * a.s_max + t];
    const uint32_t pos = a.start[(size_t)ul * a.c_max + c] + a.counts[((size_t)ul * a.n_stretch + t / a.stretch) * a.c_max + c] +
                         a.rank[(size_t)ul * a.s_max + t];
    a.order[(size_t)ul * a.s_max + pos] = t;
}

// One block per centre: sum_c = sum of llrint(x * 2^20) over its members (int64 per element, in
// registers), mu_c = sum / count (fp64 divide, rounded to fp32, then to bf16 nearest-even); an
// empty centre keeps its place.  Groups of 128 threads take the members eight at a time in
// turn (their ids are requested one round ahead of their rows); thread e of a group owns the G
// consecutive elements e*G .. e*G+G-1 of the G*128-element point, and the groups' integer sums
// are added through shared memory.  A centre of more than kPartRows members is summed by several blocks (the first
// iterations have centres of many times the average: their one block was most of the launch, 1.3 ms against 0.27):
// each adds its sums to the centre's 64-bit accumulators, and the last of them takes those and leaves zeros.
// Where a wave's values of a round are all below 128 (27 bits each), the round's eight are summed in 32 bits, five vector instructions
// an element; converted and added one by one in 64 bits, which the others still are, twelve, and those bounded the launch.  131072 points, 2048
// centres, eight KV heads of four 332 -> 300 us (now bound by the rows' 1 GB), 20000 and 600 42.7 -> 33.0; of two heads 40000 and 900
// 51 -> 38.5 (with two groups; four 44.2); of eight 50001 and 777 97 -> 94; of one 30000 and 500 29.9 -> 28.4.
// grid (c_max + ext_max, batch*g), ReduceShape<G>::NT threads
template <int G> struct ReduceShape {
    static constexpr int NG = G <= 2 ? 2 : 4, NT = 128 * NG;   // groups; a row of one or two heads is 256 or 512 bytes
};
template <int G> __global__ __launch_bounds__((ReduceShape<G>::NT)) void kmeans_reduce_kernel(KmeansArgs a)
{
    constexpr int NG = ReduceShape<G>::NG;
    __shared__ long long s_part[NG - 1][128][G];
    const int ul = blockIdx.y, b = ul / a.g, kv = ul - b * a.g;
    __shared__ uint32_t s_last;
    const int C = a.n_cent[b];
    int c = blockIdx.x;
    uint32_t p = 0;
    if (c >= a.c_max) {
        if ((uint32_t)(c - a.c_max) >= a.n_part[ul]) return;
        const uint2 cp = a.part[(size_t)ul * a.ext_max + (c - a.c_max)];
        c = (int)cp.x;
        p = cp.y;
    }
    if (c >= C) return;
    const uint32_t st = a.start[(size_t)ul * a.c_max + c];
    const uint32_t n_all = (c + 1 < C ? a.start[(size_t)ul * a.c_max + c + 1] : (uint32_t)a.ctx_lens[b]) - st;
    const uint32_t n = min(n_all - p * kPartRows, kPartRows);   // of this part
    const int32_t *ord = a.order + (size_t)ul * a.s_max + st + p * kPartRows;
    const int e = threadIdx.x & 127, grp = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 7);
    const bf16_t *base = a.q + ((size_t)a.first_row[b] * a.h + kv * G) * kD;
    const size_t rstride = (size_t)a.h * kD;
    long long acc[G];
#pragma unroll
    for (int r = 0; r < G; ++r) acc[r] = 0;
    // element r of a thread's G, with 20 added to its exponent (of normal values below 128: times 2^20, exact; of zeros and subnormals
    // still nothing)
    constexpr int NWD = (G + 1) / 2;   // words of G elements
    constexpr uint32_t kUp = 20u << 23;
    auto scaled = [&](const uint32_t (&w)[NWD], int r) __attribute__((always_inline)) {
        return __uint_as_float(r & 1 ? (w[r >> 1] & 0xffff0000u) + kUp : (w[r >> 1] << 16) + kUp);
    };
    int t[8];
    if (n) {
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = ord[min((uint32_t)(grp * 8 + u), n - 1)];
    }
    for (uint32_t m0 = grp * 8; m0 < n; m0 += NG * 8) {
        uint32_t w[8][NWD];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            w[u][NWD - 1] = 0u;
            __builtin_memcpy(w[u], base + (size_t)t[u] * rstride + (uint32_t)(e * G), G * sizeof(bf16_t));
        }
        int tn[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) tn[u] = ord[min(m0 + NG * 8 + u, n - 1)];
        typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
        u16x2_t most = {0, 0};
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int k = 0; k < NWD; ++k) most = __builtin_elementwise_max(most, __builtin_bit_cast(u16x2_t, w[u][k] & 0x7fff7fffu));
        if (__all(max((uint32_t)most.x, (uint32_t)most.y) < 0x4300u)) {   // |x| < 128
            int sum[G];
#pragma unroll
            for (int r = 0; r < G; ++r) sum[r] = 0;
            if (m0 + 8 <= n) {   // uniform
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int r = 0; r < G; ++r) sum[r] += __float2int_rn(scaled(w[u], r));
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (m0 + u < n) {
#pragma unroll
                        for (int r = 0; r < G; ++r) sum[r] += __float2int_rn(scaled(w[u], r));
                    }
            }
#pragma unroll
            for (int r = 0; r < G; ++r) acc[r] += sum[r];
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (m0 + u < n) {
#pragma unroll
                    for (int r = 0; r < G; ++r)
                        acc[r] += __float2ll_rn(__uint_as_float(r & 1 ? w[u][r >> 1] & 0xffff0000u : w[u][r >> 1] << 16) * 1048576.0f);
                }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = tn[u];
    }
    if (grp) {
#pragma unroll
        for (int r = 0; r < G; ++r) s_part[grp - 1][e][r] = acc[r];
    }
    __syncthreads();
    const uint32_t n_parts = (n_all + kPartRows - 1) / kPartRows;
    long long tot[G];
    if (grp == 0) {
#pragma unroll
        for (int r = 0; r < G; ++r) {
            tot[r] = acc[r];
#pragma unroll
            for (int y = 0; y < NG - 1; ++y) tot[r] += s_part[y][e][r];
        }
    }
    if (n_parts > 1) {
        const size_t slot = (size_t)ul * a.ext_max + a.slot[(size_t)ul * a.c_max + c];
        unsigned long long *sums = a.sums + slot * (G * 128) + e;
        if (grp == 0) {
#pragma unroll
            for (int r = 0; r < G; ++r) atomicAdd(&sums[r * 128], (unsigned long long)tot[r]);
            __threadfence();
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            const uint32_t had = atomicAdd(&a.done[slot], 1u);
            s_last = had == n_parts - 1;
            if (s_last) a.done[slot] = 0u;
            __threadfence();
        }
        __syncthreads();
        if (!s_last) return;
        if (grp == 0) {
#pragma unroll
            for (int r = 0; r < G; ++r) tot[r] = (long long)atomicExch(&sums[r * 128], 0ull);
        }
    }
    if (grp == 0 && n_all) {
#pragma unroll
        for (int r = 0; r < G; ++r) {
            const int ee = e * G + r, hh = ee >> 7, dim = ee & 127;
            float m = (float)((double)tot[r] * (1.0 / 1048576.0) / (double)n_all);
            uint32_t u = __float_as_uint(m);
            u += 0x7fffu + ((u >> 16) & 1u);
            a.centroids[(((size_t)b * a.h + kv * G + hh) * a.c_max + c) * kD + dim] = (bf16_t)(u >> 16);
        }
    }
}

}  // namespace ctkvr
