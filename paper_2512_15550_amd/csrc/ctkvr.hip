// Host side of the C ABI declared in include/ctkvr.h: argument checks, device
// memory of the index and its workspace, kernel launches.  No computation of the
// method happens on the host.
#include "../../include/ctkvr.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "kernels.hpp"
#include "kmeans.hpp"
#include "fused_args.hpp"

using namespace ctkvr;

namespace {

thread_local std::string g_err;

int fail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HIP_TRY(expr)                                                                           \
    do {                                                                                        \
        hipError_t e_ = (expr);                                                                 \
        if (e_ != hipSuccess)                                                                   \
            return fail(e_ == hipErrorOutOfMemory ? CTKVR_ENOMEM : CTKVR_EHIP, "%s: %s", #expr, \
                        hipGetErrorString(e_));                                                 \
    } while (0)

// Makes a device the calling thread's current one for a scope.  Events, the null stream, function attributes and
// device-wide waits are those of the current device, which need not be the one an index lives on.
struct DeviceScope {
    int before = -1;
    hipError_t err;
    explicit DeviceScope(int dev)
    {
        err = hipGetDevice(&before);
        if (err == hipSuccess && before == dev) before = -1;   // nothing to restore
        else err = hipSetDevice(dev);
    }
    ~DeviceScope()
    {
        if (before >= 0) (void)hipSetDevice(before);
    }
};

size_t elem_size(int dtype) { return dtype == CTKVR_BF16 ? 2 : 4; }

}  // namespace

// Scratch of the entry point that allocates nothing (ctkvr_decode_step_static): one array per GPU, held
// until the process ends.  Host code never uses the array's name as an address: the device address
// is looked up once per device and kept.  It takes every step whose buffers are 32 MiB or less with the words of a unit that atomics
// update packed, the bitmap's rows unpadded and share_tail_kernel's exchange left out, and has room for those: a cache line each and the
// padding at most 0.38 KB a unit, whose buffers take at least 28 KiB, i.e. 0.42 MiB in all; the exchange 4 KiB a unit and up to 5.7 KiB
// a block, for 128 units at most and a block a CU, i.e. 1.9 MiB on 256 CUs.
constexpr size_t kStaticStepBytes = (size_t)32 << 20;
constexpr size_t kStaticScratchBytes = kStaticStepBytes + ((size_t)4 << 20);
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned char *g_scratch_ptr[kMaxDevices] = {};

// device address of the current device's copy of `scratch`
int static_scratch(unsigned char **out)
{
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(CTKVR_EUNSUPPORTED, "device ordinal %d outside 0..%d", dev, kMaxDevices - 1);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        unsigned char *ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return fail(CTKVR_EHIP, "hipGetSymbolAddress returned a null address for the scratch array");
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return CTKVR_OK;
}

// Device memory kept between indexes.  An index and the scratch of its build are one allocation each; an index is built
// per prompt and freed per request, and hipMalloc / hipFree of what a 32K prompt takes cost 2 ms in the best case and 70 ms
// where the driver has to map and unmap 2 GB every time (7.6 to 76 ms a build, of which the kernels are 5.9).  Blocks that
// nothing uses any more are kept per device, at most kPoolMax bytes of them (the oldest go first), and handed out again: to a
// build for its scratch if it needs at least half of one, to an index, which has it as long as it lives, if that needs four fifths.
// ctkvr_release_scratch() frees them; CTKVR_BUILD_SCRATCH_CACHE=0 switches the
// keeping off.  A block enters the pool only after the work that used it has ended (a build synchronises its stream, an
// index its device), so it is idle whichever stream or host thread takes it next.  Where that wait fails -- a device cannot
// be waited for while one of its streams is being captured in global mode -- the block is set aside: nothing has it, and it is not
// freed, before a later wait for the device has succeeded (pool_settle).
constexpr size_t kPoolMax = (size_t)2 << 30;
struct PoolBlock {
    void *base;
    size_t bytes;
};
std::mutex g_pool_mu;
std::vector<PoolBlock> g_pool[kMaxDevices];   // oldest first
std::vector<PoolBlock> g_aside[kMaxDevices];  // blocks that work may still be using
int g_pool_builds[kMaxDevices] = {};          // builds that are using scratch right now

bool pool_on()
{
    const char *env = getenv("CTKVR_BUILD_SCRATCH_CACHE");
    return !(env && atoi(env) == 0);
}

// frees the current device's idle blocks (the caller holds g_pool_mu)
void pool_drop(int dev)
{
    for (PoolBlock &b : g_pool[dev]) (void)hipFree(b.base);
    g_pool[dev].clear();
}

// the work on the current device has ended
bool device_idle()
{
    if (hipDeviceSynchronize() == hipSuccess) return true;
    (void)hipGetLastError();   // (a launch's own check would report it)
    return false;
}

// an idle block into the pool, or to the runtime where it is not kept (the caller holds g_pool_mu)
void pool_keep(int dev, PoolBlock b)
{
    if (b.bytes > kPoolMax || !pool_on()) {
        (void)hipFree(b.base);
        return;
    }
    std::vector<PoolBlock> &v = g_pool[dev];
    v.push_back(b);
    size_t held = 0;
    for (PoolBlock &x : v) held += x.bytes;
    while (held > kPoolMax) {
        held -= v.front().bytes;
        (void)hipFree(v.front().base);
        v.erase(v.begin());
    }
}

// the blocks set aside on the current device, if it can be waited for now (the caller holds g_pool_mu)
void pool_settle(int dev)
{
    if (g_aside[dev].empty() || !device_idle()) return;
    for (PoolBlock &b : g_aside[dev]) pool_keep(dev, b);
    g_aside[dev].clear();
}

// a block of at least `bytes` on the current device `dev`, and of at most bytes / spare more if it was kept; out->bytes is its
// real size
int pool_get(int dev, size_t bytes, size_t spare, PoolBlock *out)
{
    const size_t grain = bytes < ((size_t)4 << 20) ? (size_t)64 << 10 : (size_t)2 << 20;
    bytes = (std::max<size_t>(bytes, 1) + grain - 1) / grain * grain;
    *out = PoolBlock{nullptr, 0};
    const bool pooled = dev >= 0 && dev < kMaxDevices;
    std::unique_lock<std::mutex> lock(g_pool_mu, std::defer_lock);
    if (pooled) {
        lock.lock();
        std::vector<PoolBlock> &v = g_pool[dev];
        for (int turn = 0; turn < 2; ++turn) {
            size_t best = v.size();
            for (size_t i = 0; i < v.size(); ++i)
                if (v[i].bytes >= bytes && v[i].bytes <= bytes + bytes / spare && (best == v.size() || v[i].bytes < v[best].bytes)) best = i;
            if (best < v.size()) {
                *out = v[best];
                v.erase(v.begin() + best);
                return CTKVR_OK;
            }
            if (turn || g_aside[dev].empty()) break;
            pool_settle(dev);   // only where nothing idle serves: a wait for the device can disturb a capture under way
        }
    }
    hipError_t e = hipMalloc(&out->base, bytes);
    if (e == hipErrorOutOfMemory && pooled && !g_pool[dev].empty()) {
        (void)hipGetLastError();
        pool_drop(dev);
        e = hipMalloc(&out->base, bytes);
    }
    if (e != hipSuccess) {
        out->base = nullptr;
        return fail(e == hipErrorOutOfMemory ? CTKVR_ENOMEM : CTKVR_EHIP, "hipMalloc(%zu): %s", bytes, hipGetErrorString(e));
    }
    out->bytes = bytes;
    return CTKVR_OK;
}

// gives a block of device `dev` back; idle: its users have been waited for
void pool_put(int dev, PoolBlock b, bool idle)
{
    if (!b.base) return;
    if (dev < 0 || dev >= kMaxDevices) {
        (void)hipFree(b.base);
        return;
    }
    std::lock_guard<std::mutex> lock(g_pool_mu);
    if (idle)
        pool_keep(dev, b);
    else
        g_aside[dev].push_back(b);
}

// Scratch of one build, given back at the end of the scope: as idle if waited() has heard of a synchronisation that succeeded.
struct BuildScratch {
    int dev = -1;
    bool idle = false;
    PoolBlock b{nullptr, 0};
    ~BuildScratch() { put(); }
    int get(int device, size_t bytes)
    {
        put();
        int rc = pool_get(device, bytes, 1, &b);
        if (rc != CTKVR_OK) return rc;
        dev = device;
        idle = false;
        if (dev >= 0 && dev < kMaxDevices) {
            std::lock_guard<std::mutex> lock(g_pool_mu);
            g_pool_builds[dev]++;
        }
        return CTKVR_OK;
    }
    void put()
    {
        if (!b.base) return;
        pool_put(dev, b, idle);
        if (dev >= 0 && dev < kMaxDevices) {
            std::lock_guard<std::mutex> lock(g_pool_mu);
            g_pool_builds[dev]--;
        }
        b = PoolBlock{nullptr, 0};
    }
    void waited(hipError_t e) { idle = e == hipSuccess; }
    unsigned char *base() const { return (unsigned char *)b.base; }
};

// Copies between pageable host memory and the device through pinned memory of the library: while a chunk is on the bus the next
// one is copied by the CPU.  Moving 16 MB to the device took 0.52 to 0.64 ms as one hipMemcpy and 0.97 ms back, the
// bus alone 0.30 ms.  One ring of kStageSlots chunks per device (8 MB, made on first use, freed by ctkvr_release_scratch); a
// caller that finds it in use takes plain copies, and so does one that finds it left by copies that could not be waited for, unless
// the device can be waited for now.
constexpr size_t kStageChunk = (size_t)1 << 20;
constexpr int kStageSlots = 8;
struct Staging {
    unsigned char *buf = nullptr;
    hipEvent_t ev[kStageSlots] = {};
    bool busy = false;
    bool unsure = false;   // copies may still be under way
};
Staging g_staging[kMaxDevices];   // (g_pool_mu)

struct CopySeg {
    void *dst;
    const void *src;
    size_t bytes;
};

void staging_drop(Staging &sg)
{
    if (sg.buf) (void)hipHostFree(sg.buf);
    for (hipEvent_t &e : sg.ev) {
        if (e) (void)hipEventDestroy(e);
        e = nullptr;
    }
    sg.buf = nullptr;
}

// the segments one after the other on `st`; on return everything has arrived
hipError_t copy_segments(int dev, const CopySeg *segs, int n, bool to_device, hipStream_t st)
{
    size_t total = 0;
    for (int i = 0; i < n; ++i) total += segs[i].bytes;
    Staging *sg = nullptr;
    if (dev >= 0 && dev < kMaxDevices && total >= ((size_t)128 << 10)) {
        std::lock_guard<std::mutex> lock(g_pool_mu);
        Staging &x = g_staging[dev];
        if (!x.busy && (!x.unsure || device_idle())) {
            x.unsure = false;
            bool ok = true;
            if (!x.buf) {
                ok = hipHostMalloc((void **)&x.buf, kStageChunk * kStageSlots, hipHostMallocDefault) == hipSuccess;
                for (hipEvent_t &e : x.ev) ok = ok && hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
                if (!ok) {
                    (void)hipGetLastError();
                    staging_drop(x);
                }
            }
            if (ok) {
                x.busy = true;
                sg = &x;
            }
        }
    }
    const hipMemcpyKind kind = to_device ? hipMemcpyHostToDevice : hipMemcpyDeviceToHost;
    hipError_t e = hipSuccess;
    if (!sg) {
        for (int i = 0; i < n && e == hipSuccess; ++i) e = hipMemcpyAsync(segs[i].dst, segs[i].src, segs[i].bytes, kind, st);
        hipError_t es = hipStreamSynchronize(st);
        return e != hipSuccess ? e : es;
    }
    struct Out {
        void *dst;
        size_t bytes;
    } out[kStageSlots] = {};   // to the host: what a slot's chunk becomes once it has arrived
    int at = 0;
    bool used[kStageSlots] = {};
    auto settle = [&](int slot) {
        if (!used[slot] || e != hipSuccess) return;
        e = hipEventSynchronize(sg->ev[slot]);
        if (e == hipSuccess && !to_device) memcpy(out[slot].dst, sg->buf + slot * kStageChunk, out[slot].bytes);
        used[slot] = false;
    };
    for (int i = 0; i < n && e == hipSuccess; ++i)
        for (size_t o = 0; o < segs[i].bytes && e == hipSuccess; o += kStageChunk, at = (at + 1) % kStageSlots) {
            const size_t m = std::min(kStageChunk, segs[i].bytes - o);
            unsigned char *pin = sg->buf + at * kStageChunk;
            settle(at);
            if (e != hipSuccess) break;
            if (to_device) {
                memcpy(pin, (const unsigned char *)segs[i].src + o, m);
                e = hipMemcpyAsync((unsigned char *)segs[i].dst + o, pin, m, kind, st);
            } else {
                e = hipMemcpyAsync(pin, (const unsigned char *)segs[i].src + o, m, kind, st);
                out[at] = Out{(unsigned char *)segs[i].dst + o, m};
            }
            if (e == hipSuccess) e = hipEventRecord(sg->ev[at], st);
            used[at] = e == hipSuccess;
        }
    for (int k = 0; k < kStageSlots; ++k) settle((at + k) % kStageSlots);
    const bool done = e == hipSuccess || hipStreamSynchronize(st) == hipSuccess;   // nothing uses the ring any more
    std::lock_guard<std::mutex> lock(g_pool_mu);
    sg->unsure = !done;
    sg->busy = false;
    return e;
}

// Lays arrays out one after the other, each 256-byte aligned; with base == nullptr only the size is computed.
struct Carver {
    unsigned char *base;
    size_t off = 0;
    void align_to(size_t a) { off = (off + a - 1) / a * a; }
    template <typename P> void take(P **ptr, size_t bytes)
    {
        if (base) *ptr = reinterpret_cast<P *>(base + off);
        off += (std::max<size_t>(bytes, 16) + 255) & ~(size_t)255;
    }
};
}  // namespace

// Buffers of one decode step for every (sequence, KV head) unit: everything ctkvr_decode_step
// writes apart from the caller's outputs.  An index owns one set; the entry point that allocates
// nothing lays the same set out in the library's static scratch array.
struct StepWs {
    float *cos = nullptr;
    int32_t *probe = nullptr, *cand = nullptr, *ncand = nullptr, *sel = nullptr, *nsel = nullptr;
    uint32_t *crow = nullptr, *srow = nullptr, *kbuf = nullptr, *gbits = nullptr, *ghist = nullptr;
    uint32_t *gbm = nullptr, *gcur = nullptr, *ginfo = nullptr;   // classify_kernel's outputs
    uint2 *glist = nullptr;
    unsigned long long *S = nullptr, *xs = nullptr;   // xs: tail_kernel's exchange slots
    float *z = nullptr, *zsel = nullptr;
    float *win = nullptr;   // window_attn_kernel's partial results
    uint32_t *m_key = nullptr;
    // single-launch step only (what its blocks hand to each other; see fused_args.hpp)
    float *part = nullptr;
    uint32_t *bar = nullptr;    // barrier counters, zero between steps
    int32_t *sid = nullptr, *slot_sure = nullptr;
    uint32_t *slot_cnt = nullptr, *slot_max = nullptr, *slot_hist = nullptr, *slot_npick = nullptr;
    unsigned long long *slot_S = nullptr;
    uint4 *slot_bkt = nullptr;
};

struct ctkvr_index {
    ctkvr_params p{};
    int G = 0, c_max = 0, s_max = 0, l_stride = 0, page_shift = 0, units = 0;
    float scale = 0.f;
    std::vector<int32_t> ctx_lens, n_cent;
    int dev = 0;
    PoolBlock mem{nullptr, 0};   // everything the index holds on the device
    // index proper
    void *centroids = nullptr;
    float *inv_norm_c = nullptr;
    int32_t *lists = nullptr;
    int32_t *d_ctx_lens = nullptr, *d_n_cent = nullptr;
    int32_t *d_first = nullptr;   // build: [batch] first row of each sequence in q_prefill
    StepWs ws;   // decode workspace
    // dynamic centroid update
    uint32_t *d_dcu_count = nullptr;   // [2]: updates so far (device side, so that captured graphs replay correctly), blocks of the running update that are done
    int32_t *dsel = nullptr, *dnsel = nullptr;   // top-rho ids of the second ranking (only when rho != rho')
    bool have_step = false;
    size_t recall_lds = 0, select_lds = 0, attn_lds = 0, build_select_lds = 0;
    size_t fused_lds = 0;   // non-zero: selection and attention run as one launch (select_attn_kernel)
    size_t dcu_lds = 0;     // non-zero: the update's ranking with a budget of its own runs as one launch (dcu_select_kernel)
    size_t tail_lds = 0;    // non-zero: everything after the scoring can run as one launch (tail_kernel)
    size_t share_lds = 0;   // non-zero: ... with a unit's recalled keys shared out over its share_nb blocks (share_tail_kernel)
    int share_nb = 1;
    bool share_pays = true; // ... and is taken for larger batches
    size_t xs_words = 0;    // exchange slots per unit
    int tail_spins = kTailSpins;
    int share_late = -1, share_late_block = -1;   // share_tail_kernel: the wait (0..3) that is given up at once, and by which block (-1: all)
    int tail = -1;          // ... : -1 chosen per batch, 0 separate launches, 1 tail_kernel and 2 share_tail_kernel whenever possible
    int keyclass = -1;      // key histogram + classification as one launch: -1 chosen per batch, 0 never, 1 always
    int attn_slices = 4;    // blocks per unit of the attention (head-dimension slices): 8 while each has a CU of its own
    int build_redone = 0;   // chunks of the matrix-core list build that the candidate route had to hand back
    int build_by_cand = 0;  // the matrix-core list build took the candidate route
    int xcd_units = -1;       // a unit's blocks on one XCD in every kernel of a step (unit_block_of; the units must be a multiple of 8):
                              // -1 for small batches, 0 never, 1 whenever possible
    int score_by_rank = -1;   // how the scoring kernel splits a unit's recalled ids over its blocks: -1 chosen per batch, 0 by id range, 1 by rank
    int sel_bits = 0, build_bits = 0;   // words for the selection's id bitmaps (0: histogram route off)
    int bitmap_words = 0, recall_split = 1, num_cu = 256;
    // single-launch step (decode_fused_kernel): blocks per unit (0: the geometry does not allow it), its shared memory,
    // the path in use (CTKVR_PATH_*), the sticky error word and the phase stamps
    int fused_bpu = 0, fused_nt = 1024, fused_stage = 0, decode_path = CTKVR_PATH_AUTO;
    size_t fused_smem = 0;
    uint32_t *d_err = nullptr;
    long long *d_prof = nullptr;
    bool prof_phases = false;
    // Groups of sequences whose steps run side by side (fork / join on streams of the library, default priority):
    // the latency-bound selection stages of one group then overlap the key streaming of another.
    int n_groups = 1;
    std::vector<hipStream_t> side;          // n_groups - 1 streams
    hipEvent_t ev_fork = nullptr;
    std::vector<hipEvent_t> ev_join;        // one per side stream
    // per-kernel timing
    std::vector<hipEvent_t> events;
    int prof_max = 0, prof_step = 0;

    ~ctkvr_index()
    {
        // the memory may be handed to another index at once, if nothing on its device uses it any more
        DeviceScope on(dev);
        pool_put(dev, mem, on.err == hipSuccess && device_idle());
        for (hipEvent_t e : events) (void)hipEventDestroy(e);
        for (hipEvent_t e : ev_join) (void)hipEventDestroy(e);
        if (ev_fork) (void)hipEventDestroy(ev_fork);
        for (hipStream_t st : side) (void)hipStreamDestroy(st);
    }
    // event slot `stage` (0 = before the first kernel) of the step being recorded
    void mark(int stage, hipStream_t st)
    {
        if (prof_step < prof_max) (void)hipEventRecord(events[(size_t)prof_step * (CTKVR_N_STAGES + 1) + stage], st);
    }
};

namespace {

#define TRY(expr)                    \
    do {                             \
        int rc_ = (expr);            \
        if (rc_ != CTKVR_OK) return rc_; \
    } while (0)

int check_params(const ctkvr_params *p, const int32_t *ctx_lens)
{
    if (!p) return fail(CTKVR_EINVAL, "params is NULL");
    if (!ctx_lens) return fail(CTKVR_EINVAL, "ctx_lens is NULL");
    if (p->batch < 1 || p->n_q_heads < 1 || p->n_kv_heads < 1) return fail(CTKVR_EINVAL, "batch/heads must be >= 1");
    if (p->n_q_heads % p->n_kv_heads) return fail(CTKVR_EINVAL, "n_q_heads %% n_kv_heads != 0");
    if (p->head_dim != 128) return fail(CTKVR_EUNSUPPORTED, "head_dim %d: only 128 is supported", p->head_dim);
    int G = p->n_q_heads / p->n_kv_heads;
    if (G != 1 && G != 2 && G != 4 && G != 8) return fail(CTKVR_EUNSUPPORTED, "group size %d: only 1, 2, 4, 8", G);
    if (p->dtype != CTKVR_F32 && p->dtype != CTKVR_BF16) return fail(CTKVR_EINVAL, "unknown dtype %d", p->dtype);
    if (p->page_size < 1 || p->page_size > 256 || (p->page_size & (p->page_size - 1)))
        return fail(CTKVR_EUNSUPPORTED, "page_size %d: powers of two up to 256", p->page_size);
    if (p->n_centroids < 0 || (p->n_centroids == 0 && p->centroid_div < 1))
        return fail(CTKVR_EINVAL, "n_centroids = 0 needs centroid_div >= 1");
    if (p->list_len < 1 || p->n_probe < 1 || p->top_k < 1) return fail(CTKVR_EINVAL, "list_len, n_probe, top_k must be >= 1");
    if (p->n_probe > 1024) return fail(CTKVR_EUNSUPPORTED, "n_probe %d > 1024", p->n_probe);
    if (p->centroid_mode != CTKVR_CENTROID_LAST_C && p->centroid_mode != CTKVR_CENTROID_KMEANS)
        return fail(CTKVR_EINVAL, "unknown centroid_mode %d", p->centroid_mode);
    if (p->build_algo != CTKVR_BUILD_EXACT && p->build_algo != CTKVR_BUILD_MFMA)
        return fail(CTKVR_EINVAL, "unknown build_algo %d", p->build_algo);
    if (!(p->sm_scale >= 0.0f)) return fail(CTKVR_EINVAL, "sm_scale must be >= 0");
    if (p->n_init < 0 || p->n_local < 0) return fail(CTKVR_EINVAL, "n_init and n_local must be >= 0");
    for (int b = 0; b < p->batch; ++b) {
        int s = ctx_lens[b];
        if (s < 1 || s > (1 << 20)) return fail(s < 1 ? CTKVR_EINVAL : CTKVR_EUNSUPPORTED, "ctx_lens[%d] = %d outside 1..2^20", b, s);
        int C = p->n_centroids ? p->n_centroids : s / p->centroid_div;
        if (C < 1 || C > s) return fail(CTKVR_EINVAL, "sequence %d: %d centroids for %d tokens", b, C, s);
        if (C > 8192) return fail(CTKVR_EUNSUPPORTED, "sequence %d: %d centroids > 8192", b, C);
        if (p->n_probe > C) return fail(CTKVR_EINVAL, "sequence %d: n_probe %d > centroids %d", b, p->n_probe, C);
        if (p->list_len > s - p->n_init - p->n_local)
            return fail(CTKVR_EINVAL, "sequence %d: list_len %d > %d keys outside the resident window", b, p->list_len,
                        s - p->n_init - p->n_local);
    }
    return CTKVR_OK;
}

// Lays the step's buffers out from `base` (each 256-byte aligned) and returns the bytes they take;
// with base == nullptr only the size is computed.  The geometry is the index's.  `packed` (size only): see kStaticStepBytes.
size_t carve_step_ws(StepWs &w, unsigned char *base, const ctkvr_index *ix, bool packed = false)
{
    Carver cv{base};
    auto take = [&](auto **ptr, size_t bytes) { cv.take(ptr, bytes); };
    const ctkvr_params &p = ix->p;
    const size_t U = ix->units, L = ix->l_stride, G = ix->G;
    const size_t bpu = std::max(1, ix->fused_bpu);
    // recalled keys of a unit: rank order (one launch per stage) or one stretch per block range (single launch)
    const size_t LS = std::max<size_t>(L, ix->fused_bpu ? (size_t)ix->fused_stage : 0);
    take(&w.cos, U * ix->c_max * 4);
    take(&w.probe, U * p.n_probe * 4);
    take(&w.cand, U * L * 4);
    take(&w.ncand, U * 4);
    take(&w.z, U * LS * G * 4);
    take(&w.m_key, U * (packed ? G : kMaxStride) * 4);
    take(&w.crow, U * LS * 4);
    take(&w.gbits, U * (size_t)(packed ? (ix->s_max + 31) / 32 : ix->bitmap_words) * 4);
    take(&w.kbuf, U * L * 4);
    take(&w.ghist, U * (size_t)kBuckets * 4);
    take(&w.gbm, U * (size_t)(2 * ((L + 63) / 64)) * 4);
    take(&w.glist, U * (size_t)kListCap * 8);
    take(&w.gcur, U * (packed ? 1 : kMaxStride) * 4);
    take(&w.ginfo, U * 16);
    take(&w.win, U * (size_t)kWinSplit * G * (2 + 128) * 4);
    take(&w.srow, U * p.top_k * 4);
    take(&w.S, U * (packed ? G : kSumStride) * 8);
    take(&w.sel, U * p.top_k * 4);
    take(&w.zsel, U * p.top_k * G * 4);
    take(&w.nsel, U * 4);
    take(&w.bar, U * (size_t)kFusedBarriers * 4);
    if (ix->fused_bpu) {
        take(&w.part, U * bpu * G * (2 + 128) * 4);
        take(&w.sid, U * LS * 4);
        take(&w.slot_cnt, U * bpu * 4);
        take(&w.slot_max, U * bpu * G * 4);
        take(&w.slot_S, U * bpu * G * 8);
        take(&w.slot_hist, U * bpu * (size_t)kFusedBins * 4);
        take(&w.slot_npick, U * bpu * 8);
        take(&w.slot_sure, U * bpu * (size_t)p.top_k * 4);
        take(&w.slot_bkt, U * bpu * (size_t)kFusedListCap * 16);
    }
    // (last: its size is no other buffer's place; 0.1 us of the 4K and 32K steps against a place before the selection's)
    take(&w.xs, U * (packed ? G * 8 : ix->xs_words) * 8);
    return cv.off;
}

// the single-launch kernel of this geometry, with its shared memory (a limit that belongs to a device)
int allow_fused(const ctkvr_index *ix)
{
    DeviceScope on(ix->dev);
    HIP_TRY(on.err);
    hipError_t e = fused_set_smem(ix->p.dtype == CTKVR_BF16, ix->G, ix->fused_nt, ix->fused_smem);
    return e == hipSuccess ? CTKVR_OK : fail(CTKVR_EHIP, "single-launch step: %s", hipGetErrorString(e));
}

// Raises a kernel's limit of dynamic shared memory to at least `bytes` on device `dev`; the runtime is asked only when
// that is more than before.
int want_lds(int dev, const void *fn, size_t bytes)
{
    static std::mutex mu;
    static std::map<std::pair<int, const void *>, size_t> limit;
    std::lock_guard<std::mutex> lock(mu);
    size_t &now = limit[{dev, fn}];
    if (bytes <= now) return CTKVR_OK;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return fail(CTKVR_EHIP, "index set-up: %s", hipGetErrorString(e));
    now = bytes;
    return CTKVR_OK;
}

// most centroids of a sequence -> cosines a thread of recall_gather_kernel holds
void (*gather_kernel_for(int c_max))(GatherArgs)
{
    return c_max <= 256    ? recall_gather_kernel<1>
           : c_max <= 512  ? recall_gather_kernel<2>
           : c_max <= 1024 ? recall_gather_kernel<4>
           : c_max <= 2048 ? recall_gather_kernel<8>
                           : recall_gather_kernel<32>;
}

template <typename T, int G> int want_decode_lds(const ctkvr_index *ix)
{
    const int dev = ix->dev;
    TRY(want_lds(dev, (const void *)gather_kernel_for(ix->c_max), ix->recall_lds));
    TRY(want_lds(dev, (const void *)rerank_select_kernel<G>, std::max(ix->select_lds, ix->build_select_lds)));
    const bool s8 = ix->attn_slices == 8;
    if (ix->fused_lds) {
        const void *fn = s8 ? (const void *)select_attn_kernel<T, G, 8> : (const void *)select_attn_kernel<T, G, 4>;
        TRY(want_lds(dev, fn, ix->fused_lds));
    }
    if (ix->dcu_lds) TRY(want_lds(dev, (const void *)dcu_select_kernel<T>, ix->dcu_lds));
    if (ix->tail_lds) {
        const void *fn = s8 ? (const void *)tail_kernel<T, G, 8> : (const void *)tail_kernel<T, G, 4>;
        TRY(want_lds(dev, fn, ix->tail_lds));
    }
    if (ix->share_lds) TRY(want_lds(dev, (const void *)share_tail_kernel<T, G>, ix->share_lds));
    return want_lds(dev, s8 ? (const void *)sparse_attn_kernel<T, G, 8> : (const void *)sparse_attn_kernel<T, G, 4>, ix->attn_lds);
}

int want_index_lds(const ctkvr_index *ix)
{
    const bool bf = ix->p.dtype == CTKVR_BF16;
    switch (ix->G) {
        case 1: return bf ? want_decode_lds<bf16_t, 1>(ix) : want_decode_lds<float, 1>(ix);
        case 2: return bf ? want_decode_lds<bf16_t, 2>(ix) : want_decode_lds<float, 2>(ix);
        case 4: return bf ? want_decode_lds<bf16_t, 4>(ix) : want_decode_lds<float, 4>(ix);
        default: return bf ? want_decode_lds<bf16_t, 8>(ix) : want_decode_lds<float, 8>(ix);
    }
}

// n host integers to device memory through kernel arguments: no staging copy, no synchronisation
int upload_ints(int32_t *dst, const int32_t *src, int n, hipStream_t st)
{
    for (int at = 0; at < n; at += IntPack::kMax) {
        IntPack pack;
        const int m = std::min(n - at, (int)IntPack::kMax);
        memcpy(pack.v, src + at, (size_t)m * 4);
        put_ints_kernel<<<1, 256, 0, st>>>(dst + at, m, pack);
    }
    HIP_TRY(hipGetLastError());
    return CTKVR_OK;
}

// Lays out and takes everything an index holds; fills the host-side geometry.  What a step expects to find zero is
// cleared on `st`; so are the tables if a later step of the build leaves rows of them unwritten (clear_tables: sequences
// with fewer than c_max centroids).  first_row (builds; else null) goes to the device with the lengths.
int create_index(const ctkvr_params *p, const int32_t *ctx_lens, const int32_t *first_row, bool clear_tables, hipStream_t st, ctkvr_index **out)
{
    ctkvr_index *ix = new (std::nothrow) ctkvr_index();
    if (!ix) return fail(CTKVR_ENOMEM, "host allocation failed");
    if (hipGetDevice(&ix->dev) != hipSuccess) {
        delete ix;
        return fail(CTKVR_EHIP, "no current device");
    }
    ix->p = *p;
    const int B = p->batch, h = p->n_q_heads, g = p->n_kv_heads;
    ix->G = h / g;
    ix->scale = p->sm_scale > 0.0f ? p->sm_scale : (float)(1.0 / sqrt(128.0));
    ix->page_shift = __builtin_ctz(p->page_size);
    ix->units = B * g;
    for (int b = 0; b < B; ++b) {
        int s = ctx_lens[b];
        int C = p->n_centroids ? p->n_centroids : s / p->centroid_div;
        ix->ctx_lens.push_back(s);
        ix->n_cent.push_back(C);
        ix->c_max = std::max(ix->c_max, C);
        ix->s_max = std::max(ix->s_max, s);
        long lm = std::min<long>(s, (long)p->n_probe * p->list_len);
        ix->l_stride = std::max<long>(ix->l_stride, lm);
    }
    const size_t es = elem_size(p->dtype);
    const size_t U = ix->units;
    {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ix->dev) == hipSuccess && cus > 0) ix->num_cu = cus;
    }
    ix->bitmap_words = (((ix->s_max + 31) / 32) + 3) & ~3;   // (rows of words on 16-byte boundaries)
    // The single-launch step needs all its blocks resident at once (one 1024-thread block per CU) and
    // its shared-memory plan to fit; up to 32 blocks work on a unit.
    if ((int)U <= ix->num_cu) {
        const int bpu = std::max(1, std::min(kFusedMaxBpu, ix->num_cu / (int)U));
        // Few recalled keys per block: four waves walk the serial parts of every phase (selections, scans,
        // reductions) faster than sixteen; many keys per block: sixteen waves keep more rows in flight.
        int nt = ix->l_stride / bpu <= 2048 ? 256 : 1024;
        if (const char *e = getenv("CTKVR_FUSED_THREADS")) {
            if (!strcmp(e, "256")) nt = 256;
            else if (!strcmp(e, "1024")) nt = 1024;
        }
        const size_t words = fused_smem_words(nt, p->n_probe, ix->s_max, bpu, p->top_k, ix->G);
        if (words * 4 <= (size_t)150 * 1024) {
            ix->fused_bpu = bpu;
            ix->fused_nt = nt;
            ix->fused_smem = words * 4;
            ix->fused_stage = bpu * fused_range_ids(ix->s_max, bpu);
        }
    }
    // Sequences of a batch are independent, and their steps can be issued as groups side by side
    // (CTKVR_DECODE_GROUPS = n at index creation).  One group is the default: on this part the split
    // measured slower on every benchmark batch (128K x 4: 131 us unsplit, 144 us as two groups, 159 us as
    // four; ragged x 16: 154 / 160 / 169 us) -- kernels of different streams take turns rather than share
    // the chip, and every group pays the per-kernel floors again.
    {
        int ng = 1;
        if (const char *e = getenv("CTKVR_DECODE_GROUPS")) ng = std::max(1, std::min(std::min(8, B), atoi(e)));
        if (const char *e = getenv("CTKVR_XCD_UNITS")) ix->xcd_units = atoi(e) != 0;
        if (const char *e = getenv("CTKVR_SCORE_BY_RANK")) ix->score_by_rank = atoi(e) != 0;
        if (const char *e = getenv("CTKVR_KEYCLASS")) ix->keyclass = atoi(e) != 0;
        if (const char *e = getenv("CTKVR_TAIL")) ix->tail = std::max(0, std::min(2, atoi(e)));
        if (const char *e = getenv("CTKVR_TAIL_SPINS")) ix->tail_spins = std::max(0, std::min((int)kTailSpins, atoi(e)));
        if (const char *e = getenv("CTKVR_SHARE_LATE")) {
            ix->share_late = std::max(-1, std::min(3, atoi(e)));
            if (const char *colon = strchr(e, ':')) ix->share_late_block = atoi(colon + 1);
        }
        ix->n_groups = ng;
    }
    if (const char *e = getenv("CTKVR_DECODE_PATH")) {
        if (!strcmp(e, "staged")) ix->decode_path = CTKVR_PATH_STAGED;
        else if (!strcmp(e, "fused") && ix->fused_bpu) ix->decode_path = CTKVR_PATH_FUSED;
    }
    // What follows the scoring, a unit's recalled keys shared out over its blocks: as many blocks as there are CUs for them, eight at
    // most (every block reads what all others of its unit publish)
    {
        int nb = 1;
        while (nb < kShareBlocks && 2 * nb * (int)U <= ix->num_cu) nb *= 2;
        ix->share_nb = nb;
        const size_t lds = share_smem_words(((ix->l_stride + 63) / 64 + nb - 1) / nb, ix->G) * 4;
        if (p->top_k <= kShareCut && lds <= 150 * 1024) ix->share_lds = lds;
        // With one block a unit the CUs that the last round of blocks leaves idle are idle for all of it, and from some length on the
        // separate launches, whose passes use the whole card, are faster.  Steps with / without, groups of four, lists of which a quarter is distinct, us:
        //   l_stride     32768       65536       131072
        //   136 units    124/137     203/207     399/387     160 units    137/152     228/234     454/443
        //   192 units    154/171     260/275     520/513     224 units    173/198     299/321
        //   264 units    227/237     380/382     (U - 256 of 256 CUs in a second round)
        // and by recalled keys L, where they cross near 20000: 160 units, l_stride 65536, L 8192, 16384 and 32768 139/151, 222/228 and 405/375; l_stride
        // 32768 all distinct 384/365.  The lines lie where a quarter to a third distinct loses nothing: l_stride 49152 where just more than half the CUs (of a round) have a block, 81920
        // where three quarters have, at most 98304.  Groups of one and two cross within 2 % of these, of eight (whose separate launches are
        // slower) nowhere; two blocks a unit and more: -2 to -13 % (72 to 128 units to 131072).
        const long long rounds = (U + ix->num_cu - 1) / ix->num_cu, cus = rounds * ix->num_cu;
        if (nb == 1 && ix->G <= 4)
            ix->share_pays = ix->l_stride <= 49152 + std::min(49152ll, 65536 * (2 * (long long)U - cus) / (cus * rounds));
        ix->xs_words = std::max<size_t>(8 * ix->G, ix->share_lds ? share_words(nb, ix->G) : 0);
    }
    // one allocation for all of it
    size_t edge = 256;
    auto lay_out = [&](unsigned char *base) {
        // (the tables and the workspace on boundaries of 2 MB, as an allocation of their own would be -- with 1 MB a 32K step took
        // 38.9 in place of 38.7 us -- or less where the three of them would come to over a fifth of the rest)
        Carver cv{base};
        cv.take(&ix->centroids, (size_t)B * h * ix->c_max * 128 * es);
        cv.align_to(edge);
        cv.take(&ix->inv_norm_c, (size_t)B * h * ix->c_max * 4);
        cv.align_to(edge);
        cv.take(&ix->lists, U * ix->c_max * p->list_len * 4);
        cv.take(&ix->d_ctx_lens, (size_t)B * 4);
        cv.take(&ix->d_n_cent, (size_t)B * 4);
        cv.take(&ix->d_first, (size_t)B * 4);
        cv.take(&ix->d_dcu_count, 8);
        cv.take(&ix->d_err, 4);
        cv.take(&ix->d_prof, 64 * 8);
        if (p->list_len != p->top_k) {
            cv.take(&ix->dsel, U * (size_t)p->list_len * 4);
            cv.take(&ix->dnsel, U * 4);
        }
        cv.align_to(edge);
        cv.off += carve_step_ws(ix->ws, base ? base + cv.off : nullptr, ix);
        return cv.off;
    };
    const size_t content = lay_out(nullptr);
    while (edge < (size_t)2 << 20 && 3 * 5 * 2 * edge <= content) edge *= 2;
    int rc = pool_get(ix->dev, lay_out(nullptr), 4, &ix->mem);
    if (rc != CTKVR_OK) {
        delete ix;
        return rc;
    }
    lay_out((unsigned char *)ix->mem.base);
    // shared-memory plan
    ix->recall_lds = ((size_t)kSelLds + p->n_probe + ix->bitmap_words) * 4;
    // selection: radix scratch, the deciding bucket's list, two id bitmaps, the picked positions;
    // where the bitmaps would not fit the histogram route is switched off
    const size_t sel_fixed = (size_t)kSelLds + 2 * kListCap;
    ix->sel_bits = 4 * ((ix->l_stride + 63) / 64);
    const size_t picks = std::max(p->top_k, p->list_len);   // the update ranks once more with budget rho
    if ((sel_fixed + ix->sel_bits + picks) * 4 > 150 * 1024) ix->sel_bits = 0;
    ix->select_lds = (sel_fixed + ix->sel_bits + picks) * 4;
    ix->build_bits = 4 * ((ix->s_max + 63) / 64);
    if ((sel_fixed + ix->build_bits + 1) * 4 > 150 * 1024) ix->build_bits = 0;
    ix->build_select_lds = (sel_fixed + ix->build_bits + 1) * 4;
    ix->attn_lds = (size_t)p->top_k * ix->G * 4;
    // The selection runs as one 1024-thread block per (sequence, KV head) and is latency-critical:
    // while there are no more such blocks than CUs, ask for over half a CU's shared memory so that
    // two never share a CU.  The recall is spread over recall_split blocks per unit.
    if ((int)U <= ix->num_cu) ix->select_lds = std::max<size_t>(ix->select_lds, 84 * 1024);
    ix->recall_split = std::max(1, std::min(8, ix->num_cu / (int)U));
    // Few enough units for every (unit, slice) block to have a CU of its own: one launch for lines 6-9.
    {
        const size_t fw = ((size_t)kSelLds + 2 * kListCap + ix->sel_bits + p->top_k + (size_t)p->top_k * ix->G) * 4;
        ix->attn_slices = 8 * (int)U <= ix->num_cu ? 8 : 4;
        if (4 * (int)U <= ix->num_cu && fw <= 150 * 1024) ix->fused_lds = fw;
        const size_t tw = tail_smem_words(ix->sel_bits, p->top_k, ix->G) * 4;
        const size_t dw = ((size_t)kSelLds + 2 * kListCap + ix->sel_bits) * 4;
        // One block per unit for the update's second ranking up to a number of recalled keys, of which l_stride is the bound
        // known here.  Update in one launch / by the chip-wide passes, G = 4, us, at 16, 29 and 53 thousand recalled keys:
        //   4 units 17.4/20.3  30/20.3  54/21.2;   8 units 13.4/18.7  23/19.7  46/21.3;   64 units 14.5/26.1  30/27.8  52/30.1
        // They cross between 19000 and 29000; the line is twice that, as for tail_kernel.
        if (ix->sel_bits && p->list_len != p->top_k && ix->l_stride <= kDcuStride) ix->dcu_lds = dw;
        if (4 * (int)U <= ix->num_cu && ix->sel_bits && tw <= 136 * 1024) ix->tail_lds = tw;
    }
    if (ix->recall_lds > 150 * 1024 || ix->select_lds > 150 * 1024 || ix->attn_lds > 128 * 1024) {
        delete ix;
        return fail(CTKVR_EUNSUPPORTED, "context, top_k or n_probe too large for the shared-memory plan");
    }
    rc = want_index_lds(ix);
    hipError_t e = hipSuccess;
    if (rc == CTKVR_OK && ix->fused_bpu && ix->decode_path == CTKVR_PATH_FUSED) rc = allow_fused(ix);
    if (rc == CTKVR_OK) {
        ZeroRanges z{};
        auto zero = [&](void *ptr, size_t words) {
            z.p[z.n] = (uint32_t *)ptr;
            z.words[z.n++] = words;
        };
        zero(ix->ws.ghist, U * (size_t)kBuckets);
        zero(ix->d_dcu_count, 2);
        zero(ix->d_err, 1);
        zero(ix->d_prof, 64 * 2);
        zero(ix->ws.bar, U * (size_t)kFusedBarriers);
        zero(ix->ws.gbits, U * (size_t)ix->bitmap_words);
        zero(ix->ws.srow, U * (size_t)p->top_k);   // always valid rows (see sparse_attn_kernel)
        size_t most = 0;
        for (int i = 0; i < z.n; ++i) most = std::max(most, z.words[i]);
        const unsigned gx = (unsigned)std::max<size_t>(1, std::min<size_t>(256, (most + 1023) / 1024));
        const int32_t *src[IntRows::kMax] = {ix->ctx_lens.data(), ix->n_cent.data(), first_row};
        int32_t *dst[IntRows::kMax] = {ix->d_ctx_lens, ix->d_n_cent, first_row ? ix->d_first : nullptr};
        if (IntRows::kMax * B <= IntPack::kMax) {   // the usual batch: one launch (of four, each some 3 us of a short build)
            IntRows rows{};
            IntPack pack;
            rows.n = B;
            for (int r = 0; r < IntRows::kMax; ++r) {
                rows.dst[r] = dst[r];
                if (dst[r]) memcpy(pack.v + r * B, src[r], (size_t)B * 4);
            }
            set_up_kernel<<<dim3(gx, z.n + 1), 256, 0, st>>>(z, rows, pack);
        } else {
            zero_ranges_kernel<<<dim3(gx, z.n), 256, 0, st>>>(z);
            for (int r = 0; r < IntRows::kMax && rc == CTKVR_OK; ++r)
                if (dst[r]) rc = upload_ints(dst[r], src[r], B, st);
        }
        e = hipGetLastError();
    }
    if (rc == CTKVR_OK && e == hipSuccess && clear_tables && *std::min_element(ix->n_cent.begin(), ix->n_cent.end()) < ix->c_max) {
        ZeroRanges z{};
        z.n = 2;
        z.p[0] = (uint32_t *)ix->lists;
        z.words[0] = U * ix->c_max * p->list_len;
        z.p[1] = (uint32_t *)ix->centroids;
        z.words[1] = (size_t)B * h * ix->c_max * 128 * es / 4;
        zero_ranges_kernel<<<dim3(1024, 2), 256, 0, st>>>(z);
        e = hipGetLastError();
    }
    if (rc != CTKVR_OK) {
        delete ix;
        return rc;
    }
    if (e == hipSuccess && ix->n_groups > 1) {
        e = hipEventCreateWithFlags(&ix->ev_fork, hipEventDisableTiming);
        for (int i = 1; i < ix->n_groups && e == hipSuccess; ++i) {
            hipStream_t sst = nullptr;
            hipEvent_t ev = nullptr;
            e = hipStreamCreateWithFlags(&sst, hipStreamNonBlocking);
            if (e == hipSuccess) ix->side.push_back(sst);
            if (e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
            if (e == hipSuccess) ix->ev_join.push_back(ev);
        }
    }
    if (e != hipSuccess) {
        delete ix;
        return fail(CTKVR_EHIP, "index set-up: %s", hipGetErrorString(e));
    }
    *out = ix;
    return CTKVR_OK;
}

Units decode_units(const ctkvr_index *ix)
{
    Units u{};
    u.g = ix->p.n_kv_heads;
    u.G = ix->G;
    u.h = ix->p.n_q_heads;
    u.build = 0;
    u.unit0 = 0;
    u.c_max = ix->c_max;
    u.n_cent = ix->d_n_cent;
    return u;
}

template <typename T> int launch_inv_norms(ctkvr_index *ix, hipStream_t st)
{
    size_t n = (size_t)ix->p.batch * ix->p.n_q_heads * ix->c_max;
    inv_norm_kernel<T><<<dim3((unsigned)((n + 15) / 16)), 256, 0, st>>>((const T *)ix->centroids, n, ix->inv_norm_c);
    HIP_TRY(hipGetLastError());
    return CTKVR_OK;
}

// shared memory of exact_list_kernel and key_list_kernel
size_t exact_list_lds(const ctkvr_index *ix) { return ((size_t)kSelLds + 2 * kListCap + 4 * ((ix->s_max + 63) / 64)) * 4; }

// Algorithm 1 lines 2-4 in the decode path's own arithmetic: for chunks of
// (sequence, KV head, centroid) units, score all keys, then per unit sum the
// denominators and select the top-rho.
template <typename T, int G>
int build_lists_exact(ctkvr_index *ix, const void *k_pages, const int32_t *block_table, int max_pages, hipStream_t st)
{
    const bool mfma = ix->p.build_algo == CTKVR_BUILD_MFMA;
    const int total_units = ix->units * ix->c_max;
    const size_t per_unit = (size_t)ix->s_max * G * 4;
    int chunk = (int)std::min<size_t>(total_units, std::max<size_t>(1, ((size_t)512 << 20) / per_unit));
    chunk = std::min(chunk, 16384);
    if (mfma) {   // whole (sequence, KV head) groups per chunk; no scores are stored, only 4-byte keys
        int nbk = (int)std::max<size_t>(1, ((size_t)8 << 30) / ((size_t)ix->s_max * 4 * ix->c_max));
        nbk = std::min(nbk, std::max(1, 16384 / ix->c_max));
        chunk = std::min(ix->units, nbk) * ix->c_max;
    }
    float *z = nullptr;
    uint32_t *m_key = nullptr;
    unsigned long long *S = nullptr;
    uint32_t *kbuf = nullptr, *ghist = nullptr;
    float *off = nullptr;     // matrix-core route: what the pairs come to
    float2 *part = nullptr;   // matrix-core route: one (maximum, sum) pair per unit, head and block of the statistics pass
    constexpr int kMaxSplits = 64;
    // Matrix-core route, candidates only (see mfma_score_kernel): when the lists are short against the contexts, so that about
    // 2 rho candidates are a small part of the keys (a 1-in-16 sample of the positions places the threshold), and the keys of
    // all lists enough to pay for the two passes and the wait that it has more, or single lists so long that the walk of one block
    // over all their keys takes longer than those.  Every key against candidates, whole builds in
    // us, C = s / 64, 8 KV heads, four query heads each unless noted:
    //   lists of 1024, one context: 16K 262 / 281, 20K (50 M keys) 363 / 364, 22K 468 / 416, 25K 597 / 482 (one head 502 / 366,
    //   eight 825 / 776), 30K 778 / 524, 40K 1307 / 820; three of 9K..30K 1128 / 859, four of 2K..30K 1194 / 900;
    //   contexts against list length: 4 x 8192 tokens, 512 centroids (8 : 1) 902 / 973, 4 x 12K (12 : 1) 578 / 545,
    //   the same with lists of 2048 (6 : 1) 594 / 633, 4 x 16K with 512 (31 : 1) 822 / 644;
    //   few lists, beyond the 32768 keys that key_list_kernel keeps in registers: 33000 tokens and 1024 lists (34 M keys) 296 / 278,
    //   40000 and 512 (20 M) 237 / 239, 65536 and 256 (17 M) 214 / 212, 512 (34 M) 308 / 250, 98304 and 16 (1.6 M) 223 / 218, 64 (6.3 M)
    //   244 / 227, 131072 and 400 (52 M) 469 / 323, 262144 and 128 (34 M) 520 / 354 (one head 596 / 468, eight 566 / 404).
    // And where the samples at the threshold with two and a half spreads of their count stand for no more keys than fit: the longer the
    // context, the more keys each stands for, and a build handed back costs a fifth where one that is not gains two thirds.  Every key /
    // candidates: 400000 tokens and 128 lists a head of 2048 1449 / 444, 440000 and 1024 lists of 1024 7240 / 1966; handed back: 400000 and 128 of
    // 1024 810 / 935, 470000 and 128 of 2048 1720 / 1979 (not taken by this line, nor are) 500000 and 128 1019 / 1303, 1024 8763 / 10021.
    // CTKVR_BUILD_CANDIDATES=0/1 forces the choice where the shared memory allows it.
    const int rho = ix->p.list_len;
    const int step_stride = std::max(16, ((ix->s_max + 31) / 32 + 255) / 256);
    const int sample_stride = ((ix->s_max + 32 * step_stride - 1) / (32 * step_stride)) * 32;
    // (2 rho + 16 step_stride or somewhat more are expected, +-6 % at rho = 2048, three times that at 1024: neighbouring positions are alike)
    const int cand_cap = std::min(kCandCap, std::max(3 * rho, 2 * rho + 2048));
    const int cand_room = 2 * std::max(cand_cap, 128 * kMaxSplits);   // entries per unit, over all segments
    const size_t cand_lds = ((size_t)2112 + kCandTies + (size_t)((ix->s_max + 31) / 32)) * 4;
    bool by_cand = false;
    if (mfma && cand_lds <= 150 * 1024 && sample_stride <= kSampleCap && cand_cap >= rho) {
        long long lists = 0, keys = 0;
        for (int b = 0; b < ix->p.batch; ++b) {
            const long long n = (long long)ix->p.n_kv_heads * ix->n_cent[b];
            lists += n;
            keys += n * ix->ctx_lens[b];
        }
        const int s_min = *std::min_element(ix->ctx_lens.begin(), ix->ctx_lens.end());
        const float n_at = (float)(2 * ((rho + step_stride - 1) / step_stride) + 16);   // samples at the threshold
        by_cand = rho >= 256 && 3 * rho <= kCandCap && (n_at + 2.5f * sqrtf(n_at)) * (float)step_stride <= (float)cand_cap &&
                  ((keys >= 60000000ll && keys >= 10ll * rho * lists) ||
                   (s_min > 32768 && s_min >= 32ll * rho && (keys >= 30000000ll || s_min >= 98304)));
        if (const char *e = getenv("CTKVR_BUILD_CANDIDATES")) by_cand = atoi(e) != 0;
    }
    ix->build_by_cand = by_cand;
    // one block per list behind the keys, where its bitmap of the context fits the shared memory (to 515072 tokens)
    const bool by_list = mfma && exact_list_lds(ix) <= 150 * 1024;
    if (by_cand) {
        // chunks of about equal size, of 8192 units at most or four (sequence, KV head) groups, whichever is more: enough to
        // fill the card in every pass, at 1.1 GB of candidates (2.1 with four groups of 4096 centroids or two of 8192).  (Four groups
        // whatever their size, each chunk waited for: 30K tokens, 468 centroids 649 us, now 524; 4 x 16K 1254, now 644)
        int groups = std::min(chunk / ix->c_max, std::max(4, 8192 / ix->c_max));
        const int n = (ix->units + groups - 1) / groups;
        groups = (ix->units + n - 1) / n;
        chunk = groups * ix->c_max;
    }
    const bool redo_always = by_cand && getenv("CTKVR_BUILD_CANDIDATES_REDO") != nullptr;   // tests: take the redo path
    uint32_t *ksamp = nullptr, *tau = nullptr, *cursor = nullptr, *d_fail = nullptr;
    uint2 *cand = nullptr;
    // one block for what every chunk needs; the redo of the candidate route takes a second one when it comes to that
    BuildScratch scratch_mem, redo_mem;
    auto lay_out_full = [&](unsigned char *base, int units) {   // the buffers of the route that keeps every key
        Carver cv{base};
        cv.take(&kbuf, (size_t)units * ix->s_max * 4);
        if (!by_list) cv.take(&ghist, (size_t)units * kBuckets * 4);
        return cv.off;
    };
    auto lay_out = [&](unsigned char *base) {
        Carver cv{base};
        if (!mfma) {
            cv.take(&m_key, (size_t)chunk * kMaxStride * 4);
            cv.take(&S, (size_t)chunk * kSumStride * 8);
        }
        if (mfma) {
            cv.take(&part, (size_t)chunk * G * kMaxSplits * sizeof(float2));
            cv.take(&off, (size_t)(by_cand ? total_units : chunk) * G * 4);   // (kept for what is handed back)
        }
        if (by_cand) {
            // a segment per block of the statistics split
            cv.take(&ksamp, (size_t)chunk * sample_stride * 4);
            cv.take(&tau, (size_t)chunk * 4);
            cv.take(&cursor, (size_t)chunk * kMaxSplits * 4);
            cv.take(&d_fail, (size_t)ix->units * 4);
            cv.take(&cand, (size_t)chunk * cand_room * sizeof(uint2));
        } else {
            if (!mfma) cv.take(&z, (size_t)chunk * per_unit);
            cv.off += lay_out_full(base ? base + cv.off : nullptr, chunk);
        }
        return cv.off;
    };
    int rc = scratch_mem.get(ix->dev, lay_out(nullptr));
    if (rc == CTKVR_OK) lay_out(scratch_mem.base());
    // a thread holds 16 candidates (cand_select_kernel)
    const bool cand_small = cand_cap <= 16 * 256;
    if (rc == CTKVR_OK && by_cand)
        rc = want_lds(ix->dev, cand_small ? (const void *)cand_select_kernel<256, 16> : (const void *)cand_select_kernel<512, kCandCap / 512>, cand_lds);
    if (rc == CTKVR_OK && by_list)
        rc = want_lds(ix->dev, ix->s_max <= 8 * 512    ? (const void *)key_list_kernel<512, 8>
                               : ix->s_max <= 32 * 512 ? (const void *)key_list_kernel<512, 32>
                               : ix->s_max <= 64 * 512 ? (const void *)key_list_kernel<512, 64>
                                                       : (const void *)key_list_kernel<1024, 32>, exact_list_lds(ix));
    // The candidate route goes through all chunks first; a second round takes the (sequence, KV head) pairs it had to hand back by
    // the route that keeps every key, with the statistics of the first.  (One flag a chunk and its statistics again, one
    // pair of eight or, of three sequences, one handed back: 30K tokens, 468 centroids 1411 us, 128K, 2048 centroids 14.7 ms, three of
    // 25K 3471 us; now 832, 9.3 ms and 2456.)
    struct Span { int u0, nu; };
    std::vector<Span> spans;
    for (int u0 = 0; u0 < total_units; u0 += chunk) spans.push_back({u0, std::min(chunk, total_units - u0)});
    bool pick = by_cand;
    for (size_t at = 0; rc == CTKVR_OK; ++at) {
        if (at == spans.size()) {
            if (!pick) break;
            std::vector<uint32_t> again(ix->units);
            hipError_t ec = hipMemcpyAsync(again.data(), d_fail, again.size() * 4, hipMemcpyDeviceToHost, st);
            if (ec == hipSuccess) ec = hipStreamSynchronize(st);
            if (ec != hipSuccess) {
                rc = fail(CTKVR_EHIP, "build: %s", hipGetErrorString(ec));
                break;
            }
            std::vector<Span> back;   // runs of pairs, inside a chunk
            int most = 0;
            for (const Span &sp : spans) {
                const size_t before = back.size();
                for (int u0 = sp.u0; u0 < sp.u0 + sp.nu; u0 += ix->c_max) {
                    if (!redo_always && !again[u0 / ix->c_max]) continue;
                    if (back.size() > before && back.back().u0 + back.back().nu == u0) back.back().nu += ix->c_max;
                    else back.push_back({u0, ix->c_max});
                    most = std::max(most, back.back().nu);
                }
                ix->build_redone += back.size() > before;
            }
            if (back.empty()) break;
            rc = redo_mem.get(ix->dev, lay_out_full(nullptr, most));
            if (rc != CTKVR_OK) break;
            lay_out_full(redo_mem.base(), most);
            spans.swap(back);
            pick = false;
            at = 0;
        }
        const int u0 = spans[at].u0, nu = spans[at].nu;
        Units u = decode_units(ix);
        u.build = 1;
        u.unit0 = u0;
        if (!mfma) {
            fill_u32_kernel<<<dim3((unsigned)((nu * kMaxStride + 255) / 256)), 256, 0, st>>>(m_key, 0u, (size_t)nu * kMaxStride);
            fill_u32_kernel<<<dim3((unsigned)((nu * kSumStride * 2 + 255) / 256)), 256, 0, st>>>((uint32_t *)S, 0u, (size_t)nu * kSumStride * 2);
        }
        if (ghist) fill_u32_kernel<<<dim3((unsigned)(((size_t)nu * kBuckets + 255) / 256)), 256, 0, st>>>(ghist, 0u, (size_t)nu * kBuckets);
        bool keys_written = false;   // kbuf holds this chunk's ranking keys (matrix-core route)
        ScoreArgs sa{};
        sa.u = u;
        sa.q = ix->centroids;
        sa.qrows = ix->c_max;
        sa.k = Paged{k_pages, block_table, max_pages, ix->page_shift};
        sa.ctx_lens = ix->d_ctx_lens;
        sa.crow = nullptr;
        sa.ncand = nullptr;
        sa.l_stride = ix->s_max;
        sa.z = z;
        sa.m_key = m_key;
        sa.scale = ix->scale;
        if constexpr (std::is_same<T, bf16_t>::value) {
            if (mfma) {
                constexpr int CT = 32 * (8 / G);
                MfmaScoreArgs ma{};
                ma.g = ix->p.n_kv_heads;
                ma.G = G;
                ma.h = ix->p.n_q_heads;
                ma.c_max = ix->c_max;
                ma.bk0 = u0 / ix->c_max;
                ma.tiles_per_bk = (ix->c_max + CT - 1) / CT;
                const int tiles = (nu / ix->c_max) * ma.tiles_per_bk;
                ma.t_splits = std::max(1, std::min({(ix->s_max + 1023) / 1024, (4 * ix->num_cu + tiles - 1) / tiles, kMaxSplits}));
                ma.n_cent = ix->d_n_cent;
                ma.ctx_lens = ix->d_ctx_lens;
                ma.centroids = (const bf16_t *)ix->centroids;
                ma.k = sa.k;
                ma.l_stride = ix->s_max;
                ma.part = part;
                ma.off = off + (by_cand ? (size_t)u0 * G : 0);
                ma.kbuf = kbuf;
                ma.n_init = ix->p.n_init;
                ma.n_local = ix->p.n_local;
                ma.scale = ix->scale;
                ma.step_stride = 1;
                // passes over the same tiles: softmax statistics first
                if (pick || !by_cand) {
                    mfma_score_kernel<G, MFMA_STAT><<<dim3(ma.t_splits, tiles), (MfmaShape<G, MFMA_STAT>::NT), 0, st>>>(ma);
                    mfma_merge_kernel<<<dim3((unsigned)((nu * G + 255) / 256)), 256, 0, st>>>(ma, nu * G);
                }
                if (pick) {
                    // keys of a sample of the positions -> a threshold per unit -> all keys again, those at or above
                    // the threshold kept -> the rho largest of them, exactly
                    ma.kbuf = ksamp;
                    ma.step_stride = step_stride;
                    ma.sample_stride = sample_stride;
                    // (one round of blocks: a sixteenth of the steps does not pay for the fragments of a second.  128K, 2048 centroids 107 ->
                    // 103 us, half a round 133; three of 9K..30K 28.3 -> 27.6)
                    MfmaScoreArgs ms = ma;
                    ms.t_splits = std::max(1, std::min(ma.t_splits, (2 * ix->num_cu + tiles - 1) / tiles));
                    mfma_score_kernel<G, MFMA_SAMPLE><<<dim3(ms.t_splits, tiles), (MfmaShape<G, MFMA_SAMPLE>::NT), 0, st>>>(ms);
                    CandArgs ca{};
                    ca.u = u;
                    ca.ctx_lens = ix->d_ctx_lens;
                    ca.rho = rho;
                    ca.step_stride = step_stride;
                    ca.sample_stride = sample_stride;
                    ca.cand_cap = cand_cap;
                    ca.n_init = ix->p.n_init;
                    ca.n_local = ix->p.n_local;
                    ca.ksamp = ksamp;
                    ca.tau = tau;
                    const int seg_cap = std::min(cand_cap, cand_room / ma.t_splits);   // candidates cluster: all the room there is
                    ca.cand = cand;
                    ca.seg_cnt = cursor;
                    ca.t_splits = ma.t_splits;
                    ca.seg_cap = seg_cap;
                    ca.lists = ix->lists;
                    ca.fail = d_fail + u0 / ix->c_max;
                    // eight samples a thread, or sixteen
                    if (sample_stride <= 2048)
                        sample_threshold_kernel<256, 8><<<dim3(nu), 256, 0, st>>>(ca);
                    else
                        sample_threshold_kernel<512, 16><<<dim3(nu), 512, 0, st>>>(ca);
                    ma.step_stride = 1;
                    ma.tau = tau;
                    ma.cand = cand;
                    ma.seg_cnt = cursor;
                    ma.seg_cap = seg_cap;
                    mfma_score_kernel<G, MFMA_PICK><<<dim3(ma.t_splits, tiles), (MfmaShape<G, MFMA_PICK>::NT), 0, st>>>(ma);
                    if (cand_small)
                        cand_select_kernel<256, 16><<<dim3(nu), 256, cand_lds, st>>>(ca);
                    else
                        cand_select_kernel<512, kCandCap / 512><<<dim3(nu), 512, cand_lds, st>>>(ca);
                } else {   // every key stored, then histogram and selection over all of them
                    ma.kbuf = kbuf;
                    mfma_score_kernel<G, MFMA_KEY><<<dim3(ma.t_splits, tiles), (MfmaShape<G, MFMA_KEY>::NT), 0, st>>>(ma);
                    keys_written = true;
                }
            } else {
                score_kernel<T, G, 16><<<dim3((ix->s_max + 255) / 256, nu), 256, 0, st>>>(sa);
            }
        } else {
            score_kernel<T, G, 16><<<dim3((ix->s_max + 255) / 256, nu), 256, 0, st>>>(sa);
        }
        if (!mfma) {
            DenomArgs da{};
            da.u = u;
            da.ctx_lens = ix->d_ctx_lens;
            da.ncand = nullptr;
            da.l_stride = ix->s_max;
            da.z = z;
            da.m_key = m_key;
            da.S = S;
            denom_kernel<G><<<dim3(std::min((ix->s_max + 1023) / 1024, 64), nu), 256, 0, st>>>(da);
        }
        if (mfma && !keys_written) {   // the candidate route has written this chunk's lists
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) rc = fail(CTKVR_EHIP, "build launch: %s", hipGetErrorString(e));
            continue;
        }
        if (by_list) {
            KeyListArgs la{};
            la.g = ix->p.n_kv_heads;
            la.c_max = ix->c_max;
            la.unit0 = u0;
            la.n_cent = ix->d_n_cent;
            la.ctx_lens = ix->d_ctx_lens;
            la.l_stride = ix->s_max;
            la.rho = rho;
            la.n_init = ix->p.n_init;
            la.n_local = ix->p.n_local;
            la.kbuf = kbuf;
            la.lists = ix->lists;
            if (ix->s_max <= 8 * 512)
                key_list_kernel<512, 8><<<dim3(nu), 512, exact_list_lds(ix), st>>>(la);
            else if (ix->s_max <= 32 * 512)
                key_list_kernel<512, 32><<<dim3(nu), 512, exact_list_lds(ix), st>>>(la);
            else if (ix->s_max <= 64 * 512)
                key_list_kernel<512, 64><<<dim3(nu), 512, exact_list_lds(ix), st>>>(la);
            else
                key_list_kernel<1024, 32><<<dim3(nu), 1024, exact_list_lds(ix), st>>>(la);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) rc = fail(CTKVR_EHIP, "build launch: %s", hipGetErrorString(e));
            continue;
        }
        KeyArgs ka{};
        ka.u = u;
        ka.ctx_lens = ix->d_ctx_lens;
        ka.ncand = nullptr;
        ka.l_stride = ix->s_max;
        ka.z = mfma ? nullptr : z;   // the matrix-core passes have written the keys: histogram only
        ka.m_key = m_key;
        ka.S = S;
        ka.kbuf = kbuf;
        ka.ghist = ghist;
        ka.n_init = ix->p.n_init;
        ka.n_local = ix->p.n_local;
        keyhist_kernel<G><<<dim3(std::min((ix->s_max + 4095) / 4096, 8), nu), 1024, 0, st>>>(ka);
        SelectArgs se{};
        se.u = u;
        se.ctx_lens = ix->d_ctx_lens;
        se.ncand = nullptr;
        se.cand = nullptr;
        se.crow = nullptr;
        se.l_stride = ix->s_max;
        se.top_k = ix->p.list_len;
        se.z = z;
        se.m_key = m_key;
        se.kbuf = kbuf;
        se.ghist = ghist;
        se.bits_words = ix->build_bits;
        se.sel = ix->lists;
        rerank_select_kernel<G><<<dim3(nu), 1024, ix->build_select_lds, st>>>(se);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) rc = fail(CTKVR_EHIP, "build launch: %s", hipGetErrorString(e));
    }
    hipError_t es = hipStreamSynchronize(st);
    scratch_mem.waited(es);
    redo_mem.waited(es);
    if (rc == CTKVR_OK && es != hipSuccess) rc = fail(CTKVR_EHIP, "build: %s", hipGetErrorString(es));
    return rc;
}

constexpr size_t kExactChunkBytes = (size_t)512 << 20;

// The same lists with the scores on the fp32 matrix cores (exact_score_kernel) and one block per list behind them
// (exact_list_kernel); needs shared memory for a bitmap of the context (to 515072 tokens).
template <typename T, int G> int build_lists_exact_mfma(ctkvr_index *ix, const void *k_pages, const int32_t *block_table, int max_pages, hipStream_t st)
{
    constexpr int CT = 32 * (8 / G);
    const int tiles_per_bk = (ix->c_max + CT - 1) / CT, tiles = ix->units * tiles_per_bk;
    const int z_stride = (ix->s_max + 3) & ~3;
    // Chunks of at most 512 MB of scores (they are read back twice, so short-lived chunks help the memory-side cache, but a
    // chunk should hold several hundred lists: one block each)
    const size_t per_tile = (size_t)CT * G * z_stride * 4;
    const int chunk = (int)std::min<size_t>(tiles, std::max<size_t>(1, kExactChunkBytes / per_tile));
    float *z = nullptr;
    uint32_t *m_part = nullptr;
    BuildScratch scratch_mem;
    auto lay_out = [&](unsigned char *base) {
        Carver cv{base};
        cv.take(&z, (size_t)chunk * per_tile);
        cv.take(&m_part, (size_t)std::max(chunk, ix->num_cu) * CT * G * 4);   // t_splits x tiles of a chunk <= CUs, or one split
        return cv.off;
    };
    TRY(scratch_mem.get(ix->dev, lay_out(nullptr)));
    lay_out(scratch_mem.base());
    const size_t lds = exact_list_lds(ix);
    // threads of a list's block by what they hold of its keys (exact_list_kernel)
    const int list_threads = ix->s_max <= 32 * 512 ? 512 : 1024;
    void (*list_kernel)(ExactListArgs) = ix->s_max <= 8 * 512    ? exact_list_kernel<G, 512, 8>
                                         : ix->s_max <= 32 * 512 ? exact_list_kernel<G, 512, 32>
                                                                 : exact_list_kernel<G, 1024, 32>;
    if constexpr (G <= 4) {
        // Two blocks of 1024 threads share a CU, at the price of spilled registers, where a chunk has a list for each: more than one a
        // CU, more than two where keys beyond the 32768 in registers are read again, through more spills.  One / two blocks, whole
        // builds in us: 2048 lists of 32768, one head 408 / 380, two 630 / 617, four 1132 / 1113; 512 of 32768, four heads 377 / 366;
        // 1024 of 40000, four heads 812 / 775; 1024 of 65536, two heads 686 / 670, of 131072, one head 860 / 747; at two lists a CU
        // and chunk, 65536 and four heads 1184 / 1229, 131072 and two 1324 / 1381; 256 of 32768, one head 168 / 178.  Eight heads (79
        // spilled): 24000 1769 / 1805, 32768 2111 / 2281, 131072 5369 / 5590.
        const long long at_once = std::min((long long)ix->units * ix->c_max, (long long)chunk * CT);
        if (ix->s_max > 32 * 512 && at_once > (ix->s_max <= 32 * 1024 ? 1 : 2) * ix->num_cu) list_kernel = exact_list_kernel<G, 1024, 32, true>;
    }
    TRY(want_lds(ix->dev, (const void *)list_kernel, lds));
    for (int t0 = 0; t0 < tiles; t0 += chunk) {
        const int nt = std::min(chunk, tiles - t0);
        ExactScoreArgs sa{};
        sa.g = ix->p.n_kv_heads;
        sa.h = ix->p.n_q_heads;
        sa.c_max = ix->c_max;
        sa.tile0 = t0;
        sa.tiles_per_bk = tiles_per_bk;
        // one round of blocks, one per CU (eight waves of 64-register fragments; a block's prologue costs as much as four of
        // its steps), of at least one step of 32 keys each (4096 tokens, 64 centroids, two KV heads: 16.8 us, of two steps 20.6)
        sa.t_splits = std::max(1, std::min((ix->s_max + 31) / 32, ix->num_cu / nt));
        sa.n_cent = ix->d_n_cent;
        sa.ctx_lens = ix->d_ctx_lens;
        sa.centroids = ix->centroids;
        sa.k = Paged{k_pages, block_table, max_pages, ix->page_shift};
        sa.z_stride = z_stride;
        sa.z = z;
        sa.m_part = m_part;
        sa.scale = ix->scale;
        exact_score_kernel<T, G><<<dim3(sa.t_splits, nt), 512, 0, st>>>(sa);
        ExactListArgs la{};
        la.g = sa.g;
        la.c_max = ix->c_max;
        la.tile0 = t0;
        la.tiles_per_bk = tiles_per_bk;
        la.ct = CT;
        la.n_cent = ix->d_n_cent;
        la.ctx_lens = ix->d_ctx_lens;
        la.z_stride = z_stride;
        la.rho = ix->p.list_len;
        la.n_init = ix->p.n_init;
        la.n_local = ix->p.n_local;
        la.z = z;
        la.t_splits = sa.t_splits;
        la.m_part = m_part;
        la.lists = ix->lists;
        list_kernel<<<dim3(nt * CT), list_threads, lds, st>>>(la);
    }
    hipError_t e = hipGetLastError();
    hipError_t es = hipStreamSynchronize(st);   // the scratch is given back
    scratch_mem.waited(es);
    if (e == hipSuccess) e = es;
    return e == hipSuccess ? CTKVR_OK : fail(CTKVR_EHIP, "build: %s", hipGetErrorString(e));
}

template <typename T>
int build_lists_dispatch(ctkvr_index *ix, const void *k_pages, const int32_t *bt, int max_pages, hipStream_t st)
{
    const bool fixed = ix->p.build_algo == CTKVR_BUILD_EXACT && exact_list_lds(ix) <= 150 * 1024;
    auto go = [&](auto g) {
        constexpr int G = decltype(g)::value;
        return fixed ? build_lists_exact_mfma<T, G>(ix, k_pages, bt, max_pages, st) : build_lists_exact<T, G>(ix, k_pages, bt, max_pages, st);
    };
    switch (ix->G) {
        case 1: return go(std::integral_constant<int, 1>{});
        case 2: return go(std::integral_constant<int, 2>{});
        case 4: return go(std::integral_constant<int, 4>{});
        default: return go(std::integral_constant<int, 8>{});
    }
}

template <typename T, int G>
int decode_launch_group(ctkvr_index *ix, const StepWs &w_all, int b0, int nb, bool whole, const void *q, const void *k_pages,
                        const void *v_pages, const int32_t *bt, int max_pages, const int32_t *cur_lens, float *out, float *out_lse,
                        int32_t *out_sel, int32_t *out_ncand, int32_t *out_probe, hipStream_t st)
{
    // The step for the sequences b0 .. b0 + nb - 1 of the batch: every per-sequence and per-unit array is entered
    // at that group's first element, and the kernels see a batch of nb sequences.  whole: the group is the batch
    // (per-kernel timing marks and the single-launch form apply to whole batches only).
    const ctkvr_params &p = ix->p;
    const int U = nb * p.n_kv_heads, u0 = b0 * p.n_kv_heads;
    const size_t es = elem_size(p.dtype);
    auto adv = [](auto *ptr, size_t n) { return ptr ? ptr + n : ptr; };
    q = (const char *)q + (size_t)b0 * p.n_q_heads * 128 * es;
    bt = bt + (size_t)b0 * max_pages;
    cur_lens = adv(cur_lens, b0);
    out = out + (size_t)b0 * p.n_q_heads * 128;
    out_lse = adv(out_lse, (size_t)b0 * p.n_q_heads);
    out_sel = adv(out_sel, (size_t)u0 * p.top_k);
    out_ncand = adv(out_ncand, u0);
    out_probe = adv(out_probe, (size_t)u0 * p.n_probe);
    const void *cen = (const char *)ix->centroids + (size_t)b0 * p.n_q_heads * ix->c_max * 128 * es;
    const float *inv_c = ix->inv_norm_c + (size_t)b0 * p.n_q_heads * ix->c_max;
    const int32_t *lists = ix->lists + (size_t)u0 * ix->c_max * p.list_len;
    const int32_t *d_n_cent = ix->d_n_cent + b0, *d_ctx_lens = ix->d_ctx_lens + b0;
    StepWs w = w_all;
    if (u0) {
        const size_t L = ix->l_stride, Gs = ix->G;
        w.cos += (size_t)u0 * ix->c_max;
        w.probe += (size_t)u0 * p.n_probe;
        w.cand += u0 * L;
        w.ncand += u0;
        w.z += u0 * L * Gs;
        w.m_key += u0 * kMaxStride;
        w.crow += u0 * L;
        w.gbits += (size_t)u0 * ix->bitmap_words;
        w.kbuf += u0 * L;
        w.ghist += (size_t)u0 * kBuckets;
        w.gbm += (size_t)u0 * (2 * ((L + 63) / 64));
        w.glist += (size_t)u0 * kListCap;
        w.gcur += u0 * kMaxStride;
        w.ginfo += (size_t)u0 * 4;
        w.win += (size_t)u0 * kWinSplit * Gs * (2 + 128);
        w.srow += (size_t)u0 * p.top_k;
        w.S += u0 * kSumStride;
        w.xs += u0 * ix->xs_words;
        w.sel += (size_t)u0 * p.top_k;
        w.zsel += (size_t)u0 * p.top_k * Gs;
        w.nsel += u0;
    }
    Units units = decode_units(ix);
    units.n_cent = d_n_cent;
    // A unit's blocks on one XCD (unit_block_of; needs a multiple of 8 units): in every kernel for small batches
    // (latency-bound: a step is a chain of dependent loads of what the previous kernel wrote); for large ones in all but
    // the two bandwidth-bound launches -- the cosines, and the scoring, whose blocks are better handed to whichever XCD is free.
    const bool xcd_small = ix->xcd_units < 0 ? (long long)ix->l_stride * U <= 2048ll * ix->num_cu : ix->xcd_units != 0;
    const int by_xcd = U % 8 == 0 && ix->xcd_units != 0;
    const int by_xcd_all = by_xcd && xcd_small;
    // lines 10-11 first: the window's share depends on q, K and V only
    const bool window = p.n_init + p.n_local > 0 || cur_lens;
    WindowArgs wa{};
    const bool one_launch = whole && ix->fused_bpu && ix->decode_path == CTKVR_PATH_FUSED;
    if (window) {
        wa.u = units;
        wa.q = q;
        wa.k = Paged{k_pages, bt, max_pages, ix->page_shift};
        wa.v_pages = v_pages;
        wa.ctx_lens = d_ctx_lens;
        wa.cur_lens = cur_lens;
        wa.n_init = p.n_init;
        wa.n_local = p.n_local;
        wa.scale = ix->scale;
        wa.win = w.win;
        wa.by_xcd = by_xcd;
        // a launch of its own before the single-launch step, and for groups of eight heads (where the window's
        // registers would cost the scoring blocks a wave per SIMD); otherwise its blocks ride in the scoring launch below
        if (one_launch || G > 4) window_attn_kernel<T, G><<<dim3(kWinSplit, U), 256, 0, st>>>(wa);
    }
    const bool stream_k = [&] {
        // key bytes the batch can touch per step: above 128 MiB (half of the 256 MB memory-side cache) few rows
        // survive to the next step, and a non-temporal hint keeps the centroid table, the lists and the step's
        // own buffers cached instead
        size_t kbytes = 0;
        for (int sl : ix->ctx_lens) kbytes += (size_t)sl * p.n_kv_heads * 128 * elem_size(p.dtype);
        return kbytes > ((size_t)128 << 20);
    }();
    if (one_launch) {
        FusedArgs fa{};
        fa.g = p.n_kv_heads;
        fa.h = p.n_q_heads;
        fa.c_max = ix->c_max;
        fa.rho = p.list_len;
        fa.n_probe = p.n_probe;
        fa.top_k = p.top_k;
        fa.l_stride = ix->l_stride;
        fa.bpu = ix->fused_bpu;
        fa.units = U;
        fa.stage = ix->fused_stage;
        fa.stream_k = stream_k;
        fa.scale = ix->scale;
        fa.n_cent = d_n_cent;
        fa.ctx_lens = d_ctx_lens;
        fa.q = q;
        fa.centroids = cen;
        fa.inv_norm_c = inv_c;
        fa.lists = lists;
        fa.k = Paged{k_pages, bt, max_pages, ix->page_shift};
        fa.v_pages = v_pages;
        fa.cos = w.cos;
        fa.probe = w.probe;
        fa.out_probe = out_probe;
        fa.sid = w.sid;
        fa.srow = w.crow;
        fa.z = w.z;
        fa.cand = w.cand;
        fa.kbuf = w.kbuf;
        fa.ncand = w.ncand;
        fa.out_ncand = out_ncand;
        fa.slot_cnt = w.slot_cnt;
        fa.slot_max = w.slot_max;
        fa.slot_S = w.slot_S;
        fa.slot_hist = w.slot_hist;
        fa.slot_npick = w.slot_npick;
        fa.slot_sure = w.slot_sure;
        fa.slot_bkt = w.slot_bkt;
        fa.part = w.part;
        fa.sel = w.sel;
        fa.nsel = w.nsel;
        fa.out_sel = out_sel;
        fa.out = out;
        fa.out_lse = out_lse;
        fa.win = window ? w.win : nullptr;
        fa.bar = w.bar;
        fa.err = ix->d_err;
        fa.prof = ix->prof_phases ? ix->d_prof : nullptr;
        if (whole) ix->mark(0, st);
        HIP_TRY(fused_launch(p.dtype == CTKVR_BF16, G, ix->fused_nt, (unsigned)(U * ix->fused_bpu), ix->fused_smem, st, fa));
        for (int k = 1; k <= 8; ++k) ix->mark(k, st);   // the whole step reads as stage 0
        if (ix->prof_step < ix->prof_max) {
            fill_u32_kernel<<<dim3(1), 64, 0, st>>>((uint32_t *)w.nsel, 0u, 0);
            if (whole) ix->mark(9, st);
            ix->prof_step++;
        }
        HIP_TRY(hipGetLastError());
        ix->have_step = &w_all == &ix->ws;
        return CTKVR_OK;
    }
    CosArgs ca{};
    ca.q = q;
    ca.centroids = cen;
    ca.inv_norm_c = inv_c;
    ca.n_cent = d_n_cent;
    ca.cos = w.cos;
    ca.m_key = w.m_key;
    ca.S = w.S;
    ca.g = p.n_kv_heads;
    ca.h = p.n_q_heads;
    ca.c_max = ix->c_max;
    ca.by_xcd = by_xcd_all;
    // Everything after the scoring as one launch (tail_kernel): for small batches, whose step is a chain of latencies,
    // and only up to a number of recalled keys: every block of a unit walks all of them, and beyond the 8192 it keeps, reads
    // them three times (one CU takes about 20 GB/s).  The number of recalled keys L is known on the device only; l_stride bounds
    // it, and neighbouring lists overlap: L is 0.2 to 0.28 of l_stride on the benchmark inputs.  Steps with tail_kernel / share_tail_kernel / the
    // separate launches, G = 4, 1024 picks, us:
    //   L           4096            8192            16384           32768           65536
    //   4 units     27.8/31.7/33.3  30.4/32.8/36.8  43.3/35.1/41.5  64.4/42.8/50.3  108/56.2/65.2   (loads from other XCDs' caches: unit_block_of)
    //   8 units     27.1/31.5/31.9  29.7/32.5/35.4  42.4/38.9/42.5  58.7/48.2/53.0  94.7/66.6/72.9
    //   16 units    29.1/33.2/34.3  35.0/37.9/41.2  48.4/45.3/49.6  70.4/60.3/66.6
    //   24 units    30.0/34.3/35.0  37.0/40.1/43.0  53.1/50.7/55.0
    //   32 units    31.8/36.1/36.6  40.1/43.3/46.0  61.5/59.8/63.9
    // (G = 1, 2 and 8 cross in the same places.)  The lines were drawn at twice the crossings with the separate launches: no loss against those
    // while at most half the probed entries are distinct.  share_tail_kernel crosses sooner, near L = 12000: at l_stride = 32768 with a quarter distinct
    // tail_kernel is still the faster (8 units 31.0/33.5, 16 34.3/37.2), at 65536 no longer (8 units 41.6/39.1).  Not where one of the
    // forms it replaces is asked for.
    const int tail_most = by_xcd ? 65536 : 32768;
    const bool tail = ix->tail_lds && ix->keyclass < 0 &&
                      (ix->tail < 0 ? (long long)ix->l_stride * U <= 2048ll * ix->num_cu && ix->l_stride <= tail_most : ix->tail == 1);
    ca.xs = w.xs;
    ca.n_xs = tail ? ix->attn_slices * G : 0;
    // Beyond that one launch all the same, with a unit's recalled keys shared out over its blocks (share_tail_kernel): 128K x 4
    // 125.8 -> 116.7 us a step, sixteen of 8K to 64K 144.9 -> 130.0, against the separate launches, which are left to budgets beyond
    // kShareCut, shares whose bitmap the shared memory does not take, and long contexts of more units than half the CUs (share_pays).  Small
    // batches would lose with it (32K 31.9 -> 34.9 us, 4K 23.5 -> 28.7: every block's chain is as long, and waits three times more for the
    // others).  Scores of little spread (logits of unit variance), 1024 picks, with / without: 32 units, l_stride 65536, L 8192, 16384 and 32768
    // 52.1/56.3, 66.0/69.8, 95.8/98.9; 128 units 114/124, 172/182, 300/300.  Lists without any overlap cost it 1 to 8 % from L = 65536 (and 128
    // units, 32768) on.
    const bool share = !tail && ix->share_lds && ix->keyclass < 0 && (ix->tail == 2 || (ix->tail != 0 && ix->share_pays));
    if (whole) ix->mark(0, st);
    centroid_cos_kernel<T, G><<<dim3((ix->c_max + 15) / 16, U), 256, 0, st>>>(ca);
    if (whole) ix->mark(1, st);

    GatherArgs ga{};
    ga.cos = w.cos;
    ga.lists = lists;
    ga.n_cent = d_n_cent;
    ga.ctx_lens = d_ctx_lens;
    ga.probe = w.probe;
    ga.out_probe = out_probe;
    ga.gbits = w.gbits;
    ga.g = p.n_kv_heads;
    ga.c_max = ix->c_max;
    ga.rho = p.list_len;
    ga.n_probe = p.n_probe;
    ga.bitmap_words = ix->bitmap_words;
    ga.by_xcd = by_xcd;
    const dim3 rgrid(ix->recall_split, U);
    gather_kernel_for(ix->c_max)<<<rgrid, 256, ix->recall_lds, st>>>(ga);
    if (whole) ix->mark(2, st);

    // lines 4-5: bitmap -> recalled ids, their rows and their scores in one launch
    Units u = units;
    RecallScoreArgs sa{};
    sa.u = u;
    sa.q = q;
    sa.k = Paged{k_pages, bt, max_pages, ix->page_shift};
    sa.ctx_lens = d_ctx_lens;
    sa.gbits = w.gbits;
    sa.bitmap_words = ix->bitmap_words;
    sa.l_stride = ix->l_stride;
    sa.cand = w.cand;
    sa.crow = w.crow;
    sa.ncand = w.ncand;
    sa.out_ncand = out_ncand;
    sa.z = w.z;
    sa.m_key = w.m_key;
    if (share) {
        sa.clear = (uint4 *)w.xs;
        sa.clear_n = (int)(ix->xs_words / 2);
    } else if (!tail) {
        sa.clear = (uint4 *)w.ghist;
        sa.clear_n = kBuckets / 4;
    }
    sa.scale = ix->scale;
    sa.by_xcd = by_xcd_all;
    {
        // Few rows per CU (a small batch): a block's rows are one round trip to memory and the slowest block
        // is the launch, so the ids are split by rank -- two blocks a CU (32K, eight units 32.9 us a step; 1.5: 34.4), those of a
        // resident window, which ride in the launch, counted in (on top of them: eight units of 32K, window of 640 and 100 decoded tokens
        // 42.7 us with the update, now 41.9; two units of 16K in fp32 40.6, now 35.2), but beyond 128 a unit 1.5 blocks a CU: each
        // reads the unit's whole bitmap, and their atomics meet on the unit's line (one and two units of 32K in bf16 33.2 and 32.2 us,
        // now 31.5 and 30.6; in fp32 34.1 and 33.2, now 32.5 and 30.9; four units, 96 or 128 blocks each: of 8192 recalled keys in bf16 31.0 and
        // 31.1, in fp32 32.4 and 31.9, of 32768 46.1 and 45.7, 52.1 and 49.6).  At least 32 per
        // unit and 64 list entries per block (128 leave CUs idle where units are few and
        // their lists short: two probes of 495, 16 units of eight heads 28.5 us, 128 29.3; four of 495, four units 31.5, 128 32.5; four of 1280,
        // four units 33.0 either way).  Otherwise by id
        // range: enough blocks to fill the chip a few times over, each owning 8..64 words of the bitmap.
        const bool by_rank = ix->score_by_rank < 0 ? (long long)ix->l_stride * U <= 2048ll * ix->num_cu : ix->score_by_rank != 0;
        const bool win_beside = window && G <= 4;
        int nbx;
        if (by_rank) {
            nbx = std::min((2 * ix->num_cu + U - 1) / U, std::max(128, (3 * ix->num_cu / 2 + U - 1) / U));
            if (win_beside) nbx = std::min(nbx, 2 * ix->num_cu / U - kWinSplit);
            nbx = std::min(std::max(32, nbx), (ix->l_stride + 63) / 64);
            nbx = std::max({1, nbx, (ix->l_stride + kRecallCap - 1) / kRecallCap});
        } else {
            const int target = std::max(32, (8 * ix->num_cu + U - 1) / U);
            const int wpb = std::max(8, std::min(kRecallWpb, (ix->bitmap_words + target - 1) / target));
            nbx = (ix->bitmap_words + wpb - 1) / wpb;
        }
        sa.nbx = nbx;
        if (by_rank) {
            // the bitmap with the ids before each word, and the block table of a sequence, where they fit 60 KB beside the block's ids (with the
            // window's own arrays 66.6 KB at most: two blocks share a CU's 160 KB, as many as the launch has for it)
            const int words = (((ix->bitmap_words + 255) / 256 + 3) & ~3) * 256;
            sa.lds.words = words <= kRecallWords ? words : 0;
            const int pages = (std::min(max_pages, ((ix->s_max - 1) >> ix->page_shift) + 1) + 255) & ~255;
            RecallLds all = sa.lds;
            all.pages = pages;
            sa.lds.pages = words && pages <= kRecallWords && all.total() * 4 <= 60 * 1024 ? pages : 0;
        } else {
            sa.lds.pages = 256;
            sa.lds.words = 0;
        }
        const size_t slds = (size_t)sa.lds.total() * 4;
        auto launch = [&](auto rank, auto stream, auto few) {
            constexpr bool RANK = decltype(rank)::value, STREAM = decltype(stream)::value, SHORT = decltype(few)::value;
            if constexpr (G <= 4) {
                if (win_beside) {
                    sa.win = wa;
                    recall_score_kernel<T, G, true, RANK, STREAM, SHORT><<<dim3(nbx + kWinSplit, U), 256, slds, st>>>(sa);
                    return;
                }
            }
            recall_score_kernel<T, G, false, RANK, STREAM, SHORT><<<dim3(nbx, U), 256, slds, st>>>(sa);
        };
        auto launch_rows = [&](auto rank, auto few) {
            if (stream_k)
                launch(rank, std::true_type{}, few);
            else
                launch(rank, std::false_type{}, few);
        };
        constexpr bool kTwo = kRankRows<T> != kShortRows;   // by rank with different numbers of rows
        if (kTwo && by_rank && (ix->l_stride <= 16 * kShortRows * nbx || (nbx * U > 2 * ix->num_cu && !win_beside)))
            launch_rows(std::bool_constant<true>{}, std::bool_constant<kTwo>{});
        else if (by_rank)
            launch_rows(std::true_type{}, std::false_type{});
        else
            launch_rows(std::false_type{}, std::false_type{});
    }
    if (whole) ix->mark(3, st);

    AttnArgs aa{};
    aa.v_pages = v_pages;
    aa.g = p.n_kv_heads;
    aa.h = p.n_q_heads;
    aa.top_k = p.top_k;
    aa.srow = w.srow;
    aa.nsel = w.nsel;
    aa.zsel = w.zsel;
    aa.out = out;
    aa.out_lse = out_lse;
    aa.win = window ? w.win : nullptr;
    aa.m_key = w.m_key;
    auto finish = [&]() -> int {
        if (whole) ix->mark(8, st);
        if (whole && ix->prof_step < ix->prof_max) {   // a null kernel between two events: what the bracketing itself costs
            fill_u32_kernel<<<dim3(1), 64, 0, st>>>((uint32_t *)w.nsel, 0u, 0);
            ix->mark(9, st);
            ix->prof_step++;
        }
        HIP_TRY(hipGetLastError());
        ix->have_step = &w_all == &ix->ws;   // the update reads the index's own workspace
        return CTKVR_OK;
    };
    if (tail) {
        TailArgs ta{};
        ta.ctx_lens = d_ctx_lens;
        ta.ncand = w.ncand;
        ta.cand = w.cand;
        ta.crow = w.crow;
        ta.l_stride = ix->l_stride;
        ta.top_k = p.top_k;
        ta.bits_words = ix->sel_bits;
        ta.z = w.z;
        ta.m_key = w.m_key;
        ta.xs = w.xs;
        ta.spins = ix->tail_spins;
        ta.gbits = w.gbits;
        ta.bitmap_words = ix->bitmap_words;
        // the update ranks once more, with another budget, from the ranking keys
        ta.kbuf = p.list_len != p.top_k && &w_all == &ix->ws ? w.kbuf : nullptr;
        ta.sel = w.sel;
        ta.nsel = w.nsel;
        ta.out_sel = out_sel;
        ta.at = aa;
        if (whole)
            for (int k = 4; k <= 7; ++k) ix->mark(k, st);   // stages of this launch: an event pair's cost each
        if (ix->attn_slices == 8)
            tail_kernel<T, G, 8><<<dim3(8 * U), kTailThreads, ix->tail_lds, st>>>(ta);
        else
            tail_kernel<T, G, 4><<<dim3(4 * U), kTailThreads, ix->tail_lds, st>>>(ta);
        return finish();
    }

    if (share) {
        ShareArgs ta{};
        ta.ctx_lens = d_ctx_lens;
        ta.ncand = w.ncand;
        ta.cand = w.cand;
        ta.crow = w.crow;
        ta.l_stride = ix->l_stride;
        ta.top_k = p.top_k;
        ta.nb = ix->share_nb;
        ta.z = w.z;
        ta.m_key = w.m_key;
        ta.xs = w.xs;
        ta.spins = (uint32_t)(ix->tail_spins + 1) / 2 * 0x01010101u;
        ta.late_spins = ix->share_late < 0 ? ta.spins : ta.spins & ~(0xffu << (8 * ix->share_late));
        ta.late_block = ix->share_late_block;
        if (ta.late_block < 0) ta.spins = ta.late_spins;
        ta.gbits = w.gbits;
        ta.bitmap_words = ix->bitmap_words;
        ta.kbuf = w.kbuf;
        ta.alone = (uint32_t *)w.zsel;
        ta.keep_keys = p.list_len != p.top_k && &w_all == &ix->ws;
        ta.sel = w.sel;
        ta.nsel = w.nsel;
        ta.out_sel = out_sel;
        ta.at = aa;
        if (whole)
            for (int k = 4; k <= 7; ++k) ix->mark(k, st);   // stages of this launch: an event pair's cost each
        share_tail_kernel<T, G><<<dim3(ix->share_nb * U), kTailThreads, ix->share_lds, st>>>(ta);
        return finish();
    }

    DenomArgs da{};
    da.u = u;
    da.ctx_lens = d_ctx_lens;
    da.ncand = w.ncand;
    da.l_stride = ix->l_stride;
    da.z = w.z;
    da.m_key = w.m_key;
    da.S = w.S;
    da.gbits = w.gbits;
    da.bitmap_words = ix->bitmap_words;
    da.gcur = w.gcur;
    da.by_xcd = by_xcd;
    const int chunks = (ix->l_stride + 1023) / 1024;
    denom_kernel<G><<<dim3(std::max(1, std::min(chunks, (4 * ix->num_cu + U - 1) / U)), U), 256, 0, st>>>(da);
    if (whole) ix->mark(4, st);

    // The separate launches.  Of small batches (that is, with budgets beyond kShareCut, or where they are asked for) the key histogram and
    // the classification pass are one, every block taking the unit's whole histogram itself (keyclass_kernel); otherwise two chip-wide ones.
    const bool keyclass = ix->sel_bits && (ix->keyclass < 0 ? (long long)ix->l_stride * U <= 2048ll * ix->num_cu : ix->keyclass != 0);
    if (keyclass) {
        KeyClassArgs kc{};
        kc.u = u;
        kc.ctx_lens = d_ctx_lens;
        kc.ncand = w.ncand;
        kc.l_stride = ix->l_stride;
        kc.top_k = p.top_k;
        kc.z = w.z;
        kc.m_key = w.m_key;
        kc.S = w.S;
        kc.kbuf = w.kbuf;
        kc.bits_stride = 2 * ((ix->l_stride + 63) / 64);
        kc.gbm = w.gbm;
        kc.glist = w.glist;
        kc.gcur = w.gcur;
        kc.ginfo = w.ginfo;
        kc.by_xcd = by_xcd;
        keyclass_kernel<G><<<dim3(std::max(1, std::min((ix->l_stride + 4095) / 4096, (2 * ix->num_cu + U - 1) / U)), U), 1024, 0, st>>>(kc);
        if (whole) ix->mark(5, st);
    } else {
    KeyArgs ka{};
    ka.u = u;
    ka.ctx_lens = d_ctx_lens;
    ka.ncand = w.ncand;
    ka.l_stride = ix->l_stride;
    ka.z = w.z;
    ka.m_key = w.m_key;
    ka.S = w.S;
    ka.kbuf = w.kbuf;
    ka.ghist = w.ghist;
    ka.gcur = w.gcur;
    ka.by_xcd = by_xcd;
    keyhist_kernel<G><<<dim3(std::max(1, std::min((ix->l_stride + 4095) / 4096, (2 * ix->num_cu + U - 1) / U)), U), 1024, 0, st>>>(ka);
    if (whole) ix->mark(5, st);
    }

    if (ix->sel_bits && !keyclass) {
        ClassifyArgs ca{};
        ca.u = u;
        ca.ctx_lens = d_ctx_lens;
        ca.ncand = w.ncand;
        ca.l_stride = ix->l_stride;
        ca.top_k = p.top_k;
        ca.kbuf = w.kbuf;
        ca.ghist = w.ghist;
        ca.bits_stride = 2 * ((ix->l_stride + 63) / 64);
        ca.gbm = w.gbm;
        ca.glist = w.glist;
        ca.gcur = w.gcur;
        ca.ginfo = w.ginfo;
        ca.by_xcd = by_xcd;
        classify_kernel<<<dim3(std::max(1, std::min(chunks, (4 * ix->num_cu + U - 1) / U)), U), 256, 0, st>>>(ca);
    }
    if (whole) ix->mark(6, st);

    SelectArgs se{};
    se.u = u;
    se.ctx_lens = d_ctx_lens;
    se.ncand = w.ncand;
    se.cand = w.cand;
    se.crow = w.crow;
    se.l_stride = ix->l_stride;
    se.top_k = p.top_k;
    se.z = w.z;
    se.m_key = w.m_key;
    se.kbuf = w.kbuf;
    se.ghist = w.ghist;
    se.bits_words = ix->sel_bits;
    if (ix->sel_bits) {
        se.gbm = w.gbm;
        se.glist = w.glist;
        se.ginfo = w.ginfo;
        se.bits_stride = 2 * ((ix->l_stride + 63) / 64);
    }
    se.sel = w.sel;
    se.srow = w.srow;
    se.zsel = w.zsel;
    se.nsel = w.nsel;
    se.out_sel = out_sel;
    if (ix->fused_lds) {
        if (whole) ix->mark(7, st);   // no separate selection launch: its stage reads as the cost of an event pair
        if (ix->attn_slices == 8)
            select_attn_kernel<T, G, 8><<<dim3(8 * U), 1024, ix->fused_lds, st>>>(se, aa);
        else
            select_attn_kernel<T, G, 4><<<dim3(4 * U), 1024, ix->fused_lds, st>>>(se, aa);
    } else {
        rerank_select_kernel<G><<<dim3(U), 1024, ix->select_lds, st>>>(se);
        if (whole) ix->mark(7, st);
        if (ix->attn_slices == 8)
            sparse_attn_kernel<T, G, 8><<<dim3(8 * U), 1024, ix->attn_lds, st>>>(aa);
        else
            sparse_attn_kernel<T, G, 4><<<dim3(4 * U), 1024, ix->attn_lds, st>>>(aa);
    }
    return finish();
}

// One step for the whole batch: a single group on the caller's stream, or (several sequences, no per-kernel
// timing, staged launches) the groups side by side -- the first on the caller's stream, the others on the
// library's streams, forked from and joined back into the caller's stream with events, so that the step is
// still one unit of work on that stream and can be captured into a graph.
template <typename T, int G>
int decode_launch(ctkvr_index *ix, const StepWs &w, const void *q, const void *k_pages, const void *v_pages, const int32_t *bt,
                  int max_pages, const int32_t *cur_lens, float *out, float *out_lse, int32_t *out_sel, int32_t *out_ncand,
                  int32_t *out_probe, hipStream_t st)
{
    const int B = ix->p.batch;
    const bool fused = ix->fused_bpu && ix->decode_path == CTKVR_PATH_FUSED;
    const int ng = (fused || ix->prof_step < ix->prof_max) ? 1 : std::min(ix->n_groups, B);
    if (ng <= 1)
        return decode_launch_group<T, G>(ix, w, 0, B, true, q, k_pages, v_pages, bt, max_pages, cur_lens, out, out_lse, out_sel,
                                         out_ncand, out_probe, st);
    HIP_TRY(hipEventRecord(ix->ev_fork, st));
    int rc = CTKVR_OK;
    for (int gi = 0; gi < ng && rc == CTKVR_OK; ++gi) {
        const int b0 = (int)((long long)B * gi / ng), b1 = (int)((long long)B * (gi + 1) / ng);
        hipStream_t gs = gi == 0 ? st : ix->side[gi - 1];
        if (gi > 0) HIP_TRY(hipStreamWaitEvent(gs, ix->ev_fork, 0));
        rc = decode_launch_group<T, G>(ix, w, b0, b1 - b0, false, q, k_pages, v_pages, bt, max_pages, cur_lens, out, out_lse,
                                       out_sel, out_ncand, out_probe, gs);
        if (gi > 0 && rc == CTKVR_OK) {
            HIP_TRY(hipEventRecord(ix->ev_join[gi - 1], gs));
            HIP_TRY(hipStreamWaitEvent(st, ix->ev_join[gi - 1], 0));
        }
    }
    return rc;
}

template <typename T>
int decode_dispatch(ctkvr_index *ix, const StepWs &w, const void *q, const void *k, const void *v, const int32_t *bt, int mp,
                    const int32_t *cur, float *out, float *lse, int32_t *sel, int32_t *ncand, int32_t *probe, hipStream_t st)
{
    switch (ix->G) {
        case 1: return decode_launch<T, 1>(ix, w, q, k, v, bt, mp, cur, out, lse, sel, ncand, probe, st);
        case 2: return decode_launch<T, 2>(ix, w, q, k, v, bt, mp, cur, out, lse, sel, ncand, probe, st);
        case 4: return decode_launch<T, 4>(ix, w, q, k, v, bt, mp, cur, out, lse, sel, ncand, probe, st);
        default: return decode_launch<T, 8>(ix, w, q, k, v, bt, mp, cur, out, lse, sel, ncand, probe, st);
    }
}

// Lloyd iterations on the centroid table (k-means centroid mode)
template <int G> int run_kmeans_g(ctkvr_index *ix, KmeansArgs ka, hipStream_t st)
{
    const int U = ix->units;
    using AS = AssignShape<G>;
    TRY(want_lds(ix->dev, (const void *)kmeans_assign_kernel<G>, AS::kLds));
    kmeans_init_kernel<<<dim3(ix->c_max, ix->p.n_q_heads, ix->p.batch), 128, 0, st>>>(ka, G);
    for (int it = 0; it < ix->p.kmeans_iters; ++it) {
        kmeans_halfnorm_kernel<G><<<dim3((ix->c_max + 15) / 16, U), 256, 0, st>>>(ka);
        kmeans_assign_kernel<G><<<dim3((ix->s_max + AS::kPoints - 1) / AS::kPoints, U), 256, AS::kLds, st>>>(ka);
        kmeans_rank_kernel<<<dim3(ka.n_stretch, U), 1024, (size_t)ix->c_max * 4, st>>>(ka);
        kmeans_offsets_kernel<<<dim3(U), 1024, (size_t)ix->c_max * 4, st>>>(ka);
        kmeans_scatter_kernel<<<dim3((ix->s_max + 255) / 256, U), 256, 0, st>>>(ka);
        kmeans_reduce_kernel<G><<<dim3(ix->c_max + ka.ext_max, U), ReduceShape<G>::NT, 0, st>>>(ka);
    }
    HIP_TRY(hipGetLastError());
    return CTKVR_OK;
}

int run_kmeans(ctkvr_index *ix, const bf16_t *q_prefill, const int32_t *d_first, const int32_t *init_pos, hipStream_t st)
{
    const size_t U = ix->units;
    KmeansArgs ka{};
    ka.g = ix->p.n_kv_heads;
    ka.h = ix->p.n_q_heads;
    ka.c_max = ix->c_max;
    ka.s_max = ix->s_max;
    ka.n_cent = ix->d_n_cent;
    ka.ctx_lens = ix->d_ctx_lens;
    ka.first_row = d_first;
    ka.q = q_prefill;
    ka.centroids = (bf16_t *)ix->centroids;
    ka.init_pos = init_pos;
    ka.ext_max = ix->s_max / (int)kPartRows + 1;
    ka.stretch = std::max(1024, (ix->s_max + kStretches - 1) / kStretches);
    ka.n_stretch = (ix->s_max + ka.stretch - 1) / ka.stretch;
    const size_t n_sums = U * ka.ext_max * ix->G * kD;
    BuildScratch scratch_mem;
    auto lay_out = [&](unsigned char *base) {
        Carver cv{base};
        cv.take(&ka.half_norm, U * ix->c_max * 4);
        cv.take(&ka.assign, U * ix->s_max * 4);
        cv.take(&ka.counts, U * ka.n_stretch * ix->c_max * 4);
        cv.take(&ka.start, U * ix->c_max * 4);
        cv.take(&ka.rank, U * ix->s_max * 4);
        cv.take(&ka.order, U * ix->s_max * 4);
        cv.take(&ka.part, U * ka.ext_max * sizeof(uint2));
        cv.take(&ka.n_part, U * 4);
        cv.take(&ka.slot, U * ix->c_max * 4);
        cv.take(&ka.sums, n_sums * 8);
        cv.take(&ka.done, U * ka.ext_max * 4);
        return cv.off;
    };
    int rc = scratch_mem.get(ix->dev, lay_out(nullptr));
    if (rc == CTKVR_OK) {
        lay_out(scratch_mem.base());
        fill_u32_kernel<<<dim3((unsigned)((n_sums * 2 + 255) / 256)), 256, 0, st>>>((uint32_t *)ka.sums, 0u, n_sums * 2);
        fill_u32_kernel<<<dim3((unsigned)((U * ka.ext_max + 255) / 256)), 256, 0, st>>>(ka.done, 0u, U * ka.ext_max);
        switch (ix->G) {
            case 1: rc = run_kmeans_g<1>(ix, ka, st); break;
            case 2: rc = run_kmeans_g<2>(ix, ka, st); break;
            case 4: rc = run_kmeans_g<4>(ix, ka, st); break;
            default: rc = run_kmeans_g<8>(ix, ka, st); break;
        }
    }
    hipError_t es = hipStreamSynchronize(st);
    scratch_mem.waited(es);
    if (rc == CTKVR_OK && es != hipSuccess) rc = fail(CTKVR_EHIP, "k-means: %s", hipGetErrorString(es));
    return rc;
}

// Algorithm 2 line 12 after a decode step: the step's ranking keys, their histogram and the
// recalled ids are still in the workspace.
template <typename T, int G> int update_launch(ctkvr_index *ix, const void *q, hipStream_t st)
{
    const ctkvr_params &p = ix->p;
    const int U = ix->units;
    DcuArgs da{};
    da.g = p.n_kv_heads;
    da.h = p.n_q_heads;
    da.G = G;
    da.c_max = ix->c_max;
    da.rho = p.list_len;
    da.n_cent = ix->d_n_cent;
    da.count = ix->d_dcu_count;
    da.q = q;
    da.centroids = ix->centroids;
    da.inv_norm_c = ix->inv_norm_c;
    da.lists = ix->lists;
    if (p.list_len == p.top_k) {   // the list is the selection of line 6
        da.src = ix->ws.sel;
        da.nsrc = ix->ws.nsel;
        da.src_stride = p.top_k;
    } else if (ix->dcu_lds) {      // the same ranking once more, with budget rho
        DcuSelectArgs ds{};
        ds.d = da;
        ds.ncand = ix->ws.ncand;
        ds.cand = ix->ws.cand;
        ds.kbuf = ix->ws.kbuf;
        ds.l_stride = ix->l_stride;
        dcu_select_kernel<T><<<dim3(U), kTailThreads, ix->dcu_lds, st>>>(ds);
        HIP_TRY(hipGetLastError());
        ix->have_step = false;
        return CTKVR_OK;
    } else {                       // ... by chip-wide passes and a selection, as in the step
        Units u = decode_units(ix);
        SelectArgs se{};
        se.u = u;
        se.ctx_lens = ix->d_ctx_lens;
        se.ncand = ix->ws.ncand;
        se.cand = ix->ws.cand;
        se.l_stride = ix->l_stride;
        se.top_k = p.list_len;
        se.z = ix->ws.z;
        se.m_key = ix->ws.m_key;
        se.kbuf = ix->ws.kbuf;
        se.ghist = ix->ws.ghist;
        se.bits_words = ix->sel_bits;
        se.sel = ix->dsel;
        se.nsel = ix->dnsel;
        se.ids_only = 1;
        if (ix->sel_bits) {
            // The keys' histogram is taken here, whatever the step left: most forms of it leave none, groups of one batch may take
            // different forms, and a replayed step leaves what it was captured with.  This launch clears the list cursors too.
            fill_u32_kernel<<<dim3((unsigned)(((size_t)U * kBuckets + 255) / 256)), 256, 0, st>>>(ix->ws.ghist, 0u, (size_t)U * kBuckets);
            KeyArgs ka{};
            ka.u = u;
            ka.ctx_lens = ix->d_ctx_lens;
            ka.ncand = ix->ws.ncand;
            ka.l_stride = ix->l_stride;
            ka.z = nullptr;   // the keys are there
            ka.kbuf = ix->ws.kbuf;
            ka.ghist = ix->ws.ghist;
            ka.gcur = ix->ws.gcur;
            keyhist_kernel<G><<<dim3(std::max(1, std::min((ix->l_stride + 4095) / 4096, (2 * ix->num_cu + U - 1) / U)), U), 1024, 0, st>>>(ka);
            ClassifyArgs ca{};
            ca.u = u;
            ca.ctx_lens = ix->d_ctx_lens;
            ca.ncand = ix->ws.ncand;
            ca.l_stride = ix->l_stride;
            ca.top_k = p.list_len;
            ca.kbuf = ix->ws.kbuf;
            ca.ghist = ix->ws.ghist;
            ca.bits_stride = 2 * ((ix->l_stride + 63) / 64);
            ca.gbm = ix->ws.gbm;
            ca.glist = ix->ws.glist;
            ca.gcur = ix->ws.gcur;
            ca.ginfo = ix->ws.ginfo;
            classify_kernel<<<dim3(std::max(1, std::min((ix->l_stride + 1023) / 1024, (4 * ix->num_cu + U - 1) / U)), U), 256, 0, st>>>(ca);
            se.gbm = ix->ws.gbm;
            se.glist = ix->ws.glist;
            se.ginfo = ix->ws.ginfo;
            se.bits_stride = ca.bits_stride;
        }
        rerank_select_kernel<G><<<dim3(U), 1024, ix->select_lds, st>>>(se);
        da.src = ix->dsel;
        da.nsrc = ix->dnsel;
        da.src_stride = p.list_len;
    }
    dcu_write_kernel<T><<<dim3(U), 256, 0, st>>>(da);
    HIP_TRY(hipGetLastError());
    ix->have_step = false;
    return CTKVR_OK;
}

template <typename T> int update_dispatch(ctkvr_index *ix, const void *q, hipStream_t st)
{
    switch (ix->G) {
        case 1: return update_launch<T, 1>(ix, q, st);
        case 2: return update_launch<T, 2>(ix, q, st);
        case 4: return update_launch<T, 4>(ix, q, st);
        default: return update_launch<T, 8>(ix, q, st);
    }
}

int min_pages_needed(const ctkvr_index *ix)
{
    return (ix->s_max + ix->p.page_size - 1) / ix->p.page_size;
}

}  // namespace

#pragma GCC visibility push(default)
extern "C" {

const char *ctkvr_last_error(void) { return g_err.c_str(); }

int ctkvr_build_index(const ctkvr_params *p, const void *q_prefill, const int32_t *cu_seqlens, int32_t q_is_tail,
                      const void *k_pages, const int32_t *block_table, int32_t max_pages, const int32_t *ctx_lens,
                      const int32_t *init_pos, void *hip_stream, ctkvr_index **out_index)
{
    if (!out_index) return fail(CTKVR_EINVAL, "out_index is NULL");
    *out_index = nullptr;
    TRY(check_params(p, ctx_lens));
    if (!q_prefill || !cu_seqlens || !k_pages || !block_table) return fail(CTKVR_EINVAL, "a required pointer is NULL");
    const bool kmeans = p->centroid_mode == CTKVR_CENTROID_KMEANS;
    if (kmeans) {
        if (p->dtype != CTKVR_BF16) return fail(CTKVR_EUNSUPPORTED, "the k-means centroid mode needs bf16 data");
        if (q_is_tail) return fail(CTKVR_EINVAL, "the k-means centroid mode needs all prompt queries (q_is_tail = 0)");
        if (!init_pos) return fail(CTKVR_EINVAL, "the k-means centroid mode needs init_pos");
        if (p->kmeans_iters < 0 || p->kmeans_iters > 1000) return fail(CTKVR_EINVAL, "kmeans_iters %d outside 0..1000", p->kmeans_iters);
    }
    if (p->build_algo == CTKVR_BUILD_MFMA && p->dtype != CTKVR_BF16)
        return fail(CTKVR_EUNSUPPORTED, "the matrix-core list build needs bf16 data");
    std::vector<int32_t> first_row(p->batch);
    for (int b = 0; b < p->batch; ++b) {
        int s = ctx_lens[b];
        int C = p->n_centroids ? p->n_centroids : s / p->centroid_div;
        int rows = cu_seqlens[b + 1] - cu_seqlens[b];
        int need = q_is_tail ? C : s;
        if (rows != need)
            return fail(CTKVR_EINVAL, "sequence %d: cu_seqlens gives %d query rows, expected %d", b, rows, need);
        if (max_pages * p->page_size < s) return fail(CTKVR_EINVAL, "max_pages %d too small for ctx_len %d", max_pages, s);
        first_row[b] = kmeans ? cu_seqlens[b] : cu_seqlens[b] + rows - C;
    }
    ctkvr_index *ix = nullptr;
    hipStream_t st = (hipStream_t)hip_stream;
    TRY(create_index(p, ctx_lens, first_row.data(), true, st, &ix));
    int rc = CTKVR_OK;
    const int32_t *d_first = ix->d_first;
    {
        dim3 grid((ix->c_max + 15) / 16, p->n_q_heads, p->batch);
        if (kmeans) {
            rc = run_kmeans(ix, (const bf16_t *)q_prefill, d_first, init_pos, st);
            if (rc == CTKVR_OK) rc = launch_inv_norms<bf16_t>(ix, st);
            if (rc == CTKVR_OK) rc = build_lists_dispatch<bf16_t>(ix, k_pages, block_table, max_pages, st);
        } else if (p->dtype == CTKVR_BF16) {
            copy_centroids_kernel<bf16_t><<<grid, 256, 0, st>>>((const bf16_t *)q_prefill, d_first, ix->d_n_cent, p->n_q_heads,
                                                                 ix->c_max, (bf16_t *)ix->centroids, ix->inv_norm_c);
            rc = build_lists_dispatch<bf16_t>(ix, k_pages, block_table, max_pages, st);
        } else {
            copy_centroids_kernel<float><<<grid, 256, 0, st>>>((const float *)q_prefill, d_first, ix->d_n_cent, p->n_q_heads,
                                                                ix->c_max, (float *)ix->centroids, ix->inv_norm_c);
            rc = build_lists_dispatch<float>(ix, k_pages, block_table, max_pages, st);
        }
    }
    if (rc == CTKVR_OK) {
        hipError_t e = hipStreamSynchronize(st);
        if (e != hipSuccess) rc = fail(CTKVR_EHIP, "build: %s", hipGetErrorString(e));
    }
    if (rc != CTKVR_OK) {
        delete ix;
        return rc;
    }
    *out_index = ix;
    return CTKVR_OK;
}

int ctkvr_index_load(const ctkvr_params *p, const int32_t *ctx_lens, const void *centroids, const int32_t *lists,
                     void *hip_stream, ctkvr_index **out_index)
{
    if (!out_index) return fail(CTKVR_EINVAL, "out_index is NULL");
    *out_index = nullptr;
    TRY(check_params(p, ctx_lens));
    if (!centroids || !lists) return fail(CTKVR_EINVAL, "a required pointer is NULL");
    ctkvr_index *ix = nullptr;
    hipStream_t st = (hipStream_t)hip_stream;
    TRY(create_index(p, ctx_lens, nullptr, false, st, &ix));
    const size_t es = elem_size(p->dtype);
    const CopySeg segs[2] = {{ix->centroids, centroids, (size_t)p->batch * p->n_q_heads * ix->c_max * 128 * es},
                             {ix->lists, lists, (size_t)ix->units * ix->c_max * p->list_len * 4}};
    hipError_t e = copy_segments(ix->dev, segs, 2, true, st);
    int rc = CTKVR_OK;
    if (e != hipSuccess) rc = fail(CTKVR_EHIP, "index upload: %s", hipGetErrorString(e));
    if (rc == CTKVR_OK) rc = p->dtype == CTKVR_BF16 ? launch_inv_norms<bf16_t>(ix, st) : launch_inv_norms<float>(ix, st);
    // every id a decode step may touch must be a valid key id of its sequence: looked through on the device (a scan of the
    // host's copy took 1.0 of 1.9 ms), the first one that is not named from the host's copy
    unsigned long long *d_bad = (unsigned long long *)ix->d_prof, bad = ~0ull;
    if (rc == CTKVR_OK) {
        fill_u32_kernel<<<1, 64, 0, st>>>((uint32_t *)d_bad, 0xffffffffu, 2);
        check_lists_kernel<<<dim3(ix->c_max, ix->units), 256, 0, st>>>(ix->lists, ix->d_ctx_lens, ix->d_n_cent, p->n_kv_heads, ix->c_max,
                                                                    p->list_len, d_bad);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipMemcpyAsync(&bad, d_bad, sizeof bad, hipMemcpyDeviceToHost, st);
        fill_u32_kernel<<<1, 64, 0, st>>>((uint32_t *)d_bad, 0u, 2);
        hipError_t e2 = hipStreamSynchronize(st);
        if (e == hipSuccess) e = e2;
        if (e != hipSuccess) rc = fail(CTKVR_EHIP, "index upload: %s", hipGetErrorString(e));
    }
    if (rc == CTKVR_OK && bad != ~0ull) {
        const size_t rho = p->list_len, row = bad / rho, unit = row / ix->c_max;
        rc = fail(CTKVR_EINVAL, "list (%d,%d,%d)[%d] = %d is not a key id of the sequence", (int)(unit / p->n_kv_heads),
                  (int)(unit % p->n_kv_heads), (int)(row % ix->c_max), (int)(bad % rho), lists[bad]);
    }
    if (rc != CTKVR_OK) {
        delete ix;
        return rc;
    }
    *out_index = ix;
    return CTKVR_OK;
}

int ctkvr_decode_step_window(ctkvr_index *idx, const void *q, const void *k_pages, const void *v_pages,
                             const int32_t *block_table, int32_t max_pages, const int32_t *cur_lens, float *out,
                             float *out_lse, int32_t *out_sel, int32_t *out_ncand, int32_t *out_probe, void *hip_stream)
{
    if (!idx) return fail(CTKVR_EINVAL, "index is NULL");
    if (!q || !k_pages || !v_pages || !block_table || !out) return fail(CTKVR_EINVAL, "a required pointer is NULL");
    if (max_pages < min_pages_needed(idx))
        return fail(CTKVR_EINVAL, "max_pages %d < %d pages of the longest sequence", max_pages, min_pages_needed(idx));
    hipStream_t st = (hipStream_t)hip_stream;
    if (idx->p.dtype == CTKVR_BF16)
        return decode_dispatch<bf16_t>(idx, idx->ws, q, k_pages, v_pages, block_table, max_pages, cur_lens, out, out_lse,
                                       out_sel, out_ncand, out_probe, st);
    return decode_dispatch<float>(idx, idx->ws, q, k_pages, v_pages, block_table, max_pages, cur_lens, out, out_lse, out_sel,
                                  out_ncand, out_probe, st);
}

int ctkvr_decode_step(ctkvr_index *idx, const void *q, const void *k_pages, const void *v_pages,
                      const int32_t *block_table, int32_t max_pages, float *out, float *out_lse, int32_t *out_sel,
                      int32_t *out_ncand, int32_t *out_probe, void *hip_stream)
{
    return ctkvr_decode_step_window(idx, q, k_pages, v_pages, block_table, max_pages, nullptr, out, out_lse, out_sel,
                                    out_ncand, out_probe, hip_stream);
}

int ctkvr_decode_step_static(ctkvr_index *idx, const void *q, const void *k_pages, const void *v_pages,
                             const int32_t *block_table, int32_t max_pages, float *out, float *out_lse, int32_t *out_sel,
                             int32_t *out_ncand, int32_t *out_probe, void *hip_stream)
{
    if (!idx) return fail(CTKVR_EINVAL, "index is NULL");
    if (!q || !k_pages || !v_pages || !block_table || !out) return fail(CTKVR_EINVAL, "a required pointer is NULL");
    if (max_pages < min_pages_needed(idx))
        return fail(CTKVR_EINVAL, "max_pages %d < %d pages of the longest sequence", max_pages, min_pages_needed(idx));
    StepWs w;
    const size_t need = carve_step_ws(w, nullptr, idx, true);
    if (need > kStaticStepBytes || carve_step_ws(w, nullptr, idx) > kStaticScratchBytes)   // (the second follows from the first)
        return fail(CTKVR_EUNSUPPORTED, "the step's workspace (%zu bytes) exceeds the static scratch of %zu bytes", need,
                    kStaticStepBytes);
    unsigned char *base = nullptr;
    TRY(static_scratch(&base));
    carve_step_ws(w, base, idx);
    hipStream_t st = (hipStream_t)hip_stream;
    // The array keeps the last call's contents, possibly of another index: what a step expects to find
    // zero is cleared here (fill kernels, so that a captured call replays correctly): the recall bitmap, and
    // the selected rows (slots beyond the selection are read as valid row numbers).
    const size_t nbits = (size_t)idx->units * idx->bitmap_words, nrow = (size_t)idx->units * idx->p.top_k;
    const size_t nbar = (size_t)idx->units * kFusedBarriers;
    zero3_u32_kernel<<<dim3((unsigned)((nbits + nrow + nbar + 255) / 256)), 256, 0, st>>>(w.gbits, nbits, w.srow, nrow, w.bar, nbar);
    if (idx->p.dtype == CTKVR_BF16)
        return decode_dispatch<bf16_t>(idx, w, q, k_pages, v_pages, block_table, max_pages, nullptr, out, out_lse, out_sel,
                                       out_ncand, out_probe, st);
    return decode_dispatch<float>(idx, w, q, k_pages, v_pages, block_table, max_pages, nullptr, out, out_lse, out_sel,
                                  out_ncand, out_probe, st);
}

int ctkvr_centroid_update(ctkvr_index *idx, const void *q, void *hip_stream)
{
    if (!idx) return fail(CTKVR_EINVAL, "index is NULL");
    if (!q) return fail(CTKVR_EINVAL, "q is NULL");
    if (!idx->have_step) return fail(CTKVR_EINVAL, "no decode step since the index was built or last updated");
    hipStream_t st = (hipStream_t)hip_stream;
    if (idx->p.dtype == CTKVR_BF16) return update_dispatch<bf16_t>(idx, q, st);
    return update_dispatch<float>(idx, q, st);
}

void ctkvr_free(ctkvr_index *idx)
{
    delete idx;   // synchronises the index's device
}

int ctkvr_profile_enable(ctkvr_index *idx, int32_t max_steps)
{
    if (!idx || max_steps < 0) return fail(CTKVR_EINVAL, "bad argument");
    DeviceScope on(idx->dev);
    HIP_TRY(on.err);
    HIP_TRY(hipDeviceSynchronize());
    for (hipEvent_t e : idx->events) (void)hipEventDestroy(e);
    idx->events.clear();
    idx->prof_max = idx->prof_step = 0;
    for (size_t i = 0; i < (size_t)max_steps * (CTKVR_N_STAGES + 1); ++i) {
        hipEvent_t e;
        HIP_TRY(hipEventCreate(&e));
        idx->events.push_back(e);
    }
    idx->prof_max = max_steps;
    return CTKVR_OK;
}

int ctkvr_profile_collect(ctkvr_index *idx, float *ms_host, int32_t capacity_steps, int32_t *n_steps)
{
    if (!idx || !ms_host || !n_steps) return fail(CTKVR_EINVAL, "NULL argument");
    DeviceScope on(idx->dev);
    HIP_TRY(on.err);
    HIP_TRY(hipDeviceSynchronize());
    int n = std::min<int>(idx->prof_step, capacity_steps);
    for (int s = 0; s < n; ++s)
        for (int k = 0; k < CTKVR_N_STAGES; ++k) {
            const hipEvent_t *ev = &idx->events[(size_t)s * (CTKVR_N_STAGES + 1)];
            HIP_TRY(hipEventElapsedTime(&ms_host[(size_t)s * CTKVR_N_STAGES + k], ev[k], ev[k + 1]));
        }
    *n_steps = n;
    idx->prof_step = 0;
    return CTKVR_OK;
}

int ctkvr_index_set_decode_path(ctkvr_index *idx, int32_t path)
{
    if (!idx) return fail(CTKVR_EINVAL, "index is NULL");
    if (path != CTKVR_PATH_AUTO && path != CTKVR_PATH_STAGED && path != CTKVR_PATH_FUSED)
        return fail(CTKVR_EINVAL, "unknown decode path %d", path);
    if (path == CTKVR_PATH_FUSED && !idx->fused_bpu)
        return fail(CTKVR_EUNSUPPORTED, "the single-launch step does not fit this geometry (%d units on %d CUs, or its shared memory)",
                    idx->units, idx->num_cu);
    if (path == CTKVR_PATH_FUSED) TRY(allow_fused(idx));
    idx->decode_path = path;
    return CTKVR_OK;
}

int ctkvr_release_scratch(void)
{
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return CTKVR_OK;
    std::lock_guard<std::mutex> lock(g_pool_mu);
    if (g_pool_builds[dev]) return fail(CTKVR_EINVAL, "an index build is using the scratch");
    pool_settle(dev);
    pool_drop(dev);
    if (!g_staging[dev].busy && (!g_staging[dev].unsure || device_idle())) {
        g_staging[dev].unsure = false;
        staging_drop(g_staging[dev]);
    }
    return CTKVR_OK;
}

int ctkvr_index_build_route(const ctkvr_index *idx, int32_t *by_candidates_host, int32_t *chunks_redone_host)
{
    if (!idx) return fail(CTKVR_EINVAL, "null index");
    if (by_candidates_host) *by_candidates_host = idx->build_by_cand;
    if (chunks_redone_host) *chunks_redone_host = idx->build_redone;
    return CTKVR_OK;
}

int ctkvr_index_decode_path(const ctkvr_index *idx)
{
    if (!idx) return fail(CTKVR_EINVAL, "index is NULL");
    return (idx->fused_bpu && idx->decode_path == CTKVR_PATH_FUSED) ? CTKVR_PATH_FUSED : CTKVR_PATH_STAGED;
}

int ctkvr_index_check(ctkvr_index *idx)
{
    if (!idx) return fail(CTKVR_EINVAL, "index is NULL");
    DeviceScope on(idx->dev);
    HIP_TRY(on.err);
    HIP_TRY(hipDeviceSynchronize());
    uint32_t e = 0;
    HIP_TRY(hipMemcpy(&e, idx->d_err, 4, hipMemcpyDeviceToHost));
    if (e)
        return fail(CTKVR_EHIP, "a single-launch decode step gave up waiting for its sibling blocks (were two such steps "
                                "running on this GPU at once?); results since then are invalid");
    return CTKVR_OK;
}

int ctkvr_profile_phases(ctkvr_index *idx, int32_t enable, long long *ticks_host)
{
    if (!idx) return fail(CTKVR_EINVAL, "index is NULL");
    DeviceScope on(idx->dev);
    HIP_TRY(on.err);
    HIP_TRY(hipDeviceSynchronize());
    if (ticks_host) HIP_TRY(hipMemcpy(ticks_host, idx->d_prof, 64 * sizeof(long long), hipMemcpyDeviceToHost));
    idx->prof_phases = enable != 0;
    return CTKVR_OK;
}

int ctkvr_measure_dispatch_floor(int32_t n_launches, float *us_per_launch_host, void *hip_stream)
{
    if (n_launches < 1 || n_launches > 100000 || !us_per_launch_host) return fail(CTKVR_EINVAL, "bad argument");
    hipStream_t st = nullptr;
    (void)hip_stream;
    HIP_TRY(hipStreamCreate(&st));   // capture needs a stream of its own (not the legacy default stream)
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int rc = CTKVR_OK;
    auto step = [&](hipError_t e, const char *what) {
        if (rc == CTKVR_OK && e != hipSuccess) rc = fail(CTKVR_EHIP, "%s: %s", what, hipGetErrorString(e));
        return rc == CTKVR_OK;
    };
    if (step(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal), "begin capture")) {
        for (int i = 0; i < n_launches; ++i) fill_u32_kernel<<<dim3(1), 64, 0, st>>>(nullptr, 0u, 0);
        step(hipStreamEndCapture(st, &graph), "end capture");
    }
    if (rc == CTKVR_OK) step(hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0), "instantiate");
    if (rc == CTKVR_OK) step(hipEventCreate(&e0), "event");
    if (rc == CTKVR_OK) step(hipEventCreate(&e1), "event");
    if (rc == CTKVR_OK) step(hipGraphLaunch(exec, st), "warm-up launch");
    if (rc == CTKVR_OK) step(hipStreamSynchronize(st), "sync");
    if (rc == CTKVR_OK) step(hipEventRecord(e0, st), "record");
    if (rc == CTKVR_OK) step(hipGraphLaunch(exec, st), "launch");
    if (rc == CTKVR_OK) step(hipEventRecord(e1, st), "record");
    if (rc == CTKVR_OK) step(hipEventSynchronize(e1), "sync");
    float ms = 0.0f;
    if (rc == CTKVR_OK) step(hipEventElapsedTime(&ms, e0, e1), "elapsed");
    if (rc == CTKVR_OK) *us_per_launch_host = ms * 1e3f / (float)n_launches;
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    (void)hipStreamDestroy(st);
    return rc;
}

int ctkvr_selftest_exp(uint64_t *mismatches_host, void *stream)
{
    if (!mismatches_host) return fail(CTKVR_EINVAL, "NULL argument");
    hipStream_t st = (hipStream_t)stream;
    unsigned long long *bad = nullptr;
    HIP_TRY(hipMalloc(&bad, sizeof(*bad)));
    fill_u32_kernel<<<1, 64, 0, st>>>((uint32_t *)bad, 0u, 2);
    // the negative values from -0 down to -32 have the bit patterns 0x80000000 .. 0xC2000000; then +0
    exp_selftest_kernel<<<4096, 256, 0, st>>>(0x80000000u, 0x42000001u, bad);
    exp_selftest_kernel<<<1, 256, 0, st>>>(0u, 1u, bad);
    unsigned long long h = ~0ull;
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(&h, bad, sizeof(h), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(bad);
    if (e != hipSuccess) return fail(CTKVR_EHIP, "exp self-check: %s", hipGetErrorString(e));
    *mismatches_host = h;
    return CTKVR_OK;
}

int ctkvr_index_info(const ctkvr_index *idx, ctkvr_index_info_t *out)
{
    if (!idx || !out) return fail(CTKVR_EINVAL, "NULL argument");
    out->batch = idx->p.batch;
    out->n_q_heads = idx->p.n_q_heads;
    out->n_kv_heads = idx->p.n_kv_heads;
    out->head_dim = idx->p.head_dim;
    out->dtype = idx->p.dtype;
    out->c_max = idx->c_max;
    out->list_len = idx->p.list_len;
    out->n_probe = idx->p.n_probe;
    out->top_k = idx->p.top_k;
    out->l_stride = idx->l_stride;
    out->index_bytes = (int64_t)idx->units * idx->c_max * idx->p.list_len * 4;
    out->device_bytes = (int64_t)idx->mem.bytes;
    return CTKVR_OK;
}

int ctkvr_index_lists(const ctkvr_index *idx, int32_t *dst_host)
{
    if (!idx || !dst_host) return fail(CTKVR_EINVAL, "NULL argument");
    DeviceScope on(idx->dev);
    HIP_TRY(on.err);
    HIP_TRY(hipDeviceSynchronize());
    const CopySeg seg{dst_host, idx->lists, (size_t)idx->units * idx->c_max * idx->p.list_len * 4};
    HIP_TRY(copy_segments(idx->dev, &seg, 1, false, nullptr));
    return CTKVR_OK;
}

int ctkvr_index_centroids(const ctkvr_index *idx, void *dst_host)
{
    if (!idx || !dst_host) return fail(CTKVR_EINVAL, "NULL argument");
    DeviceScope on(idx->dev);
    HIP_TRY(on.err);
    HIP_TRY(hipDeviceSynchronize());
    const CopySeg seg{dst_host, idx->centroids,
                      (size_t)idx->p.batch * idx->p.n_q_heads * idx->c_max * 128 * elem_size(idx->p.dtype)};
    HIP_TRY(copy_segments(idx->dev, &seg, 1, false, nullptr));
    return CTKVR_OK;
}

int ctkvr_index_last_candidates(const ctkvr_index *idx, int32_t *dst_host)
{
    if (!idx || !dst_host) return fail(CTKVR_EINVAL, "NULL argument");
    DeviceScope on(idx->dev);
    HIP_TRY(on.err);
    HIP_TRY(hipDeviceSynchronize());
    HIP_TRY(hipMemcpy(dst_host, idx->ws.cand, (size_t)idx->units * idx->l_stride * 4, hipMemcpyDeviceToHost));
    return CTKVR_OK;
}

#ifdef CTKVR_TRACE
int ctkvr_debug_trace_read(long long *dst_host)
{
    HIP_TRY(hipDeviceSynchronize());
    HIP_TRY(hipMemcpyFromSymbol(dst_host, HIP_SYMBOL(ctkvr::g_trace), sizeof(long long) * 128));
    return CTKVR_OK;
}
int ctkvr_debug_blk_read(long long *dst_host)
{
    HIP_TRY(hipDeviceSynchronize());
    HIP_TRY(hipMemcpyFromSymbol(dst_host, HIP_SYMBOL(ctkvr::g_blk), sizeof(long long) * 8 * 2048));
    return CTKVR_OK;
}
#endif

}  // extern "C"
#pragma GCC visibility pop
