// A stand-in for the HIP runtime, for tests of the library's host code without a GPU: two devices whose memory is host
// memory, kernels that do nothing (but for the one that fills words), and calls that fail when a test asks for it or when they mix objects of two devices.  Loaded with
// its symbols global before libctkvr.so, whose HIP calls then come here.  Fresh device memory reads as ones in every bit.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>

namespace {
enum { kOk = 0, kBadValue = 1, kBadDevice = 101, kBadHandle = 400, kCapturing = 900 };
struct Stream {
    int dev;
};
struct Event {
    int dev;
};
struct Dim3 {
    uint32_t x, y, z;
};
struct Block {
    size_t bytes;
    int dev;
};
std::recursive_mutex mu;
std::map<void *, Block> blocks;
thread_local int cur = 0, last = kOk;
thread_local struct {
    Dim3 grid, block;
    size_t lds;
    void *stream;
} call;
int n_malloc = 0, n_free = 0, n_launch = 0, n_record = 0, n_pinned = 0, n_sync[2] = {}, attr_dev = -1, n_attr = 0;
int refuse_device_sync = 0, refuse_stream_sync = 0;
std::map<const void *, void *> symbols;
const void *fill_words = nullptr;

int ret(int e)
{
    if (e != kOk) last = e;
    return e;
}
int dev_of(void *st) { return st ? ((Stream *)st)->dev : cur; }
int malloc_on(void **p, size_t n)
{
    std::lock_guard<std::recursive_mutex> l(mu);
    *p = aligned_alloc(4096, (n + 4095) / 4096 * 4096);
    memset(*p, 0xff, n);
    blocks[*p] = Block{n, cur};
    n_malloc++;
    return kOk;
}
}  // namespace

extern "C" {
// --- what a test sets and reads ---
void fake_refuse_syncs(int device, int stream)
{
    refuse_device_sync = device;
    refuse_stream_sync = stream;
}
int fake_mallocs() { return n_malloc; }
int fake_frees() { return n_free; }
int fake_launches() { return n_launch; }
int fake_records() { return n_record; }
int fake_pinned() { return n_pinned; }
int fake_syncs(int dev) { return n_sync[dev]; }
int fake_attr_calls() { return n_attr; }
int fake_attr_device() { return attr_dev; }   // current device at the last hipFuncSetAttribute
size_t fake_live_bytes(int dev)
{
    std::lock_guard<std::recursive_mutex> l(mu);
    size_t n = 0;
    for (auto &b : blocks)
        if (b.second.dev == dev) n += b.second.bytes;
    return n;
}

// --- the runtime ---
int hipGetDevice(int *d) { return *d = cur, kOk; }
int hipSetDevice(int d)
{
    if (d < 0 || d > 1) return ret(kBadDevice);
    cur = d;
    return kOk;
}
int hipDeviceGetAttribute(int *v, int, int) { return *v = 256, kOk; }
int hipGetLastError()
{
    int e = last;
    last = kOk;
    return e;
}
const char *hipGetErrorString(int e) { return e == kBadHandle ? "invalid handle" : e == kCapturing ? "refused during capture" : e ? "error" : "ok"; }
int hipMalloc(void **p, size_t n) { return malloc_on(p, n); }
int hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = malloc(n);
    n_pinned++;
    return kOk;
}
int hipHostFree(void *p)
{
    n_pinned--;
    return free(p), kOk;
}
int hipFree(void *p)
{
    std::lock_guard<std::recursive_mutex> l(mu);
    if (!p) return kOk;
    if (!blocks.erase(p)) return ret(kBadValue);
    free(p);
    n_free++;
    return kOk;
}
int hipDeviceSynchronize()
{
    if (refuse_device_sync) return ret(kCapturing);
    n_sync[cur]++;
    return kOk;
}
int hipStreamSynchronize(void *) { return refuse_stream_sync ? ret(kCapturing) : kOk; }
int hipStreamCreate(void **s) { return *s = new Stream{cur}, kOk; }
int hipStreamCreateWithFlags(void **s, unsigned) { return *s = new Stream{cur}, kOk; }
int hipStreamDestroy(void *s) { return delete (Stream *)s, kOk; }
int hipStreamWaitEvent(void *, void *, unsigned) { return kOk; }
int hipEventCreate(void **e) { return *e = new Event{cur}, kOk; }
int hipEventCreateWithFlags(void **e, unsigned) { return *e = new Event{cur}, kOk; }
int hipEventDestroy(void *e) { return delete (Event *)e, kOk; }
int hipEventRecord(void *e, void *s)
{
    n_record++;
    return ((Event *)e)->dev == dev_of(s) ? kOk : ret(kBadHandle);
}
int hipEventSynchronize(void *) { return refuse_stream_sync ? ret(kCapturing) : kOk; }
int hipEventElapsedTime(float *ms, void *, void *) { return *ms = 0.0f, kOk; }
int hipMemcpy(void *d, const void *s, size_t n, int) { return memcpy(d, s, n), kOk; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { return memcpy(d, s, n), kOk; }
int hipFuncSetAttribute(const void *, int, int)
{
    attr_dev = cur;
    n_attr++;
    return kOk;
}
int hipGetSymbolAddress(void **p, const void *sym)
{
    std::lock_guard<std::recursive_mutex> l(mu);
    void *&at = symbols[sym];
    if (!at) at = calloc(1, (size_t)33 << 20);
    *p = at;
    return kOk;
}
int hipLaunchKernel(const void *fn, Dim3, Dim3, void **args, size_t, void *)
{
    n_launch++;
    if (fn == fill_words) {
        uint32_t *p = *(uint32_t **)args[0], v = *(uint32_t *)args[1];
        for (size_t i = 0, n = *(size_t *)args[2]; i < n; ++i) p[i] = v;
    }
    return kOk;
}
int hipStreamBeginCapture(void *, int) { return ret(kBadValue); }
int hipStreamEndCapture(void *, void **) { return ret(kBadValue); }
int hipGraphInstantiate(void **, void *, void **, char *, size_t) { return ret(kBadValue); }
int hipGraphLaunch(void *, void *) { return ret(kBadValue); }
int hipGraphDestroy(void *) { return kOk; }
int hipGraphExecDestroy(void *) { return kOk; }
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void *st)
{
    call = {g, b, lds, st};
    return kOk;
}
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *lds, void **st)
{
    *g = call.grid;
    *b = call.block;
    *lds = call.lds;
    *st = call.stream;
    return kOk;
}
void **__hipRegisterFatBinary(const void *) { return (void **)calloc(1, sizeof(void *)); }
void __hipRegisterFunction(void **, const void *fn, char *, const char *name, unsigned, void *, void *, Dim3 *, Dim3 *, int *)
{
    if (strstr(name, "fill_u32_kernel")) fill_words = fn;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
}
