// The HIP calls that libiso makes, without a device: memory from malloc, streams and events as numbers, and a record of what was
// enqueued in which order.  Loaded before libiso it takes the runtime's place, so that a test can look at the host side (what is
// allocated, launched and ordered, and what follows a call that fails) on a machine without a GPU.
#include <stdlib.h>
#include <string.h>
#include <unistd.h>

#include <map>
#include <mutex>
#include <set>
#include <string>

struct dim3 { unsigned x, y, z; };
typedef void *stream_t;

static std::mutex g_lock;
static std::string g_log;                       // one line per call: what, stream, detail
static std::map<const void *, std::string> &names() { static std::map<const void *, std::string> m; return m; }
static size_t g_refuse;                         // hipMalloc of this many bytes fails
static int g_last, g_launch_us, g_capturing, g_arg = -1;
static std::set<const void *> g_pinned;
static long g_handles = 0x100;
struct Call { dim3 grid, block; size_t lds; stream_t s; };
static thread_local Call t_call;

static void note(const std::string &what, stream_t s, const std::string &detail) {
    const std::lock_guard<std::mutex> hold(g_lock);
    g_log += what + " " + std::to_string((long)s) + " " + detail + "\n";
}

extern "C" {
void fake_refuse(size_t bytes) { g_refuse = bytes; }
void fake_launch_us(int us) { g_launch_us = us; }
void fake_capturing(int on) { g_capturing = on; }
void fake_int_argument(int i) { g_arg = i; }     // note the i-th argument of every launch, an int (-1: none)
const char *fake_log() { return g_log.c_str(); }
void fake_clear() { g_log.clear(); }

void **__hipRegisterFatBinary(const void *) { static void *m; return &m; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { names()[host] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, stream_t s) { t_call = Call{g, b, lds, s}; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, stream_t *s) { *g = t_call.grid; *b = t_call.block; *lds = t_call.lds; *s = t_call.s; return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3, void **args, size_t, stream_t s) {
    note("kernel", s, names()[f] + " " + std::to_string(g.x) + "x" + std::to_string(g.y) + "x" + std::to_string(g.z) +
                          (g_arg < 0 ? "" : " " + std::to_string(*(int *)args[g_arg])));
    if (g_launch_us) usleep(g_launch_us);
    return 0;
}
int hipMalloc(void **p, size_t n) {
    if (g_refuse && n == g_refuse) { note("refused", 0, std::to_string(n)); *p = nullptr; return g_last = 2; }
    *p = aligned_alloc(256, (n + 255) / 256 * 256);
    note("malloc", 0, std::to_string(n));
    return 0;
}
int hipFree(void *p) { free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { *p = aligned_alloc(4096, (n + 4095) / 4096 * 4096); g_pinned.insert(*p); return 0; }
int hipHostFree(void *p) { g_pinned.erase(p); free(p); return 0; }
int hipMemset(void *p, int v, size_t n) { memset(p, v, n); note("memset", 0, std::to_string(n)); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *, const void *, size_t n, int, stream_t s) { note("copy", s, std::to_string(n)); return 0; }
int hipMemcpy2DAsync(void *, size_t, const void *, size_t, size_t w, size_t h, int, stream_t s) { note("copy2d", s, std::to_string(w) + "x" + std::to_string(h)); return 0; }
int hipGetLastError() { const int e = g_last; g_last = 0; return e; }
const char *hipGetErrorString(int) { return "fake error"; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipDeviceSynchronize() { note("device_sync", 0, ""); return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetSymbolAddress(void **p, const void *) { static char array[64]; *p = array; return 0; }
struct Attributes { int type, device; void *device_pointer, *host_pointer; };
int hipPointerGetAttributes(Attributes *a, const void *p) {       // knows the start of a pinned allocation
    if (!g_pinned.count(p)) return g_last = 1;
    *a = Attributes{1, 0, (void *)p, (void *)p};
    return 0;
}
int hipStreamCreateWithFlags(stream_t *s, unsigned) { *s = (stream_t)g_handles++; return 0; }
int hipStreamDestroy(stream_t) { return 0; }
int hipStreamSynchronize(stream_t) { return 0; }
int hipStreamIsCapturing(stream_t, int *c) { *c = g_capturing; return 0; }
int hipThreadExchangeStreamCaptureMode(int *) { return 0; }
int hipStreamWaitEvent(stream_t s, void *e, unsigned) { note("wait", s, std::to_string((long)e)); return 0; }
int hipEventCreate(void **e) { *e = (void *)g_handles++; return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = (void *)g_handles++; return 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *e, stream_t s) { note("record", s, std::to_string((long)e)); return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 0; return 0; }
}
