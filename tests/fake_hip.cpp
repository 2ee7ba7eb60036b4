// A HIP runtime without a GPU, for tests of what libdz's host side decides: it hands out addresses, refuses memory beyond a
// budget, answers "this stream is being captured" as told, and writes down every launch.  Loaded before libdz.so with
// RTLD_GLOBAL, its symbols are the ones that libdz binds.  No kernel runs and no address is ever read.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <vector>

struct Dim3 { uint32_t x, y, z; };
struct Launch { std::string name; Dim3 grid; size_t lds; int watched; };

static std::map<const void *, std::string> g_names;         // host stub -> mangled kernel name
static std::map<const void *, size_t> g_lds;                // dynamic LDS a kernel has been allowed beyond 64 KB
static std::map<uintptr_t, size_t> g_live;
static std::vector<Launch> g_launches;
static uintptr_t g_next = 0x100000000000ull;
static size_t g_room = ~(size_t)0;
static unsigned long long g_capture = 0;                    // id of the running capture, 0 = none
static int g_last = 0, g_refused = 0;
static std::string g_watch;
static int g_watch_arg = 0;
static struct { Dim3 grid, block; size_t lds; void *stream; } g_config;

static int fail(int e) { return g_last = e; }

extern "C" {

void fake_room(size_t bytes) { g_room = bytes; }
void fake_capture(unsigned long long id) { g_capture = id; }
void fake_watch(const char *kernel, int arg) { g_watch = kernel; g_watch_arg = arg; }      // note 4 bytes of this argument
int fake_refused() { return g_refused; }
size_t fake_live_bytes() { size_t n = 0; for (auto &a : g_live) n += a.second; return n; }
void fake_clear() { g_launches.clear(); }
int fake_launches() { return (int)g_launches.size(); }
const char *fake_name(int i) { return g_launches[i].name.c_str(); }
unsigned fake_grid(int i) { return g_launches[i].grid.x; }
size_t fake_lds(int i) { return g_launches[i].lds; }
int fake_watched(int i) { return g_launches[i].watched; }

int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipDeviceSynchronize() { return 0; }
int hipGetLastError() { const int e = g_last; g_last = 0; return e; }
const char *hipGetErrorString(int e) { static char t[32]; snprintf(t, sizeof t, "error %d", e); return t; }

int hipMalloc(void **p, size_t n)
{
    if (g_capture) return fail(900);
    if (fake_live_bytes() + n > g_room) { ++g_refused; return fail(2); }
    *p = (void *)g_next;
    g_live[g_next] = n;
    g_next += (n + 0x1fffff) / 0x100000 * 0x100000;
    return 0;
}
int hipFree(void *p) { return !p || g_live.erase((uintptr_t)p) ? 0 : fail(1); }
int hipMemset(void *, int, size_t) { return 0; }
int hipMemcpyAsync(void *dst, const void *, size_t n, int kind, void *) { if (kind == 2) memset(dst, 0, n); return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = (void *)8; return 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = (void *)0x200000000000ull; return 0; }
int hipStreamIsCapturing(void *, int *s) { *s = g_capture ? 1 : 0; return 0; }
int hipStreamGetCaptureInfo(void *, int *s, unsigned long long *id) { *s = g_capture ? 1 : 0; *id = g_capture; return 0; }
int hipFuncSetAttribute(const void *f, int, int v) { g_lds[f] = (size_t)v; return 0; }

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *stub, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    g_names[stub] = name;
}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void *stream)
{
    g_config = {grid, block, lds, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *lds, void **stream)
{
    *grid = g_config.grid; *block = g_config.block; *lds = g_config.lds; *stream = g_config.stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim3 grid, Dim3, void **args, size_t lds, void *)
{
    Launch l{g_names[f], grid, lds, 0};
    const size_t allowed = g_lds.count(f) ? g_lds[f] : 65536;
    if (lds > allowed) return fail(1);
    if (!g_watch.empty() && l.name.find(g_watch) != std::string::npos) memcpy(&l.watched, args[g_watch_arg], 4);
    g_launches.push_back(l);
    return 0;
}

}  // extern "C"
