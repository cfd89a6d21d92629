// A stand-in for the HIP runtime on a machine without a device, loaded before the library
// (LD_PRELOAD): device and pinned memory come from the host and are counted, copies are made, and
// kernels are not run but written to a log, so the library's host side -- what it allocates, frees,
// launches, captures and waits for, and what it does when memory runs out -- can be tested.  As in
// the HIP runtime, an error stays until hipGetLastError reads it.  Plain C++, no HIP headers.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Dim3 { unsigned x, y, z; };
struct Stream { bool busy = false; };
struct Graph { std::vector<std::string> nodes; };
struct Exec { std::vector<std::string> nodes; Stream *on = nullptr; };

std::map<void *, size_t> dev, pinned;
size_t dev_used = 0, dev_mallocs = 0, pinned_used = 0, dev_limit = SIZE_MAX, refuse_at_least = SIZE_MAX, refuse_below = SIZE_MAX;
std::map<const void *, std::string> kernels;
std::string text;
Stream *capturing = nullptr;
Graph *graph = nullptr;
int last_error = 0;
struct Config { Dim3 g, b; size_t shm; void *s; } config;

int fail(int e) { return last_error = e; }
void note(const std::string &s) { text += s + "\n"; }
int launch(const void *f, void *s) {
    std::string name = kernels.count(f) ? kernels[f] : "?";
    if (capturing == s && graph) graph->nodes.push_back(name);
    else { note("run " + name); if (s) ((Stream *)s)->busy = true; }
    return 0;
}
void *take(std::map<void *, size_t> &m, size_t &used, size_t n) {
    void *p = std::aligned_alloc(4096, (n + 4095) / 4096 * 4096);
    m[p] = n;
    used += n;
    return p;
}
void give(std::map<void *, size_t> &m, size_t &used, void *p) {
    auto i = m.find(p);
    if (i == m.end()) { if (p) note("BAD FREE"); return; }
    used -= i->second;
    m.erase(i);
    std::free(p);
}
}  // namespace

extern "C" {
// controls of the tests
void fake_limit(size_t bytes) { dev_limit = bytes; }
void fake_refuse(size_t from, size_t below) { refuse_at_least = from; refuse_below = below; }
size_t fake_used(void) { return dev_used; }
size_t fake_mallocs(void) { return dev_mallocs; }
size_t fake_pinned(void) { return pinned_used; }
const char *fake_log(void) { static std::string out; out.swap(text); text.clear(); return out.c_str(); }

int hipMalloc(void **p, size_t n) {
    if (dev_used + n > dev_limit || (n >= refuse_at_least && n < refuse_below)) return fail(2);
    *p = take(dev, dev_used, n);
    ++dev_mallocs;
    return 0;
}
int hipFree(void *p) { give(dev, dev_used, p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { *p = take(pinned, pinned_used, n); return 0; }
int hipHostFree(void *p) { give(pinned, pinned_used, p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int) { std::memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) {
    note("copy " + std::to_string(n));
    std::memcpy(d, s, n);
    return 0;
}
int hipMemsetAsync(void *p, int v, size_t n, void *) {   // (no kernel reads a field)
    if (n <= 4096) std::memset(p, v, n);
    return 0;
}
int hipGetLastError(void) { int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int e) { return e == 2 ? "out of memory" : e ? "error" : "no error"; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetSymbolAddress(void **p, const void *s) { *p = const_cast<void *>(s); return 0; }

int hipStreamCreateWithFlags(void **s, unsigned) { *s = new Stream; return 0; }
int hipStreamDestroy(void *s) { delete (Stream *)s; return 0; }
int hipStreamSynchronize(void *s) { if (s) ((Stream *)s)->busy = false; return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipEventCreate(void **e) { *e = std::malloc(1); return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = std::malloc(1); return 0; }
int hipEventDestroy(void *e) { std::free(e); return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 1.0f; return 0; }
int hipEventQuery(void *) { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }

int hipStreamBeginCapture(void *s, int) { capturing = (Stream *)s; graph = new Graph; return 0; }
int hipStreamEndCapture(void *, void **g) { *g = graph; graph = nullptr; capturing = nullptr; return 0; }
int hipGraphDestroy(void *g) { delete (Graph *)g; return 0; }
int hipGraphInstantiate(void **x, void *g, void **, char *, size_t) {
    note("instantiate");
    *x = new Exec{((Graph *)g)->nodes};
    return 0;
}
int hipGraphLaunch(void *x, void *s) {
    for (auto &n : ((Exec *)x)->nodes) note("run " + n);
    ((Exec *)x)->on = (Stream *)s;
    if (s) ((Stream *)s)->busy = true;
    return 0;
}
int hipGraphExecDestroy(void *x) {
    if (((Exec *)x)->on && ((Exec *)x)->on->busy) note("GRAPH DESTROYED IN FLIGHT");
    delete (Exec *)x;
    return 0;
}

int hipLaunchKernel(const void *f, Dim3, Dim3, void **, size_t, void *s) { return launch(f, s); }
int hipExtLaunchKernel(const void *f, Dim3, Dim3, void **, size_t, void *s, void *, void *, int) { return launch(f, s); }
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shm, void *s) { config = {g, b, shm, s}; return 0; }
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *shm, void **s) {
    *g = config.g; *b = config.b; *shm = config.shm; *s = config.s;
    return 0;
}
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *) {
    kernels[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
}
