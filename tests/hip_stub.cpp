// A HIP runtime without a device, for tests of the library's host side on the CPU (tests/test_host_runtime.py loads
// it before libepi.so, whose HIP calls then land here).  Device memory is host memory, copies are done at once, and
// kernels are not run: a launch is checked against the limits of the hardware's dispatch packet, noted, and counted
// as queued until the next wait.  The kernels whose results steer the host leave the numbers a test asks for.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

struct Dim3 {
    uint32_t x, y, z;
};
struct Launch {
    std::string name;
    Dim3 grid, block;
    void *arg0;
};
static std::map<const void *, std::string> names;
static std::map<char *, size_t> blocks;  // device memory
static std::map<char *, int> home;       // and the device it is on
static int device = 0;                   // the current one, of two
static std::vector<Launch> launches;
static std::string fail_kernel;
static int64_t limit = INT64_MAX, used = 0, most = 0, queued_on[2] = {}, total = 0;
#define queued queued_on[device]
static int err = 0;
static char *first = nullptr;
static struct {
    Dim3 grid, block;
    size_t shared;
    void *stream;
} call;

static int set(int e) { return e ? err = e : 0; }
enum { kInvalid = 1, kNoMemory = 2, kConfig = 9, kLaunch = 719 };

extern "C" {
// what the tests ask for and read
void stub_reset() { launches.clear(); fail_kernel.clear(); limit = INT64_MAX; most = used; first = nullptr; }
void stub_limit(int64_t bytes) { limit = bytes; }
void stub_fail_kernel(const char *part) { fail_kernel = part; }
void stub_total(int64_t v) { total = v; }
int64_t stub_queued() { return queued_on[0]; }
int64_t stub_used_on(int d) {
    int64_t n = 0;
    for (auto &b : blocks) n += home[b.first] == d ? (int64_t)b.second : 0;
    return n;
}
int64_t stub_used() { return used; }
int64_t stub_most() { return most; }
void *stub_first_block() { return first; }
int64_t stub_launches() { return (int64_t)launches.size(); }
const char *stub_launch_name(int64_t i) { return launches[i].name.c_str(); }
int64_t stub_launch_grid(int64_t i) { return (int64_t)launches[i].grid.x * launches[i].grid.y; }
void *stub_launch_arg(int64_t i) { return launches[i].arg0; }
void *stub_device_block(int64_t bytes, int fill) {
    char *p = (char *)std::calloc(1, bytes);
    std::memset(p, fill, bytes);
    blocks[p] = bytes;
    home[p] = device;
    used += bytes;
    return p;
}

int hipMalloc(void **p, size_t n) {
    if (used + (int64_t)n > limit) return set(kNoMemory);
    char *q = (char *)std::calloc(1, n ? n : 1);
    if (!q) return set(kNoMemory);
    if (!first) first = q;
    blocks[q] = n;
    home[q] = device;
    used += n;
    most = used > most ? used : most;
    *p = q;
    return 0;
}
int hipFree(void *p) {
    if (!p) return 0;
    auto it = blocks.find((char *)p);
    if (it == blocks.end()) return set(kInvalid);
    used -= it->second;
    std::free(p);
    blocks.erase(it);
    queued_on[home[(char *)p]] = 0;  // (waits for the device)
    home.erase((char *)p);
    return 0;
}
int hipMemGetAddressRange(void **base, size_t *size, void *p) {
    auto it = blocks.upper_bound((char *)p);
    if (it == blocks.begin() || (char *)p >= (--it)->first + it->second) return set(kInvalid);
    *base = it->first;
    *size = it->second;
    return 0;
}
// the first fields of hipPointerAttribute_t: type (1 host, 2 device, 0 unregistered), device
int hipPointerGetAttributes(void *out, const void *p) {
    void *base;
    size_t size;
    const int e = err;
    const bool dev = hipMemGetAddressRange(&base, &size, (void *)p) == 0;
    err = e;
    std::memset(out, 0, 2 * sizeof(int));
    ((int *)out)[0] = dev ? 2 : 0;
    return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned) { return (*p = std::calloc(1, n)) ? 0 : set(kNoMemory); }
int hipHostFree(void *p) { std::free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int) { std::memmove(d, s, n); queued = 0; return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) {
    for (const char *p : {(const char *)s, (const char *)d}) {  // (a range that leaves its block is refused)
        auto it = blocks.upper_bound((char *)p);
        if (it != blocks.begin() && p < (--it)->first + it->second && p + n > it->first + it->second) return set(kInvalid);
    }
    std::memmove(d, s, n);
    ++queued;
    return 0;
}
int hipMemset(void *d, int v, size_t n) { std::memset(d, v, n); queued = 0; return 0; }
int hipMemsetAsync(void *d, int v, size_t n, void *) { std::memset(d, v, n); ++queued; return 0; }
int hipDeviceSynchronize() { queued = 0; return 0; }
int hipStreamSynchronize(void *) { queued = 0; return 0; }
int hipGetDeviceCount(int *n) { *n = 2; return 0; }
int hipGetDevice(int *d) { *d = device; return 0; }
int hipSetDevice(int d) { device = d; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipGetLastError() { const int e = err; err = 0; return e; }
const char *hipGetErrorString(int e) { return e == kNoMemory ? "out of memory" : "stub error"; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 8; return 0; }
int hipGetSymbolAddress(void **p, const void *) {
    static void *room = std::calloc(1, size_t(64) << 20);
    *p = room;
    return 0;
}
static int handle(void **p) { *p = std::malloc(1); return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { return handle(s); }
int hipStreamDestroy(void *s) { std::free(s); return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipStreamBeginCapture(void *, int) { return 0; }
int hipStreamEndCapture(void *, void **g) { return handle(g); }
int hipEventCreate(void **e) { return handle(e); }
int hipEventCreateWithFlags(void **e, unsigned) { return handle(e); }
int hipEventDestroy(void *e) { std::free(e); return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { queued = 0; return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 0; return 0; }
int hipGraphInstantiate(void **x, void *, void *, char *, size_t) { return handle(x); }
int hipGraphLaunch(void *, void *) { ++queued; return 0; }
int hipGraphDestroy(void *g) { std::free(g); return 0; }
int hipGraphExecDestroy(void *g) { std::free(g); return 0; }

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *fn, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) {
    names[fn] = name;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void *stream) {
    call = {grid, block, shared, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *shared, void **stream) {
    *grid = call.grid;
    *block = call.block;
    *shared = call.shared;
    *stream = call.stream;
    return 0;
}
int hipLaunchKernel(const void *fn, Dim3 grid, Dim3 block, void **args, size_t shared, void *) {
    const std::string &name = names[fn];
    auto bad = [](uint32_t g, uint32_t b) { return g == 0 || b == 0 || (uint64_t)g * b >= uint64_t(1) << 32; };
    if (bad(grid.x, block.x) || bad(grid.y, block.y) || bad(grid.z, block.z) ||
        (uint64_t)block.x * block.y * block.z > 1024 || shared > 160 * 1024)
        return set(kConfig);
    if (!fail_kernel.empty() && name.find(fail_kernel) != std::string::npos) return set(kLaunch);
    launches.push_back({name, grid, block, *(void **)args[0]});
    ++queued;
    auto is = [&](const char *part) { return name.find(part) != std::string::npos; };
    int64_t *sum = is("k_scan_small") ? *(int64_t **)args[3] : is("k_scan_apply64") ? *(int64_t **)args[5] : nullptr;
    if (sum) *sum = total;
    if (is("k_type_off"))  // 1000 events of every type
        for (int32_t k = 0; k <= *(int32_t *)args[1]; ++k) (*(int32_t **)args[2])[k] = 1000 * k;
    if (is("k_gap_init"))
        for (uint32_t k = 0; k < block.x; ++k) (*(int64_t **)args[0])[k] = INT64_MAX;
    if (is("k_level1I"))
        for (uint32_t k = 0; k < grid.x; ++k) (*(int32_t **)args[3])[k] = 1000;
    return 0;
}
}
