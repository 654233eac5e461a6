// A stand-in for the HIP runtime, for CPU tests of the transport world's host code: device memory
// is host memory, copies are copies, kernels do not run.  Launches are recorded by name with the
// arguments asked for (stub_watch); the two kernels that only move counters are carried out, with
// counts that the test sets (stub_counts).  Preloaded ahead of the real runtime.
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>
#include <vector>

namespace {

struct Dim3 {
    uint32_t x, y, z;
};
struct Launch {
    std::string name;
    Dim3 grid, block;
    std::vector<uint64_t> args;      // the first 8 bytes of each argument watched
};
struct Watch {
    std::string name;
    int arg;
};

std::map<const void *, std::string> names;
std::vector<Launch> launches;
std::vector<Watch> watches;
std::vector<uint64_t> counts, restored;
int64_t copied[5];                   // bytes of asynchronous copies by kind (1: to the device, 2: back)
int64_t pinned = 0;
int fail_syncs = 0;
Dim3 grid0, block0;
size_t shared0;
void *stream0;

uint64_t word(void **args, int i)
{
    uint64_t v;
    memcpy(&v, args[i], 8);
    return v;
}

}  // namespace

extern "C" {

void stub_watch(const char *name, int arg) { watches.push_back({name, arg}); }
void stub_counts(const uint64_t *v, int n) { counts.assign(v, v + n); }
void stub_fail_syncs(int n) { fail_syncs = n; }
void stub_clear()
{
    launches.clear();
    restored.clear();
    memset(copied, 0, sizeof copied);
}
int stub_launches() { return (int)launches.size(); }
const char *stub_name(int i) { return launches[i].name.c_str(); }
uint32_t stub_grid(int i) { return launches[i].grid.x; }
uint32_t stub_block(int i) { return launches[i].block.x; }
uint64_t stub_arg(int i, int k) { return launches[i].args.at(k); }
int stub_restored() { return (int)restored.size(); }
uint64_t stub_restored_word(int i) { return restored[i]; }
int64_t stub_copied(int kind) { return copied[kind]; }
int64_t stub_pinned() { return pinned; }

void **__hipRegisterFatBinary(const void *)
{
    static void *module;
    return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *)
{
    names[host] = name;
}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shared, void *stream)
{
    grid0 = g;
    block0 = b;
    shared0 = shared;
    stream0 = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *shared, void **stream)
{
    *g = grid0;
    *b = block0;
    *shared = shared0;
    *stream = stream0;
    return 0;
}

int hipLaunchKernel(const void *f, Dim3 g, Dim3 b, void **args, size_t, void *)
{
    Launch l{names[f], g, b, {}};
    for (const Watch &w : watches)
        if (l.name.find(w.name) != std::string::npos) l.args.push_back(word(args, w.arg));
    if (l.name.find("finish_kernel") != std::string::npos) {
        uint64_t *ctr = (uint64_t *)word(args, 0), *other = (uint64_t *)word(args, 1);
        uint64_t *host = (uint64_t *)word(args, 4);
        const int n = (int)word(args, 5);
        for (int i = 0; i < n; ++i) {
            ctr[i] = host[i] = i < (int)counts.size() ? counts[i] : 0;
            other[i] = 0;
        }
    } else if (l.name.find("reset_kernel") != std::string::npos) {
        const uint64_t *alive = (const uint64_t *)word(args, 0);
        uint64_t *ctr = (uint64_t *)word(args, 1), *other = (uint64_t *)word(args, 2);
        const int n = (int)word(args, 4);
        restored.assign(alive, alive + n);
        for (int i = 0; i < n; ++i) {
            ctr[i] = alive[i];
            other[i] = 0;
        }
    }
    launches.push_back(l);
    return 0;
}

int hipStreamSynchronize(void *)
{
    if (fail_syncs == 0) return 0;
    --fail_syncs;
    return 900;          // hipErrorStreamCaptureUnsupported
}
int hipDeviceSynchronize() { return 0; }
int hipGetDevice(int *d) { return *d = 0; }
int hipDeviceGetAttribute(int *v, int, int)
{
    *v = 256;
    return 0;
}
const char *hipGetErrorString(int) { return "stub"; }
int hipGetLastError() { return 0; }
int hipMalloc(void **p, size_t n) { return (*p = calloc(1, n)) ? 0 : 2; }
int hipFree(void *p)
{
    free(p);
    return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned)
{
    pinned += (int64_t)n;
    return hipMalloc(p, n);
}
int hipHostFree(void *p) { return hipFree(p); }
int hipMemset(void *p, int v, size_t n)
{
    memset(p, v, n);
    return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int)
{
    memcpy(d, s, n);
    return 0;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *)
{
    copied[kind] += (int64_t)n;
    memcpy(d, s, n);
    return 0;
}

}  // extern "C"
