// A HIP runtime without a device, for tests of the library's host code: memory
// is the host's, kernels are not run but noted (name, grid, workgroup, LDS
// bytes), and calls can be made to fail.  Loaded with RTLD_GLOBAL before the
// library, whose references then find these definitions first.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

struct dim3 {
    uint32_t x, y, z;
};
namespace {
std::mutex m;
std::map<const void *, std::string> kernels;
std::string notes;
thread_local int last_error;
int fail_pinned;  // hipHostMalloc fails
int capturing;    // calls that a global-mode capture forbids fail, but for threads in relaxed mode
thread_local int mode;
struct Config {
    dim3 grid, block;
    size_t lds;
    void *stream;
};
thread_local std::vector<Config> configs;
int result(int e) {
    if (e) last_error = e;
    return e;
}
void note(const std::string &s) {
    std::lock_guard<std::mutex> l(m);
    notes += s + "\n";
}
}  // namespace

extern "C" {
void fake_hip_set(int pinned_fails, int in_capture) {
    fail_pinned = pinned_fails;
    capturing = in_capture;
}
// the notes so far, and forgets them
const char *fake_hip_notes() {
    static std::string out;
    std::lock_guard<std::mutex> l(m);
    out.swap(notes);
    notes.clear();
    return out.c_str();
}

void **__hipRegisterFatBinary(const void *) {
    static void *h;
    return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) {
    kernels[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream) {
    configs.push_back({grid, block, lds, stream});
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream) {
    const Config c = configs.back();
    configs.pop_back();
    *grid = c.grid, *block = c.block, *lds = c.lds, *stream = c.stream;
    return 0;
}
int hipLaunchKernel(const void *host, dim3 grid, dim3 block, void **args, size_t lds, void *) {
    const std::string &name = kernels[host];
    note(name + " " + std::to_string(grid.x) + " " + std::to_string(block.x) + " " + std::to_string(lds));
    // the reduction's result: a number of its own for every launch
    if (name.find("k_reduce") != std::string::npos) {
        static double n;
        double *out = *(double **)args[2];
        std::lock_guard<std::mutex> l(m);
        n += 1;
        for (int i = 0; i < 8; ++i) out[i] = i == 5 || i == 6 ? 0.0 : n;
    }
    return 0;
}

int hipGetLastError() {
    const int e = last_error;
    last_error = 0;
    return e;
}
const char *hipGetErrorString(int e) { return e ? "fake error" : "no error"; }
int hipGetDevice(int *d) {
    *d = 0;
    return 0;
}
int hipGetSymbolAddress(void **p, const void *) {
    static void *mem = calloc(1, 32 << 20);
    *p = mem;
    return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned) {
    note("hipHostMalloc " + std::to_string(n));
    if (capturing && mode != 2) return result(900);  // hipErrorStreamCaptureUnsupported
    if (fail_pinned) return result(2);               // hipErrorOutOfMemory
    *p = calloc(1, n);
    return 0;
}
int hipHostFree(void *p) {  // waits for the device
    note("hipHostFree");
    free(p);
    return 0;
}
int hipThreadExchangeStreamCaptureMode(int *to) {
    const int was = mode;
    mode = *to;
    *to = was;
    return 0;
}
int hipMemcpyAsync(void *to, const void *from, size_t n, int, void *) {
    memcpy(to, from, n);
    return 0;
}
int hipStreamSynchronize(void *) { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) {
    *s = calloc(1, 8);
    return 0;
}
int hipStreamDestroy(void *s) {
    free(s);
    return 0;
}
int hipStreamBeginCapture(void *, int) { return 0; }
int hipStreamEndCapture(void *, void **g) {
    *g = calloc(1, 8);
    return 0;
}
int hipGraphInstantiate(void **e, void *, void **, char *, size_t) {
    *e = calloc(1, 8);
    return 0;
}
int hipGraphLaunch(void *, void *) { return 0; }
int hipGraphDestroy(void *g) {
    free(g);
    return 0;
}
int hipGraphExecDestroy(void *e) {
    free(e);
    return 0;
}
}
