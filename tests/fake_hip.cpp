/* The HIP runtime calls that liblgf.so makes, without a GPU: launches are
 * written to a log instead of run, device memory is an address and nothing
 * else, events and streams are always done.  Loaded with RTLD_GLOBAL before
 * liblgf.so it takes the place of the runtime, so the host side of the library
 * (which kernels it launches, in what order, what it waits for) can be looked
 * at on a machine without a GPU.
 *
 * The final sums of a lattice give the F and theta of fake_result(F, theta,
 * factor), theta times the factor after each of them.
 * The device has fake_memory(bytes) bytes free from now on.
 * hipEventElapsedTime gives 1 ms, or 0.5 ms where the last sweep launched has
 * the text of fake_fast(text) in its line. */
#include <cxxabi.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <vector>

struct Dim {
    uint32_t x, y, z;
};

namespace {
std::string text;            // the log, a line per call
std::map<const void *, std::string> kernels;
Dim cfg_grid, cfg_block;
size_t cfg_lds;
void *cfg_stream;
bool capturing = false;
double result[2] = {0.5, 1.0}, factor = 1.0;
uint64_t next_address = 1ull << 40, next_object = 1, free_bytes = 1ull << 50;
std::map<void *, uint64_t> sizes;
std::string fast, last_sweep;
size_t new_bytes = 0;
int own = 0;  // inside the stand-in, whose own strings do not count
struct Own {
    Own() { ++own; }
    ~Own() { --own; }
};
std::map<size_t, std::string> copied;  // the last host-to-device copy of a size

void line(const std::string &s)
{
    Own guard;
    text += s + "\n";
}
std::string num(const void *p) { return std::to_string((uintptr_t)p); }

// n 32-bit words of an argument
std::string words(const void *arg, int n)
{
    std::string s;
    for (int i = 0; i < n; ++i) {
        uint32_t w;
        std::memcpy(&w, (const char *)arg + 4 * i, 4);
        s += " " + std::to_string(w);
    }
    return s;
}
}  // namespace

// what the library's own C++ allocations take
void *operator new(size_t n)
{
    if (!own) new_bytes += n;
    if (void *p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

extern "C" {

const char *fake_log() { return text.c_str(); }
// the names of the library's kernels, one a line
const char *fake_kernels()
{
    static std::string all;
    all.clear();
    for (const auto &k : kernels) all += k.second + "\n";
    return all.c_str();
}
void fake_clear() { text.clear(); }
void fake_result(double F, double theta, double f) { result[0] = F; result[1] = theta; factor = f; }
void fake_memory(uint64_t bytes) { free_bytes = bytes; }
void fake_fast(const char *s) { fast = s; }
const char *fake_copied(size_t n) { return copied.count(n) ? copied[n].data() : nullptr; }
size_t fake_new_bytes() { const size_t n = new_bytes; new_bytes = 0; return n; }

void **__hipRegisterFatBinary(const void *) { static void *module = nullptr; return &module; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *,
                           void *, int *)
{
    int st = 0;
    char *d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    std::string s = d ? d : name;
    std::free(d);
    for (const char *prefix : {"void ", "lgf::", "(anonymous namespace)::"})
        if (s.compare(0, std::strlen(prefix), prefix) == 0) s.erase(0, std::strlen(prefix));
    const size_t open = s.find('(');  // "kernel<...>(arguments"
    if (open != std::string::npos) s.erase(open);
    for (char &c : s)
        if (c == ' ') c = '_';
    kernels[host] = s;
}
int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void *stream)
{
    cfg_grid = grid;
    cfg_block = block;
    cfg_lds = lds;
    cfg_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim *grid, Dim *block, size_t *lds, void **stream)
{
    *grid = cfg_grid;
    *block = cfg_block;
    *lds = cfg_lds;
    *stream = cfg_stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim grid, Dim block, void **args, size_t, void *)
{
    Own guard;
    const std::string &k = kernels[f];
    std::string s = std::string(capturing ? "record " : "launch ") + k + " grid " + std::to_string(grid.x) + " " +
                    std::to_string(grid.y) + " block " + std::to_string(block.x);
    const bool fixed = k.find("fixed_sweep_kernel") == 0;
    if (k.find("sweep_kernel") == 0 || k.find("sweep_coulomb_kernel") == 0) s += " order" + words(args[4], 1);
    else if (k.find("anneal_kernel") != std::string::npos) s += " order" + words(args[8], 1);
    else if (fixed) s += " order" + words(args[5], 14);  // the whole TileOrder
    if (fixed || k.find("sweep") == 0) last_sweep = s;
    if (!capturing && k.find("finish_measure_kernel") == 0) {
        std::memcpy(*(double **)args[3], result, sizeof result);
        result[1] *= factor;
    }
    if (!capturing && k.find("finish_coulomb_kernel") == 0) {
        for (uint32_t t = 0; t < grid.x; ++t) std::memcpy(*(double **)args[3] + 2 * t, result, sizeof result);
        result[1] *= factor;
    }
    line(s);
    return 0;
}

int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "error"; }
int hipGetSymbolAddress(void **p, const void *) { *p = (void *)0x1000; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 2; return 0; }

int hipMalloc(void **p, size_t n)
{
    Own guard;
    if (n > free_bytes) return 2;
    free_bytes -= n;
    *p = (void *)next_address;
    sizes[*p] = n;
    next_address += (n + 4095) / 4096 * 4096 + 4096;
    line("malloc " + num(*p) + " " + std::to_string(n));
    return 0;
}
int hipFree(void *p)
{
    Own guard;
    line("free " + num(p));
    if (sizes.count(p)) free_bytes += sizes[p];
    sizes.erase(p);
    return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned) { *p = std::calloc(1, n); return *p ? 0 : 2; }
int hipHostFree(void *p) { std::free(p); return 0; }
int hipMemcpyAsync(void *dst, const void *src, size_t n, int kind, void *)
{
    Own guard;
    line("copy " + std::to_string(n) + " kind " + std::to_string(kind));
    if (kind == 1) copied[n] = std::string((const char *)src, n);
    if (kind == 2) std::memset(dst, 0, n);
    return 0;
}

int hipStreamCreate(void **s) { *s = (void *)next_object++; return 0; }
int hipStreamDestroy(void *) { return 0; }
int hipStreamSynchronize(void *) { line("wait"); return 0; }
int hipEventCreate(void **e) { *e = (void *)next_object++; return 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *e, void *) { line("mark " + num(e)); return 0; }
int hipEventSynchronize(void *e) { line("wait"); (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *, void *)
{
    *ms = (!fast.empty() && last_sweep.find(fast) != std::string::npos) ? 0.5f : 1.0f;
    return 0;
}

int hipStreamBeginCapture(void *, int) { capturing = true; return 0; }
int hipStreamEndCapture(void *, void **g) { capturing = false; *g = (void *)next_object++; return 0; }
int hipGraphDestroy(void *) { return 0; }
int hipGraphInstantiate(void **e, void *, void *, char *, size_t)
{
    *e = (void *)next_object++;
    line("graph_new " + num(*e));
    return 0;
}
int hipGraphLaunch(void *e, void *) { line("graph_launch " + num(e)); return 0; }
int hipGraphExecDestroy(void *e) { line("graph_destroy " + num(e)); return 0; }

}  // extern "C"
