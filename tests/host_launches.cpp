// Host-side double of the HIP runtime: runs the library's C ABI without a
// device and records what it launches.  The executable defines the runtime
// functions the library imports, so its definitions take their place (link
// with -rdynamic); device pointers are never dereferenced by host code.
//
//   host_launches LIB < commands
//
//   gemm ENTRY LAYOUT M N K A_BLK B_BLK OUT KIND STREAM CAPTURING
//       one product (ENTRY gemm, ex, noalloc or pm) on fake operands; STREAM
//       a small integer (0: the null stream).  Prints "STATUS" and then, per
//       launch, " | kernel<...> grid block".
//   amax NUMEL STREAM CAPTURING
//   together THREADS REPS <one gemm or amax command>
//       the same call REPS times from each of THREADS host threads at once.
//       Prints "STATUS runs N split S": S of the N calls had another call's
//       launch between their own.
//
// A launch of 2^32 work-items or more in one dimension is refused, as the
// device runtime does.
#include <cxxabi.h>
#include <dlfcn.h>
#include <unistd.h>

#include <atomic>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <iostream>
#include <map>
#include <mutex>
#include <sstream>
#include <string>
#include <thread>
#include <vector>

struct dim3 {
    uint32_t x, y, z;
};

namespace {
struct Launch {
    int call;
    std::string text;
};
std::mutex g_mu;
std::map<const void*, std::string>* g_names;      // kernel stub -> name (filled while the library loads)
std::vector<Launch> g_launches;
std::atomic<int> g_calls{0};
thread_local int t_call = 0;
std::atomic<int> g_capturing{0};
std::atomic<uintptr_t> g_next{0x7000000000};
bool g_slow = false;                              // widen the gap between a call's launches

thread_local dim3 t_grid, t_block;
thread_local size_t t_shmem;
thread_local void* t_stream;

std::string kernel_name(const char* mangled) {
    int st = 0;
    char* d = abi::__cxa_demangle(mangled, nullptr, nullptr, &st);
    std::string s = st == 0 && d ? d : mangled;
    free(d);
    // the kernel and its template arguments, without scope and parameters
    size_t end = s.find('<');
    const size_t paren = s.find('(', s.find("anonymous namespace") == std::string::npos ? 0 : s.find(")::") + 3);
    if (end == std::string::npos || end > paren) end = paren;
    size_t start = s.rfind("::", end);
    start = start == std::string::npos ? 0 : start + 2;
    return s.substr(start, (paren == std::string::npos ? s.size() : paren) - start);
}
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* stub, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
    if (g_names == nullptr) g_names = new std::map<const void*, std::string>;
    (*g_names)[stub] = kernel_name(name);
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, void* stream) {
    t_grid = grid; t_block = block; t_shmem = shmem; t_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, void** stream) {
    *grid = t_grid; *block = t_block; *shmem = t_shmem; *stream = t_stream;
    return 0;
}
thread_local int t_error = 0;
int hipLaunchKernel(const void* stub, dim3 grid, dim3 block, void**, size_t, void*) {
    const uint64_t lim = (uint64_t)1 << 32;
    if ((uint64_t)grid.x * block.x >= lim || (uint64_t)grid.y * block.y >= lim || grid.x == 0)
        return t_error = 9;                       // invalid configuration
    {
        std::lock_guard<std::mutex> lock(g_mu);
        g_launches.push_back({t_call, (*g_names)[stub] + " " + std::to_string(grid.x) + " " + std::to_string(block.x)});
    }
    if (g_slow) usleep(300);
    return 0;
}
int hipGetLastError() {
    const int e = t_error;
    t_error = 0;
    return e;
}
int hipGetDevice(int* dev) { *dev = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }   // compute units
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 2; return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = reinterpret_cast<void*>((uintptr_t)0x5000000000); return 0; }
int hipMalloc(void** p, size_t bytes) {
    if (g_capturing) return t_error = 900;
    *p = reinterpret_cast<void*>(g_next.fetch_add((bytes + 0xFFF) & ~(size_t)0xFFF));
    return 0;
}
int hipStreamIsCapturing(void*, int* status) { *status = g_capturing; return 0; }
}

namespace {
void* g_lib;
template <typename F>
F sym(const char* name) {
    void* p = dlsym(g_lib, name);
    if (p == nullptr) { fprintf(stderr, "no %s\n", name); exit(2); }
    return reinterpret_cast<F>(p);
}

struct Call {
    std::string what, entry;
    int layout = 0, a_blk = 0, b_blk = 0, out = 0, kind = 0, capturing = 0;
    int64_t M = 0, N = 0, K = 0;
    uintptr_t stream = 0;

    int run() const {
        char* const f = reinterpret_cast<char*>((uintptr_t)0x100000);
        void* const s = reinterpret_cast<void*>(stream);
        if (what == "amax")
            return sym<int (*)(const void*, int64_t, void*, int, void*)>("ue5m3_amax_accumulate")(f, M, f, 1, s);
        if (entry == "ex")
            return sym<int (*)(int, int64_t, int64_t, int64_t, void*, void*, int, void*, void*, void*, int, void*, void*,
                               int, int, void*)>("ue5m3_gemm_ex")(layout, M, N, K, f, f, a_blk, f, f, f, b_blk, f, f,
                                                                  out, kind, s);
        if (entry == "pm")
            return sym<int (*)(int, int64_t, int64_t, int64_t, void*, void*, int, void*, void*, void*, int, void*, void*,
                               int, int, int, void*)>("ue5m3_gemm_pm")(layout, M, N, K, f, f, a_blk, f, f, f, b_blk, f,
                                                                       f, out, kind, 1024, s);
        return sym<int (*)(int, int64_t, int64_t, int64_t, void*, void*, int, void*, void*, void*, int, void*, void*, int,
                           void*)>(entry == "noalloc" ? "ue5m3_gemm_noalloc" : "ue5m3_gemm")(
            layout, M, N, K, f, f, a_blk, f, f, f, b_blk, f, f, out, s);
    }
};

bool parse(std::istream& in, Call& c) {
    if (!(in >> c.what)) return false;
    if (c.what == "amax") return (bool)(in >> c.M >> c.stream >> c.capturing);
    return c.what == "gemm" && (bool)(in >> c.entry >> c.layout >> c.M >> c.N >> c.K >> c.a_blk >> c.b_blk >> c.out >>
                                      c.kind >> c.stream >> c.capturing);
}
}  // namespace

int main(int argc, char** argv) {
    if (argc != 2) return 2;
    g_lib = dlopen(argv[1], RTLD_NOW);
    if (g_lib == nullptr) { fprintf(stderr, "%s\n", dlerror()); return 2; }
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        int threads = 0, reps = 0;
        if (line.rfind("together", 0) == 0) {
            std::string word;
            in >> word >> threads >> reps;
        }
        Call c;
        if (!parse(in, c)) { fprintf(stderr, "bad command: %s\n", line.c_str()); return 2; }
        g_launches.clear();
        g_capturing = c.capturing;
        if (threads == 0) {
            printf("%d", c.run());
            for (const auto& l : g_launches) printf(" | %s", l.text.c_str());
            printf("\n");
        } else {
            g_slow = true;
            std::atomic<int> status{0};
            std::vector<std::thread> ts;
            for (int t = 0; t < threads; ++t)
                ts.emplace_back([&] {
                    for (int r = 0; r < reps; ++r) {
                        t_call = ++g_calls;
                        const int st = c.run();
                        if (st != 0) status = st;
                    }
                });
            for (auto& t : ts) t.join();
            g_slow = false;
            std::map<int, std::pair<size_t, size_t>> span;   // call -> first and last launch
            std::map<int, size_t> count;
            for (size_t i = 0; i < g_launches.size(); ++i) {
                const int id = g_launches[i].call;
                if (count[id]++ == 0) span[id].first = i;
                span[id].second = i;
            }
            size_t split = 0;
            for (const auto& s : span) split += s.second.second - s.second.first + 1 != count[s.first];
            printf("%d runs %zu split %zu\n", (int)status, span.size(), split);
        }
        fflush(stdout);
    }
    return 0;
}
