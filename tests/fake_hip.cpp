// A HIP runtime without a GPU for host-side tests: device memory is host
// memory with checked bounds, kernels are reported instead of run, and every
// launch knows which earlier ones it is ordered behind (streams, events and
// synchronizations), so that a race between two launches, a copy out of its
// block or a launch the hardware cannot take shows on the CPU.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>

using Set = std::set<int>;
using Callback = void (*)(int index, const char* kernel, uint64_t grid, uint64_t block, void** args);

namespace {

enum { OK = 0, INVALID_VALUE = 1, OUT_OF_MEMORY = 2, INVALID_CONFIG = 9, CAPTURE_UNSUPPORTED = 900 };

std::map<char*, size_t> blocks;             // device allocations
std::map<const void*, std::string> names;   // kernel handle -> device name
std::map<void*, Set> done;                  // launches a stream's next one is ordered behind
std::map<void*, Set> marks;                 // the same, at an event
std::map<int, Set> before;
std::map<void*, int> capture;               // capturing stream -> mode (0 global, 1 thread, 2 relaxed)
Set all;
Callback callback = nullptr;
int bad_copies = 0, last_error = 0, frees = 0, launches = 0;
uintptr_t handles = 0x1000;

int fail(int e)
{
    last_error = e;
    return e;
}

bool inside(const void* p, size_t n)
{
    char* c = static_cast<char*>(const_cast<void*>(p));
    auto it = blocks.upper_bound(c);
    if (it == blocks.begin()) return false;
    --it;
    return c + n <= it->first + it->second;
}

// An unsafe call (one that may synchronize) while a capture forbids it.
bool forbidden()
{
    for (const auto& c : capture)
        if (c.second != 2) return true;
    return false;
}

int copy(void* dst, const void* src, size_t n, int kind)
{
    if ((kind == 1 && !inside(dst, n)) || (kind == 2 && !inside(src, n))) {
        ++bad_copies;
        return fail(INVALID_VALUE);
    }
    std::memcpy(dst, src, n);
    return OK;
}

void* handle() { return reinterpret_cast<void*>(handles += 16); }

struct Dim {
    uint32_t x, y, z;
};

}  // namespace

extern "C" {

void fake_on_launch(Callback f) { callback = f; }
int fake_ordered(int a, int b) { return (int)before[b].count(a); }   // a ends before b begins
int fake_bad_copies() { return bad_copies; }
int fake_frees() { return frees; }
int fake_blocks() { return (int)blocks.size(); }
void* fake_stream() { return handle(); }
void fake_capture(void* s, int mode)
{
    if (mode < 0) capture.erase(s);
    else capture[s] = mode;
}

void** __hipRegisterFatBinary(const void*) { return reinterpret_cast<void**>(handle()); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    names[f] = name;
}
static Dim cfg_grid, cfg_block;
static size_t cfg_lds;
static void* cfg_stream;
int __hipPushCallConfiguration(Dim g, Dim b, size_t lds, void* s)
{
    cfg_grid = g;
    cfg_block = b;
    cfg_lds = lds;
    cfg_stream = s;
    return OK;
}
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* lds, void** s)
{
    *g = cfg_grid;
    *b = cfg_block;
    *lds = cfg_lds;
    *s = cfg_stream;
    return OK;
}
int hipLaunchKernel(const void* f, Dim g, Dim b, void** args, size_t, void* s)
{
    if ((uint64_t)g.x * b.x >= 1ull << 32) return fail(INVALID_CONFIG);   // work-items of one dimension: 32 bits
    const int i = launches++;
    before[i] = done[s];
    done[s].insert(i);
    all.insert(i);
    if (callback) callback(i, names[f].c_str(), g.x, b.x, args);
    return OK;
}

int hipMalloc(void** p, size_t n)
{
    if (forbidden()) return fail(CAPTURE_UNSUPPORTED);
    *p = std::calloc(1, n + 64);
    if (!*p) return fail(OUT_OF_MEMORY);
    blocks[static_cast<char*>(*p)] = n;
    return OK;
}
int hipFree(void* p)
{
    if (forbidden()) return fail(CAPTURE_UNSUPPORTED);
    if (p) {
        blocks.erase(static_cast<char*>(p));
        std::free(p);
        ++frees;
    }
    return OK;
}
int hipHostMalloc(void** p, size_t n, unsigned)
{
    *p = std::calloc(1, n);
    return OK;
}
int hipHostFree(void* p)
{
    std::free(p);
    return OK;
}
int hipMemcpy(void* d, const void* s, size_t n, int kind) { return forbidden() ? fail(CAPTURE_UNSUPPORTED) : copy(d, s, n, kind); }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void*) { return copy(d, s, n, kind); }
int hipMemset(void* d, int v, size_t n)
{
    if (!inside(d, n)) return fail(INVALID_VALUE);
    std::memset(d, v, n);
    return OK;
}

int hipStreamCreateWithFlags(void** s, unsigned)
{
    *s = handle();
    return OK;
}
int hipStreamDestroy(void*) { return OK; }
int hipStreamSynchronize(void* s)
{
    if (capture.count(s)) return fail(CAPTURE_UNSUPPORTED);
    for (auto& d : done) d.second.insert(done[s].begin(), done[s].end());
    return OK;
}
int hipDeviceSynchronize()
{
    if (!capture.empty()) return fail(CAPTURE_UNSUPPORTED);
    for (auto& d : done) d.second = all;
    return OK;
}
int hipStreamIsCapturing(void* s, int* status)
{
    *status = capture.count(s) ? 1 : 0;
    return OK;
}
int hipStreamWaitEvent(void* s, void* e, unsigned)
{
    done[s].insert(marks[e].begin(), marks[e].end());
    return OK;
}
// A captured graph's launches: the ones before the capture do not count as
// ordered behind by the stream alone, only through edges of the graph.
int hipStreamBeginCapture(void* s, int mode)
{
    capture[s] = mode;
    done.clear();
    marks.clear();
    return OK;
}
int hipStreamEndCapture(void* s, void** graph)
{
    capture.erase(s);
    *graph = handle();
    return OK;
}
int hipGraphInstantiate(void** x, void*, void*, char*, size_t)
{
    *x = handle();
    return OK;
}
int hipGraphLaunch(void*, void*) { return OK; }
int hipGraphDestroy(void*) { return OK; }
int hipGraphExecDestroy(void*) { return OK; }

int hipEventCreate(void** e)
{
    *e = handle();
    return OK;
}
int hipEventCreateWithFlags(void** e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void*) { return OK; }
int hipEventRecord(void* e, void* s)
{
    marks[e] = done[s];
    return OK;
}
int hipEventSynchronize(void*) { return OK; }
int hipEventElapsedTime(float* ms, void*, void*)
{
    *ms = 1.0f;
    return OK;
}

int hipGetDevice(int* d)
{
    *d = 0;
    return OK;
}
int hipSetDevice(int) { return OK; }
int hipDeviceGetAttribute(int* v, int, int)
{
    *v = 256;
    return OK;
}
int hipFuncSetAttribute(const void*, int, int) { return OK; }
int hipGetSymbolAddress(void** p, const void*)
{
    static char memory[1 << 20];
    *p = memory;
    return OK;
}
int hipGetLastError()
{
    const int e = last_error;
    last_error = OK;
    return e;
}
const char* hipGetErrorString(int) { return "fake HIP error"; }

}  // extern "C"
