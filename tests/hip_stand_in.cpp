// A stand-in for the HIP calls that the library's host code makes, for tests
// without a GPU.  Loaded with RTLD_GLOBAL before libstencil.so, its symbols are
// the ones the library binds to.  Nothing runs on a device: launches are noted
// (on a capturing stream in its graph, and again at every launch of that
// graph), memory is host memory, and every handle is checked, so that a use
// after destruction, a second destruction, an unjoined capture or an event
// waited for before it was recorded ends the process with a message.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

namespace {

struct Dim3 {
    uint32_t x, y, z;
};
struct Launch {
    std::string name;
    Dim3 grid, block;
    const void* stream;
    unsigned char arg0[128];   // the first argument's first bytes (sweep descriptors only)
};
struct Graph {
    std::vector<Launch> work;
};
struct Capture {
    void* origin;
    Graph graph;
    std::set<void*> streams;         // streams in this capture
    std::map<void*, bool> pending;   // a forked stream's work is not joined yet
};
struct Event {
    bool recorded = false;
    Capture* capture = nullptr;
    void* stream = nullptr;
};

std::map<const void*, std::string> kernels;
std::map<const void*, size_t> vars;
std::map<const void*, void*> var_memory;
std::vector<Launch> noted;
std::set<void*> streams, blocks;
std::map<void*, Event> events;
std::set<Graph*> graphs, execs;
std::map<void*, Capture*> capturing;   // stream -> capture
int begun = 0, instantiated = 0, replayed = 0, syncs = 0;
std::string failing;   // the call that returns an error, once
int device = 0;        // the current device
std::set<std::pair<const void*, int>> large_lds;   // kernels allowed more than 64 KiB of LDS, by device

struct Config {
    Dim3 grid, block;
    size_t shared;
    void* stream;
};
thread_local std::vector<Config> configs;

[[noreturn]] void die(const char* what) {
    std::fprintf(stderr, "stand-in: %s\n", what);
    std::fflush(stderr);
    std::abort();
}

void check_stream(void* s) {
    if (s && !streams.count(s)) die("a stream that does not exist");
}

bool fails(const char* call) {
    if (failing != call) return false;
    failing.clear();
    return true;
}

void note(const Launch& l) {
    auto it = capturing.find(const_cast<void*>(l.stream));
    if (it == capturing.end()) {
        noted.push_back(l);
        return;
    }
    it->second->graph.work.push_back(l);
    if (l.stream != it->second->origin) it->second->pending[const_cast<void*>(l.stream)] = true;
}

}  // namespace

#define API extern "C" __attribute__((visibility("default")))

// ------------------------------------------------------------- the HIP calls
API void** __hipRegisterFatBinary(const void*) {
    static void* handle = nullptr;
    return &handle;
}
API void __hipUnregisterFatBinary(void**) {}
API void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                               int*) {
    kernels[host] = name;
}
API void __hipRegisterVar(void**, void* var, char*, char*, int, size_t size, int, int) { vars[var] = size; }
API int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void* stream) {
    configs.push_back({grid, block, shared, stream});
    return 0;
}
API int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shared, void** stream) {
    if (configs.empty()) die("no launch configuration");
    *grid = configs.back().grid;
    *block = configs.back().block;
    *shared = configs.back().shared;
    *stream = configs.back().stream;
    configs.pop_back();
    return 0;
}
API int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void** args, size_t shared, void* stream) {
    check_stream(stream);
    if (!kernels.count(f)) die("a kernel that was not registered");
    if (shared > 65536 && !large_lds.count({f, device})) die("more than 64 KiB of LDS, not enabled on this device");
    if (fails("hipLaunchKernel")) return 1;
    Launch l{kernels[f], grid, block, stream, {}};
    for (const char* swept : {"k_step2d", "k_march2d", "k_zbrickI", "k_zmarchI"})
        if (l.name.find(swept) != std::string::npos) std::memcpy(l.arg0, args[0], sizeof l.arg0);
    note(l);
    return 0;
}
API int hipModuleLaunchKernel(void*, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned, void*, void**,
                              void**) {
    die("module launches are not covered");
}
API int hipGetLastError() { return 0; }
API const char* hipGetErrorString(int) { return "stand-in error"; }
API int hipGetDevice(int* d) {
    *d = device;
    return 0;
}
API int hipDeviceGetAttribute(int* v, int, int) {
    *v = 256;
    return 0;
}
API int hipGetDevicePropertiesR0600(void*, int) { return 1; }
API int hipFuncSetAttribute(const void* f, int, int) {
    large_lds.insert({f, device});
    return 0;
}
API int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    *n = 8 >> device;   // a device holds half as many as the one before
    return 0;
}
API int hipDeviceSynchronize() {
    if (!capturing.empty()) die("hipDeviceSynchronize while a stream is capturing");
    syncs++;
    return 0;
}
API int hipMalloc(void** p, size_t n) {
    if (fails("hipMalloc")) return 2;
    *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
    blocks.insert(*p);
    return 0;
}
API int hipFree(void* p) {
    if (!blocks.erase(p)) die("hipFree of memory that is not allocated");
    std::free(p);
    return 0;
}
API int hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::calloc(1, n);
    return 0;
}
API int hipHostFree(void* p) {
    std::free(p);
    return 0;
}
API int hipMemcpy(void* d, const void* s, size_t n, int) {
    if (!capturing.empty()) die("hipMemcpy while a stream is capturing");
    std::memcpy(d, s, n);
    return 0;
}
API int hipMemcpyAsync(void*, const void*, size_t, int, void* s) {
    check_stream(s);
    return 0;
}
API int hipGetSymbolAddress(void** p, const void* symbol) {
    if (!vars.count(symbol)) die("a symbol that was not registered");
    void*& m = var_memory[symbol];
    if (!m) m = std::aligned_alloc(256, (vars[symbol] + 255) / 256 * 256);
    *p = m;
    return 0;
}
API int hipStreamCreateWithFlags(void** s, unsigned) {
    *s = std::malloc(1);
    streams.insert(*s);
    return 0;
}
API int hipStreamDestroy(void* s) {
    if (capturing.count(s)) die("a capturing stream destroyed");
    if (!streams.erase(s)) die("a stream destroyed twice");
    return 0;
}
API int hipStreamSynchronize(void* s) {
    check_stream(s);
    if (capturing.count(s)) return 900;
    syncs++;
    return 0;
}
API int hipStreamIsCapturing(void* s, int* status) {
    check_stream(s);
    *status = capturing.count(s) ? 1 : 0;
    return 0;
}
API int hipStreamBeginCapture(void* s, int) {
    check_stream(s);
    if (!s) return 1;
    if (capturing.count(s)) die("a capture begun twice on a stream");
    if (fails("hipStreamBeginCapture")) return 1;
    Capture* c = new Capture;
    c->origin = s;
    c->streams.insert(s);
    capturing[s] = c;
    begun++;
    return 0;
}
API int hipStreamEndCapture(void* s, Graph** out) {
    check_stream(s);
    *out = nullptr;
    auto it = capturing.find(s);
    if (it == capturing.end()) return 901;
    Capture* c = it->second;
    if (c->origin != s) die("a capture ended on another stream than its own");
    bool joined = true;
    for (auto& p : c->pending) joined &= !p.second;
    for (void* t : c->streams) capturing.erase(t);
    for (auto& e : events)
        if (e.second.capture == c) e.second.capture = nullptr, e.second.recorded = false;
    if (joined) {
        *out = new Graph(c->graph);
        graphs.insert(*out);
    }
    delete c;
    return joined ? 0 : 904;
}
API int hipStreamWaitEvent(void* s, void* e, unsigned) {
    check_stream(s);
    auto it = events.find(e);
    if (it == events.end()) die("an event that does not exist");
    if (!it->second.recorded) die("an event waited for before it was recorded");
    Capture* c = it->second.capture;
    auto in = capturing.find(s);
    if (c) {
        if (in != capturing.end() && in->second != c) die("two captures meet");
        c->streams.insert(s);
        capturing[s] = c;
        c->pending[it->second.stream] = false;
    } else if (in != capturing.end()) {
        die("a capturing stream waits for work outside its capture");
    }
    return 0;
}
static int event_create(void** e) {
    *e = std::malloc(1);
    events[*e] = Event{};
    return 0;
}
API int hipEventCreate(void** e) { return event_create(e); }
API int hipEventCreateWithFlags(void** e, unsigned) { return event_create(e); }
API int hipEventDestroy(void* e) {
    if (!events.erase(e)) die("an event destroyed twice");
    return 0;
}
API int hipEventRecord(void* e, void* s) {
    check_stream(s);
    auto it = events.find(e);
    if (it == events.end()) die("an event that does not exist");
    auto in = capturing.find(s);
    it->second = Event{true, in == capturing.end() ? nullptr : in->second, s};
    return 0;
}
API int hipEventSynchronize(void* e) {
    if (!events.count(e)) die("an event that does not exist");
    return 0;
}
API int hipEventElapsedTime(float* ms, void*, void*) {
    *ms = 1.f;
    return 0;
}
API int hipGraphInstantiate(Graph** x, Graph* g, void*, void*, size_t) {
    if (!graphs.count(g)) die("a graph that does not exist");
    if (fails("hipGraphInstantiate")) return 2;
    *x = new Graph(*g);
    execs.insert(*x);
    instantiated++;
    return 0;
}
API int hipGraphDestroy(Graph* g) {
    if (!graphs.erase(g)) die("a graph destroyed twice");
    delete g;
    return 0;
}
API int hipGraphExecDestroy(Graph* x) {
    if (!execs.erase(x)) die("an executable graph destroyed twice");
    delete x;
    return 0;
}
API int hipGraphLaunch(Graph* x, void* s) {
    check_stream(s);
    if (!execs.count(x)) die("an executable graph that does not exist");
    if (capturing.count(s)) die("a graph launched into a capture");
    for (const Launch& l : x->work) noted.push_back(l);
    replayed++;
    return 0;
}

// ------------------------------------------------------- what the tests read
API int stand_in_launches() { return (int)noted.size(); }
API const char* stand_in_name(int i) { return noted[(size_t)i].name.c_str(); }
API const void* stand_in_arg0(int i) { return noted[(size_t)i].arg0; }
API unsigned stand_in_grid(int i) { return noted[(size_t)i].grid.x; }
API void stand_in_device(int d) { device = d; }
API void stand_in_clear() { noted.clear(); }
API void stand_in_fail(const char* call) { failing = call; }
// captures begun, graphs instantiated, graphs launched, synchronisations;
// alive: executable graphs, graphs, events, streams, allocations
API void stand_in_counts(int* out) {
    const int c[9] = {begun,        instantiated,       replayed,           syncs,           (int)execs.size(),
                      (int)graphs.size(), (int)events.size(), (int)streams.size(), (int)blocks.size()};
    std::memcpy(out, c, sizeof c);
}
