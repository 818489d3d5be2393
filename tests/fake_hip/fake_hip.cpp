// A HIP runtime without a GPU, for tests of the library's host code: the library is loaded with these symbols in front
// of the real ones.  Memory is host memory (reserved, touched on use), copies are memcpy, kernels do not run - their
// launches are checked against the documented limits and logged.  A few kernels of the M-step can be imitated, and a
// call can be made to fail.  Two devices; objects belong to the one that was current when they were made.  Accesses to the
// buffers of the chunks that are streamed are followed: two of them, one a write, that neither streams nor events nor waits put in order
// are counted as a race.
#include <malloc.h>
#include <sys/mman.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

// Host memory in use by way of operator new, the library's included, and what it may grow to.
static std::atomic<int64_t> new_bytes{0}, new_limit{INT64_MAX};
void *operator new(size_t n) {
    void *p = new_bytes.load() + (int64_t)n <= new_limit.load() ? malloc(n ? n : 1) : nullptr;
    if (!p) throw std::bad_alloc();
    new_bytes += (int64_t)malloc_usable_size(p);
    return p;
}
void operator delete(void *p) noexcept { if (p) new_bytes -= (int64_t)malloc_usable_size(p); free(p); }
void operator delete(void *p, size_t) noexcept { operator delete(p); }

namespace {
enum { kOk = 0, kInvalidValue = 1, kOutOfMemory = 2, kInvalidConfiguration = 9, kInvalidDevice = 101, kInvalidHandle = 400 };
struct Dim { uint32_t x, y, z; };
using Clock = std::map<int, int64_t>;              // of every stream, how many of its operations lie before
struct Object { int device; int64_t launches; int id; bool blocking; Clock seen; };   // (an event: launches in front of it)
struct Launch { std::string name; Dim grid, block; };
struct Config { Dim grid, block; size_t lds; Object *stream; };

std::mutex mu;
std::map<void *, size_t> blocks;
std::map<const void *, std::string> kernels;
std::map<const void *, size_t> vars;
std::map<const void *, void *> var_mem;
std::vector<Launch> launches;
std::map<std::string, int64_t> calls;
int64_t mallocs_on[2] = {};
std::string fail_name;
int fail_at = 0, imitate = 0, cus = 256;
int64_t host_bytes = 0;
int last_stream = 0;
std::map<Object *, bool> streams;
Clock host_seen;
struct Access { int stream; int64_t at; std::string what; };
struct Accesses { Access write; std::vector<Access> reads; };
std::map<void *, Accesses> accesses;
int64_t races = 0;
std::string first_race;
thread_local int device = 0, last_error = 0;
thread_local std::vector<Config> configs;

// the call that fake_fail() chose fails
bool fails(const std::string &name) {
    std::lock_guard<std::mutex> lock(mu);
    calls[name]++;
    return fail_at > 0 && name.find(fail_name) != std::string::npos && --fail_at == 0;
}
int result(int e) { if (e) last_error = e; return e; }
void *reserve(size_t bytes) {
    void *p = mmap(nullptr, bytes ? bytes : 1, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == MAP_FAILED) return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    blocks[p] = bytes ? bytes : 1;
    return p;
}
int release(void *p) {
    if (!p) return kOk;
    std::lock_guard<std::mutex> lock(mu);
    auto it = blocks.find(p);
    if (it == blocks.end()) return kInvalidValue;
    munmap(p, it->second);
    blocks.erase(it);
    accesses.erase(p);
    return kOk;
}
template <typename T> T arg(void **args, int i) { T v; memcpy(&v, args[i], sizeof(v)); return v; }

// ---- order of accesses (mu is held) ----
void join(Clock &into, const Clock &from) { for (const auto &c : from) into[c.first] = std::max(into[c.first], c.second); }
// an operation on stream s, or (null) one of the host: its clock
const Clock &begin_op(Object *s) {
    if (!s) {                          // the null stream waits for the streams that do not opt out, and the host for it
        for (auto &o : streams) if (o.first->blocking) join(host_seen, o.first->seen);
        host_seen[0]++;
        return host_seen;
    }
    join(s->seen, host_seen);
    s->seen[s->id]++;
    return s->seen;
}
void touch(Object *s, const Clock &now, const void *p, bool write, const std::string &what) {
    auto it = blocks.upper_bound(const_cast<void *>(p));
    if (it == blocks.begin()) return;
    --it;
    if ((const char *)p >= (const char *)it->first + it->second) return;
    Accesses &a = accesses[it->first];
    auto before = [&](const Access &x) {
        const auto c = now.find(x.stream);
        if (x.at == 0 || (c != now.end() && c->second >= x.at)) return;
        if (!races++) first_race = what + " after " + x.what;
    };
    before(a.write);
    const int id = s ? s->id : 0;
    const Access mine{id, now.at(id), what};
    if (!write) { a.reads.push_back(mine); return; }
    for (const Access &x : a.reads) before(x);
    a.write = mine;
    a.reads.clear();
}
// what kernels read and write of the buffers of chunks
void follow(Object *s, const std::string &name, void **a) {
    auto is = [&](const char *n) { return name.find(n) != std::string::npos; };
    const Clock &now = begin_op(s);
    auto reads = [&](const void *p) { if (p) touch(s, now, p, false, name); };
    auto writes = [&](const void *p) { if (p) touch(s, now, p, true, name); };
    if (is("expand_tok_doc_kernel")) { reads(arg<void *>(a, 0)); writes(arg<void *>(a, 5)); }
    else if (is("scatter_zwm_kernel")) { reads(arg<void *>(a, 1)); writes(arg<void *>(a, 3)); }
    else if (is("fill_zwm_kernel")) { reads(arg<void *>(a, 1)); reads(arg<void *>(a, 2)); }
    else if (is("init_z_kernel")) writes(arg<void *>(a, 0));
    else if (is("count_dz_kernel")) reads(((void *const *)a[0])[2]);   // SegGroup: list, ptr, z
    else if (is("estep_kernel")) {     // EStepParams: tiles, tok_doc, tok_t, docrec, cd_rows, four sizes, phi, l3, l3_64, sumphi, z
        void *const *p = (void *const *)a[0];
        reads(p[1]); reads(p[2]);
        if (is("estep_kernelILi0E")) writes(p[11]);
    }
}

// what the M-step's accumulators hold: B, the topic totals
struct VzItem { int32_t row, count; int64_t begin; };
struct PhiRow { int32_t word, count; int64_t begin; };
template <typename Z> void count_slabs(Dim grid, void **a) {
    const Z *z = arg<const Z *>(a, 0), *z_wm = arg<const Z *>(a, 6);
    const int64_t T = arg<int64_t>(a, 1), per_block = arg<int64_t>(a, 2);
    const int n_tot = arg<int>(a, 3), Kpad = arg<int>(a, 9);
    for (int b = 0; b < (int)grid.x; b++) {
        if (b < n_tot) {
            for (int64_t t = b * per_block; t < std::min(T, (b + 1) * per_block); t++) arg<unsigned long long *>(a, 4)[z[t]]++;
        } else {
            const VzItem it = arg<const VzItem *>(a, 5)[b - n_tot];
            for (int64_t t = it.begin; t < it.begin + it.count; t++) arg<int32_t *>(a, 7)[(size_t)it.row * Kpad + z_wm[t]]++;
        }
    }
}
void run(const std::string &name, Dim grid, void **a) {
    auto is = [&](const char *s) { return name.find(s) != std::string::npos; };
    if (is("fill_u32_kernel")) std::fill_n(arg<uint32_t *>(a, 0), arg<size_t>(a, 2), arg<uint32_t>(a, 1));
    else if (is("count_slabs_kernelIt")) count_slabs<uint16_t>(grid, a);
    else if (is("count_slabs_kernelIi")) count_slabs<int32_t>(grid, a);
    else if (is("denominators_kernel")) {
        unsigned long long *acc = arg<unsigned long long *>(a, 0), *ck = arg<unsigned long long *>(a, 1);
        for (int k = 0; k < arg<int>(a, 3); k++) { ck[k] = acc[k]; acc[k] = 0; }
    } else if (is("phi_tree_kernel")) {
        const int Kpad = arg<int>(a, 8);
        for (uint32_t r = 0; r < grid.x; r++)
            if (arg<const PhiRow *>(a, 0)[r].count < 0) memset(arg<int32_t *>(a, 2) + (size_t)r * Kpad, 0, sizeof(int32_t) * Kpad);
    }
}
}  // namespace

extern "C" {
// ---- for the tests ----
void fake_fail(const char *name, int nth) { std::lock_guard<std::mutex> lock(mu); fail_name = name; fail_at = nth; }   // the nth call (launch) whose name contains `name`
int fake_fail_pending() { std::lock_guard<std::mutex> lock(mu); return fail_at; }
void fake_imitate(int on) { imitate = on; }
void fake_cus(int n) { cus = n; }
int64_t fake_races(char *first, int64_t size) {   // accesses to buffers of chunks that nothing puts in order; the first one's names
    std::lock_guard<std::mutex> lock(mu);
    if (size) { strncpy(first, first_race.c_str(), (size_t)size - 1); first[size - 1] = 0; }
    return races;
}
void fake_clear() { std::lock_guard<std::mutex> lock(mu); launches.clear(); calls.clear(); host_bytes = 0; mallocs_on[0] = mallocs_on[1] = 0; }
int64_t fake_mallocs_on(int d) { std::lock_guard<std::mutex> lock(mu); return mallocs_on[d]; }   // of device memory, with device d current
void fake_new_limit(int64_t bytes) { new_limit = bytes < 0 ? INT64_MAX : new_bytes + bytes; }   // operator new: so many bytes more than now
int64_t fake_host_bytes() { return host_bytes; }   // of pinned memory asked for
int64_t fake_calls(const char *name) { std::lock_guard<std::mutex> lock(mu); return calls[name]; }   // of those that can be made to fail
int64_t fake_launches(const char *name, uint64_t *most_threads) {   // launches of kernels whose name contains `name`
    std::lock_guard<std::mutex> lock(mu);
    int64_t n = 0;
    *most_threads = 0;
    for (const Launch &l : launches)
        if (l.name.find(name) != std::string::npos) { n++; *most_threads = std::max(*most_threads, (uint64_t)l.grid.x * l.block.x); }
    return n;
}
uint64_t fake_blocks(const char *name) {   // workgroups of all of them
    std::lock_guard<std::mutex> lock(mu);
    uint64_t n = 0;
    for (const Launch &l : launches) if (l.name.find(name) != std::string::npos) n += (uint64_t)l.grid.x * l.grid.y;
    return n;
}
int fake_block(const char *name) {   // threads per workgroup of the last of them
    std::lock_guard<std::mutex> lock(mu);
    int n = 0;
    for (const Launch &l : launches) if (l.name.find(name) != std::string::npos) n = (int)l.block.x;
    return n;
}

// ---- the runtime ----
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { kernels[host] = name; }
void __hipRegisterVar(void **, void *var, char *, char *, int, size_t size, int, int) { vars[var] = size; }
int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, Object *stream) { configs.push_back({grid, block, lds, stream}); return kOk; }
int __hipPopCallConfiguration(Dim *grid, Dim *block, size_t *lds, Object **stream) {
    const Config c = configs.back();
    configs.pop_back();
    *grid = c.grid; *block = c.block; *lds = c.lds; *stream = c.stream;
    return kOk;
}
int hipLaunchKernel(const void *fn, Dim grid, Dim block, void **args, size_t lds, Object *s) {
    const std::string name = kernels[fn];
    if (fails(name)) return result(kOutOfMemory);
    // threads per grid dimension below 2^32, at most 1,024 per workgroup, at least one
    if (!grid.x || !grid.y || !grid.z || !block.x || (uint64_t)block.x * block.y * block.z > 1024 || lds > 160 * 1024 ||
        (uint64_t)grid.x * block.x >> 32 || (uint64_t)grid.y * block.y >> 32) return result(kInvalidConfiguration);
    { std::lock_guard<std::mutex> lock(mu); launches.push_back({name, grid, block}); follow(s, name, args); }
    if (imitate) run(name, grid, args);
    return kOk;
}
int hipGetLastError() { const int e = last_error; last_error = kOk; return e; }
const char *hipGetErrorString(int) { return "error of the stand-in runtime"; }
int hipGetDeviceCount(int *n) { *n = 2; return kOk; }
int hipGetDevice(int *d) { *d = device; return kOk; }
int hipSetDevice(int d) { if (d < 0 || d > 1) return result(kInvalidDevice); device = d; return kOk; }
int hipDeviceGetAttribute(int *v, int what, int) { *v = what == 63 ? cus : 160 * 1024; return kOk; }   // CUs; LDS of one
int hipFuncGetAttributes(void *attr, const void *) { memset(attr, 0, 56); return kOk; }
int hipFuncSetAttribute(const void *, int, int) { return kOk; }
int hipGetSymbolAddress(void **p, const void *var) {
    if (!vars.count(var)) return result(kInvalidValue);
    if (!var_mem[var]) var_mem[var] = reserve(vars[var]);
    *p = var_mem[var];
    return kOk;
}
int hipMemGetInfo(size_t *f, size_t *t) { *f = *t = (size_t)288 << 30; return kOk; }
int hipMalloc(void **p, size_t n) {
    if (fails("hipMalloc")) return result(kOutOfMemory);
    { std::lock_guard<std::mutex> lock(mu); mallocs_on[device]++; }
    *p = reserve(n);
    return *p ? kOk : result(kOutOfMemory);
}
int hipFree(void *p) { return result(release(p)); }
int hipHostMalloc(void **p, size_t n, unsigned) { if (fails("hipHostMalloc")) return result(kOutOfMemory); host_bytes += (int64_t)n; *p = reserve(n); return *p ? kOk : result(kOutOfMemory); }
int hipHostFree(void *p) { return result(release(p)); }
static void copy(void *d, const void *m, size_t n, Object *s) {
    std::lock_guard<std::mutex> lock(mu);
    const Clock &now = begin_op(s);
    if (n) { touch(s, now, m, false, "a copy"); touch(s, now, d, true, "a copy"); }
    memcpy(d, m, n);
}
int hipMemcpy(void *d, const void *m, size_t n, int) { if (fails("hipMemcpy:")) return result(kInvalidValue); copy(d, m, n, nullptr); return kOk; }
int hipMemcpyAsync(void *d, const void *m, size_t n, int, Object *s) { if (fails("hipMemcpyAsync")) return result(kInvalidValue); copy(d, m, n, s); return kOk; }
int hipMemsetAsync(void *d, int v, size_t n, Object *) { memset(d, v, n); return kOk; }
static Object *new_stream(bool blocking) {
    std::lock_guard<std::mutex> lock(mu);
    Object *s = new Object{device, 0, ++last_stream, blocking, {}};
    streams[s] = true;
    return s;
}
int hipStreamCreate(Object **s) { if (fails("hipStreamCreate")) return result(kOutOfMemory); *s = new_stream(true); return kOk; }
int hipStreamCreateWithFlags(Object **s, unsigned flags) { if (fails("hipStreamCreate")) return result(kOutOfMemory); *s = new_stream(!(flags & 1)); return kOk; }
int hipStreamDestroy(Object *s) { { std::lock_guard<std::mutex> lock(mu); streams.erase(s); } delete s; return kOk; }
int hipStreamSynchronize(Object *s) { std::lock_guard<std::mutex> lock(mu); if (s) join(host_seen, s->seen); return kOk; }
int hipStreamWaitEvent(Object *s, Object *e, unsigned) {
    if (fails("hipStreamWaitEvent")) return result(kInvalidValue);
    std::lock_guard<std::mutex> lock(mu);
    if (s) join(s->seen, e->seen);
    return kOk;
}
int hipEventCreate(Object **e) { if (fails("hipEventCreate")) return result(kOutOfMemory); *e = new Object{device, 0, 0, false, {}}; return kOk; }
int hipEventCreateWithFlags(Object **e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(Object *e) { delete e; return kOk; }
int hipEventRecord(Object *e, Object *s) {   // both have to belong to one device
    if (fails("hipEventRecord")) return result(kInvalidValue);
    { std::lock_guard<std::mutex> lock(mu); e->launches = (int64_t)launches.size(); if (s) { join(s->seen, host_seen); e->seen = s->seen; } }
    return e->device == (s ? s->device : device) ? kOk : result(kInvalidHandle);
}
int hipEventSynchronize(Object *e) { std::lock_guard<std::mutex> lock(mu); join(host_seen, e->seen); return kOk; }
int hipEventElapsedTime(float *ms, Object *a, Object *b) { *ms = (float)(b->launches - a->launches); return kOk; }   // a launch takes a millisecond
}
