// The library's host path on a stub of the HIP runtime (no GPU).  This
// program defines the runtime functions that libswe_hip.so calls, so that
// they are taken instead of the installed ones: device memory is host
// memory, copies happen at once, kernels are only recorded.  What the stub
// does keep is what the host path has to get right: which stream an operation
// was queued on (hipStreamPerThread names another stream in every thread),
// what has been waited for, which device is current, and what memory was
// asked for.  The two kernels that carry fields between device and pinned
// memory are carried out (their arguments are the pointers and sizes of
// XferFields in swe_xfer.hpp), so that a state can be read back.
//
//   host_runtime <scenario>      exit code 0: as it should be
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>

#include <dlfcn.h>
#include <unistd.h>

#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <future>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "../include/swe.h"

// ---------------------------------------------------------------- the stub

namespace {

struct Stream {
    int device = 0;
    bool per_thread = false, blocked = false, capturing = false;
    long long queued = 0, done = 0, work = 0, piece = 0;   // last operations of either kind
};
struct Event {
    int device = 0;
    Stream* on = nullptr;
    long long seq = 0;
};

std::mutex mu;
std::condition_variable cv;
thread_local int current_device = 0;
thread_local Stream* thread_stream = nullptr;
std::vector<Stream*> streams;
int violations = 0;               // operations queued without waiting for another thread's stream
bool no_pinned = false;           // hipHostMalloc fails
std::map<void*, size_t> device_mem, pinned_mem;
size_t device_bytes = 0, pinned_bytes = 0;
long long launches = 0;

Stream* make_stream(bool per_thread) {
    Stream* s = new Stream;
    s->device = current_device;
    s->per_thread = per_thread;
    streams.push_back(s);
    return s;
}
// (mu held)
Stream* stream_of(hipStream_t st) {
    static Stream* null_stream = make_stream(false);
    if (!st) return null_stream;
    if (st != hipStreamPerThread) return reinterpret_cast<Stream*>(st);
    if (!thread_stream) thread_stream = make_stream(true);
    return thread_stream;
}
// Pieces of one transfer may run beside each other on several threads'
// streams; everything else needs the other threads' operations to be done.
void queue(hipStream_t st, bool piece) {
    std::lock_guard<std::mutex> lk(mu);
    Stream* s = stream_of(st);
    if (s->capturing) return;
    if (s->per_thread)
        for (Stream* o : streams)
            if (o != s && o->per_thread && (o->work > o->done || (!piece && o->piece > o->done))) ++violations;
    ++s->queued;
    (piece ? s->piece : s->work) = s->queued;
}
// Wait until the operations of s up to `seq` are done; work takes a while.
void wait_done(std::unique_lock<std::mutex>& lk, Stream* s, long long seq) {
    if (s->work > s->done && seq >= s->work) {
        lk.unlock();
        std::this_thread::sleep_for(std::chrono::milliseconds(5));
        lk.lock();
    }
    cv.wait(lk, [&] { return !s->blocked; });
    if (s->done < seq) s->done = seq;
}
void block(hipStream_t st, bool on) {
    std::lock_guard<std::mutex> lk(mu);
    reinterpret_cast<Stream*>(st)->blocked = on;
    cv.notify_all();
}
hipError_t allocate(std::map<void*, size_t>& of, size_t& bytes, void** p, size_t n) {
    std::lock_guard<std::mutex> lk(mu);
    *p = calloc(1, n ? n : 1);
    of[*p] = n;
    bytes += n;
    return hipSuccess;
}
void wait_for_all() {   // what freeing memory does
    std::unique_lock<std::mutex> lk(mu);
    for (Stream* s : std::vector<Stream*>(streams)) cv.wait(lk, [&] { return !s->blocked; });
}
hipError_t release(std::map<void*, size_t>& of, size_t& bytes, void* p) {
    wait_for_all();
    std::lock_guard<std::mutex> lk(mu);
    auto it = of.find(p);
    if (it == of.end()) return hipErrorInvalidValue;
    bytes -= it->second;
    of.erase(it);
    free(p);
    return hipSuccess;
}

// k_export / k_import<real, N>: a[q], b[q] per field, then host[q]; the
// stub's grids are in layer 0, buffer a
void carry(const std::string& name, unsigned fields, void** args) {
    const size_t size = name.find("portIf") != std::string::npos ? 4 : 8, N = name.find("Li3E") != std::string::npos ? 3 : 1;
    char* const* const f = static_cast<char* const*>(args[0]);
    if (name.find("k_import") != std::string::npos) {
        const size_t first = *static_cast<size_t*>(args[1]), cnt = *static_cast<size_t*>(args[2]);
        for (unsigned q = 0; q < fields; ++q)
            for (int k = 0; k < 2; ++k) memcpy(f[2 * q + k] + first * size, f[2 * N + q], cnt * size);
        return;
    }
    const size_t pitch = *static_cast<int*>(args[2]), x0 = *static_cast<int*>(args[3]), y0 = *static_cast<int*>(args[4]),
                 w = *static_cast<int*>(args[5]), first = *static_cast<size_t*>(args[6]), cnt = *static_cast<size_t*>(args[7]);
    for (unsigned q = 0; q < fields; ++q)
        for (size_t k = 0; k < cnt; ++k)
            memcpy(f[2 * N + q] + k * size, f[2 * q] + ((y0 + (first + k) / w) * pitch + x0 + (first + k) % w) * size, size);
}

thread_local bool no_memory = false;   // operator new throws in this thread, but for the stub's own
struct StubsOwn {
    const bool was = no_memory;
    StubsOwn() { no_memory = false; }
    ~StubsOwn() { no_memory = was; }
};

struct Config { dim3 grid, block; size_t shared; hipStream_t stream; };
thread_local std::vector<Config> configs;

}  // namespace

void* operator new(size_t n) {
    void* p = no_memory ? nullptr : malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

extern "C" {

hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
    const StubsOwn own;
    configs.push_back({grid, block, shared, stream});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
    const Config c = configs.back();
    configs.pop_back();
    *grid = c.grid; *block = c.block; *shared = c.shared; *stream = c.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t st) {
    const StubsOwn own;
    Dl_info info;
    const std::string name = dladdr(f, &info) && info.dli_sname ? info.dli_sname : "";
    const bool piece = name.find("k_export") != std::string::npos || name.find("k_import") != std::string::npos ||
                       name.find("k_crops_in") != std::string::npos;
    queue(st, piece);
    if (piece && name.find("port") != std::string::npos) carry(name, grid.y, args);
    std::lock_guard<std::mutex> lk(mu);
    ++launches;
    return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void* f, dim3 g, dim3 b, void** a, size_t s, hipStream_t st, hipEvent_t,
                              hipEvent_t, int) {
    return hipLaunchKernel(f, g, b, a, s, st);
}
hipError_t hipMalloc(void** p, size_t n) { return allocate(device_mem, device_bytes, p, n); }
hipError_t hipFree(void* p) { return p ? release(device_mem, device_bytes, p) : hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    if (no_pinned) return hipErrorOutOfMemory;
    return allocate(pinned_mem, pinned_bytes, p, n);
}
hipError_t hipHostFree(void* p) { return p ? release(pinned_mem, pinned_bytes, p) : hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
    queue(st, false);
    memmove(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    memmove(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, hipMemcpyKind,
                            hipStream_t st) {
    queue(st, false);
    for (size_t k = 0; k < h; ++k) memmove((char*)d + k * dp, (const char*)s + k * sp, w);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) {
    queue(st, false);
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) {
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* st, unsigned) {
    std::lock_guard<std::mutex> lk(mu);
    *st = reinterpret_cast<hipStream_t>(make_stream(false));
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t st, hipDevice_t* dev) {
    std::lock_guard<std::mutex> lk(mu);
    *dev = stream_of(st)->device;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t st) {
    std::unique_lock<std::mutex> lk(mu);
    Stream* s = stream_of(st);
    wait_done(lk, s, s->queued);
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t st, hipStreamCaptureMode) {
    std::lock_guard<std::mutex> lk(mu);
    stream_of(st)->capturing = true;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t st, hipGraph_t* g) {
    std::lock_guard<std::mutex> lk(mu);
    stream_of(st)->capturing = false;
    *g = reinterpret_cast<hipGraph_t>(new int);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    *e = reinterpret_cast<hipGraphExec_t>(new int);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t st) {
    queue(st, false);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete reinterpret_cast<int*>(g); return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { delete reinterpret_cast<int*>(e); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    const StubsOwn own;
    Event* v = new Event;
    v->device = current_device;
    *e = reinterpret_cast<hipEvent_t>(v);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<Event*>(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) {
    std::lock_guard<std::mutex> lk(mu);
    Event* v = reinterpret_cast<Event*>(e);
    Stream* s = stream_of(st);
    if (v->device != s->device) return hipErrorInvalidHandle;
    v->on = s;
    v->seq = s->queued;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    std::unique_lock<std::mutex> lk(mu);
    Event* v = reinterpret_cast<Event*>(e);
    if (!v->on) return hipSuccess;
    wait_done(lk, v->on, v->seq);
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = current_device; return hipSuccess; }
hipError_t hipSetDevice(int d) { current_device = d; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 2; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }

}  // extern "C"

// ---------------------------------------------------------------- scenarios

namespace {

#define EXPECT(c)                                                                                          \
    do {                                                                                                   \
        if (!(c)) { printf("line %d: %s   (%s)\n", __LINE__, #c, swe_last_error()); fflush(stdout); _exit(1); } \
    } while (0)

swe_params params(int precision, void* stream, const std::vector<double>& H) {
    swe_params p;
    memset(&p, 0, sizeof p);
    p.precision = precision;
    p.g = 9.81; p.cfl = 0.4; p.eps = 1e-4; p.h_wind = 0.1; p.skip_dry = 1;
    p.stream = stream;
    p.H0 = H.data();
    return p;
}

// A grid of n x n cells: with n = 1024 its state takes 12 MB in FP32, which
// several host threads move; with n = 64 one piece on the calling thread.
struct Grid {
    int n;
    std::vector<double> b, H, Q, R;
    swe_t* s = nullptr;
    Grid(int side, int precision, void* stream) : n(side), b((size_t)side * side), H(b.size(), 1.0), Q(b.size()), R(b.size()) {
        for (size_t k = 0; k < Q.size(); ++k) { Q[k] = (double)(k % 1000) / 8.0; R[k] = -Q[k]; H[k] = 1.0 + Q[k]; }
        swe_params p = params(precision, stream, H);
        p.Qx0 = Q.data();
        p.Qy0 = R.data();
        s = swe_create(n, n, 1.0, b.data(), nullptr, &p);
    }
    int get() { return swe_get_state(s, H.data(), Q.data(), R.data()); }
    bool kept() const {   // the layer that was set comes back
        for (size_t k = 0; k < Q.size(); ++k)
            if (Q[k] != (double)(k % 1000) / 8.0 || R[k] != -Q[k] || H[k] != 1.0 + Q[k]) return false;
        return true;
    }
    int set() { return swe_set_state(s, H.data(), Q.data(), R.data()); }
};

struct Crops {
    int tile, n;
    size_t in, out;
    std::vector<double> x, y, m, o;
    swe_lc_t* c = nullptr;
    Crops(int tile_, int n_, void* stream) : tile(tile_), n(n_), in((size_t)(tile + 9) * (tile + 9) * 6),
        out((size_t)(tile + 1) * (tile + 1) * 6), x(in * n), y(out * n), m(out * n, 1.0), o(out * n) {
        for (size_t k = 0; k < x.size(); ++k) x[k] = (double)(k % 97) / 16.0;
        const double one[6] = {1, 1, 1, 1, 1, 1};
        c = swe_lc_create(tile, n, one, one, stream);
    }
    int train() { double loss; return swe_lc_train_step(c, n, x.data(), y.data(), m.data(), 1e-3, &loss); }
};

// Everything that a caller on hipStreamPerThread queued is done before a
// piece of a transfer touches the memory, and the pieces before what follows.
int per_thread_stream() {
    void* const st = (void*)hipStreamPerThread;
    Grid g(1024, 32, st);
    EXPECT(g.s);
    EXPECT(swe_enqueue(g.s, 3) == 0 && g.get() == 0);
    EXPECT(swe_enqueue(g.s, 2) == 0 && g.set() == 0);
    EXPECT(swe_step(g.s) == 0 && g.get() == 0 && g.kept());
    Crops c(32, 40, st);
    EXPECT(c.c && c.train() == 0 && c.train() == 0);
    EXPECT(swe_lc_forward(c.c, c.n, c.x.data(), c.o.data()) == 0);
    EXPECT(swe_lc_infer(c.c, c.n, c.x.data(), c.o.data()) == 0);
    if (violations) printf("%d operations were not ordered\n", violations);
    EXPECT(violations == 0);
    return 0;
}

// Calls that wait for one handle's queued work hold up no other handle: its
// transfers, a network's calls and its creation go on while a hundred threads
// wait.  What the pool pins is bounded and given back with the last handle.
int independent_handles() {
    auto make = [] {
        hipStream_t st;
        (void)hipStreamCreateWithFlags(&st, 0);
        return st;
    };
    std::vector<hipStream_t> slow;
    std::vector<std::thread> waiting;
    std::vector<Grid*> grids;
    int bad = 0;
    auto wait = [&](int n, std::function<bool(Grid&)> call) {
        slow.push_back(make());
        Grid* g = new Grid(n, 32, slow.back());
        grids.push_back(g);
        EXPECT(g->s && swe_enqueue(g->s, 1) == 0);
        block(slow.back(), true);
        waiting.emplace_back([&, g, call] { if (!call(*g)) ++bad; });
    };
    Grid b(1024, 32, make()), small(48, 64, make());
    hipStream_t net_stream = make();
    Crops net(32, 40, net_stream), other(32, 40, make());
    EXPECT(b.s && small.s && net.c && other.c && net.train() == 0);
    auto goes_on = [&](const char* what) {
        auto f = std::async(std::launch::async, [&] {
            Grid& fresh = *new Grid(256, 32, make());
            grids.push_back(&fresh);   // (freeing device memory waits for the device)
            return b.set() == 0 && b.get() == 0 && b.kept() && small.set() == 0 && small.get() == 0 &&
                   small.kept() && swe_run(b.s, 1) == 0 && swe_time(small.s) == 0.0 && other.train() == 0 && fresh.s &&
                   fresh.get() == 0 && fresh.kept();
        });
        if (f.wait_for(std::chrono::seconds(20)) != std::future_status::ready) {
            printf("held up while another handle's %s waits\n", what);
            fflush(stdout);
            _exit(1);
        }
        return f.get();
    };
    wait(1024, [](Grid& g) { return g.get() == 0; });
    EXPECT(goes_on("large state read"));
    wait(1024, [](Grid& g) { return g.set() == 0; });
    EXPECT(goes_on("large state set"));
    wait(64, [](Grid& g) { return g.get() == 0 && g.set() == 0; });
    EXPECT(goes_on("small state read"));
    wait(64, [](Grid& g) { return swe_run(g.s, 1) == 0; });
    EXPECT(goes_on("run"));
    block(net_stream, true);
    slow.push_back(net_stream);
    waiting.emplace_back([&] { if (net.train() != 0) ++bad; });
    EXPECT(goes_on("training step"));
    for (int k = 0; k < 100; ++k) wait(32, [](Grid& g) { return std::isfinite(swe_time(g.s)); });
    EXPECT(goes_on("hundred clock reads"));
    EXPECT(pinned_bytes <= (size_t(128) << 20));
    for (hipStream_t st : slow) block(st, false);
    for (std::thread& t : waiting) t.join();
    EXPECT(bad == 0);
    for (Grid* g : grids) swe_destroy(g->s);
    swe_destroy(b.s);
    swe_destroy(small.s);
    swe_lc_destroy(net.c);
    EXPECT(pinned_bytes > 0);
    swe_lc_destroy(other.c);
    EXPECT(pinned_bytes == 0);
    return 0;
}

// A device array of n elements that holds exactly `want`.
template <typename T> bool on_device(const std::vector<T>& want) {
    std::lock_guard<std::mutex> lk(mu);
    for (auto& m : device_mem)
        if (m.second == want.size() * sizeof(T) && !memcmp(m.first, want.data(), m.second)) return true;
    return false;
}

// Without any pinned memory every transfer works through ordinary memory:
// states of one piece and of several, a patch's interior, a network's crops
// and parameters.
int no_pinned_memory() {
    no_pinned = true;
    for (int n : {64, 1500})
        for (int precision : {32, 64}) {
            Grid g(n, precision, nullptr);
            EXPECT(g.s && g.get() == 0 && g.kept());
            EXPECT(g.set() == 0 && swe_run(g.s, 3) == 0 && swe_time(g.s) == 0.0);
            std::vector<double> only(g.b.size());
            EXPECT(swe_get_state(g.s, nullptr, only.data(), nullptr) == 0 && only == g.Q);
            swe_destroy(g.s);
        }
    {
        const int n = 40, r = 3, cw = 9, ch = 7, w = r * cw, h = r * ch;
        std::vector<double> b(n * n), H(n * n, 1.0), bf((w + 2 * SWE_NEST_FRAME) * (h + 2 * SWE_NEST_FRAME)), Hf(w * h), o(w * h);
        for (size_t k = 0; k < Hf.size(); ++k) Hf[k] = 1.0 + (double)k;
        swe_params p = params(32, nullptr, H);
        swe_patch q = {10, 12, cw, ch, bf.data(), nullptr, Hf.data(), nullptr, nullptr};
        swe_nest_t* s = swe_nest_create(n, n, 1.0, b.data(), nullptr, &p, r, 1, 1, &q);
        EXPECT(s && swe_nest_get_patch(s, 0, o.data(), nullptr, nullptr) == 0 && o == Hf);
    }
    Crops c(16, 5, nullptr);
    EXPECT(c.c && c.train() == 0);
    std::vector<unsigned short> x(c.x.size() / 6 * 16);   // (the values are exact in bf16)
    for (size_t k = 0; k < c.x.size(); ++k) {
        const float f = (float)c.x[k];
        unsigned u;
        memcpy(&u, &f, 4);
        x[k / 6 * 16 + k % 6] = (unsigned short)(u >> 16);
    }
    EXPECT(on_device(x) && on_device(std::vector<float>(c.m.begin(), c.m.end())));
    EXPECT(swe_lc_forward(c.c, c.n, c.x.data(), c.o.data()) == 0 && swe_lc_infer(c.c, c.n, c.x.data(), c.o.data()) == 0);
    std::vector<double> par(swe_lc_nparams(), 0.5), got(par.size());
    EXPECT(swe_lc_set_params(c.c, par.data()) == 0 && swe_lc_get_params(c.c, got.data()) == 0 && got == par);
    return 0;
}

// Pinned memory is asked for as a transfer needs it: little for small grids
// and networks, the whole of a large transfer only for a large one, once.
int memory_by_need() {
    Grid small(64, 32, nullptr);
    EXPECT(small.s && swe_run(small.s, 1) == 0 && small.get() == 0);
    EXPECT(pinned_bytes <= (size_t(256) << 10));
    Crops c(32, 24, nullptr);   // 2.2 MB of crops, labels and mask
    EXPECT(c.c && c.train() == 0 && c.train() == 0);
    EXPECT(pinned_bytes <= (size_t(256) << 10) + (size_t(4) << 20));
    const size_t before = pinned_bytes;
    Grid large(2048, 32, nullptr);
    EXPECT(large.s && large.get() == 0 && large.kept() && large.set() == 0);
    Grid odd(1500, 64, nullptr);
    EXPECT(odd.s && odd.get() == 0 && odd.kept());
    EXPECT(pinned_bytes <= before + (size_t(32) << 20));
    return 0;
}

// A network holds the partials of as large a training step as it can take.
int network_memory() {
    Crops one(32, 1, nullptr);
    EXPECT(one.c && device_bytes <= (size_t(12) << 20));
    const size_t created = device_bytes;
    EXPECT(one.train() == 0 && one.train() == 0 && device_bytes == created);
    Crops many(32, 64, nullptr);
    EXPECT(many.c && many.train() == 0);
    swe_lc_destroy(many.c);
    swe_lc_destroy(one.c);
    EXPECT(device_bytes == 0);
    return 0;
}

// Where a thread cannot be started for want of memory, the calling one does
// its share.
int no_memory_for_threads() {
    Grid g(1024, 32, nullptr);
    EXPECT(g.s);
    no_memory = true;
    const int get = g.get(), set = g.set(), again = g.get();
    no_memory = false;
    EXPECT(get == 0 && set == 0 && again == 0 && g.kept());
    return 0;
}

// A handle's transfers work whichever device is current, and leave it so.
int another_device() {
    for (int n : {64, 1024}) {
        Grid g(n, 32, nullptr);
        EXPECT(g.s);
        (void)hipSetDevice(1);
        EXPECT(g.get() == 0 && g.kept() && g.set() == 0 && g.get() == 0 && g.kept());
        EXPECT(current_device == 1);
        (void)hipSetDevice(0);
    }
    return 0;
}

const std::map<std::string, std::function<int()>> scenarios = {
    {"another_device", another_device},
    {"no_memory_for_threads", no_memory_for_threads},
    {"network_memory", network_memory},
    {"memory_by_need", memory_by_need},
    {"independent_handles", independent_handles},
    {"no_pinned_memory", no_pinned_memory},
    {"per_thread_stream", per_thread_stream},
};

}  // namespace

int main(int argc, char** argv) {
    if (argc < 2 || !scenarios.count(argv[1])) {
        for (auto& s : scenarios) printf("%s\n", s.first.c_str());
        return 2;
    }
    const int rc = scenarios.at(argv[1])();
    fflush(stdout);
    _exit(rc);
}
