// swe_xfer.hpp -- transfers between the caller's FP64 arrays and the stencil
// type's fields on the device.
//
// The caller's arrays are pageable, so a copy straight to or from them goes
// through the runtime's staging in small pieces, one host thread converting
// after each array: 4 GB/s on a 4096^2 state.  Here a kernel moves a piece of
// a field between device memory and pinned host memory at the link's rate
// (it picks the current layer of a ping-pong pair from the step count itself,
// so that no round trip for the control block comes first), and several host
// threads convert pieces while others are on the way.  Transfers of less than
// XFER_THREADED bytes take one launch, one wait and the calling thread.  Where
// there is no pinned memory to be had, fields are copied to and from ordinary
// memory in pieces instead.
//
// The handle of the caller's stream may name another stream in every thread
// (hipStreamPerThread).  Other threads launch pieces only after the calling one
// has waited for what it had queued, and each waits for its own pieces; where
// pieces are only queued, the calling thread launches all of them on that
// handle.
//
// The pinned memory is one pool per process: buffers leased to one transfer
// each, allocated when none that is free is large enough and given back when
// the last handle is destroyed; at most XFER_BUFFERS of them and XFER_TOTAL
// bytes.  No transfer waits for another one: the pool's lock is held for the
// bookkeeping alone, a large transfer takes its buffer only once the work
// queued before it is done, and one that finds none left goes without.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <sys/mman.h>

#include <climits>
#include <cstring>
#include <exception>
#include <mutex>
#include <new>
#include <thread>

#include "swe_step.hpp"

namespace swe {

// One field as a ping-pong pair (b = a for a single buffer).
template <typename real> struct FieldPair { real* a; real* b; };

template <typename real, int N> struct XferFields {
    FieldPair<real> f[N];
    real* host[N];
};

// Copy cells [first, first + cnt) of the w-wide rectangle at (x0, y0) of each
// field's current layer (rows of `pitch` cells) into host[q].
template <typename real, int N>
__global__ __launch_bounds__(256) void k_export(XferFields<real, N> x, const Ctrl* ctrl, int pitch, int x0, int y0,
                                                int w, size_t first, size_t cnt) {
    const int q = blockIdx.y;
    const real* src = (ctrl->step & 1) ? x.f[q].b : x.f[q].a;
    real* dst = x.host[q];
    const size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x, nt = (size_t)gridDim.x * blockDim.x;
    if (w == pitch) {
        src += (size_t)y0 * pitch + first;
        constexpr int V = 16 / sizeof(real);
        size_t done = 0;
        if ((((uintptr_t)src | (uintptr_t)dst) & 15) == 0) {
            const size_t nv = cnt / V;
            for (size_t k = t; k < nv; k += nt)
                reinterpret_cast<uint4*>(dst)[k] = reinterpret_cast<const uint4*>(src)[k];
            done = nv * V;
        }
        for (size_t k = done + t; k < cnt; k += nt) dst[k] = src[k];
    } else {
        for (size_t k = t; k < cnt; k += nt) {
            const size_t c = first + k;
            dst[k] = src[(y0 + c / w) * pitch + x0 + c % w];
        }
    }
}

// Cells [first, first + cnt) of each field, both buffers of its pair, from
// host[q].
template <typename real, int N>
__global__ __launch_bounds__(256) void k_import(XferFields<real, N> x, size_t first, size_t cnt) {
    const int q = blockIdx.y;
    real* a = x.f[q].a + first;
    real* b = x.f[q].b + first;
    const real* src = x.host[q];
    const size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x, nt = (size_t)gridDim.x * blockDim.x;
    constexpr int V = 16 / sizeof(real);
    size_t done = 0;
    if ((((uintptr_t)a | (uintptr_t)b | (uintptr_t)src) & 15) == 0) {
        const size_t nv = cnt / V;
        for (size_t k = t; k < nv; k += nt) {
            const uint4 v = reinterpret_cast<const uint4*>(src)[k];
            reinterpret_cast<uint4*>(a)[k] = v;
            if (b != a) reinterpret_cast<uint4*>(b)[k] = v;
        }
        done = nv * V;
    }
    for (size_t k = done + t; k < cnt; k += nt) { a[k] = src[k]; b[k] = src[k]; }
}

}  // namespace swe

namespace {

constexpr int XFER_SLOTS = 8;                    // pieces in flight = host threads of a large transfer
constexpr size_t XFER_SLOT = size_t(4) << 20;
constexpr size_t XFER_THREADED = size_t(2) << 20;
constexpr size_t XFER_PAGEABLE = size_t(1) << 20;   // elements of a piece without pinned memory

constexpr int XFER_BUFFERS = 64;
// smallest buffer (others are powers of two times it): a 128^2 grid's state, so
// that a small grid allocates one (each allocation takes some 30 us)
constexpr size_t XFER_LEAST = size_t(256) << 10;
constexpr size_t XFER_TOTAL = size_t(128) << 20;

struct XferPool {
    struct Buffer {
        unsigned char* p = nullptr;   // null: none allocated (or being allocated while busy)
        size_t size = 0;
        bool busy = false;
    };
    std::mutex mu;   // held for bookkeeping only
    Buffer buf[XFER_BUFFERS];
    size_t total = 0;
    int users = 0;   // live handles
};
XferPool& xfer_pool() {
    static XferPool* p = new XferPool;   // never destroyed: handles may be freed at process exit
    return *p;
}
void xfer_retain() {
    XferPool& p = xfer_pool();
    std::lock_guard<std::mutex> lk(p.mu);
    ++p.users;
}
void xfer_release() {
    XferPool& p = xfer_pool();
    unsigned char* gone[XFER_BUFFERS];
    int n = 0;
    {
        std::lock_guard<std::mutex> lk(p.mu);
        if (--p.users > 0) return;
        for (XferPool::Buffer& b : p.buf)
            if (b.p && !b.busy) {
                gone[n++] = b.p;
                p.total -= b.size;
                b = XferPool::Buffer();
            }
    }
    for (int k = 0; k < n; ++k) (void)hipHostFree(gone[k]);   // (may wait for the device: not under the lock)
}

// A buffer of the pool, leased while this lives.  The holder waits for what
// the device does with it before letting it go.
struct XferHold {
    XferPool::Buffer* at = nullptr;
    XferHold() {}
    ~XferHold() { drop(); }
    XferHold(const XferHold&) = delete;
    void drop() {
        if (!at) return;
        std::lock_guard<std::mutex> lk(xfer_pool().mu);
        at->busy = false;
        at = nullptr;
    }
    // pinned memory for `bytes`; the largest piece there is where no more is
    // to be had.  Returns its size, 0 for none.
    size_t get(size_t bytes, unsigned char** base) {
        drop();
        XferPool& p = xfer_pool();
        size_t size = XFER_LEAST;
        while (size < bytes) size *= 2;
        std::unique_lock<std::mutex> lk(p.mu);
        XferPool::Buffer *fit = nullptr, *most = nullptr, *empty = nullptr;
        for (XferPool::Buffer& b : p.buf) {
            if (b.busy) continue;
            if (!b.p) { empty = &b; continue; }
            if (b.size >= bytes && (!fit || b.size < fit->size)) fit = &b;
            if (!most || b.size > most->size) most = &b;
        }
        if (!fit && empty && p.total + size <= XFER_TOTAL) {
            empty->busy = true;
            p.total += size;
            lk.unlock();
            void* q = nullptr;
            const hipError_t e = hipHostMalloc(&q, size, hipHostMallocPortable | hipHostMallocMapped);
            if (e != hipSuccess) (void)hipGetLastError();
            lk.lock();
            if (e == hipSuccess) {
                empty->p = (unsigned char*)q;
                empty->size = size;
                fit = empty;
            } else {
                empty->busy = false;
                p.total -= size;
                if (most && most->busy) most = nullptr;   // taken meanwhile
            }
        }
        at = fit ? fit : most;
        *base = at ? at->p : nullptr;
        if (!at) return 0;
        at->busy = true;
        return at->size;
    }
};

// The stream's device as the current one while this lives: events belong to
// the device that is current when they are made, and are recorded only on
// streams of that device.
struct XferDevice {
    int was = -1;
    explicit XferDevice(hipStream_t st) {
        int now = 0;
        hipDevice_t dev = 0;
        if (hipGetDevice(&now) == hipSuccess && hipStreamGetDevice(st, &dev) == hipSuccess && (int)dev != now &&
            hipSetDevice((int)dev) == hipSuccess)
            was = now;
    }
    ~XferDevice() {
        if (was >= 0) (void)hipSetDevice(was);
    }
    XferDevice(const XferDevice&) = delete;
};

// Run job(t) for every t < T <= XFER_SLOTS on host threads (the caller is
// number 0) and, on the calling thread and in order, then(t) once job(t) is
// done.  Returns the first error, after which the caller starts no more.
template <class Job, class Then>
hipError_t xfer_team(int T, Job job, Then then) {
    int dev = 0;
    const hipError_t e0 = hipGetDevice(&dev);
    if (e0 != hipSuccess) return e0;
    hipError_t err[XFER_SLOTS] = {}, e = hipSuccess;
    std::thread th[XFER_SLOTS];
    int started = 1;
    try {
        for (; started < T; ++started)
            th[started] = std::thread([&, t = started] {
                err[t] = hipSetDevice(dev);
                if (err[t] == hipSuccess) err[t] = job(t);
            });
    } catch (const std::exception&) {   // no more threads, or no memory for one: the caller takes the rest
    }
    for (int t = 0; t < T; ++t) {
        if (t > 0 && t < started) th[t].join();
        else if (e == hipSuccess) err[t] = job(t);
        if (e == hipSuccess) e = err[t] == hipSuccess ? then(t) : err[t];
    }
    return e;
}

// Run job(chunk, slot) for every chunk on up to `threads` <= XFER_SLOTS host
// threads, thread t taking chunks t, t + T, ... and slot t.
template <class Job>
hipError_t xfer_parallel(int chunks, int threads, Job job) {
    const int T = chunks < threads ? chunks : threads;
    return xfer_team(
        T,
        [&](int t) {
            hipError_t e = hipSuccess;
            for (int c = t; c < chunks && e == hipSuccess; c += T) e = job(c, t);
            return e;
        },
        [](int) { return hipSuccess; });
}

inline int xfer_grid(size_t cells) {
    const size_t b = (cells + 1023) / 1024;
    return (int)(b < 1 ? 1 : b > 1024 ? 1024 : b);
}

// Pages of a fresh array are faulted in by one call per piece instead of one
// trap per 4 KB page (1.3 us each here: 11 ms for 32 MB, against 0.9 ms to
// convert into them); pages already there, or an older kernel: no effect.
inline void xfer_populate(void* p, size_t bytes) {
#ifdef MADV_POPULATE_WRITE
    const uintptr_t page = 4096, lo = ((uintptr_t)p + page - 1) & ~(page - 1), hi = ((uintptr_t)p + bytes) & ~(page - 1);
    if (hi > lo) (void)madvise((void*)lo, hi - lo, MADV_POPULATE_WRITE);
#else
    (void)p; (void)bytes;
#endif
}

// Ordinary host memory for a transfer that gets no pinned memory.
template <typename T> struct XferHeap {
    T* p;
    explicit XferHeap(size_t n) : p(new (std::nothrow) T[n ? n : 1]) {}
    ~XferHeap() { delete[] p; }
    XferHeap(const XferHeap&) = delete;
};

// A transfer of nf <= 3 fields of n cells through the pool: in one piece where
// that is small, else split over threads with an event each; without pinned
// memory neither (base stays null).
struct XferPlan {
    XferHold hold;
    unsigned char* base = nullptr;
    bool whole = false;
    size_t piece = 0, slot = 0;
    int per = 0, threads = 0;
    hipEvent_t ev[XFER_SLOTS] = {};
    hipError_t prepare(int nf, size_t n, size_t rsize) {
        const size_t all = nf * n * rsize;
        if (all <= XFER_THREADED) {
            whole = hold.get(all, &base) >= all;
            if (!whole) base = nullptr;
            return hipSuccess;
        }
        const size_t most = XFER_SLOTS * XFER_SLOT, size = hold.get(all < most ? all : most, &base);
        threads = XFER_SLOTS;
        slot = size / threads / (1024 * rsize) * (1024 * rsize);
        if (!slot) {   // none, or too little to split
            base = nullptr;
            return hipSuccess;
        }
        piece = (n * nf + threads - 1) / threads;   // about one piece a thread, at least 32768 cells, at most a slot
        if (piece < 32768) piece = 32768;
        piece = (piece + 1023) / 1024 * 1024;
        if (piece > slot / rsize) piece = slot / rsize;
        per = (int)((n + piece - 1) / piece);
        for (int t = 0; t < threads; ++t) {
            const hipError_t e = hipEventCreateWithFlags(&ev[t], hipEventDisableTiming);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    ~XferPlan() {
        for (hipEvent_t v : ev)
            if (v) (void)hipEventDestroy(v);
    }
};

// xfer_get and xfer_put without pinned memory, in pieces of about
// XFER_PAGEABLE cells, each copied and waited for.
template <typename real, class Convert>
hipError_t xfer_get_pageable(hipStream_t st, const swe::Ctrl* ctrl, real* const (&a)[3], real* const (&b)[3], int pitch,
                             int x0, int y0, int w, int h, double* const (&out)[3], Convert convert) {
    long long step = 0;
    hipError_t e = hipMemcpyAsync(&step, &ctrl->step, sizeof step, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return e;
    const size_t n = (size_t)w * h;
    // whole rows of a rectangle, any cells of a whole layer
    const size_t rows = XFER_PAGEABLE / w > 1 ? XFER_PAGEABLE / w : 1, most = w == pitch ? XFER_PAGEABLE : rows * w;
    XferHeap<real> buf(n < most ? n : most);
    if (!buf.p) return hipErrorOutOfMemory;
    for (int q = 0; q < 3; ++q) {
        if (!out[q]) continue;
        const real* src = ((step & 1) ? b[q] : a[q]) + (size_t)y0 * pitch + x0;
        for (size_t first = 0; first < n; first += most) {
            const size_t cnt = n - first < most ? n - first : most;
            if (w == pitch)
                e = hipMemcpyAsync(buf.p, src + first, cnt * sizeof(real), hipMemcpyDeviceToHost, st);
            else
                e = hipMemcpy2DAsync(buf.p, w * sizeof(real), src + first / w * pitch, pitch * sizeof(real),
                                     w * sizeof(real), cnt / w, hipMemcpyDeviceToHost, st);
            const hipError_t s = hipStreamSynchronize(st);
            if (e == hipSuccess) e = s;
            if (e != hipSuccess) return e;
            convert(out[q] + first, buf.p, cnt);
        }
    }
    return hipSuccess;
}
template <typename real, class Fill>
hipError_t xfer_put_pageable(hipStream_t st, int nf, const swe::FieldPair<real>* f, size_t n, Fill fill) {
    XferHeap<real> buf(n < XFER_PAGEABLE ? n : XFER_PAGEABLE);
    if (!buf.p) return hipErrorOutOfMemory;
    for (int q = 0; q < nf; ++q)
        for (size_t first = 0; first < n; first += XFER_PAGEABLE) {
            const size_t cnt = n - first < XFER_PAGEABLE ? n - first : XFER_PAGEABLE;
            fill(q, first, cnt, buf.p);
            hipError_t e = hipMemcpyAsync(f[q].a + first, buf.p, cnt * sizeof(real), hipMemcpyHostToDevice, st);
            if (e == hipSuccess && f[q].b != f[q].a)
                e = hipMemcpyAsync(f[q].b + first, buf.p, cnt * sizeof(real), hipMemcpyHostToDevice, st);
            const hipError_t s = hipStreamSynchronize(st);
            if (e == hipSuccess) e = s;
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

// The rectangle (x0, y0, w x h) of up to three fields' current layers into
// FP64 host arrays (null: not wanted), after everything queued on `st`.
template <typename real>
hipError_t xfer_get(hipStream_t st, const swe::Ctrl* ctrl, real* const (&a)[3], real* const (&b)[3], int pitch, int x0,
                    int y0, int w, int h, double* const (&out)[3]) {
    int want[3], nf = 0;
    for (int q = 0; q < 3; ++q)
        if (out[q]) want[nf++] = q;
    const size_t n = (size_t)w * h;
    if (nf == 0) return hipStreamSynchronize(st);
    auto convert = [](double* dst, const real* src, size_t cnt) {
        if constexpr (sizeof(real) == 8) std::memcpy(dst, src, cnt * 8);
        else for (size_t k = 0; k < cnt; ++k) dst[k] = (double)src[k];
    };
    const XferDevice current(st);
    hipError_t e = hipSuccess;
    // (a small one is queued behind it: on a new stream this wait takes 20 us)
    if (nf * n * sizeof(real) > XFER_THREADED && (e = hipStreamSynchronize(st)) != hipSuccess) return e;
    XferPlan pl;
    if ((e = pl.prepare(nf, n, sizeof(real))) != hipSuccess) return e;
    if (!pl.base) return xfer_get_pageable(st, ctrl, a, b, pitch, x0, y0, w, h, out, convert);
    if (pl.whole) {
        real* base = (real*)pl.base;
        swe::XferFields<real, 3> x{};
        for (int k = 0; k < nf; ++k) {
            x.f[k] = {a[want[k]], b[want[k]]};
            x.host[k] = base + k * n;
        }
        hipLaunchKernelGGL((swe::k_export<real, 3>), dim3(xfer_grid(n), nf), dim3(256), 0, st, x, ctrl, pitch, x0, y0, w,
                           (size_t)0, n);
        if ((e = hipGetLastError()) != hipSuccess || (e = hipStreamSynchronize(st)) != hipSuccess) return e;
        for (int k = 0; k < nf; ++k) convert(out[want[k]], base + k * n, n);
        return hipSuccess;
    }
    return xfer_parallel(nf * pl.per, pl.threads, [&](int c, int t) -> hipError_t {
        const int q = want[c / pl.per];
        const size_t first = (size_t)(c % pl.per) * pl.piece, cnt = n - first < pl.piece ? n - first : pl.piece;
        real* slot = (real*)(pl.base + t * pl.slot);
        const swe::XferFields<real, 1> x{{{a[q], b[q]}}, {slot}};
        hipLaunchKernelGGL((swe::k_export<real, 1>), dim3(xfer_grid(cnt)), dim3(256), 0, st, x, ctrl, pitch, x0, y0, w,
                           first, cnt);
        hipError_t s = hipGetLastError();
        if (s == hipSuccess) s = hipEventRecord(pl.ev[t], st);
        xfer_populate(out[q] + first, cnt * sizeof(double));   // while the piece is on its way
        if (s == hipSuccess) s = hipEventSynchronize(pl.ev[t]);
        if (s == hipSuccess) convert(out[q] + first, slot, cnt);
        else (void)hipStreamSynchronize(st);   // no piece is under way when the pool is let go
        return s;
    });
}

// Fields of n cells each from fill(q, first, cnt, dst), which writes cells
// [first, first + cnt) of field q in the stencil type; both buffers of each
// pair.  Returns once the device has them.
template <typename real, class Fill>
hipError_t xfer_put(hipStream_t st, int nf, const swe::FieldPair<real>* f, size_t n, Fill fill) {
    const XferDevice current(st);
    hipError_t e = hipSuccess;
    // (a small one is queued behind it: on a new stream this wait takes 20 us)
    if (nf * n * sizeof(real) > XFER_THREADED && (e = hipStreamSynchronize(st)) != hipSuccess) return e;
    XferPlan pl;
    if ((e = pl.prepare(nf, n, sizeof(real))) != hipSuccess) return e;
    if (!pl.base) return xfer_put_pageable(st, nf, f, n, fill);
    if (pl.whole) {
        real* base = (real*)pl.base;
        swe::XferFields<real, 3> x{};
        for (int q = 0; q < nf; ++q) {
            fill(q, (size_t)0, n, base + q * n);
            x.f[q] = f[q];
            x.host[q] = base + q * n;
        }
        hipLaunchKernelGGL((swe::k_import<real, 3>), dim3(xfer_grid(n), nf), dim3(256), 0, st, x, (size_t)0, n);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        return hipStreamSynchronize(st);
    }
    return xfer_parallel(nf * pl.per, pl.threads, [&](int c, int t) -> hipError_t {
        const int q = c / pl.per;
        const size_t first = (size_t)(c % pl.per) * pl.piece, cnt = n - first < pl.piece ? n - first : pl.piece;
        real* slot = (real*)(pl.base + t * pl.slot);
        fill(q, first, cnt, slot);
        const swe::XferFields<real, 1> x{{f[q]}, {slot}};
        hipLaunchKernelGGL((swe::k_import<real, 1>), dim3(xfer_grid(cnt)), dim3(256), 0, st, x, first, cnt);
        hipError_t s = hipGetLastError();
        if (s == hipSuccess) s = hipEventRecord(pl.ev[t], st);
        if (s == hipSuccess) s = hipEventSynchronize(pl.ev[t]);
        if (s != hipSuccess) (void)hipStreamSynchronize(st);
        return s;
    });
}

// Whether every x[i], i < n, lies in [lo, hi] (false for NaN), on host threads
// for a large n; a null x does.
inline bool xfer_within(const double* x, size_t n, double lo, double hi) {
    if (!x) return true;
    constexpr size_t PART = size_t(1) << 18;
    auto bad = [=](size_t i0, size_t i1) {
        int v = 0;   // no early exit: the loop vectorises
        for (size_t i = i0; i < i1; ++i) v |= !((x[i] >= lo) & (x[i] <= hi));
        return v;
    };
    const size_t parts = (n + PART - 1) / PART;
    int found[XFER_SLOTS] = {};
    if (parts < 2 || parts > (size_t)INT_MAX ||
        xfer_parallel((int)parts, XFER_SLOTS, [&](int c, int t) -> hipError_t {
            const size_t i0 = c * PART;
            found[t] |= bad(i0, n - i0 < PART ? n : i0 + PART);
            return hipSuccess;
        }) != hipSuccess)
        return !bad(0, n);
    for (int f : found)
        if (f) return false;
    return true;
}

// A few bytes of device memory after everything queued on `st`, through a
// buffer of the pool (a pageable destination costs 9 us more); straight where
// there is none.
inline hipError_t xfer_read(void* dst, const void* src, size_t bytes, hipStream_t st) {
    XferHold hold;
    unsigned char* base = nullptr;
    void* const to = hold.get(bytes, &base) >= bytes ? base : dst;
    hipError_t e = hipMemcpyAsync(to, src, bytes, hipMemcpyDeviceToHost, st);
    if (e != hipSuccess || (e = hipStreamSynchronize(st)) != hipSuccess) return e;
    if (to != dst) std::memcpy(dst, to, bytes);
    return hipSuccess;
}

}  // namespace
