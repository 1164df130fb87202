// Serving loop of libcrb: continuous (iteration-level) batching of frames that
// arrive over time, the GPU analogue of CRBLASTER's director polling its actors
// (Section 6.2: the director collects subimages as actors finish, without a
// barrier).
//
// Requests wait FIFO.  A request is admitted when a slot is free and its device footprint
// (image, mask, workspace) fits the HBM budget; one from host memory is uploaded on a copy
// stream, one from device memory is cleaned in the caller's buffers.  Each round runs ONE
// iteration for every admitted frame, each at its own iteration index, with the batched
// kernels over a descriptor table rebuilt per round (its tile lists on the device: writing
// those of 24 frames on the host took 70 us a round), so frames that arrive while others are
// on the GPU join at the next round.  A frame leaves after niter iterations or when an
// iteration selects no new pixel (early stop, result-neutral); results for host memory are
// copied back on the copy stream.  Progress is observed only by
// polling events: no call blocks on the device.  A server is used from one thread.
#include "api_internal.h"

#include <string.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <deque>
#include <map>
#include <mutex>
#include <new>
#include <functional>
#include <thread>
#include <vector>

namespace crb {

static double now_s() {
    return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch())
        .count();
}

enum ReqState { kWaiting, kActive, kDraining };

// Host copies between the caller's buffers and pinned staging, split over a few
// threads (a single core copies well below the host link's bandwidth).
class CopyPool {
  public:
    explicit CopyPool(unsigned n) {
        for (unsigned i = 0; i < n; ++i)
            threads_.emplace_back([this] { run(); });
    }
    ~CopyPool() {
        {
            std::lock_guard<std::mutex> g(mu_);
            stop_ = true;
        }
        cv_.notify_all();
        for (auto &t : threads_)
            t.join();
    }
    void copy(void *dst, const void *src, size_t n) {
        const size_t chunk = (size_t)4 << 20;
        if (threads_.empty() || n <= chunk) {
            memcpy(dst, src, n);
            return;
        }
        const size_t parts = (n + chunk - 1) / chunk;
        std::atomic<size_t> next{0}, done{0};
        auto work = [&] {
            for (size_t p; (p = next.fetch_add(1)) < parts;) {
                const size_t off = p * chunk, len = off + chunk < n ? chunk : n - off;
                memcpy((char *)dst + off, (const char *)src + off, len);
                done.fetch_add(1);
            }
        };
        {
            std::lock_guard<std::mutex> g(mu_);
            job_ = work;
            ++gen_;
        }
        cv_.notify_all();
        work();                                   // the calling thread helps
        while (done.load() < parts)
            std::this_thread::yield();
        // retire the job and wait until no worker still holds it (it refers to this frame)
        std::unique_lock<std::mutex> g(mu_);
        job_ = nullptr;
        cv_done_.wait(g, [&] { return busy_ == 0; });
    }

  private:
    void run() {
        uint64_t seen = 0;
        std::unique_lock<std::mutex> g(mu_);
        for (;;) {
            cv_.wait(g, [&] { return stop_ || gen_ != seen; });
            if (stop_)
                return;
            seen = gen_;
            if (!job_)
                continue;
            auto job = job_;
            ++busy_;
            g.unlock();
            job();
            g.lock();
            --busy_;
            cv_done_.notify_all();
        }
    }
    std::vector<std::thread> threads_;
    std::mutex mu_;
    std::condition_variable cv_;
    std::condition_variable cv_done_;
    std::function<void()> job_;
    uint64_t gen_ = 0;
    int busy_ = 0;
    bool stop_ = false;
};

struct Request {
    int64_t id = 0;
    int32_t H = 0, W = 0;
    float gain = 0, readnoise = 0, sky = 0, sigclip = 0, sigfrac = 0, objlim = 0;
    int32_t niter = 0;
    const float *host_img = nullptr;   // caller's input, valid until completion
    bool direct = false;               // caller's buffers are pinned or on the device:
                                       // transferred without staging copies
    bool on_device = false;            // caller's buffers are device memory
    bool idle = false;                 // the caller's stream was idle at submit
    bool in_buffers = false;           // cleaned in the caller's device buffers, no copies
    bool copied = false;               // niter 0: the result is written
    bool shared = false;               // a buffer that it or another request writes is also
                                       // that other's (device requests)
    size_t alloc_bytes = 0;            // device memory taken from the server
    float *host_clean = nullptr;
    uint8_t *host_mask = nullptr;
    double t_submit = 0;
    size_t pin_bytes = 0, dev_bytes = 0;
    char *pin = nullptr;               // staging: image (4HW), then mask (HW)
    char *dev = nullptr;               // device: J (4HW) | mask (HW) | workspace
    DevFrame df;
    int k_next = 1;                    // next iteration to run
    ReqState state = kWaiting;
    hipEvent_t ev_h2d = nullptr;       // upload finished
    hipEvent_t ev_d2h = nullptr;       // download finished
    bool need_wait = false;            // next round must wait for ev_h2d
};

// A device buffer of a request in the server, kept by its first byte.
struct Span {
    uintptr_t end;
    Request *r;
    bool output;
};
using Spans = std::multimap<uintptr_t, Span>;

}  // namespace crb

using namespace crb;

struct crb_server {
    size_t budget = 0, in_use = 0, allocated = 0;
    int32_t max_slots = 0;
    int device = 0;
    hipStream_t compute = nullptr, copy = nullptr;
    int64_t next_id = 1;
    std::deque<Request *> waiting;
    std::vector<Request *> active;     // admitted, state kActive
    std::vector<Request *> draining;   // results being copied back
    Spans spans;                       // device buffers of the requests not yet reported
    size_t longest = 0;                // the largest of them so far
    // round in flight
    bool round_busy = false;
    std::vector<Request *> round_members;
    hipEvent_t ev_round = nullptr;
    // per-round tables: pinned host copies and device buffers
    size_t tab_cap = 0;                // bytes of each table buffer
    char *h_tab = nullptr, *d_tab = nullptr;
    // memory pools keyed by exact size
    std::multimap<size_t, char *> dev_free, pin_free;
    std::vector<hipEvent_t> event_pool;
    CopyPool *copies = nullptr;
};

namespace crb {

static crb_status get_event(crb_server *s, hipEvent_t *ev) {
    if (!s->event_pool.empty()) {
        *ev = s->event_pool.back();
        s->event_pool.pop_back();
        return CRB_OK;
    }
    return hip_status(hipEventCreateWithFlags(ev, hipEventDisableTiming), "hipEventCreate");
}

static void put_event(crb_server *s, hipEvent_t ev) {
    if (ev)
        s->event_pool.push_back(ev);
}

static crb_status pin_alloc(crb_server *s, size_t bytes, char **out) {
    auto it = s->pin_free.find(bytes);
    if (it != s->pin_free.end()) {
        *out = it->second;
        s->pin_free.erase(it);
        return CRB_OK;
    }
    hipError_t e = hipHostMalloc((void **)out, bytes, hipHostMallocDefault);
    if (e != hipSuccess) {
        *out = nullptr;
        (void)hipGetLastError();
        return fail(CRB_ENOMEM, "pinned staging of %zu bytes: %s", bytes, hipGetErrorString(e));
    }
    return CRB_OK;
}

// device memory within the budget; pooled blocks of other sizes are released first
static crb_status dev_alloc(crb_server *s, size_t bytes, char **out) {
    auto it = s->dev_free.find(bytes);
    if (it != s->dev_free.end()) {
        *out = it->second;
        s->dev_free.erase(it);
        return CRB_OK;
    }
    while (s->allocated + bytes > s->budget && !s->dev_free.empty()) {
        auto victim = s->dev_free.begin();
        (void)hipFree(victim->second);
        s->allocated -= victim->first;
        s->dev_free.erase(victim);
    }
    if (s->allocated + bytes > s->budget)
        return CRB_EBUSY;
    hipError_t e = hipMalloc((void **)out, bytes);
    if (e != hipSuccess) {
        *out = nullptr;
        (void)hipGetLastError();
        return CRB_EBUSY;   // the device is fuller than the budget assumed: retry later
    }
    s->allocated += bytes;
    return CRB_OK;
}

// the kind of memory p points to: 0 pageable host memory (unknown to HIP), 1 page-locked
// host memory the device can read and write directly, 2 device memory of `device`,
// -1 another device's memory
static int memory_kind(const void *p, int device) {
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    if (a.type == hipMemoryTypeHost)
        return 1;
    if (a.type == hipMemoryTypeDevice)
        return a.device == device ? 2 : -1;
    return 0;
}

static size_t frame_dev_bytes(int32_t H, int32_t W) {
    const size_t n = (size_t)H * (size_t)W;
    const size_t img = (4 * n + 255) / 256 * 256;
    const size_t msk = (n + 255) / 256 * 256;
    return img + msk + ws_layout(H, W).total;
}

static void leave_spans(crb_server *s, const Request *r);

static void release_request(crb_server *s, Request *r) {
    if (r->on_device)
        leave_spans(s, r);
    if (r->dev) {
        s->dev_free.emplace(r->alloc_bytes, r->dev);
        s->in_use -= r->dev_bytes;
        r->dev = nullptr;
    }
    if (r->pin) {
        s->pin_free.emplace(r->pin_bytes, r->pin);
        r->pin = nullptr;
    }
    put_event(s, r->ev_h2d);
    put_event(s, r->ev_d2h);
    delete r;
}

static bool overlap(const void *a, size_t na, const void *b, size_t nb) {
    const uintptr_t pa = (uintptr_t)a, pb = (uintptr_t)b;
    return pa < pb + nb && pb < pa + na;
}

struct Buffer {
    const void *p;
    size_t bytes;
    bool output;
};
static std::array<Buffer, 3> buffers(const Request *r) {
    const size_t n = (size_t)r->H * (size_t)r->W;
    return {{{r->host_img, 4 * n, false}, {r->host_clean, 4 * n, true}, {r->host_mask, n, true}}};
}
// Whether an output of q overlaps a buffer of r.
static bool writes_into(const Request *q, const Request *r) {
    for (const Buffer &a : buffers(q))
        for (const Buffer &b : buffers(r))
            if (a.output && overlap(a.p, a.bytes, b.p, b.bytes))
                return true;
    return false;
}

// Enters a device request's buffers, and marks it and the requests still waiting where one
// writes what is also the other's.
static void enter_spans(crb_server *s, Request *r) {
    for (const Buffer &b : buffers(r)) {
        const uintptr_t p = (uintptr_t)b.p, e = p + b.bytes;
        for (auto it = s->spans.lower_bound(p > s->longest ? p - s->longest : 0);
             it != s->spans.end() && it->first < e; ++it)
            if (it->second.end > p && it->second.r != r && (b.output || it->second.output))
                r->shared = it->second.r->shared = true;
    }
    for (const Buffer &b : buffers(r)) {
        s->spans.emplace((uintptr_t)b.p, Span{(uintptr_t)b.p + b.bytes, r, b.output});
        s->longest = std::max(s->longest, b.bytes);
    }
}
static void leave_spans(crb_server *s, const Request *r) {
    for (const Buffer &b : buffers(r)) {
        const auto range = s->spans.equal_range((uintptr_t)b.p);
        for (auto it = range.first; it != range.second;)
            it = it->second.r == r ? s->spans.erase(it) : std::next(it);
    }
}

// Whether a device request can be cleaned in the caller's own buffers, its outputs written from
// its first round on: no buffer may overlap another (a request in place would leave neither its
// input nor its result behind if the server were destroyed), no other request in the server may
// share a buffer that either writes, and no work that the caller's stream still held at submit
// may use the outputs' memory (an allocator hands a block on as soon as work on its former
// tensor is enqueued).  Otherwise the request is copied in at admission and out at completion.
static bool clean_in_buffers(const Request *r) {
    if (!r->on_device || !r->idle || r->shared)
        return false;
    const size_t n = (size_t)r->H * (size_t)r->W;
    return !overlap(r->host_img, 4 * n, r->host_clean, 4 * n) &&
           !overlap(r->host_mask, n, r->host_img, 4 * n) &&
           !overlap(r->host_mask, n, r->host_clean, 4 * n);
}

// Whether r has to wait for a request before it that is being cleaned in buffers which r reads
// or writes too (r was submitted after that one's admission, so neither knew of the other), or
// for a niter 0 copy that does the same.
static bool must_wait(const crb_server *s, const Request *r) {
    if (!r->shared)
        return false;
    for (const Request *q : s->active)
        if (q->in_buffers && (writes_into(q, r) || (r->niter == 0 && writes_into(r, q))))
            return true;
    for (const Request *q : s->waiting) {
        if (q == r)
            break;
        if (q->niter == 0 && !q->copied && (writes_into(q, r) || writes_into(r, q)))
            return true;
    }
    return false;
}

// The result of a device request with niter == 0, on the copy stream.
static hipError_t copy_niter0(crb_server *s, const Request *r) {
    const size_t n = (size_t)r->H * (size_t)r->W;
    hipError_t e = hipMemcpyAsync(r->host_clean, r->host_img, 4 * n, hipMemcpyDeviceToDevice,
                                  s->copy);
    if (e == hipSuccess)
        e = hipMemsetAsync(r->host_mask, 0, n, s->copy);
    return e;
}
// Enqueues those that had to wait at submit and need not any more.
static crb_status start_niter0(crb_server *s) {
    for (auto it = s->waiting.begin(); it != s->waiting.end();) {
        Request *r = *it;
        if (r->niter > 0 || r->copied || must_wait(s, r)) {
            ++it;
            continue;
        }
        crb_status st = get_event(s, &r->ev_d2h);
        if (st != CRB_OK)
            return st;
        hipError_t e = copy_niter0(s, r);
        if (e == hipSuccess)
            e = hipEventRecord(r->ev_d2h, s->copy);
        if (e != hipSuccess)
            return hip_status(e, "niter 0 copy");
        r->copied = true;
        r->state = kDraining;
        s->draining.push_back(r);
        it = s->waiting.erase(it);
    }
    return CRB_OK;
}

// Admit waiting requests (FIFO) while slots and budget allow, at most a few per
// call: staging an admitted frame is a host copy, and the next round should start
// while later frames are still being staged.
constexpr int kAdmitPerPoll = 4;

static crb_status admit(crb_server *s) {
    // a cap on staged admissions only: direct transfers cost the host nothing
    for (int staged = 0; staged < kAdmitPerPoll;) {
        // (a request with niter == 0 has its results since submit and waits to be reported: a
        // round has nothing to run for it and would not clear its mask)
        const auto next = std::find_if(s->waiting.begin(), s->waiting.end(),
                                       [](const Request *q) { return q->niter > 0; });
        if (next == s->waiting.end())
            return CRB_OK;
        Request *r = *next;
        const int held = (int)(s->active.size() + s->draining.size());
        if (held >= s->max_slots || s->in_use + r->dev_bytes > s->budget || must_wait(s, r))
            return CRB_OK;
        const size_t n = (size_t)r->H * (size_t)r->W;
        const size_t img = (4 * n + 255) / 256 * 256;
        const size_t msk = (n + 255) / 256 * 256;
        const FrameWs L = ws_layout(r->H, r->W);
        r->in_buffers = clean_in_buffers(r);
        r->alloc_bytes = r->in_buffers ? L.lists : r->dev_bytes;
        char *dev = nullptr;
        crb_status st = dev_alloc(s, r->alloc_bytes, &dev);
        if (st == CRB_EBUSY)
            return CRB_OK;
        if (st != CRB_OK)
            return st;
        if (!r->in_buffers && (st = get_event(s, &r->ev_h2d)) != CRB_OK) {
            s->dev_free.emplace(r->alloc_bytes, dev);
            return st;
        }
        if (!r->direct) {
            if ((st = pin_alloc(s, r->pin_bytes, &r->pin)) != CRB_OK) {
                s->dev_free.emplace(r->alloc_bytes, dev);
                return st;
            }
            s->copies->copy(r->pin, r->host_img, 4 * n);
            ++staged;
        }
        float *J = r->in_buffers ? r->host_clean : reinterpret_cast<float *>(dev);
        uint8_t *mask = r->in_buffers ? r->host_mask : reinterpret_cast<uint8_t *>(dev + img);
        r->dev = dev;
        s->in_use += r->dev_bytes;
        r->df = make_devframe(r->in_buffers ? r->host_img : J, J, mask,
                              r->in_buffers ? dev : dev + img + msk, L, r->H, r->W, r->gain,
                              r->readnoise, r->sky, r->sigclip, r->sigfrac, r->objlim, r->niter,
                              kFreshMask);
        if (!r->in_buffers) {
            hipError_t e = hipMemcpyAsync(J, r->direct ? (const void *)r->host_img : r->pin, 4 * n,
                                          r->on_device ? hipMemcpyDeviceToDevice
                                                       : hipMemcpyHostToDevice,
                                          s->copy);
            if (e == hipSuccess)
                e = hipEventRecord(r->ev_h2d, s->copy);
            if (e != hipSuccess)
                return hip_status(e, "upload");
        }
        r->need_wait = !r->in_buffers;
        r->k_next = 1;
        r->state = kActive;
        s->waiting.erase(next);
        s->active.push_back(r);
    }
    return CRB_OK;
}

static crb_status ensure_tables(crb_server *s, size_t bytes) {
    if (s->tab_cap >= bytes)
        return CRB_OK;
    size_t cap = s->tab_cap ? s->tab_cap : 1 << 16;
    while (cap < bytes)
        cap *= 2;
    if (s->h_tab)
        (void)hipHostFree(s->h_tab);
    if (s->d_tab)
        (void)hipFree(s->d_tab);
    s->h_tab = nullptr;
    s->d_tab = nullptr;
    s->tab_cap = 0;
    hipError_t e = hipHostMalloc((void **)&s->h_tab, cap, hipHostMallocDefault);
    if (e == hipSuccess)
        e = hipMalloc((void **)&s->d_tab, cap);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(CRB_ENOMEM, "round tables of %zu bytes: %s", cap, hipGetErrorString(e));
    }
    // the active list's counters: each round leaves them at zero
    e = hipMemsetAsync(s->d_tab, 0, (size_t)kListSegments * kTicketStride * 4, s->compute);
    if (e != hipSuccess)
        return hip_status(e, "hipMemsetAsync");
    s->tab_cap = cap;
    return CRB_OK;
}

// The tables of a round over `members`, on the device: the active list's counters (at the
// start, whatever the round), the frames (from the host), the tiles of the frames at iteration
// 1 and of the others, the list of those that have work, and the results (back to the host).
struct RoundTables {
    static constexpr size_t kCounters = (size_t)kListSegments * kTicketStride * 4;
    size_t nnew = 0, nold = 0, max_tiles = 0;      // tiles of either kind
    size_t o_frames = kCounters, o_new, o_old, o_active, o_st, bytes;
    explicit RoundTables(const std::vector<Request *> &members) {
        const size_t n = members.size();
        for (const Request *r : members) {
            const size_t t = (size_t)detect_tiles(r->H, r->W, kSumTY);
            if (r->k_next == 1)
                nnew += t;
            else
                nold += (t + 63) / 64 * 64;        // (launch_tiles: in groups of 64)
            max_tiles = t > max_tiles ? t : max_tiles;
        }
        auto al = [](size_t x) { return (x + 255) / 256 * 256; };
        o_new = o_frames + al(n * sizeof(DevFrame));
        o_old = o_new + al(nnew * sizeof(TileRef));
        o_active = o_old + al(nold * sizeof(TileRef));
        o_st = o_active + al(kListSegments * tile_list_cap(nold) * 4);
        bytes = o_st + al(2 * n * sizeof(long long));
    }
};

// one iteration for every active frame, at its own iteration index
static crb_status launch_round(crb_server *s) {
    const int n = (int)s->active.size();
    if (n == 0)
        return CRB_OK;
    const RoundTables t(s->active);
    crb_status st = ensure_tables(s, t.bytes);
    if (st != CRB_OK)
        return st;
    DevFrame *hf = reinterpret_cast<DevFrame *>(s->h_tab + t.o_frames);
    size_t inew = 0, iold = 0;
    bool narrow = false;
    for (int i = 0; i < n; ++i) {
        Request *r = s->active[i];
        narrow = narrow || r->df.narrow != 0;
        hf[i] = r->df;
        hf[i].k = r->k_next;
        const size_t nt = (size_t)detect_tiles(r->H, r->W, kSumTY);
        hf[i].list_base[0] = hf[i].list_base[1] = hf[i].list_base[2] = -1;
        if (r->k_next == 1) {
            hf[i].list_base[1] = (int)inew;
            inew += nt;
        } else {
            hf[i].tile_base = (int)iold;
            iold += (nt + 63) / 64 * 64;
        }
        if (r->need_wait) {
            hipError_t e = hipStreamWaitEvent(s->compute, r->ev_h2d, 0);
            if (e != hipSuccess)
                return hip_status(e, "hipStreamWaitEvent");
            r->need_wait = false;
        }
    }
    const DevFrame *dfr = reinterpret_cast<const DevFrame *>(s->d_tab + t.o_frames);
    TileRef *dnew = reinterpret_cast<TileRef *>(s->d_tab + t.o_new);
    TileRef *dold = reinterpret_cast<TileRef *>(s->d_tab + t.o_old);
    long long *dst = reinterpret_cast<long long *>(s->d_tab + t.o_st);
    const TileList active = {reinterpret_cast<unsigned int *>(s->d_tab + t.o_active),
                             reinterpret_cast<unsigned int *>(s->d_tab), kListSegments,
                             (int)tile_list_cap(t.nold)};
    DevFrame none;
    memset(&none, 0, sizeof(none));
    hipError_t e = hipMemcpyAsync(s->d_tab + t.o_frames, hf, n * sizeof(DevFrame),
                                  hipMemcpyHostToDevice, s->compute);
    // Rounds mix frames at different iterations.  Those at iteration 1 take the first detection
    // and then every tile; the others the tiles their marks name.
    const LaunchCfg cfg;
    const StepLists lists = {};
    if (e == hipSuccess)
        e = launch_tiles(dfr, n, t.max_tiles, nullptr, dnew, nullptr, dold, active, nullptr, 0,
                         s->compute);
    if (e == hipSuccess && t.nnew)
        e = launch_detect(dfr, dnew, (int)t.nnew, none, cfg, narrow, lists, nullptr, s->compute);
    if (e == hipSuccess && t.nnew)
        e = launch_step(dfr, dnew, (int)t.nnew, none, 1, false, narrow, lists, nullptr, s->compute);
    if (e == hipSuccess && t.nold)
        e = launch_step_active(dfr, dold, t.nold, narrow, active, s->compute);
    if (e == hipSuccess)
        e = launch_round_stats(dfr, n, dst, active, s->compute);
    if (e == hipSuccess)
        e = hipMemcpyAsync(s->h_tab + t.o_st, dst, 2 * n * sizeof(long long),
                           hipMemcpyDeviceToHost, s->compute);
    if (e == hipSuccess)
        e = hipEventRecord(s->ev_round, s->compute);
    if (e != hipSuccess)
        return hip_status(e, "round launch");
    s->round_members = s->active;
    s->round_busy = true;
    return CRB_OK;
}

// the round finished: advance frames, start downloads of finished ones
static crb_status finish_round(crb_server *s) {
    const int n = (int)s->round_members.size();
    const long long *stats = reinterpret_cast<const long long *>(
        s->h_tab + RoundTables(s->round_members).o_st);
    std::vector<Request *> still;
    for (int i = 0; i < n; ++i) {
        Request *r = s->round_members[i];
        const int k = r->k_next;
        const bool done = k >= r->niter || stats[2 * i] == 0;
        if (!done) {
            r->k_next = k + 1;
            still.push_back(r);
            continue;
        }
        r->state = kDraining;
        s->draining.push_back(r);
        if (r->in_buffers)
            continue;                  // (no event: the results are where they belong)
        // download the cleaned image and the mask once the round is complete
        crb_status st = get_event(s, &r->ev_d2h);
        if (st != CRB_OK)
            return st;
        const size_t npx = (size_t)r->H * r->W;
        hipError_t e = hipStreamWaitEvent(s->copy, s->ev_round, 0);
        void *dst_clean = r->direct ? (void *)r->host_clean : (void *)r->pin;
        void *dst_mask = r->direct ? (void *)r->host_mask : (void *)(r->pin + 4 * npx);
        const hipMemcpyKind kind = r->on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
        if (e == hipSuccess)
            e = hipMemcpyAsync(dst_clean, r->df.J, 4 * npx, kind, s->copy);
        if (e == hipSuccess)
            e = hipMemcpyAsync(dst_mask, r->df.mask, npx, kind, s->copy);
        if (e == hipSuccess)
            e = hipEventRecord(r->ev_d2h, s->copy);
        if (e != hipSuccess)
            return hip_status(e, "download");
    }
    // frames admitted while the round ran were appended after its members
    for (size_t i = s->round_members.size(); i < s->active.size(); ++i)
        still.push_back(s->active[i]);
    s->active.swap(still);
    s->round_members.clear();
    s->round_busy = false;
    return CRB_OK;
}

// completed requests: results in place, or their download finished
static crb_status collect(crb_server *s, int64_t *done_ids, double *done_latency,
                          int32_t max_done, int32_t *n_done) {
    for (size_t i = 0; i < s->draining.size() && *n_done < max_done;) {
        Request *r = s->draining[i];
        const hipError_t q = r->in_buffers ? hipSuccess : hipEventQuery(r->ev_d2h);
        if (q == hipErrorNotReady) {
            ++i;
            continue;
        }
        if (q != hipSuccess)
            return hip_status(q, "download event");
        const size_t npx = (size_t)r->H * r->W;
        if (!r->direct) {
            s->copies->copy(r->host_clean, r->pin, 4 * npx);
            s->copies->copy(r->host_mask, r->pin + 4 * npx, npx);
        }
        done_ids[*n_done] = r->id;
        done_latency[*n_done] = now_s() - r->t_submit;
        ++*n_done;
        s->draining.erase(s->draining.begin() + i);
        release_request(s, r);
    }
    return CRB_OK;
}

}  // namespace crb

extern "C" {

crb_status crb_server_create(size_t hbm_budget, int32_t max_slots, crb_server **out) {
    if (!out)
        return fail(CRB_EINVAL, "null out");
    *out = nullptr;
    if (hbm_budget == 0 || max_slots < 1)
        return fail(CRB_EINVAL, "budget must be > 0 and max_slots >= 1");
    crb_server *s = new (std::nothrow) crb_server();
    if (!s)
        return fail(CRB_ENOMEM, "host allocation failed");
    s->budget = hbm_budget;
    s->max_slots = max_slots;
    {
        unsigned hw = std::thread::hardware_concurrency();
        unsigned n = hw > 1 ? (hw < 9 ? hw - 1 : 7) : 0;
        s->copies = new (std::nothrow) CopyPool(n);
        if (!s->copies) {
            delete s;
            return fail(CRB_ENOMEM, "host allocation failed");
        }
    }
    hipError_t e = hipGetDevice(&s->device);
    if (e == hipSuccess)
        e = hipStreamCreateWithFlags(&s->compute, hipStreamNonBlocking);
    if (e == hipSuccess)
        e = hipStreamCreateWithFlags(&s->copy, hipStreamNonBlocking);
    if (e == hipSuccess)
        e = hipEventCreateWithFlags(&s->ev_round, hipEventDisableTiming);
    if (e != hipSuccess) {
        crb_server_destroy(s);
        return hip_status(e, "server setup");
    }
    *out = s;
    return ok();
}

crb_status crb_server_submit(crb_server *s, const float *host_img, int32_t H, int32_t W,
                             float gain, float readnoise, float sky, float sigclip, float sigfrac,
                             float objlim, int32_t niter, float *host_clean, uint8_t *host_mask,
                             int64_t *out_id) {
    const double t0 = now_s();
    if (!s || !host_img || !host_clean || !host_mask || !out_id)
        return fail(CRB_EINVAL, "null argument");
    crb_status st = check_frame_args(H, W, gain, readnoise, sky, sigclip, sigfrac, objlim, niter);
    if (st != CRB_OK)
        return st;
    const size_t npx = (size_t)H * (size_t)W;
    Request *r = new (std::nothrow) Request();
    if (!r)
        return fail(CRB_ENOMEM, "host allocation failed");
    r->H = H;
    r->W = W;
    r->gain = gain;
    r->readnoise = readnoise;
    r->sky = sky;
    r->sigclip = sigclip;
    r->sigfrac = sigfrac;
    r->objlim = objlim;
    r->niter = niter;
    r->host_clean = host_clean;
    r->host_mask = host_mask;
    r->t_submit = t0;
    r->dev_bytes = frame_dev_bytes(H, W);
    if (r->dev_bytes > s->budget) {
        delete r;
        return fail(CRB_EBUSY, "frame needs %zu bytes of device memory, budget is %zu",
                    frame_dev_bytes(H, W), s->budget);
    }
    r->pin_bytes = 5 * npx;
    r->host_img = host_img;
    const int ki = memory_kind(host_img, s->device), kc = memory_kind(host_clean, s->device),
              km = memory_kind(host_mask, s->device);
    if (ki < 0 || kc < 0 || km < 0 || (ki == 2) != (kc == 2) || (ki == 2) != (km == 2)) {
        delete r;
        return fail(CRB_EINVAL, "the image and both outputs must all be host memory or all "
                                "device memory of the server's device");
    }
    r->on_device = ki == 2;
    r->direct = ki > 0 && kc > 0 && km > 0;
    if (r->on_device) {
        const hipStream_t ts = thread_stream();
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        r->idle = hipStreamIsCapturing(ts, &cap) == hipSuccess &&
                  cap == hipStreamCaptureStatusNone && hipStreamQuery(ts) == hipSuccess;
        (void)hipGetLastError();
    }
    if (r->on_device)
        enter_spans(s, r);
    if (niter == 0 && r->on_device) {
        // nothing to compute: the result is the input, copied on the device (at once, unless
        // a request in the server is being cleaned in one of these buffers)
        if (!must_wait(s, r)) {
            hipError_t e = copy_niter0(s, r);
            if (e == hipSuccess)
                e = hipStreamSynchronize(s->copy);
            if (e != hipSuccess) {
                leave_spans(s, r);
                delete r;
                return hip_status(e, "niter 0 copy");
            }
            r->copied = true;
        }
    } else if (niter == 0) {       // nothing to compute: the result is the input
        memcpy(host_clean, host_img, 4 * npx);
        memset(host_mask, 0, npx);
        r->copied = true;
    }
    r->id = s->next_id++;
    *out_id = r->id;
    s->waiting.push_back(r);
    return ok();
}

crb_status crb_server_poll(crb_server *s, int64_t *done_ids, double *done_latency,
                           int32_t max_done, int32_t *n_done) {
    if (!s || !n_done || max_done < 0 || (max_done > 0 && (!done_ids || !done_latency)))
        return fail(CRB_EINVAL, "bad arguments");
    *n_done = 0;
    crb_status st;
    // requests with niter == 0 complete at once
    for (auto it = s->waiting.begin(); it != s->waiting.end();) {
        Request *r = *it;
        if (r->copied && *n_done < max_done) {
            done_ids[*n_done] = r->id;
            done_latency[*n_done] = now_s() - r->t_submit;
            ++*n_done;
            it = s->waiting.erase(it);
            release_request(s, r);
        } else {
            ++it;
        }
    }
    if ((st = collect(s, done_ids, done_latency, max_done, n_done)) != CRB_OK)
        return st;
    // the round in flight
    if (s->round_busy) {
        hipError_t q = hipEventQuery(s->ev_round);
        if (q == hipErrorNotReady) {
            if ((st = admit(s)) != CRB_OK)     // uploads overlap the running round
                return st;
            return ok();
        }
        if (q != hipSuccess)
            return hip_status(q, "round event");
        if ((st = finish_round(s)) != CRB_OK || (st = start_niter0(s)) != CRB_OK ||
            (st = collect(s, done_ids, done_latency, max_done, n_done)) != CRB_OK)
            return st;
    }
    if ((st = admit(s)) != CRB_OK)
        return st;
    if ((st = launch_round(s)) != CRB_OK)
        return st;
    return ok();
}

int32_t crb_server_pending(crb_server *s) {
    if (!s)
        return 0;
    return (int32_t)(s->waiting.size() + s->active.size() + s->draining.size());
}

void crb_server_destroy(crb_server *s) {
    if (!s)
        return;
    if (s->compute)
        (void)hipStreamSynchronize(s->compute);
    if (s->copy)
        (void)hipStreamSynchronize(s->copy);
    for (Request *r : s->waiting)
        release_request(s, r);
    for (Request *r : s->active)
        release_request(s, r);
    for (Request *r : s->draining)
        release_request(s, r);
    for (auto &kv : s->dev_free)
        (void)hipFree(kv.second);
    for (auto &kv : s->pin_free)
        (void)hipHostFree(kv.second);
    for (hipEvent_t ev : s->event_pool)
        (void)hipEventDestroy(ev);
    if (s->ev_round)
        (void)hipEventDestroy(s->ev_round);
    if (s->h_tab)
        (void)hipHostFree(s->h_tab);
    if (s->d_tab)
        (void)hipFree(s->d_tab);
    if (s->compute)
        (void)hipStreamDestroy(s->compute);
    if (s->copy)
        (void)hipStreamDestroy(s->copy);
    delete s->copies;
    delete s;
}

}  // extern "C"
