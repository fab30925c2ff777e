// Host bookkeeping of U(1) block-sparse tensors: sector tables and the block
// layouts declared in include/pdmrg.h.
#include "common.hpp"
#include "kernels.hpp"

#include <atomic>
#include <mutex>

namespace pdmrg {

static thread_local std::string g_last_error;
void set_last_error(const std::string &msg) { g_last_error = msg; }
const char *last_error_cstr() { return g_last_error.c_str(); }

Bond::Bond(const std::vector<int> &qs, const std::vector<int> &dims) : q(qs), dim(dims) {
    PD_REQUIRE(q.size() == dim.size(), PDMRG_EINVAL, "bond: charge / dimension count mismatch");
    off.resize(q.size());
    int64_t o = 0;
    for (size_t k = 0; k < q.size(); ++k) {
        PD_REQUIRE(dim[k] > 0, PDMRG_EINVAL, "bond: sector dimension must be positive");
        PD_REQUIRE(k == 0 || q[k] > q[k - 1], PDMRG_EINVAL, "bond: charges must be strictly ascending");
        off[k] = o;
        o += dim[k];
    }
    PD_REQUIRE(o < (1 << 30), PDMRG_EINVAL, "bond: dimension too large");
    total = (int)o;
    const int64_t range = q.empty() ? 0 : (int64_t)q.back() - q[0] + 1;
    if (range <= 8 * (int64_t)q.size() + 64) {
        at_.assign((size_t)range, -1);
        for (size_t k = 0; k < q.size(); ++k) at_[q[k] - q[0]] = (int32_t)k;
    }
}

Bond Bond::from(const pdmrg_bond *b) {
    PD_REQUIRE(b != nullptr && b->nsec >= 0, PDMRG_EINVAL, "bond: null descriptor");
    PD_REQUIRE(b->nsec == 0 || (b->q && b->dim), PDMRG_EINVAL, "bond: null arrays");
    return Bond(std::vector<int>(b->q, b->q + b->nsec), std::vector<int>(b->dim, b->dim + b->nsec));
}

Phys Phys::from(const pdmrg_phys *p) {
    PD_REQUIRE(p != nullptr && p->d > 0 && p->q != nullptr, PDMRG_EINVAL, "phys: bad descriptor");
    Phys r;
    r.q.assign(p->q, p->q + p->d);
    return r;
}

MpoSite MpoSite::from(const pdmrg_mpo_site *s) {
    PD_REQUIRE(s && s->W && s->dl && s->dr && s->Dl > 0 && s->Dr > 0 && s->d > 0, PDMRG_EINVAL,
               "mpo site: bad descriptor");
    MpoSite m;
    m.Dl = s->Dl; m.Dr = s->Dr; m.d = s->d;
    m.W.assign(s->W, s->W + (size_t)s->Dl * s->d * s->d * s->Dr);
    m.dl.assign(s->dl, s->dl + s->Dl);
    m.dr.assign(s->dr, s->dr + s->Dr);
    return m;
}

static SiteLayout generic_site_layout(const Bond &bl, const Bond &br, const Phys &p, bool two) {
    const int d = p.d();
    SiteLayout L;
    L.nphys = two ? d * d : d;
    const int ns = bl.nsec();
    L.base.resize(ns);
    L.rows.resize(ns);
    L.cols.resize(ns);
    L.colo.assign((size_t)ns * L.nphys, -1);
    L.width.assign((size_t)ns * L.nphys, 0);
    int64_t o = 0;
    for (int i = 0; i < ns; ++i) {
        int c = 0;
        for (int s = 0; s < L.nphys; ++s) {
            const int dq = two ? p.q[s / d] + p.q[s % d] : p.q[s];
            const int k = br.find(bl.q[i] + dq);
            if (k < 0) continue;
            L.colo[(size_t)i * L.nphys + s] = c;
            L.width[(size_t)i * L.nphys + s] = br.dim[k];
            c += br.dim[k];
        }
        L.base[i] = o;
        L.rows[i] = bl.dim[i];
        L.cols[i] = c;
        o += (int64_t)bl.dim[i] * c;
    }
    L.size = o;
    return L;
}

SiteLayout site_layout(const Bond &bl, const Bond &br, const Phys &p) {
    return generic_site_layout(bl, br, p, false);
}
SiteLayout two_site_layout(const Bond &bl, const Bond &br, const Phys &p) {
    return generic_site_layout(bl, br, p, true);
}

static EnvLayout generic_env_layout(const Bond &b, const std::vector<int> &deltas, int sign) {
    // L (sign +1): per ket sector q', rows = bra states of q' + delta_w;
    // R (sign -1): per bra sector q, rows = ket states of q - delta_w.
    EnvLayout E;
    E.D = (int)deltas.size();
    const int ns = b.nsec();
    E.base.resize(ns);
    E.rows.resize(ns);
    E.cols.resize(ns);
    E.rowo.assign((size_t)ns * E.D, -1);
    int64_t o = 0;
    for (int j = 0; j < ns; ++j) {
        int r = 0;
        for (int w = 0; w < E.D; ++w) {
            const int k = b.find(b.q[j] + sign * deltas[w]);
            if (k < 0) continue;
            E.rowo[(size_t)j * E.D + w] = r;
            r += b.dim[k];
        }
        E.base[j] = o;
        E.rows[j] = r;
        E.cols[j] = b.dim[j];
        o += (int64_t)r * b.dim[j];
    }
    E.size = o;
    return E;
}

EnvLayout env_l_layout(const Bond &b, const std::vector<int> &deltas) { return generic_env_layout(b, deltas, +1); }
EnvLayout env_r_layout(const Bond &b, const std::vector<int> &deltas) { return generic_env_layout(b, deltas, -1); }

// Caching device allocator behind DevBuf.  Sizes are rounded up to a size
// class: powers of two up to 1 MiB, above that multiples of one eighth of the
// power of two below the request (at most 12.5 % over the request, so a
// 1.8 GB environment takes 1.88 GB, not 2 GiB).  Released blocks go to a
// pending list and become reusable only after one device-wide
// synchronisation, so a block can never be handed out while a kernel launched
// before its release still uses it.  That synchronisation waits for every
// stream (concurrent regions included), so it is taken only once the pending
// blocks hold kRecycleBytes; below that a miss allocates a new block.  Cached
// blocks are kept until the process ends.
//
// The mutex guards only the host lists: hipMalloc, hipFree and the device
// synchronisation run with it released, so a thread that allocates never
// holds up the HIP calls of the other region threads.  Blocks moved out of
// the pending list are owned by the thread that synchronises; ones released
// meanwhile stay pending for the next round.
std::atomic<bool> g_alloc_poison{false};

namespace {
std::mutex g_cache_mu;   // the allocator serves every host thread of the process

// debugging aid: NaN bytes in a buffer about to be handed out
void poison(void *ptr, size_t bytes) {
    if (!g_alloc_poison.load(std::memory_order_relaxed)) return;
    HIP_OK(hipDeviceSynchronize());
    HIP_OK(hipMemset(ptr, 0xFF, bytes));
    HIP_OK(hipDeviceSynchronize());
}
constexpr size_t kRecycleBytes = size_t(2) << 30;
using BlockMap = std::map<std::pair<int, size_t>, std::vector<void *>>;
struct DeviceCache {
    BlockMap free_, pending_;
    size_t pending_bytes = 0;
    int64_t in_use = 0, peak = 0, cached = 0;   // bytes (size classes)
};
DeviceCache &cache() {
    static DeviceCache *c = new DeviceCache();   // never destroyed: no hipFree after runtime teardown
    return *c;
}
}  // namespace

size_t size_class(size_t n) {
    size_t c = 256;
    while (c < n && c < (size_t(1) << 20)) c <<= 1;
    if (c >= n) return c;
    size_t p = size_t(1) << 20;
    while (p * 2 <= n) p <<= 1;
    const size_t step = p / 8;
    return (n + step - 1) / step * step;
}

// The idle blocks behind ListBuf (below): freed, and their bytes.
void list_pool_trim();
int64_t list_pool_idle();

namespace {
void count_in_use(int64_t bytes) {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    DeviceCache &c = cache();
    c.in_use += bytes;
    c.peak = std::max(c.peak, c.in_use);
}
// under g_cache_mu: a cached block of class `cls` on `dev`, or null
void *take_free(DeviceCache &c, int dev, size_t cls) {
    auto it = c.free_.find(std::make_pair(dev, cls));
    if (it == c.free_.end() || it->second.empty()) return nullptr;
    void *p = it->second.back();
    it->second.pop_back();
    return p;
}
void merge_into(BlockMap &dst, BlockMap &src) {
    for (auto &kv : src) {
        auto &d = dst[kv.first];
        d.insert(d.end(), kv.second.begin(), kv.second.end());
    }
    src.clear();
}
}  // namespace

void DevBuf::alloc(size_t n) {
    if (n == 0) n = 16;
    int dev = 0;
    HIP_OK(hipGetDevice(&dev));
    const size_t cls = size_class(n);
    DeviceCache &c = cache();
    void *p = nullptr;
    BlockMap recycled;
    {
        std::lock_guard<std::mutex> lk(g_cache_mu);
        p = take_free(c, dev, cls);
        if (!p && c.pending_bytes >= kRecycleBytes) {
            recycled.swap(c.pending_);
            c.pending_bytes = 0;
        }
    }
    if (!recycled.empty()) {
        // every kernel that used these blocks was launched before they were
        // released, hence before this synchronisation
        HIP_OK(hipDeviceSynchronize());
        std::lock_guard<std::mutex> lk(g_cache_mu);
        merge_into(c.free_, recycled);
        p = take_free(c, dev, cls);
    }
    if (!p) {
        hipError_t e = hipMalloc(&p, cls);
        if (e != hipSuccess) {
            // out of memory: give every cached block back to the runtime and retry once
            (void)hipGetLastError();
            BlockMap all;
            {
                std::lock_guard<std::mutex> lk(g_cache_mu);
                merge_into(all, c.free_);
                merge_into(all, c.pending_);
                c.pending_bytes = 0;
            }
            HIP_OK(hipDeviceSynchronize());
            for (auto &kv : all)
                for (void *q : kv.second) (void)hipFree(q);
            list_pool_trim();
            p = nullptr;
            e = hipMalloc(&p, cls);
        }
        if (e != hipSuccess) {
            ptr = nullptr;
            bytes = 0;
            throw Error(PDMRG_ENOMEM, "hipMalloc of " + std::to_string(cls) + " bytes failed: " + hipGetErrorString(e));
        }
    }
    ptr = p;
    bytes = cls;
    count_in_use((int64_t)cls);
    poison(ptr, cls);
}

void alloc_stats(int64_t *in_use, int64_t *peak, int64_t *cached) {
    int64_t held = list_pool_idle();
    std::lock_guard<std::mutex> lk(g_cache_mu);
    DeviceCache &c = cache();
    for (auto *m : {&c.free_, &c.pending_})
        for (auto &kv : *m) held += (int64_t)kv.first.second * (int64_t)kv.second.size();
    if (in_use) *in_use = c.in_use;
    if (peak) *peak = c.peak;
    if (cached) *cached = held;
}

void alloc_reset_peak() {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    cache().peak = cache().in_use;
}

void DevBuf::release() {
    if (ptr) {
        int dev = 0;
        if (hipGetDevice(&dev) == hipSuccess) {
            std::lock_guard<std::mutex> lk(g_cache_mu);
            DeviceCache &c = cache();
            c.pending_[std::make_pair(dev, bytes)].push_back(ptr);
            c.pending_bytes += bytes;
            c.in_use -= (int64_t)bytes;
        }
    }
    ptr = nullptr;
    bytes = 0;
}

// ---------------------------------------------------------------- work lists to the device, small results back
// A plan's lists come to some 0.1 to 1 MB in 8 to 10 arrays.  Copied one by one
// from pageable memory they cost 20 to 50 us each (the runtime stages them and
// waits); packed and read by a kernel they cost one memcpy, a launch and the bus.
// (24 x 8 cylinder, m = 2000, one environment update: 0.23 ms of copies; with the
// lists of later products built while the first one runs, the call went from
// 0.89 ms to 0.30, of which the kernels are 0.26.)  Results of a few words or kilobytes that the host waits for come back the
// same way.
//
// Pinned blocks are reused once the event behind their last copy has passed.
// All of them together are bounded; a list that finds no block, or is larger
// than one, goes through the runtime's pageable copy and waits for it; idle
// blocks of other sizes make room first.  The device side of lists
// that live within one call (ListBuf) is kept by stream, also bounded: a block
// from the allocator above would be a new one each time (75 us of hipMalloc for
// 0.5 MB), for it has to wait for the whole device before it is used again.  The
// blocks of a stream go with the last context on it, all of them when memory is
// short.
namespace {
constexpr size_t kPinnedBytes = size_t(64) << 20, kPinnedBlock = size_t(8) << 20;
constexpr size_t kListBytes = size_t(256) << 20, kListBlock = size_t(8) << 20;
struct Pinned {
    void *ptr = nullptr;
    hipEvent_t done = nullptr;
    int dev = 0;
    size_t bytes = 0;
};
std::mutex g_pin_mu;
struct ListBlock {
    void *ptr;
    size_t bytes;
    int dev;
    hipStream_t s;
};
struct PinPool {
    std::vector<Pinned> blocks;     // not in use by a thread, oldest copy first
    size_t bytes = 0;               // of all blocks
    std::vector<ListBlock> lists;   // device blocks, free for lists on their stream
    size_t list_bytes = 0;          // of all of them
    std::map<std::pair<int, hipStream_t>, int> users;   // contexts on a stream
    int holders = 0;
};
PinPool &pins() {
    static PinPool *p = new PinPool();
    return *p;
}

void pin_free(Pinned &b) {
    (void)hipEventSynchronize(b.done);
    (void)hipEventDestroy(b.done);
    (void)hipHostFree(b.ptr);
}

// A block of at least n bytes whose last copy has ended, or one without ptr.
Pinned pin_take(int dev, size_t n) {
    size_t cls = size_t(64) << 10;
    while (cls < n) cls <<= 2;
    cls = std::min(cls, kPinnedBlock);
    std::vector<Pinned> idle;
    bool room = false;
    {
        std::lock_guard<std::mutex> lk(g_pin_mu);
        PinPool &p = pins();
        int busy = 0;
        for (size_t k = 0; k < p.blocks.size() && busy < 4; ++k) {
            if (p.blocks[k].dev != dev || p.blocks[k].bytes != cls) continue;
            if (hipEventQuery(p.blocks[k].done) == hipSuccess) {
                Pinned b = p.blocks[k];
                p.blocks.erase(p.blocks.begin() + (ptrdiff_t)k);
                return b;
            }
            (void)hipGetLastError();   // not ready; the later ones hardly are
            ++busy;
        }
        for (size_t k = 0; k < p.blocks.size() && p.bytes + cls > kPinnedBytes;) {
            if (hipEventQuery(p.blocks[k].done) != hipSuccess) {
                (void)hipGetLastError();
                ++k;
                continue;
            }
            idle.push_back(p.blocks[k]);
            p.bytes -= p.blocks[k].bytes;
            p.blocks.erase(p.blocks.begin() + (ptrdiff_t)k);
        }
        room = p.bytes + cls <= kPinnedBytes;
        if (room) p.bytes += cls;
    }
    for (Pinned &b : idle) pin_free(b);
    if (!room) return Pinned{};
    Pinned b;
    b.dev = dev;
    b.bytes = cls;
    if (hipHostMalloc(&b.ptr, cls, hipHostMallocCoherent) != hipSuccess) {
        b.ptr = nullptr;
    } else if (hipEventCreateWithFlags(&b.done, hipEventDisableTiming) != hipSuccess) {
        (void)hipHostFree(b.ptr);
        b.ptr = nullptr;
    }
    if (!b.ptr) {
        (void)hipGetLastError();
        std::lock_guard<std::mutex> lk(g_pin_mu);
        pins().bytes -= cls;
    }
    return b;
}

// Out of the pool, under g_pin_mu: the idle list blocks that `which` chooses.
template <class F>
std::vector<ListBlock> lists_out(F which) {
    PinPool &p = pins();
    std::vector<ListBlock> out;
    for (size_t k = p.lists.size(); k-- > 0;) {
        if (!which(p.lists[k])) continue;
        out.push_back(p.lists[k]);
        p.list_bytes -= p.lists[k].bytes;
        p.lists.erase(p.lists.begin() + (ptrdiff_t)k);
    }
    return out;
}
}  // namespace

void list_pool_trim() {
    std::vector<ListBlock> lists;
    {
        std::lock_guard<std::mutex> lk(g_pin_mu);
        lists = lists_out([](const ListBlock &) { return true; });
    }
    for (ListBlock &b : lists) (void)hipFree(b.ptr);   // waits for the device
}
int64_t list_pool_idle() {
    std::lock_guard<std::mutex> lk(g_pin_mu);
    int64_t n = 0;
    for (const ListBlock &b : pins().lists) n += (int64_t)b.bytes;
    return n;
}

StageHold::StageHold() {
    std::lock_guard<std::mutex> lk(g_pin_mu);
    ++pins().holders;
}
void StageHold::bind(int device, hipStream_t stream) {
    std::lock_guard<std::mutex> lk(g_pin_mu);
    dev = device;
    s = stream;
    bound = true;
    ++pins().users[{dev, s}];
}
StageHold::~StageHold() {
    std::vector<Pinned> all;
    std::vector<ListBlock> lists;
    {
        std::lock_guard<std::mutex> lk(g_pin_mu);
        PinPool &p = pins();
        const bool last = --p.holders == 0;
        bool dead = false;   // no context left on its stream
        if (bound && --p.users[{dev, s}] == 0) {
            p.users.erase({dev, s});
            dead = true;
        }
        lists = lists_out([&](const ListBlock &b) { return last || (dead && b.dev == dev && b.s == s); });
        if (last) all.swap(p.blocks);
        for (const Pinned &b : all) p.bytes -= b.bytes;
    }
    for (Pinned &b : all) pin_free(b);
    for (ListBlock &b : lists) (void)hipFree(b.ptr);   // waits for the device
}

void ListBuf::ensure(size_t n, hipStream_t stream) {
    if (ptr && n <= bytes && s == stream) return;
    release();
    int d = 0;
    HIP_OK(hipGetDevice(&d));
    size_t cls = size_t(4) << 10;
    while (cls < n) cls <<= 1;
    // hipStreamPerThread is one handle for as many streams as there are threads:
    // a block freed on one is not ordered before the list copies of another
    if (cls > kListBlock || stream == hipStreamPerThread) {
        large.ensure(n);
        ptr = large.ptr;
        bytes = large.bytes;
        s = stream;
        return;
    }
    bool room = false;
    {
        std::lock_guard<std::mutex> lk(g_pin_mu);
        PinPool &p = pins();
        for (size_t k = p.lists.size(); k-- > 0 && !ptr;) {
            const ListBlock &b = p.lists[k];
            if (b.dev != d || b.s != stream || b.bytes != cls) continue;
            ptr = b.ptr;
            p.lists.erase(p.lists.begin() + (ptrdiff_t)k);
        }
        room = ptr || p.list_bytes + cls <= kListBytes;
        if (!ptr && room) p.list_bytes += cls;
    }
    if (!ptr && room && hipMalloc(&ptr, cls) != hipSuccess) {
        (void)hipGetLastError();
        ptr = nullptr;
        room = false;
        std::lock_guard<std::mutex> lk(g_pin_mu);
        pins().list_bytes -= cls;
    }
    if (!room) {   // from the allocator, which gives its cache back when memory is short
        large.ensure(cls);
        ptr = large.ptr;
    }
    bytes = cls;
    dev = d;
    s = stream;
    if (large.ptr) return;
    count_in_use((int64_t)cls);
    poison(ptr, cls);
}

void ListBuf::release() {
    if (ptr && !large.ptr) {
        count_in_use(-(int64_t)bytes);
        std::lock_guard<std::mutex> lk(g_pin_mu);
        pins().lists.push_back(ListBlock{ptr, bytes, dev, s});
    }
    large.release();
    ptr = nullptr;
    bytes = 0;
}

namespace {
// Back to the pool; what used the block on `s` has been launched.
void pin_give(const Pinned &b, hipStream_t s) {
    const bool ok = hipEventRecord(b.done, s) == hipSuccess;
    if (!ok) (void)hipStreamSynchronize(s);   // no event to wait for
    {
        std::lock_guard<std::mutex> lk(g_pin_mu);
        pins().blocks.push_back(b);
    }
    PD_REQUIRE(ok, PDMRG_EHIP, "pinned copy: event record failed");
}
}  // namespace

void read_back(const std::vector<HostCopy> &parts, hipStream_t s) {
    size_t total = 0;
    for (const HostCopy &p : parts) total += (p.bytes + 255) & ~size_t(255);
    int dev = 0;
    HIP_OK(hipGetDevice(&dev));
    Pinned b;
    if (total > 0 && total <= kPinnedBlock) b = pin_take(dev, total);
    size_t at = 0;
    hipError_t e = hipSuccess;
    for (const HostCopy &p : parts) {
        if (p.bytes == 0 || e != hipSuccess) continue;
        e = b.ptr ? launch_list_copy(static_cast<char *>(b.ptr) + at, p.src, p.bytes, s)
                  : hipMemcpyAsync(p.dst, p.src, p.bytes, hipMemcpyDeviceToHost, s);
        at += (p.bytes + 255) & ~size_t(255);
    }
    const hipError_t es = hipStreamSynchronize(s);
    if (e == hipSuccess) e = es;
    if (b.ptr) {
        at = 0;
        for (const HostCopy &p : parts) {
            if (e != hipSuccess) break;
            if (p.bytes) std::memcpy(p.dst, static_cast<char *>(b.ptr) + at, p.bytes);
            at += (p.bytes + 255) & ~size_t(255);
        }
        std::lock_guard<std::mutex> lk(g_pin_mu);   // its event has passed: no copy of it is under way
        pins().blocks.push_back(b);
    }
    HIP_OK(e);
}

void ListStage::flush(DevBuf &buf, hipStream_t s) {
    buf.ensure(std::max<size_t>(total_, 16));
    copy(buf.as<char>(), s);
}
void ListStage::flush(ListBuf &buf, hipStream_t s) {
    buf.ensure(std::max<size_t>(total_, 16), s);
    copy(buf.as<char>(), s);
}

void ListStage::copy(char *dst, hipStream_t s) {
    int dev = 0;
    HIP_OK(hipGetDevice(&dev));
    Pinned b;
    if (total_ > 0 && total_ <= kPinnedBlock) b = pin_take(dev, total_);
    hipError_t e = hipSuccess;
    for (const Part &pt : parts_) {
        *pt.dst = dst + pt.at;
        if (pt.bytes == 0) continue;
        if (b.ptr) std::memcpy(static_cast<char *>(b.ptr) + pt.at, pt.src, pt.bytes);
        else if (e == hipSuccess) e = hipMemcpyAsync(dst + pt.at, pt.src, pt.bytes, hipMemcpyHostToDevice, s);
    }
    if (b.ptr) {
        e = launch_list_copy(dst, b.ptr, total_, s);
        pin_give(b, s);
    } else if (total_ > 0) {
        // the runtime may still be reading the host arrays
        const hipError_t es = hipStreamSynchronize(s);
        if (e == hipSuccess) e = es;
    }
    parts_.clear();
    total_ = 0;
    HIP_OK(e);
}

void check_grid(int64_t blocks, int threads, const char *what) {
    PD_REQUIRE(blocks >= 0 && blocks * (int64_t)threads < (int64_t(1) << 32), PDMRG_ESHAPE,
               std::string(what) + ": launch grid beyond 2^32 work-items");
}

// ---------------------------------------------------------------- worker pool
WorkerPool::~WorkerPool() {
    {
        std::lock_guard<std::mutex> lk(mu_);
        quit_ = true;
    }
    cv_work_.notify_all();
    for (auto &t : threads_) t.join();
}

void WorkerPool::loop(int k) {
    std::unique_lock<std::mutex> lk(mu_);
    while (true) {
        cv_work_.wait(lk, [&] { return quit_ || ready_[k]; });
        if (!ready_[k]) return;   // quit with nothing left to run
        const std::function<void(int)> *fn = job_[k];
        ready_[k] = 0;
        lk.unlock();
        (void)hipSetDevice(device_);   // jobs select the device again and report a failure
        (*fn)(k);
        lk.lock();
        if (--pending_ == 0) cv_done_.notify_all();
    }
}

void WorkerPool::run(int n, const std::function<void(int)> &fn) {
    if (n <= 0) return;
    std::unique_lock<std::mutex> lk(mu_);
    while ((int)threads_.size() < n) {
        const int k = (int)threads_.size();
        job_.push_back(nullptr);
        ready_.push_back(0);
        threads_.emplace_back([this, k] { loop(k); });
    }
    for (int k = 0; k < n; ++k) {
        job_[k] = &fn;
        ready_[k] = 1;
    }
    pending_ = n;
    cv_work_.notify_all();
    cv_done_.wait(lk, [&] { return pending_ == 0; });
}

}  // namespace pdmrg
