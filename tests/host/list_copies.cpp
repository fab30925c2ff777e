// Host checks of the list and result copies of csrc/layout.cpp on a stand-in
// for the HIP runtime: device memory is host memory, and what is launched on a
// stream waits in that stream's queue until the check runs it, so every order
// that the real streams allow can be tried.  hipStreamPerThread stands for a
// queue of each thread, as in the runtime.  One check per run: argv[1].
#include "../../paper_1301_3494_amd/csrc/common.hpp"
#include "../../paper_1301_3494_amd/csrc/kernels.hpp"

#include <cstdio>
#include <cstdlib>
#include <deque>
#include <set>

using namespace pdmrg;

// ---------------------------------------------------------------- the stand-in
namespace {
using Queue = std::deque<std::function<void()>>;
std::mutex g_mu;
std::map<std::pair<hipStream_t, std::thread::id>, Queue> g_queues;
std::map<void *, size_t> g_device;     // live allocations
std::set<void *> g_pinned;
size_t g_device_bytes = 0, g_device_limit = size_t(-1);
int g_pageable = 0;                    // copies past the pinned blocks

Queue &queue(hipStream_t s) {
    return g_queues[{s, s == hipStreamPerThread ? std::this_thread::get_id() : std::thread::id()}];
}
void push(hipStream_t s, std::function<void()> f) {
    std::lock_guard<std::mutex> lk(g_mu);
    queue(s).push_back(std::move(f));
}
void run_one(Queue &q) {
    if (q.empty()) return;
    auto f = std::move(q.front());
    q.pop_front();
    f();
}
void run_all(Queue &q) {
    while (!q.empty()) run_one(q);
}
struct Event {
    bool recorded = false, passed = true;
};

#define CHECK(c)                                                                   \
    do {                                                                           \
        if (!(c)) {                                                                \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #c);                    \
            std::exit(1);                                                          \
        }                                                                          \
    } while (0)
}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (g_device_bytes + n > g_device_limit) return hipErrorOutOfMemory;
    g_device[*p = std::malloc(n)] = n;
    g_device_bytes += n;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
    std::lock_guard<std::mutex> lk(g_mu);
    for (auto &q : g_queues) run_all(q.second);
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    (void)hipDeviceSynchronize();
    std::lock_guard<std::mutex> lk(g_mu);
    CHECK(g_device.count(p) == 1);
    g_device_bytes -= g_device[p];
    g_device.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemset(void *p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_pinned.insert(*p = std::malloc(n));
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    std::lock_guard<std::mutex> lk(g_mu);
    CHECK(g_pinned.erase(p) == 1);
    std::free(p);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = reinterpret_cast<hipEvent_t>(new Event());
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<Event *>(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    auto *ev = reinterpret_cast<Event *>(e);
    ev->passed = false;
    push(s, [ev] { ev->passed = true; });
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) { return reinterpret_cast<Event *>(e)->passed ? hipSuccess : hipErrorNotReady; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipDeviceSynchronize(); }
hipError_t hipStreamSynchronize(hipStream_t s) {
    std::lock_guard<std::mutex> lk(g_mu);
    run_all(queue(s));
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind, hipStream_t s) {
    ++g_pageable;
    push(s, [=] { std::memcpy(dst, src, n); });
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in error"; }
}

namespace pdmrg {
bool g_fail_copies = false;
hipError_t launch_list_copy(void *dst, const void *src, size_t n, hipStream_t s) {
    if (g_fail_copies) return hipErrorLaunchFailure;
    push(s, [=] { std::memcpy(dst, src, n); });
    return hipSuccess;
}
}  // namespace pdmrg

// ---------------------------------------------------------------- the checks
namespace {
// A "kernel" on s that reads the list behind `list` into `out`.
void launch_reader(const int *list, std::vector<int> &out, hipStream_t s) {
    push(s, [=, &out] { std::copy(list, list + out.size(), out.begin()); });
}

// Two threads with a context each on hipStreamPerThread: one thread's list is
// released once its kernel is launched, the other's copy runs between the first
// one's copy and kernel.
void per_thread_streams() {
    StageHold hold;
    const hipStream_t s = hipStreamPerThread;
    std::vector<int> list_a(100, 1), list_b(100, 2), seen_a(100), seen_b(100);
    {
        ListBuf d;
        upload_list(d, list_a, s);
        launch_reader(d.as<int>(), seen_a, s);
    }
    run_one(queue(s));   // A's copy
    std::thread b([&] {
        ListBuf d;
        upload_list(d, list_b, s);
        launch_reader(d.as<int>(), seen_b, s);
        CHECK(hipStreamSynchronize(s) == hipSuccess);
    });
    b.join();
    CHECK(hipStreamSynchronize(s) == hipSuccess);   // A's kernel
    CHECK(seen_a == list_a && seen_b == list_b);
}

// The same on ordinary streams: the block of a released list goes to the next
// list on its stream and to no other stream's.
void ordinary_streams() {
    StageHold hold;
    int h1, h2;
    const auto s1 = reinterpret_cast<hipStream_t>(&h1), s2 = reinterpret_cast<hipStream_t>(&h2);
    std::vector<int> a(100, 1), b(100, 2), c(100, 3), seen_a(100), seen_b(100), seen_c(100);
    void *pa, *pb, *pc;
    {
        ListBuf d;
        upload_list(d, a, s1);
        pa = d.ptr;
        launch_reader(d.as<int>(), seen_a, s1);
    }
    {
        ListBuf d;
        upload_list(d, b, s2);
        pb = d.ptr;
        launch_reader(d.as<int>(), seen_b, s2);
    }
    run_all(queue(s2));
    {
        ListBuf d;
        upload_list(d, c, s1);
        pc = d.ptr;
        launch_reader(d.as<int>(), seen_c, s1);
    }
    run_all(queue(s1));
    CHECK(pa != pb && pa == pc);
    CHECK(seen_a == a && seen_b == b && seen_c == c);
}

// A copy that could not be launched is an error, not the last copy's contents;
// its block is there for the next one.
void failed_copies() {
    StageHold hold;
    double src = 7.0, dst = 0.0;
    read_back({{&dst, &src, sizeof dst}}, nullptr);
    CHECK(dst == 7.0 && g_pinned.size() == 1);
    auto throws = [](auto &&f) {
        try {
            f();
        } catch (const Error &e) {
            return e.code == PDMRG_EHIP;
        }
        return false;
    };
    src = 8.0;
    g_fail_copies = true;
    dst = 1.0;
    CHECK(throws([&] { read_back({{&dst, &src, sizeof dst}}, nullptr); }) && dst == 1.0);
    CHECK(throws([&] {
        ListBuf d;
        upload_list(d, std::vector<int>(10, 1), nullptr);
    }));
    g_fail_copies = false;
    CHECK(hipDeviceSynchronize() == hipSuccess);
    read_back({{&dst, &src, sizeof dst}}, nullptr);
    CHECK(dst == 8.0 && g_pinned.size() == 1);
}

// The host arrays are free once the lists are on their way, whichever way that
// is: through a pinned block, or past it for lists that no block holds and once
// all blocks are in use.
void host_arrays_are_free() {
    StageHold hold;
    auto check = [](size_t n) {
        std::vector<int> list(n, 5), seen(n);
        ListBuf d;
        upload_list(d, list, nullptr);
        launch_reader(d.as<int>(), seen, nullptr);
        std::fill(list.begin(), list.end(), -1);
        CHECK(hipStreamSynchronize(nullptr) == hipSuccess);
        CHECK(seen == std::vector<int>(n, 5));
    };
    check(1000);
    check(size_t(5) << 20);   // 20 MB
    // pinned blocks whose copies have not run
    int h;
    const auto busy = reinterpret_cast<hipStream_t>(&h);
    std::vector<std::unique_ptr<ListBuf>> bufs;
    const std::vector<int> big(size_t(3) << 19, 1);   // 6 MB
    for (int k = 0; k < 12; ++k) {
        bufs.emplace_back(new ListBuf());
        upload_list(*bufs.back(), big, busy);
        check(1000);
        check(size_t(1) << 20);
    }
    CHECK(hipDeviceSynchronize() == hipSuccess);
}

// Contexts that come and go on streams of their own while one lives on: the
// blocks of a stream go with the last context on it, and lists do not end up in
// the allocator.
void dead_streams() {
    StageHold keep;
    keep.bind(0, nullptr);
    const std::vector<int> list(size_t(1) << 20, 3);   // 4 MB
    std::vector<int> handles(200);
    auto use = [&](hipStream_t s) {
        ListBuf d;
        upload_list(d, list, s);
        CHECK(!d.large.ptr);
    };
    use(nullptr);
    const size_t mine = g_device_bytes;
    for (int &h : handles) {
        const auto s = reinterpret_cast<hipStream_t>(&h);
        StageHold one;
        one.bind(0, s);
        use(s);
        {
            StageHold two;   // another context on that stream
            two.bind(0, s);
            use(s);
        }
        CHECK(hipStreamSynchronize(s) == hipSuccess);
        CHECK(g_device_bytes == 2 * mine);
    }
    CHECK(g_device_bytes == mine);
    use(nullptr);
    CHECK(g_device_bytes == mine);
}

// Idle list blocks are counted as held for reuse, blocks in use as in use, and
// they are given back when an allocation fails.
void list_memory() {
    StageHold hold;
    int64_t in_use, peak, cached;
    {
        ListBuf d;
        upload_list(d, std::vector<int>(size_t(1) << 20, 3), nullptr);   // 4 MB
        alloc_stats(&in_use, &peak, &cached);
        CHECK(in_use == int64_t(4) << 20 && peak == in_use && cached == 0);
    }
    alloc_stats(&in_use, &peak, &cached);
    CHECK(in_use == 0 && cached == int64_t(4) << 20);
    g_device_limit = size_t(6) << 20;
    DevBuf b(size_t(5) << 20);
    CHECK(b.ptr && g_device_bytes == size_t(5) << 20);
    alloc_stats(&in_use, &peak, &cached);
    CHECK(in_use == int64_t(5) << 20 && cached == 0);
    // and a list that finds no memory of its own takes it from the allocator's cache
    b.release();
    ListBuf d;
    upload_list(d, std::vector<int>(size_t(1) << 20, 3), nullptr);
    CHECK(d.ptr && g_device_bytes <= g_device_limit);
}

// Large lists that have used up the pinned memory leave it to small ones.
void pinned_sizes() {
    StageHold hold;
    const std::vector<int> big(size_t(3) << 19, 1), small(100, 2);   // 6 MB
    {
        std::vector<std::unique_ptr<ListBuf>> bufs;
        for (int k = 0; k < 8; ++k) {
            bufs.emplace_back(new ListBuf());
            upload_list(*bufs.back(), big, nullptr);
        }
    }
    CHECK(g_pageable == 0 && g_pinned.size() == 8);
    CHECK(hipDeviceSynchronize() == hipSuccess);
    for (int k = 0; k < 3; ++k) {
        ListBuf d;
        upload_list(d, small, nullptr);
    }
    CHECK(g_pageable == 0);
}
}  // namespace

int main(int argc, char **argv) {
    const std::map<std::string, void (*)()> checks = {
        {"per_thread_streams", per_thread_streams},
        {"ordinary_streams", ordinary_streams},
        {"failed_copies", failed_copies},
        {"host_arrays_are_free", host_arrays_are_free},
        {"dead_streams", dead_streams},
        {"list_memory", list_memory},
        {"pinned_sizes", pinned_sizes},
    };
    const auto it = checks.find(argc > 1 ? argv[1] : "");
    CHECK(it != checks.end());
    it->second();
    std::printf("ok\n");
    return 0;
}
