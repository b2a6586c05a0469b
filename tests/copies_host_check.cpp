// copies_to_host (csrc/host.hpp) on the CPU, against a model of the HIP calls it
// makes: streams are queues whose work runs when somebody waits for them, and
// hipStreamPerThread is another queue in every thread, and an event can be recorded
// only on streams of the device on which it was created.  usage: <exe> <case>
#include "../paper_1511_04633_amd/csrc/host.hpp"

#include <cstdarg>
#include <cstdio>
#include <deque>
#include <functional>
#include <map>
#include <mutex>

namespace {

struct Queue {
    std::deque<std::function<void()>> work;
    size_t pushed = 0, done = 0;
};
std::mutex lock;
std::map<std::pair<hipStream_t, std::thread::id>, Queue> queues;

Queue &queue_of(hipStream_t s)
{
    return queues[{s, s == hipStreamPerThread ? std::this_thread::get_id() : std::thread::id()}];
}
void push(hipStream_t s, std::function<void()> f)
{
    std::lock_guard<std::mutex> g(lock);
    Queue &q = queue_of(s);
    q.work.push_back(std::move(f));
    ++q.pushed;
}
void run(Queue &q, size_t upto)  // with the lock held
{
    while (q.done < upto) {
        q.work.front()();
        q.work.pop_front();
        ++q.done;
    }
}
thread_local int device = 0;
std::map<const void *, size_t> pinned;  // by the caller: begin, bytes
size_t staged = 0;                      // bytes of pinned memory that the code allocated
size_t waits = 0;                       // for a stream
std::map<hipStream_t, int> device_of;  // 0 for a stream not in it
struct Event {
    int device;
    Queue *q = nullptr;
    size_t at = 0;
};

}  // namespace

extern "C" {
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    push(st, [=] { std::memcpy(d, s, n); });
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s)
{
    std::lock_guard<std::mutex> g(lock);
    Queue &q = queue_of(s);
    run(q, q.pushed);
    ++waits;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    *e = reinterpret_cast<hipEvent_t>(new Event{device});
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    std::lock_guard<std::mutex> g(lock);
    Event *ev = reinterpret_cast<Event *>(e);
    if (ev->device != device_of[s])
        return hipErrorInvalidHandle;
    ev->q = &queue_of(s);
    ev->at = ev->q->pushed;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    std::lock_guard<std::mutex> g(lock);
    Event *ev = reinterpret_cast<Event *>(e);
    if (ev->q)
        run(*ev->q, ev->at);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e)
{
    delete reinterpret_cast<Event *>(e);
    return hipSuccess;
}
hipError_t hipSetDevice(int d)
{
    device = d;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = device;
    return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t *d)
{
    std::lock_guard<std::mutex> g(lock);
    *d = device_of[s];
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = std::malloc(n);
    staged += n;
    return hipSuccess;
}
hipError_t hipHostFree(void *p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    for (const auto &r : pinned)
        if (p >= r.first && p < static_cast<const char *>(r.first) + r.second) {
            a->type = hipMemoryTypeHost;
            return hipSuccess;
        }
    return hipErrorInvalidValue;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
}

namespace lbmx {
namespace host {
lbmx_status fail(lbmx_status s, const char *fmt, ...)
{
    va_list a;
    va_start(a, fmt);
    std::vfprintf(stderr, fmt, a);
    va_end(a);
    return s;
}
}  // namespace host
}  // namespace lbmx

using namespace lbmx::host;

// Arrays of doubles that work enqueued on `s` fills, copied to the host (the first
// `pins` of them into memory that the caller has pinned): exit status 0 where each
// arrives whole and as it was filled.
static int copies(hipStream_t s, const std::vector<size_t> &sizes, size_t pins = 0)
{
    std::vector<std::vector<double>> dev, host;
    for (size_t n : sizes) {
        dev.emplace_back(n, -1.0);
        host.emplace_back(n, -2.0);
        if (host.size() <= pins)
            pinned[host.back().data()] = n * sizeof(double);
    }
    push(s, [&] {
        for (size_t k = 0; k < dev.size(); ++k)
            for (size_t i = 0; i < dev[k].size(); ++i)
                dev[k][i] = double(k * 1e9 + i);
    });
    std::vector<HostCopy> list;
    for (size_t k = 0; k < dev.size(); ++k)
        list.push_back({host[k].data(), dev[k].data(), dev[k].size() * sizeof(double)});
    Staging staging;
    if (copies_to_host(s, staging, list.data(), int(list.size())) != LBMX_OK || hipStreamSynchronize(s) != hipSuccess)
        return 2;
    return host == dev && host[0][0] == 0.0 ? 0 : 1;
}

// Several threads read through one handle's staging memory at once.
static int together(hipStream_t s, int count)
{
    Staging staging;
    const std::vector<size_t> sizes = {700001, 2500003};
    std::atomic<int> bad{0};
    std::vector<std::thread> pool;
    for (int t = 0; t < count; ++t)
        pool.emplace_back([&, t] {
            for (int round = 0; round < 4; ++round) {
                std::vector<double> dev(sizes[(t + round) % 2], 1000.0 * t + round), host(dev.size(), -1.0);
                const HostCopy c{host.data(), dev.data(), dev.size() * sizeof(double)};
                if (copies_to_host(s, staging, &c, 1) != LBMX_OK || hipStreamSynchronize(s) != hipSuccess || host != dev)
                    ++bad;
            }
        });
    for (std::thread &t : pool)
        t.join();
    return bad.load() ? 1 : 0;
}

int main(int argc, char **argv)
{
    const std::string c = argc > 1 ? argv[1] : "";
    const hipStream_t own = reinterpret_cast<hipStream_t>(0x1000);
    const std::vector<size_t> small = {1000, 3}, large = {1000003, 700001, 1, 900001};
    if (c == "small")  // waits for nothing: several passes of them follow each other
        return copies(own, small) + (waits == 1 ? 0 : 4);
    if (c == "large")
        return copies(own, large);
    if (c == "per_thread_stream")
        return copies(hipStreamPerThread, large) + copies(hipStreamPerThread, small);
    if (c == "several_threads")
        return together(own, 4);
    if (c == "pinned")  // nothing is staged
        return copies(own, large, large.size()) + (staged == 0 ? 0 : 4);
    if (c == "partly_pinned")
        return copies(own, {900001, 2500003, 700001}, 1) + (staged > 0 ? 0 : 4);
    if (c == "other_device") {  // the handle's stream on device 1, the caller on device 0
        device_of[own] = 1;
        return copies(own, large) + (device == 0 ? 0 : 4);
    }
    return 3;
}
