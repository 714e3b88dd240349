// Transfers between host arrays and the kernels that read or write a
// lattice's state.  The kernels work on pinned host memory directly (mapped,
// over PCIe), chunk by chunk in a ring, while a few host threads move the
// chunks before and after to or from the caller's arrays.  Measured: the
// kernels reach 56 GB/s on pinned memory, as the copy engine does; one host
// thread fills fresh pages at 14 GB/s, eight at 68 GB/s.  256^3 moments
// (537 MB) in a sampling loop 58 -> 14.4 ms, D3Q27 96^3 FP16 populations in
// and out 27 -> 7.3 ms.
#pragma once

#include <hip/hip_runtime.h>
#include <unistd.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstddef>
#include <memory>
#include <mutex>
#include <thread>

namespace ptrt {

// Host threads and pinned memory shared by the live handles of the process:
// made on first use, given back with the last handle.  Any thread may use
// it at any time: a job's caller works on its own job until it is done, so
// no caller waits for another one's.
class HostPool {
public:
    // nullptr when out of host memory
    static std::shared_ptr<HostPool> shared() noexcept
    try {
        // never destroyed: handles may outlive static destruction
        static std::mutex *m = new std::mutex;
        static std::weak_ptr<HostPool> *w = new std::weak_ptr<HostPool>;
        std::lock_guard<std::mutex> lock(*m);
        std::shared_ptr<HostPool> p = w->lock();
        if (!p) *w = p = std::shared_ptr<HostPool>(new HostPool, &HostPool::release);
        return p;
    } catch (...) {
        return nullptr;
    }

    // In a forked child the threads do not exist, and what they hold and wait
    // for is as it was: the child leaves an inherited pool alone.
    static void release(HostPool *p)
    {
        if (p->own_process()) delete p;
    }
    bool own_process() const { return getpid() == pid_; }

    ~HostPool()
    {
        {
            std::lock_guard<std::mutex> lock(mutex_);
            stop_ = true;
        }
        work_.notify_all();
        for (int k = 0; k < threads_; ++k) thread_[k].join();
        for (int k = 0; k < kept_; ++k) (void)hipHostFree(keep_[k].ptr);
    }

    // A transfer of this many bytes begins: the pinned bytes for its ring, about
    // a tenth of all transfers so far, from 4 to 64 MB.  Pinned memory that
    // is new costs the host 380 us a megabyte in page faults, so that large
    // rings have to be earned: a handle on 64^3 nodes, made, read once and
    // freed, takes 1.1 ms with pageable copies, 2.7 with a ring of 16 MB and
    // 0.9 with 4.
    static constexpr long long LEAST = 4 << 20, MOST = 64 << 20;
    long long ring_bytes(long long bytes)
    {
        std::lock_guard<std::mutex> lock(mutex_);
        moved_ += bytes;
        long long r = LEAST;
        while (r < MOST && r <= moved_ / 16) r *= 2;
        return r;
    }

    // f(i) for i = 0 ... n - 1, on the caller and the pool's threads.
    template <class F>
    void parallel(int n, const F &f)
    {
        if (n <= 1 || !own_process() || !ready(n)) {
            for (int i = 0; i < n; ++i) f(i);
            return;
        }
        Job job;
        job.call = [](const void *g, int i) { (*static_cast<const F *>(g))(i); };
        job.f = &f;
        job.n = n;
        {
            std::lock_guard<std::mutex> lock(mutex_);
            job.link = jobs_;
            jobs_ = &job;
        }
        work_.notify_all();
        job.run();
        std::unique_lock<std::mutex> lock(mutex_);
        for (Job **j = &jobs_; *j; j = &(*j)->link)
            if (*j == &job) {
                *j = job.link;
                break;
            }
        idle_.wait(lock, [&] { return job.users == 0; });
    }

    struct Stage {
        char *ptr = nullptr;
        size_t bytes = 0;
    };
    // Pinned memory of at least `bytes`; nullptr when it cannot be had.
    Stage take(size_t bytes)
    {
        {
            std::lock_guard<std::mutex> lock(mutex_);
            int best = -1;
            for (int k = 0; k < kept_; ++k)
                if (keep_[k].bytes >= bytes && (best < 0 || keep_[k].bytes < keep_[best].bytes)) best = k;
            if (best >= 0) {
                const Stage s = keep_[best];
                keep_[best] = keep_[--kept_];
                return s;
            }
        }
        Stage s;
        s.bytes = 64 << 10;
        while (s.bytes < bytes) s.bytes *= 2;
        if (hipHostMalloc((void **)&s.ptr, s.bytes, hipHostMallocPortable | hipHostMallocCoherent) !=
            hipSuccess) {
            (void)hipGetLastError();
            s.ptr = nullptr;
        }
        return s;
    }
    // Back to the pool, which keeps at most KEEP blocks (the smallest goes).
    void give(Stage s)
    {
        if (!s.ptr) return;
        {
            std::lock_guard<std::mutex> lock(mutex_);
            if (kept_ < KEEP) {
                keep_[kept_++] = s;
                return;
            }
            int least = 0;
            for (int k = 1; k < KEEP; ++k)
                if (keep_[k].bytes < keep_[least].bytes) least = k;
            if (keep_[least].bytes < s.bytes) std::swap(keep_[least], s);
        }
        (void)hipHostFree(s.ptr);
    }

private:
    struct Job {
        void (*call)(const void *, int) = nullptr;
        const void *f = nullptr;
        int n = 0, users = 0;
        std::atomic<int> next{0};
        Job *link = nullptr;
        void run()
        {
            for (int i; (i = next.fetch_add(1, std::memory_order_relaxed)) < n;) call(f, i);
        }
    };
    static constexpr int MAX_THREADS = 15, KEEP = 2;

    HostPool() = default;

    // Whether there are threads for n pieces: up to n - 1, one per two megabytes
    // of the transfers so far and none below 8 MB, so that a handle that is
    // made, read once and freed does not pay for threads that it hardly uses.
    // Starting and joining one takes 67 us, fifteen 285 us, as long as the
    // caller alone takes for 1 and 4 MB into fresh pages (made, one step, read,
    // freed, us: 56^3 FP32 864 with pageable copies, 646 without threads, 740
    // with one per 4 MB; 32^3, ten steps, 388, 270 and, with fifteen threads
    // at once, 739).  Fewer, or none, where the system refuses.
    bool ready(int n)
    {
        std::lock_guard<std::mutex> lock(mutex_);
        const long long mb = moved_ >> 20;
        if (mb >= 8 && most_ < 0) most_ = std::min(MAX_THREADS, (int)std::thread::hardware_concurrency() - 1);
        const int want = mb < 8 ? 0 : (int)std::min<long long>(std::min(most_, n - 1), mb / 2);
        try {
            while (!refused_ && threads_ < want) {
                thread_[threads_] = std::thread([this] { serve(); });
                ++threads_;
            }
        } catch (...) {
            refused_ = true;
        }
        return threads_ > 0;
    }

    void serve()
    {
        std::unique_lock<std::mutex> lock(mutex_);
        for (;;) {
            Job *job = nullptr;
            work_.wait(lock, [&] {
                for (job = jobs_; job && job->next.load(std::memory_order_relaxed) >= job->n;) job = job->link;
                return stop_ || job;
            });
            if (stop_) return;
            ++job->users;
            lock.unlock();
            job->run();
            lock.lock();
            if (--job->users == 0) idle_.notify_all();
        }
    }

    const pid_t pid_ = getpid();
    int most_ = -1; // threads at most; not looked up yet
    std::mutex mutex_;
    std::condition_variable work_, idle_;
    Job *jobs_ = nullptr;
    std::thread thread_[MAX_THREADS];
    int threads_ = 0;
    long long moved_ = 0; // bytes of all transfers
    bool refused_ = false, stop_ = false;
    Stage keep_[KEEP];
    int kept_ = 0;
};

// A ring of up to four chunks of a lattice's nodes in pinned memory.
class StageRing {
public:
    static constexpr int RING = 4;
    // per_node: bytes of one node.  Up to 2 MB in one chunk; more in a ring of
    // the pool's choice, of two chunks at its least size and four beyond, that
    // overlap, of 2 MB at least (2.2 MB as two chunks of 1.1: 62 x 1448 read in
    // a loop 190 us for 150).  The host's share, page faults of the caller's fresh arrays
    // above all, is the longer one, and larger chunks keep more threads busy:
    // 256^3 moments in a sampling loop 17.8 ms with chunks of 8 MB and 8
    // threads, 14.6 with 16 and 16.
    StageRing(const std::shared_ptr<HostPool> &pool, long long nodes, size_t per_node, hipStream_t stream)
        : pool_(pool), nodes_(nodes), per_node_(per_node), stream_(stream)
    {
        const long long total = nodes * (long long)per_node, ring = pool->ring_bytes(total);
        const int most = ring == HostPool::LEAST ? 2 : RING;
        const long long chunk = std::max(HostPool::LEAST / 2, std::min(ring, total) / most);
        step_ = std::min(nodes, std::max(1LL, chunk / (long long)per_node));
        chunks_ = (nodes + step_ - 1) / step_;
        slots_ = (int)std::min<long long>(most, chunks_);
    }
    ~StageRing()
    {
        // the kernels that use the memory have run
        if (stage_.ptr && !idle_) (void)hipStreamSynchronize(stream_);
        for (hipEvent_t e : event_)
            if (e) (void)hipEventDestroy(e);
        pool_->give(stage_);
    }
    StageRing(const StageRing &) = delete;
    StageRing &operator=(const StageRing &) = delete;

    // Out: launch(buffer, n0, count) enqueues the kernel that writes a
    // chunk, copy(buffer, n0, count, a, b) hands its nodes a ... b - 1 to the
    // caller's arrays.
    template <class Launch, class Copy>
    hipError_t out(Launch launch, Copy copy)
    {
        hipError_t e = open();
        for (long long c = 0; c < slots_ && e == hipSuccess; ++c) e = enqueue(launch, c);
        for (long long c = 0; c < chunks_ && e == hipSuccess; ++c) {
            e = wait(c);
            if (e != hipSuccess) break;
            move(copy, c);
            if (c + slots_ < chunks_) e = enqueue(launch, c + slots_);
        }
        idle_ = e == hipSuccess;
        return e;
    }
    // In: fill(buffer, n0, count, a, b) takes nodes a ... b - 1 from the
    // caller's arrays, launch(buffer, n0, count) enqueues the kernel that
    // reads the chunk.
    template <class Fill, class Launch>
    hipError_t in(Fill fill, Launch launch)
    {
        hipError_t e = open();
        for (long long c = 0; c < chunks_ && e == hipSuccess; ++c) {
            if (c >= slots_) e = wait(c - slots_);
            if (e != hipSuccess) break;
            move(fill, c);
            e = enqueue(launch, c);
        }
        if (e == hipSuccess) e = hipStreamSynchronize(stream_);
        idle_ = e == hipSuccess;
        return e;
    }

private:
    hipError_t open()
    {
        // smaller chunks where no more pinned memory can be had
        while (!(stage_ = pool_->take((size_t)step_ * per_node_ * (size_t)slots_)).ptr) {
            if (step_ == 1 || (size_t)step_ * per_node_ <= (32u << 10)) return hipErrorOutOfMemory;
            step_ = (step_ + 1) / 2;
            chunks_ = (nodes_ + step_ - 1) / step_;
            slots_ = (int)std::min<long long>(2, chunks_);
        }
        for (int k = 0; k < slots_ && chunks_ > 1; ++k) {
            const hipError_t e = hipEventCreateWithFlags(&event_[k], hipEventDisableTiming);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    char *buffer(long long c) const { return stage_.ptr + (size_t)(c % slots_) * (size_t)step_ * per_node_; }
    long long first(long long c) const { return c * step_; }
    long long count(long long c) const { return std::min(step_, nodes_ - c * step_); }
    template <class Launch>
    hipError_t enqueue(Launch &launch, long long c)
    {
        launch(buffer(c), first(c), count(c));
        hipError_t e = hipGetLastError();
        if (e == hipSuccess && event_[c % slots_]) e = hipEventRecord(event_[c % slots_], stream_);
        return e;
    }
    hipError_t wait(long long c)
    {
        return event_[c % slots_] ? hipEventSynchronize(event_[c % slots_]) : hipStreamSynchronize(stream_);
    }
    template <class Move>
    void move(Move &f, long long c)
    {
        const long long n = count(c);
        char *b = buffer(c);
        const int pieces = (int)std::max(1LL, std::min(64LL, n * (long long)per_node_ / (256 << 10)));
        pool_->parallel(pieces, [&](int i) {
            f(b, first(c), n, n * i / pieces, n * (i + 1) / pieces);
        });
    }

    std::shared_ptr<HostPool> pool_;
    long long nodes_, step_ = 1, chunks_ = 0;
    size_t per_node_;
    int slots_ = 0;
    hipStream_t stream_;
    HostPool::Stage stage_;
    bool idle_ = false; // no kernel uses the memory
    hipEvent_t event_[RING] = {nullptr, nullptr, nullptr, nullptr};
};

} // namespace ptrt
