// Output maps on their way to pageable host memory (host side).
//
// A copy into pageable memory goes through the runtime's own staging, one map
// at a time, and the first touch of a new buffer's pages is taken by one
// thread. Here the kernel that forms the maps writes them to pinned memory that
// the context keeps, and after the step's one wait the maps are copied out, by
// several threads if they are large. 64 mixed sequences, 59 MB of maps into new
// arrays: 32.9 ms per frame step, 26.5 without maps, 40.8 with a copy per map
// (36.7 with one thread beside the caller, 34.1 with three, 31.6 with fifteen).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstring>
#include <functional>
#include <mutex>
#include <thread>
#include <vector>

namespace pv {

// pinned memory of a context for its maps: taken when a step first asks for
// maps in host memory, grown if a later one needs more, freed by release()
class MapStage {
public:
    // room for n floats, or null (more than kMaxBytes, or no memory): the maps
    // then take the runtime's copies
    float* reserve(size_t n) {
        if (n > kMaxBytes / sizeof(float)) return nullptr;
        if (n <= n_) return buf_;
        release();
        if (hipHostMalloc((void**)&buf_, n * sizeof(float)) != hipSuccess) {
            (void)hipGetLastError();
            buf_ = nullptr;
            return nullptr;
        }
        n_ = n;
        return buf_;
    }
    void release() {
        if (buf_) (void)hipHostFree(buf_);
        buf_ = nullptr;
        n_ = 0;
    }

private:
    static constexpr size_t kMaxBytes = (size_t)256 << 20;   // what one context may pin
    float* buf_ = nullptr;
    size_t n_ = 0;
};

// Whether a frame's map of n floats goes to `dst` by a copy of the runtime's: a
// large one to memory that is itself pinned, where the device's copy engine
// writes it at the link's rate and a second copy by the host only costs time.
// Both maps of a frame read out into pinned memory without iterating, copied
// directly and through the context's: 256 x 256 55 and 51 us, 320 x 320 61 and
// 66, 384 x 384 70 and 84, 640 x 480 98 and 141, 1920 x 1080 414 and 612.
inline bool copied_directly(const float* dst, size_t n) {
    constexpr size_t kMinDirect = (size_t)1 << 17;
    if (n < kMinDirect) return false;
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, dst) != hipSuccess) {
        (void)hipGetLastError();   // memory that the runtime does not know
        return false;
    }
    return a.type == hipMemoryTypeHost;
}

struct MapJob {
    float* dst;
    const float* src;
    size_t n;
};

// whether any two destinations have memory in common (sorts them)
inline bool destinations_overlap(std::vector<MapJob>& maps) {
    std::sort(maps.begin(), maps.end(), [](const MapJob& a, const MapJob& b) { return std::less<float*>()(a.dst, b.dst); });
    for (size_t i = 1; i < maps.size(); ++i)
        if (std::less<float*>()(maps[i].dst, maps[i - 1].dst + maps[i - 1].n)) return true;
    return false;
}

// Copies maps from pinned memory to where they belong. The workers are started
// before the wait for the device (so that it hides their start) and wait for
// run(); destroyed without it, nothing is copied. Destinations that overlap are
// written by the calling thread alone, in order.
class MapCopier {
public:
    MapCopier(const MapJob* jobs, int n_jobs) : jobs_(jobs), n_jobs_(n_jobs) {
        size_t total = 0;
        for (int i = 0; i < n_jobs; ++i) {
            total += jobs[i].n;
            chunks_ += chunks_of(jobs[i]);
        }
        size_t want = total * sizeof(float) / kBytesPerWorker;
        if (want > kWorkers) want = kWorkers;
        if (want > 0 && (n_jobs > kMaxJobs || overlapping())) want = 0;
        try {
            for (; (size_t)n_ < want; ++n_) pool_[n_] = std::thread([this] { wait_and_copy(); });
        } catch (...) {
            // fewer workers: the calling thread copies what they do not
        }
    }
    ~MapCopier() { finish(false); }
    void run() { finish(true); }

private:
    static constexpr int kWorkers = 7;
    static constexpr size_t kBytesPerWorker = (size_t)4 << 20;
    static constexpr int kMaxJobs = 2048;   // whose destinations are compared, each with each
    static constexpr size_t kChunk = (size_t)1 << 17;   // floats

    static size_t chunks_of(const MapJob& j) { return (j.n + kChunk - 1) / kChunk; }

    bool overlapping() const {
        for (int i = 0; i < n_jobs_; ++i)
            for (int k = 0; k < i; ++k)
                if (jobs_[i].dst < jobs_[k].dst + jobs_[k].n && jobs_[k].dst < jobs_[i].dst + jobs_[i].n) return true;
        return false;
    }

    void copy() {
        for (size_t c; (c = next_.fetch_add(1)) < chunks_;) {
            const MapJob* j = jobs_;
            for (size_t m; c >= (m = chunks_of(*j)); ++j) c -= m;
            const size_t at = c * kChunk, left = j->n - at;
            std::memcpy(j->dst + at, j->src + at, (left < kChunk ? left : kChunk) * sizeof(float));
        }
    }

    void wait_and_copy() {
        {
            std::unique_lock<std::mutex> lock(m_);
            cv_.wait(lock, [this] { return state_ != 0; });
            if (state_ < 0) return;
        }
        copy();
    }

    void finish(bool copy_maps) {
        if (finished_) return;
        finished_ = true;
        {
            std::lock_guard<std::mutex> lock(m_);
            state_ = copy_maps ? 1 : -1;
        }
        cv_.notify_all();
        if (copy_maps) copy();
        for (int k = 0; k < n_; ++k) pool_[k].join();
    }

    const MapJob* jobs_;
    int n_jobs_;
    size_t chunks_ = 0;
    std::atomic<size_t> next_{0};
    std::mutex m_;
    std::condition_variable cv_;
    int state_ = 0;         // 0: wait, 1: copy, -1: end
    bool finished_ = false;
    int n_ = 0;
    std::thread pool_[kWorkers];
};

}  // namespace pv
