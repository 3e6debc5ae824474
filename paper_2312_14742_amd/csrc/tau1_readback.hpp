// tau1_readback.hpp -- state readback through pinned host memory.
//
// The export kernel writes FP64 values straight into pinned host slots over
// PCIe; worker threads copy each finished slot to the caller's arrays while the
// next ones are written.  Copying is spread over threads because the caller's
// pages are usually touched for the first time here, and one thread faults and
// fills them at about 10 GB/s.  Measured against copies from a device staging
// area into the caller's pageable memory: 128^3 5.7 -> 1.7 ms, 256^3 51 -> 13
// ms, 512^3 (4.3 GB) 408 -> 97 ms.
#pragma once

#include <hip/hip_runtime.h>

#include <condition_variable>
#include <cstring>
#include <mutex>
#include <thread>
#include <utility>
#include <vector>

namespace tau1 {

constexpr int kReadSlots = 4;
constexpr int64_t kReadNodes = int64_t(1) << 18;                 // nodes per slot
// Workers: the caller alone for small samples (it needs no other thread to be
// woken), then one per 12 MiB up to eight.  Measured: 47-67 MB 1.8-2.5 ms with
// one, 1.5 ms with three to twelve; 537 MB 40 ms with one, 22 with two, 14 with
// four, 11-13 with eight.
constexpr int kReadWorkers = 8;
constexpr size_t kBytesPerWorker = size_t(12) << 20;

// What the host reads while later kernels of the stream still run has to be
// visible to it: the blocks are coherent (with Portable alone that would be up
// to HIP_HOST_COHERENT), and a slot's event, recorded behind the kernel that
// writes it, releases to the system.
constexpr unsigned kReadPinned = hipHostMallocPortable | hipHostMallocCoherent;
constexpr unsigned kReadEvent = hipEventDisableTiming | hipEventReleaseToSystem;

// Pinned blocks, shared by the contexts of the process: a call takes one that is
// large enough for its duration (at most kReadSlots slots, 32 MiB), up to
// kKeep idle ones are kept for the next, and the last context to go gives them
// back.  Blocks are no larger than a power of two above what was asked, since
// pinning costs about 40 us a MiB at the first call.
// hipHostFree waits until the whole device is idle, also for streams that have
// nothing to do with this library, so a thread of the pool's own calls it.
// Both calls are made in relaxed capture mode: neither touches a stream, and
// another thread may be capturing.
class ReadPool {
public:
    struct Block {
        void* p = nullptr;
        size_t bytes = 0;
    };
    static ReadPool& get() {
        static ReadPool pool;
        return pool;
    }
    void add_context() {
        std::lock_guard<std::mutex> l(m_);
        ++contexts_;
    }
    void drop_context() {
        std::lock_guard<std::mutex> l(m_);
        if (--contexts_ == 0)
            for (auto& b : idle_) retire(b);
    }
    ~ReadPool() {
        if (freer_.joinable()) freer_.join();
    }
    // A block of at least `bytes`; p is null when pinned memory cannot be had.
    Block take(size_t bytes) {
        Block b;
        {
            std::lock_guard<std::mutex> l(m_);
            for (auto& i : idle_)
                if (i.bytes >= bytes && (!b.p || i.bytes < b.bytes)) std::swap(b, i);
        }
        if (b.p) return b;
        b.bytes = size_t(1) << 16;
        while (b.bytes < bytes) b.bytes *= 2;
        const RelaxedCapture relaxed;
        if (hipHostMalloc(&b.p, b.bytes, kReadPinned) != hipSuccess) {
            (void)hipGetLastError();
            b.p = nullptr;
        }
        return b;
    }
    void give(Block b) {
        {
            std::lock_guard<std::mutex> l(m_);
            if (contexts_ > 0)  // the larger blocks stay
                for (auto& i : idle_)
                    if (i.bytes < b.bytes) std::swap(i, b);
            retire(b);
        }
        if (b.p) (void)hipHostFree(b.p);  // no memory to note it down
    }

private:
    struct RelaxedCapture {
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
        ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    };
    // Leaves b to the freeing thread (m_ held); where none can be started it
    // waits for the next call's, and where it cannot be noted down b is kept.
    void retire(Block& b) {
        if (!b.p) return;
        try {
            retired_.push_back(b);
            b = Block{};
            if (freeing_) return;
            if (freer_.joinable()) freer_.join();  // it has left its loop
            freer_ = std::thread([this] { free_retired(); });
            freeing_ = true;
        } catch (...) {
        }
    }
    void free_retired() {
        const RelaxedCapture relaxed;
        std::unique_lock<std::mutex> l(m_);
        while (!retired_.empty()) {
            const Block b = retired_.back();
            retired_.pop_back();
            l.unlock();
            (void)hipHostFree(b.p);
            l.lock();
        }
        freeing_ = false;
    }

    static constexpr size_t kKeep = 2;
    std::mutex m_;
    Block idle_[kKeep];
    std::vector<Block> retired_;
    std::thread freer_;
    bool freeing_ = false;
    int contexts_ = 0;
};

// A block for the duration of a call: `slots` slots of `slot_doubles` values,
// then a few values for flags and results.
struct ReadBlock {
    explicit ReadBlock(int slots = 0, size_t slot_doubles = 0)
        : stride(slot_doubles), end(slots * slot_doubles),
          b(ReadPool::get().take((end + 8) * sizeof(double))) {}
    ReadBlock(const ReadBlock&) = delete;
    ~ReadBlock() {
        if (b.p) ReadPool::get().give(b);
    }
    double* slot(int i) const { return static_cast<double*>(b.p) + i * stride; }
    double* tail() const { return static_cast<double*>(b.p) + end; }
    const size_t stride, end;
    const ReadPool::Block b;
};

// Threads that copy finished slots to the caller's arrays.  Chunk c (nodes
// [c * kReadNodes, ...)) lies in slot c % kReadSlots as `arrays` runs of its
// node count; run a goes to dst[a].
class SlotCopy {
public:
    SlotCopy(const ReadBlock& b, int64_t n, int arrays, double* const* dst)
        : b_(b), n_(n), arrays_(arrays), dst_(dst) {
        const size_t bytes = (size_t)n * arrays * sizeof(double);
        size_t want = bytes / kBytesPerWorker;
        if (want > (size_t)kReadWorkers) want = kReadWorkers;
        const unsigned cpus = std::thread::hardware_concurrency();
        if (cpus && want > cpus) want = cpus;
        if (want < 2) return;
        // the slices depend on the number of workers: they start once it is known
        try {
            threads_.reserve(want);
            for (size_t i = 0; i < want; ++i) threads_.emplace_back([this, i] { work((int)i); });
        } catch (...) {  // as many as could be started
        }
        std::lock_guard<std::mutex> l(m_);
        workers_ = (int)threads_.size();
        started_ = true;
        cv_.notify_all();
    }
    ~SlotCopy() {
        {
            std::lock_guard<std::mutex> l(m_);
            stop_ = true;
            cv_.notify_all();
        }
        for (auto& t : threads_) t.join();
    }
    // Chunk c, the next in order, is in its slot.
    void ready(int64_t c) {
        if (threads_.empty()) {
            copy(c, 0, 1);
            done_slot(c);
            return;
        }
        std::lock_guard<std::mutex> l(m_);
        ready_ = c + 1;
        cv_.notify_all();
    }
    // Whether chunk c has left its slot.
    bool left(int64_t c) {
        std::lock_guard<std::mutex> l(m_);
        return copied_[c % kReadSlots] > c;
    }
    // Waits until it has.
    void wait(int64_t c) {
        std::unique_lock<std::mutex> l(m_);
        cv_.wait(l, [&] { return copied_[c % kReadSlots] > c; });
    }

private:
    void work(int w) {
        int workers;
        {
            std::unique_lock<std::mutex> l(m_);
            cv_.wait(l, [&] { return started_ || stop_; });
            workers = workers_;
        }
        const int64_t chunks = (n_ + kReadNodes - 1) / kReadNodes;
        for (int64_t c = 0; c < chunks; ++c) {
            {
                std::unique_lock<std::mutex> l(m_);
                cv_.wait(l, [&] { return ready_ > c || stop_; });
                if (ready_ <= c) return;
            }
            copy(c, w, workers);
            std::lock_guard<std::mutex> l(m_);
            if (++parts_[c % kReadSlots] == workers) {
                parts_[c % kReadSlots] = 0;
                copied_[c % kReadSlots] = c + 1;
                cv_.notify_all();
            }
        }
    }
    void done_slot(int64_t c) {
        std::lock_guard<std::mutex> l(m_);
        copied_[c % kReadSlots] = c + 1;
    }
    // Part w of `parts` of chunk c.
    void copy(int64_t c, int w, int parts) {
        const int64_t i0 = c * kReadNodes, len = n_ - i0 < kReadNodes ? n_ - i0 : kReadNodes;
        const int64_t a = len * w / parts, b = len * (w + 1) / parts;
        const double* src = b_.slot((int)(c % kReadSlots));
        for (int k = 0; k < arrays_; ++k)
            std::memcpy(dst_[k] + i0 + a, src + k * len + a, sizeof(double) * (size_t)(b - a));
    }

    const ReadBlock& b_;
    const int64_t n_;
    const int arrays_;
    double* const* const dst_;
    std::vector<std::thread> threads_;
    std::mutex m_;
    std::condition_variable cv_;
    int workers_ = 0;
    bool started_ = false, stop_ = false;
    int64_t ready_ = 0;
    int64_t copied_[kReadSlots] = {};
    int parts_[kReadSlots] = {};
};

}  // namespace tau1
