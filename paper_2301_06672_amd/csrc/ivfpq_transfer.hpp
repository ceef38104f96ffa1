// Large copies from the device to ordinary host memory: the arrays travel in pieces through a small ring of pinned slots, and several
// threads copy slot to array.
//
// A copy to ordinary memory is staged by one thread of the runtime: 48 MB took 2,970 us, to pinned memory 890 us (54 GB/s).  Pinning the
// arrays themselves costs more than the copy, so the ring (16 MB) is made for one transfer.  A piece of 1 MB took 40 us with its event,
// one of 4 MB 85 us, hence 4 MB, of which each thread copies an eighth.  (The other way a ring was slower in a program's first uploads,
// 3,300 against 2,200 us, and 1,750 against 2,150 us later: the runtime's copies serve.)
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cstring>
#include <memory>
#include <thread>
#include <vector>

#include "ivfpq_hip_util.hpp"

namespace {

class HostTransfer {
public:
    static constexpr size_t kPiece = (size_t)4 << 20;
    static constexpr int kSlots = 4, kThreads = 8;
    static constexpr size_t kParts = 8, kSmall = 2 * kPiece; // below kSmall the runtime's own copies are as fast

    explicit HostTransfer(hipStream_t st) : st_(st) {}
    ~HostTransfer() { (void)end(); }
    HostTransfer(const HostTransfer&) = delete;
    HostTransfer& operator=(const HostTransfer&) = delete;

    // Appends a copy of `bytes` device bytes.  `widen`: 32-bit numbers, of which the host array takes each as 64 bits.
    void add(void* host, const void* dev, size_t bytes, bool widen = false) {
        for (size_t at = 0; at < bytes; at += kPiece)
            pieces_.push_back({(char*)host + (widen ? 2 * at : at), (const char*)dev + at, std::min(kPiece, bytes - at), widen});
        total_ += bytes;
    }

    // Queues the copies on the stream, in order, and waits for them; called once.
    int run() {
        const RelaxedCapture relaxed;
        const bool ring = total_ >= kSmall && start();
        const int s = ring ? run_ring() : run_plain();
        const hipError_t e = end();
        if (s != IVFPQ_OK) return s;
        HIP_TRY(e);
        if (!ring) widen_plain();
        return IVFPQ_OK;
    }

private:
    struct Piece { char* host; const char* dev; size_t bytes; bool widen; };

    // While another thread captures a graph, allocations and waits on events are neither refused nor do they end its capture.
    struct RelaxedCapture {
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        bool ok;
        RelaxedCapture() : ok(hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess) {}
        ~RelaxedCapture() { if (ok) (void)hipThreadExchangeStreamCaptureMode(&mode); }
    };

    struct Ring {
        void* slots = nullptr;
        hipEvent_t moved[kSlots] = {};
        ~Ring() {
            for (hipEvent_t e : moved)
                if (e) (void)hipEventDestroy(e);
            if (slots) (void)hipHostFree(slots);
        }
    };

    // False: no ring to be had (memory, events or threads); the plain copies serve.
    bool start() {
        ring_.reset(new Ring);
        bool ok = hipHostMalloc(&ring_->slots, kSlots * kPiece, 0) == hipSuccess;
        for (int i = 0; ok && i < kSlots; ++i) ok = hipEventCreateWithFlags(&ring_->moved[i], hipEventDisableTiming) == hipSuccess;
        if (ok) {
            parts_done_.reset(new std::atomic<uint32_t>[pieces_.size()]());
            const unsigned hw = std::thread::hardware_concurrency();
            const int want = hw == 0 ? kThreads : (int)std::min<unsigned>(kThreads, hw);
            try {
                while (started_ < want) {
                    pool_[started_] = std::thread([this] { work(); });
                    ++started_;
                }
            } catch (...) {                                  // fewer threads than wished for
            }
            ok = started_ > 0;
        }
        if (!ok) {
            (void)hipGetLastError();
            ring_.reset();
        }
        return ok;
    }

    // The threads first, then the stream: a copy may still be on its way to a slot.
    hipError_t end() {
        if (ended_) return hipSuccess;
        ended_ = true;
        quit_.store(true);
        for (int t = 0; t < started_; ++t) pool_[t].join();
        const hipError_t e = hipStreamSynchronize(st_);
        ring_.reset();
        return e;
    }

    // A thread takes parts in order and waits for the part's piece to be queued and moved.  run_ring waits, before it queues a piece, for
    // the parts of the piece that was in the slot before.  Each wait is for something earlier in the order, so it ends, or ends with quit_.
    void work() {
        const RelaxedCapture relaxed;
        for (;;) {
            const size_t part = next_.fetch_add(1), p = part / kParts;
            if (p >= pieces_.size()) return;
            while (queued_.load(std::memory_order_acquire) <= p) {
                if (quit_.load()) return;
                std::this_thread::yield();
            }
            if (hipEventSynchronize(ring_->moved[p % kSlots]) != hipSuccess) {
                failed_.store(true);
                return;
            }
            const Piece& c = pieces_[p];
            const size_t step = (c.bytes / kParts + 63) / 64 * 64;
            const size_t from = std::min(c.bytes, part % kParts * step), to = part % kParts + 1 == kParts ? c.bytes : std::min(c.bytes, from + step);
            const char* pinned = (const char*)ring_->slots + p % kSlots * kPiece + from;
            if (c.widen) {
                const uint32_t* src = (const uint32_t*)pinned;
                int64_t* dst = (int64_t*)(c.host + 2 * from);
                for (size_t i = 0, n = (to - from) / 4; i < n; ++i) dst[i] = (int64_t)src[i];
            } else {
                std::memcpy(c.host + from, pinned, to - from);
            }
            parts_done_[p].fetch_add(1, std::memory_order_release);
        }
    }

    int wait_done(size_t p) {
        while (parts_done_[p].load(std::memory_order_acquire) < kParts) {
            if (failed_.load()) return fail(IVFPQ_EHIP, "waiting for a copy to the host failed");
            std::this_thread::yield();
        }
        return IVFPQ_OK;
    }

    int run_ring() {
        const size_t n = pieces_.size();
        for (size_t p = 0; p < n; ++p) {
            if (p >= kSlots)
                if (int s = wait_done(p - kSlots)) return s;
            HIP_TRY(hipMemcpyAsync((char*)ring_->slots + p % kSlots * kPiece, pieces_[p].dev, pieces_[p].bytes, hipMemcpyDeviceToHost, st_));
            HIP_TRY(hipEventRecord(ring_->moved[p % kSlots], st_));
            queued_.store(p + 1, std::memory_order_release);
        }
        for (size_t p = n - std::min<size_t>(kSlots, n); p < n; ++p)
            if (int s = wait_done(p)) return s;
        return IVFPQ_OK;
    }

    // A piece to be widened arrives in the upper half of its place; widen_plain spreads it from there.
    int run_plain() {
        for (const Piece& c : pieces_)
            HIP_TRY(hipMemcpyAsync(c.widen ? c.host + c.bytes : c.host, c.dev, c.bytes, hipMemcpyDeviceToHost, st_));
        return IVFPQ_OK;
    }
    void widen_plain() {
        for (const Piece& c : pieces_)
            for (size_t i = 0, n = c.widen ? c.bytes / 4 : 0; i < n; ++i) {
                uint32_t v;
                std::memcpy(&v, c.host + c.bytes + 4 * i, 4);
                const int64_t w = (int64_t)v;
                std::memcpy(c.host + 8 * i, &w, 8);          // ends at 8 i + 8 <= 4 n + 4 (i + 1): what lies above is still unread
            }
    }

    const hipStream_t st_;
    std::vector<Piece> pieces_;
    size_t total_ = 0;
    std::unique_ptr<Ring> ring_;
    std::unique_ptr<std::atomic<uint32_t>[]> parts_done_;
    std::thread pool_[kThreads];
    int started_ = 0;
    bool ended_ = false;
    std::atomic<size_t> next_{0}, queued_{0};
    std::atomic<bool> quit_{false}, failed_{false};
};

}  // namespace
