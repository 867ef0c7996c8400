// Copies between device memory and the caller's (pageable) host memory.
//
// The runtime's copy of pageable memory pins the caller's pages piece by piece
// on one thread: 11 GB/s into memory just allocated, 18 GB/s into memory in
// use.  Large copies go through pinned buffers of this library instead, a few
// threads moving the pieces between them and the caller's memory while the
// next ones are on the bus: 30 GB/s on four threads (134 MB 12.3 -> 4.4 ms,
// 50 MB 4.6 -> 1.7 ms, 8 MB 0.78 -> 0.43 ms; two threads 22 GB/s, eight as
// four).  Below kStagedMin the threads cost what they save, and memory that is
// pinned already needs none of it.  The buffers live
// for one call (allocating them takes 0.12 ms).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <thread>

namespace lbfss {

constexpr size_t kStagedMin = size_t(6) << 20;
constexpr size_t kStagePiece = size_t(1) << 20;
constexpr int kStageWorkers = 4;

class HostStage {
  public:
    HostStage(hipStream_t stream, int device) : stream_(stream), device_(device) {}
    HostStage(const HostStage &) = delete;
    ~HostStage() {
        if (!pin_) return;
        (void)hipStreamSynchronize(stream_);  // no copy may still use the buffers
        (void)hipHostFree(pin_);
    }
    // Small copies are queued on the stream; large ones are done on return
    // (to_host) or have left host memory (to_device).
    hipError_t to_host(void *dst, const void *src, size_t bytes) { return move((char *)dst, (char *)src, bytes, true); }
    hipError_t to_device(void *dst, const void *src, size_t bytes) { return move((char *)src, (char *)dst, bytes, false); }

  private:
    struct OnDevice {
        int was = -1;
        hipError_t err;
        explicit OnDevice(int device) {
            err = hipGetDevice(&was);
            if (err == hipSuccess && was != device) err = hipSetDevice(device);
            else was = -1;
        }
        ~OnDevice() {
            if (was >= 0) (void)hipSetDevice(was);
        }
    };
    // Memory that the runtime knows (pinned, managed, a device's) it copies in
    // one piece and faster, 45 to 56 GB/s: 128^3 density into a pinned array
    // 0.37 ms, through the pieces 0.78 ms; 192^3 populations 19.1, 35.9 ms.
    static bool known(const void *p) {
        hipPointerAttribute_t a{};
        if (hipPointerGetAttributes(&a, p) == hipSuccess) return a.type != hipMemoryTypeUnregistered;
        (void)hipGetLastError();
        return false;
    }
    hipError_t plain(char *host, char *dev, size_t bytes, bool down) {
        return down ? hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, stream_)
                    : hipMemcpyAsync(dev, host, bytes, hipMemcpyHostToDevice, stream_);
    }
    hipError_t move(char *host, char *dev, size_t bytes, bool down) {
        if (bytes < kStagedMin || known(host)) return plain(host, dev, bytes, down);
        // the buffers and the first worker's events are the stream's device's,
        // whichever is current on the caller's thread
        OnDevice on(device_);
        if (on.err != hipSuccess) return on.err;
        if (!pin_ && hipHostMalloc((void **)&pin_, 2 * kStageWorkers * kStagePiece, hipHostMallocDefault) != hipSuccess) {
            pin_ = nullptr;
            (void)hipGetLastError();
            return plain(host, dev, bytes, down);
        }
        std::atomic<size_t> next{0};
        std::atomic<int> err{(int)hipSuccess};
        auto work = [&](int w) { worker(w, host, dev, bytes, down, next, err); };
        std::thread extra[kStageWorkers - 1];
        for (int w = 1; w < kStageWorkers; ++w) {
            try {
                extra[w - 1] = std::thread(work, w);
            } catch (...) {
                break;  // the workers there are take all pieces
            }
        }
        work(0);
        for (auto &t : extra)
            if (t.joinable()) t.join();
        if (err.load() != (int)hipSuccess) (void)hipStreamSynchronize(stream_);
        return (hipError_t)err.load();
    }
    // Takes pieces until none is left, two buffers each: a piece moves between
    // its buffer and the caller's memory while the other buffer's is copied.
    void worker(int w, char *host, char *dev, size_t bytes, bool down, std::atomic<size_t> &next,
                std::atomic<int> &err) {
        const size_t pieces = (bytes + kStagePiece - 1) / kStagePiece;
        char *buf[2] = {pin_ + 2 * w * kStagePiece, pin_ + (2 * w + 1) * kStagePiece};
        hipEvent_t ev[2] = {nullptr, nullptr};
        hipError_t e = w > 0 ? hipSetDevice(device_) : hipSuccess;
        for (int k = 0; k < 2 && e == hipSuccess; ++k) e = hipEventCreateWithFlags(&ev[k], hipEventDisableTiming);
        size_t held[2] = {pieces, pieces};  // the piece a buffer holds (pieces: none)
        auto finish = [&](int k) {          // wait for a buffer's copy; down: hand its piece over
            if (held[k] == pieces) return;
            e = hipEventSynchronize(ev[k]);
            const size_t o = held[k] * kStagePiece;
            if (e == hipSuccess && down) std::memcpy(host + o, buf[k], std::min(kStagePiece, bytes - o));
            held[k] = pieces;
        };
        int k = 0;
        while (e == hipSuccess && err.load() == (int)hipSuccess) {
            const size_t c = next.fetch_add(1);
            if (c >= pieces) break;
            const size_t o = c * kStagePiece, n = std::min(kStagePiece, bytes - o);
            if (!down) {
                finish(k);
                if (e == hipSuccess) std::memcpy(buf[k], host + o, n);
            }
            if (e == hipSuccess) e = plain(buf[k], dev + o, n, down);
            if (e == hipSuccess) e = hipEventRecord(ev[k], stream_);
            if (e != hipSuccess) break;
            held[k] = c;
            k ^= 1;
            if (down) finish(k);
        }
        for (int i = 0; i < 2 && e == hipSuccess; ++i) finish(k ^ i);
        for (hipEvent_t v : ev)
            if (v) (void)hipEventDestroy(v);
        if (e != hipSuccess) {
            int none = (int)hipSuccess;
            (void)err.compare_exchange_strong(none, (int)e);
        }
    }

    hipStream_t stream_;
    int device_;
    char *pin_ = nullptr;
};

}  // namespace lbfss
