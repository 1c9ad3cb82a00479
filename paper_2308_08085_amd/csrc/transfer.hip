// transfer.hip -- device data to the caller's host memory.  That memory is
// pageable, so data goes through pinned memory that the kernels (or a copy)
// write directly; while the GPU fills the next chunks, host threads move the
// finished ones on.
//
// What bounds it: PCIe carries 55 GB/s into pinned memory, one host thread
// copies into freshly mapped memory at 5-14 GB/s, eight at 24-92 GB/s (4 KiB /
// 2 MiB pages).  The HIP runtime's own path for pageable destinations is one
// thread behind a 1 MB bounce buffer: 10 GB/s, and 0.4 ms for 1 MB.
//
// Pinned memory: kPinBytes per handle, for counters and small reads, from the
// kPinFrom-th transfer on (pinning and unpinning it takes as long as 30 small
// transfers save: a short run never pays that); and one ring of kSlots x
// kSlotBytes (32 MB) in the process, made when a handle has read kRingFrom bytes
// in all (0.4 ms) and given back when the last handle is destroyed.  One
// transfer uses the ring at a time; others meanwhile, and all if pinned memory
// cannot be had, take the runtime's path.
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

#include "runtime_internal.h"

namespace amr {

namespace {

constexpr uint64_t kRingFrom = uint64_t(4) << 20;
constexpr int kPinFrom = 32;
constexpr int kSlots = 8, kMaxWorkers = 6;
constexpr size_t kWorkerBytes = size_t(2) << 20;  // one host thread per this much of a transfer: starting one takes 20 us

struct Ring {
    std::mutex use;    // held by the transfer that uses the ring
    std::mutex count;  // guards `users`
    int users = 0;
    char *mem = nullptr;  // written with `use` held
};
Ring g_ring;

// Host threads that move finished chunks; chunk i may be overwritten when done(i).
class Workers {
  public:
    Workers(int n_chunks, int n_threads) : done_(n_chunks, 0) {
        try {
            for (int k = 0; k < n_threads; k++) threads_.emplace_back([this] { loop(); });
        } catch (...) {  // fewer threads, or none: give() then copies itself
        }
    }
    ~Workers() {
        {
            std::lock_guard<std::mutex> l(m_);
            end_ = true;
        }
        ready_.notify_all();
        for (auto &t : threads_) t.join();
    }
    void give(int i, const Piece &p, const char *from, char *dst) {
        if (threads_.empty()) {
            memcpy(dst + p.at, from + p.offset, p.bytes);
            done_[i] = 1;
            return;
        }
        {
            std::lock_guard<std::mutex> l(m_);
            jobs_.push_back({i, p, from, dst});
        }
        ready_.notify_one();
    }
    bool done(int i) {
        std::lock_guard<std::mutex> l(m_);
        return done_[i] != 0;
    }
    void wait(int i) {
        std::unique_lock<std::mutex> l(m_);
        moved_.wait(l, [&] { return done_[i] != 0; });
    }

  private:
    struct Job {
        int i;
        Piece p;
        const char *from;
        char *dst;
    };
    void loop() {
        std::unique_lock<std::mutex> l(m_);
        for (;;) {
            ready_.wait(l, [&] { return next_ < jobs_.size() || end_; });
            if (next_ >= jobs_.size()) return;
            const Job j = jobs_[next_++];
            l.unlock();
            memcpy(j.dst + j.p.at, j.from + j.p.offset, j.p.bytes);
            l.lock();
            done_[j.i] = 1;
            moved_.notify_all();
        }
    }
    std::mutex m_;
    std::condition_variable ready_, moved_;
    std::vector<Job> jobs_;
    size_t next_ = 0;
    std::vector<char> done_;
    bool end_ = false;
    std::vector<std::thread> threads_;
};

// whether a piece of a chunk lies in the chunk and in the destination
bool fits(const Piece &p, uint64_t total, size_t chunk) {
    return p.at <= total && p.bytes <= total - p.at && p.offset <= chunk && p.bytes <= chunk - p.offset;
}
amr_status misfit(const Piece &p, uint64_t total) {
    return fail(AMR_ERR_DEVICE, "field transfer: %llu bytes at %llu of %llu", (unsigned long long)p.bytes,
                (unsigned long long)p.at, (unsigned long long)total);
}

// through the ring (held by the caller)
amr_status through_ring(amr_handle *h, char *dst, int n, uint64_t total,
                        const std::function<hipError_t(int, char *)> &fill,
                        const std::function<Piece(int, const int64_t *)> &piece) {
    hipStream_t st = h->c.stream;
    const int slots = n < kSlots ? n : kSlots;
    hipEvent_t ev[kSlots] = {nullptr};
    hipError_t e = hipSuccess;
    amr_status s = AMR_OK;
    for (int k = 0; k < slots && e == hipSuccess; k++) e = hipEventCreateWithFlags(&ev[k], hipEventDisableTiming);
    try {
        const uint64_t want = total / kWorkerBytes;
        Workers w(n, n > 1 && want > 1 ? (int)(want < kMaxWorkers ? want : kMaxWorkers) : 0);
        int launched = 0;
        for (int i = 0; i < n && e == hipSuccess && s == AMR_OK; i++) {
            while (launched < n && launched < i + slots && e == hipSuccess) {
                const int before = launched - slots;  // the chunk this slot held
                if (before >= 0 && !w.done(before)) {
                    if (launched > i) break;
                    w.wait(before);
                }
                e = fill(launched, g_ring.mem + (size_t)(launched % slots) * kSlotBytes);
                if (e == hipSuccess) e = hipEventRecord(ev[launched % slots], st);
                launched++;
            }
            if (e == hipSuccess) e = hipEventSynchronize(ev[i % slots]);
            if (e != hipSuccess) break;
            const char *from = g_ring.mem + (size_t)(i % slots) * kSlotBytes;
            const Piece p = piece(i, (const int64_t *)from);
            if (fits(p, total, kSlotBytes)) w.give(i, p, from, dst);
            else s = misfit(p, total);
        }
    } catch (...) {
        e = hipErrorOutOfMemory;
    }
    if (e != hipSuccess || s != AMR_OK) (void)hipStreamSynchronize(st);  // nothing writes the ring once it is free again
    for (int k = 0; k < slots; k++)
        if (ev[k]) hipEventDestroy(ev[k]);
    return e == hipSuccess ? s : fail(AMR_ERR_DEVICE, "field transfer: %s", hipGetErrorString(e));
}

}  // namespace

void transfer_add_user(amr_handle *) {
    std::lock_guard<std::mutex> l(g_ring.count);
    g_ring.users++;
}

void transfer_drop_user(amr_handle *h) {
    if (h->pin) hipHostFree(h->pin);
    h->pin = nullptr;
    std::lock_guard<std::mutex> l(g_ring.count);
    if (--g_ring.users > 0) return;
    std::lock_guard<std::mutex> u(g_ring.use);
    if (g_ring.mem) hipHostFree(g_ring.mem);
    g_ring.mem = nullptr;
}

size_t transfer_chunk(const amr_handle *h, uint64_t total) {
    size_t c = (size_t)(total / kSlots);
    if (c < (size_t(256) << 10)) c = size_t(256) << 10;
    if (c > kSlotBytes) c = kSlotBytes;
    return c < h->c.staging_bytes ? c : h->c.staging_bytes;
}

amr_status transfer_out(amr_handle *h, void *dst_, int n, uint64_t total,
                        const std::function<hipError_t(int, char *)> &fill,
                        const std::function<Piece(int, const int64_t *)> &piece,
                        const std::function<hipError_t()> &plain) {
    hipStream_t st = h->c.stream;
    char *dst = (char *)dst_;
    // a kernel that was to make the data and was refused: no later call says so
    HIP_TRY(hipGetLastError());
    if (n <= 0) {
        HIP_TRY(hipStreamSynchronize(st));
        return AMR_OK;
    }
    h->read_total += total;
    if (!h->pin && ++h->reads == kPinFrom) {
        void *p = nullptr;
        if (hipHostMalloc(&p, kPinBytes, hipHostMallocPortable) == hipSuccess) h->pin = (char *)p;
        else (void)hipGetLastError();
    }
    if (n == 1 && total + kHeadBytes <= kPinBytes && h->pin) {
        HIP_TRY(fill(0, h->pin));
        HIP_TRY(hipStreamSynchronize(st));
        const Piece p = piece(0, (const int64_t *)h->pin);
        if (!fits(p, total, kPinBytes)) return misfit(p, total);
        memcpy(dst + p.at, h->pin + p.offset, p.bytes);
        return AMR_OK;
    }
    std::unique_lock<std::mutex> use(g_ring.use, std::try_to_lock);
    if (use.owns_lock()) {
        if (!g_ring.mem && h->read_total >= kRingFrom) {
            void *p = nullptr;
            if (hipHostMalloc(&p, kSlots * kSlotBytes, hipHostMallocPortable) == hipSuccess) g_ring.mem = (char *)p;
            else (void)hipGetLastError();
        }
        if (g_ring.mem) return through_ring(h, dst, n, total, fill, piece);
        use.unlock();
    }
    if (plain) {
        HIP_TRY(plain());
        HIP_TRY(hipStreamSynchronize(st));
        return AMR_OK;
    }
    for (int i = 0; i < n; i++) {  // through the staging area and the runtime's own pinned memory
        int64_t head[kHeadBytes / 8];
        HIP_TRY(fill(i, (char *)h->c.staging));
        HIP_TRY(hipMemcpyAsync(head, h->c.staging, sizeof(head), hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
        const Piece p = piece(i, head);
        if (!fits(p, total, h->c.staging_bytes)) return misfit(p, total);
        HIP_TRY(hipMemcpyAsync(dst + p.at, (char *)h->c.staging + p.offset, p.bytes, hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
    }
    return AMR_OK;
}

amr_status copy_out(amr_handle *h, void *dst, const void *dev, size_t bytes) {
    hipStream_t st = h->c.stream;
    const size_t chunk = bytes + kHeadBytes <= kPinBytes ? bytes : transfer_chunk(h, bytes);
    const auto size = [&](int i) { return bytes - (size_t)i * chunk < chunk ? bytes - (size_t)i * chunk : chunk; };
    return transfer_out(
        h, dst, bytes ? (int)((bytes + chunk - 1) / chunk) : 0, bytes,
        [&](int i, char *to) {
            return hipMemcpyAsync(to, (const char *)dev + (size_t)i * chunk, size(i), hipMemcpyDefault, st);
        },
        [&](int i, const int64_t *) { return Piece{(uint64_t)i * chunk, 0, size(i)}; },
        [&] { return hipMemcpyAsync(dst, dev, bytes, hipMemcpyDeviceToHost, st); });
}

}  // namespace amr
