// transfer.hip -- device data to the caller's memory.  Pageable host memory is
// reached through pinned memory that the kernels (or a copy) write directly;
// while the GPU fills the next chunks, host threads move the finished ones on.
// Memory that the GPU can write by itself needs no such help.
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
//
// us to pageable memory, runtime's path and ring:
//   copy of 1.3 MB   80 and 110      rho, u of 0.13 MB   75 and  20
//           3.2 MB  200 and 190                  2.1 MB  205 and 130
//          10.6 MB  620 and 415                 28.3 MB 1840 and 820
// (3.2 MB to memory that was never touched 240 and 210),
// and to pinned memory, staging area and ring:
//   rho, u of 0.13 MB  70 and 20, 1.0 MB 43 and 87, 28.3 MB 545 and 822.
#include <algorithm>
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
// Which way is faster (figures above): plain copies to pageable memory take the
// ring up to kRingCopySmall (one or two chunks, which this thread copies: 0.22 MB
// 25 us, the runtime 19 to 98) and from kRingCopyLarge on (several threads);
// gathers always, but into pinned memory of the caller only below
// kPinnedDirectFrom.
constexpr uint64_t kRingCopySmall = uint64_t(512) << 10, kRingCopyLarge = uint64_t(3) << 20;
constexpr uint64_t kPinnedDirectFrom = uint64_t(1) << 20;
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

size_t ring_chunk(uint64_t total) {
    const size_t c = (size_t)(total / kSlots);
    return std::min(kSlotBytes, std::max(size_t(256) << 10, c));
}

// through the ring (held by the caller)
amr_status through_ring(amr_handle *h, char *dst, uint64_t total, const Source &src) {
    hipStream_t st = h->c.stream;
    const int n = src.split(ring_chunk(total));
    const int slots = n < kSlots ? n : kSlots;
    // The host reads what the kernels wrote once the chunk's event has passed; pinned
    // memory is not promised to be coherent (HIP_HOST_COHERENT), so the event releases
    // to the host.
    constexpr unsigned kEventFlags = hipEventDisableTiming | hipEventReleaseToSystem;
    hipEvent_t ev[kSlots] = {nullptr};
    hipError_t e = hipSuccess;
    amr_status s = AMR_OK;
    for (int k = 0; k < slots && e == hipSuccess; k++) e = hipEventCreateWithFlags(&ev[k], kEventFlags);
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
                e = src.fill(launched, g_ring.mem + (size_t)(launched % slots) * kSlotBytes);
                if (e == hipSuccess) e = hipEventRecord(ev[launched % slots], st);
                launched++;
            }
            if (e == hipSuccess) e = hipEventSynchronize(ev[i % slots]);
            if (e != hipSuccess) break;
            const char *from = g_ring.mem + (size_t)(i % slots) * kSlotBytes;
            const Piece p = src.piece(i, n > 1 ? (const int64_t *)from : nullptr);
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

// through the staging area and the runtime's own pinned memory, or directly to
// memory of the caller that the GPU can write
amr_status through_staging(amr_handle *h, char *dst, uint64_t total, const Source &src) {
    hipStream_t st = h->c.stream;
    const int n = src.split(h->c.staging_bytes);
    for (int i = 0; i < n; i++) {
        int64_t head[kHeadBytes / 8];
        HIP_TRY(src.fill(i, (char *)h->c.staging));
        if (n > 1) {
            HIP_TRY(hipMemcpyAsync(head, h->c.staging, sizeof(head), hipMemcpyDeviceToHost, st));
            HIP_TRY(hipStreamSynchronize(st));
        }
        const Piece p = src.piece(i, n > 1 ? head : nullptr);
        if (!fits(p, total, h->c.staging_bytes)) return misfit(p, total);
        HIP_TRY(hipMemcpyAsync(dst + p.at, (char *)h->c.staging + p.offset, p.bytes, hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
    }
    return AMR_OK;
}

// Memory that the GPU writes by itself: the caller's pinned memory, or a GPU's.
enum class Memory { Pageable, Pinned, Device };
Memory memory_of(const void *p) {
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return Memory::Pageable;
    }
    return a.type == hipMemoryTypeUnregistered ? Memory::Pageable
           : a.type == hipMemoryTypeHost       ? Memory::Pinned
                                               : Memory::Device;
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

bool host_memory(const void *p) { return memory_of(p) != Memory::Device; }

amr_status transfer_out(amr_handle *h, void *dst_, uint64_t total, const Source &src) {
    StepReplay::waited();  // every way below waits for the stream
    hipStream_t st = h->c.stream;
    char *dst = (char *)dst_;
    // a kernel that was to make the data and was refused: no later call says so
    HIP_TRY(hipGetLastError());
    if (total == 0) {
        HIP_TRY(hipStreamSynchronize(st));
        return AMR_OK;
    }
    h->read_total += total;
    if (!h->pin && ++h->reads == kPinFrom) {
        void *p = nullptr;
        if (hipHostMalloc(&p, kPinBytes, hipHostMallocPortable) == hipSuccess) h->pin = (char *)p;
        else (void)hipGetLastError();
    }
    const Memory to = memory_of(dst);
    if (total + kHeadBytes <= kPinBytes && h->pin && to != Memory::Device) {
        if (src.split(kPinBytes) != 1) return fail(AMR_ERR_DEVICE, "field transfer: more than one chunk");
        HIP_TRY(src.fill(0, h->pin));
        HIP_TRY(hipStreamSynchronize(st));
        const Piece p = src.piece(0, nullptr);
        if (!fits(p, total, kPinBytes)) return misfit(p, total);
        memcpy(dst + p.at, h->pin + p.offset, p.bytes);
        return AMR_OK;
    }
    const bool ring = to == Memory::Pageable
                          ? !src.plain || total <= kRingCopySmall || total >= kRingCopyLarge
                          : to == Memory::Pinned && !src.plain && total < kPinnedDirectFrom;
    if (ring) {
        std::unique_lock<std::mutex> use(g_ring.use, std::try_to_lock);
        if (use.owns_lock()) {
            if (!g_ring.mem && h->read_total >= kRingFrom) {
                void *p = nullptr;
                if (hipHostMalloc(&p, kSlots * kSlotBytes, hipHostMallocPortable) == hipSuccess) g_ring.mem = (char *)p;
                else (void)hipGetLastError();
            }
            if (g_ring.mem) return through_ring(h, dst, total, src);
        }
    }
    if (!src.plain) return through_staging(h, dst, total, src);
    HIP_TRY(src.plain());
    HIP_TRY(hipStreamSynchronize(st));
    return AMR_OK;
}

amr_status copy_out(amr_handle *h, void *dst, const void *dev, size_t bytes) {
    hipStream_t st = h->c.stream;
    size_t chunk = bytes;
    const auto size = [&](int i) { return std::min(chunk, bytes - (size_t)i * chunk); };
    const Source src = {
        [&](size_t c) {
            chunk = c;
            return (int)((bytes + c - 1) / c);
        },
        [&](int i, char *to) {
            return hipMemcpyAsync(to, (const char *)dev + (size_t)i * chunk, size(i), hipMemcpyDefault, st);
        },
        [&](int i, const int64_t *) { return Piece{(uint64_t)i * chunk, 0, size(i)}; },
        [&] { return hipMemcpyAsync(dst, dev, bytes, hipMemcpyDeviceToHost, st); }};
    return transfer_out(h, dst, bytes, src);
}

}  // namespace amr
