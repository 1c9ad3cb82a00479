// Host test of csrc/transfer.hip: the HIP calls it makes are replaced by ones
// that work on host memory and of which one can be told to fail.  Every failure
// of a call, a launch that was refused, and a chunk head that names rows outside
// the destination must come back as an error, with nothing written past it.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <atomic>

#include "runtime_internal.h"

using namespace amr;

namespace {
std::atomic<int> g_calls{0};    // fallible calls so far
int g_fail_at = -1;             // the one that fails
bool g_no_pinned = false;       // pinned memory cannot be had
hipMemoryType g_type = hipMemoryTypeUnregistered;  // of the caller's memory
hipError_t g_last = hipSuccess;  // of refused launches
hipError_t call() { return g_calls++ == g_fail_at ? hipErrorInvalidValue : hipSuccess; }
}  // namespace

extern "C" {
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    const hipError_t e = call();
    if (e == hipSuccess) memcpy(d, s, n);
    return e;
}
hipError_t hipStreamSynchronize(hipStream_t) { return call(); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    const hipError_t r = call();
    *e = r == hipSuccess ? (hipEvent_t)malloc(1) : nullptr;
    return r;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return call(); }
hipError_t hipEventSynchronize(hipEvent_t) { return call(); }
hipError_t hipEventDestroy(hipEvent_t e) {
    free((void *)e);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    *p = g_no_pinned ? nullptr : malloc(n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p) {
    free(p);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *) {
    a->type = g_type;
    if (g_type != hipMemoryTypeUnregistered) return hipSuccess;
    return g_last = hipErrorInvalidValue;  // as for memory that the runtime does not know
}
hipError_t hipGetLastError(void) {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "error"; }
}

namespace amr {
amr_status fail(amr_status code, const char *, ...) { return code; }
uint64_t StepReplay::next_id() { return 1; }
void StepReplay::waited() {}
}  // namespace amr

namespace {

int g_bad = 0;
void expect(bool ok, const char *what, size_t bytes, int at) {
    if (ok) return;
    g_bad++;
    printf("FAILED: %s, %zu bytes, call %d\n", what, bytes, at);
}

enum Fault { kNone_, kEarlier, kRefused, kHeadHigh, kHeadNegative };

struct Run {
    amr_status s;
    bool right, guards;
    int chunks;
};

// one transfer of `bytes`; rows: as a gather with heads, else a copy
Run transfer(size_t bytes, bool rows, bool pin, bool ring, Fault fault) {
    amr_handle h;
    std::vector<char> staging(size_t(1) << 20), data(bytes), out(bytes + 2048, 7);
    h.c.staging = staging.data();
    h.c.staging_bytes = staging.size();
    for (size_t i = 0; i < bytes; i++) data[i] = (char)(i * 2654435761u >> 13);
    transfer_add_user(&h);
    g_no_pinned = false;
    if (pin) h.pin = (char *)malloc(kPinBytes);
    if (ring) h.read_total = uint64_t(1) << 30;
    else g_no_pinned = true;
    char *dst = out.data() + 1024;
    if (fault == kEarlier) g_last = hipErrorInvalidConfiguration;
    Run r{};
    if (rows) {
        const size_t row = 32;
        const int64_t all = (int64_t)(bytes / row);
        int64_t per = 1;
        int n = 0;
        const Source src = {
            [&](size_t chunk) {
                per = (int64_t)((chunk - kHeadBytes) / row);
                return n = (int)((all + per - 1) / per);
            },
            [&](int i, char *to) {
                if (fault == kRefused && i == n - 1) return hipErrorInvalidConfiguration;  // and nothing written
                const int64_t first = i * per, end = std::min(all, (i + 1) * per);
                int64_t head[2] = {first, end - first};
                if (i == n - 1 && fault == kHeadHigh) head[0] += 1;
                if (i == n - 1 && fault == kHeadNegative) head[0] = -1;
                memcpy(to, head, sizeof(head));
                memcpy(to + kHeadBytes, data.data() + first * row, (end - first) * row);
                return hipSuccess;
            },
            [&](int, const int64_t *head) {
                expect((n == 1) == (head == nullptr), "head", bytes, n);
                return head ? Piece{(uint64_t)head[0] * row, kHeadBytes, (size_t)head[1] * row}
                            : Piece{0, kHeadBytes, bytes};
            },
            nullptr};
        r.s = transfer_out(&h, dst, bytes, src);
        r.chunks = n;
    } else {
        r.s = copy_out(&h, dst, data.data(), bytes);
    }
    r.right = bytes == 0 || memcmp(dst, data.data(), bytes) == 0;
    r.guards = true;
    for (int i = 0; i < 1024; i++) r.guards = r.guards && out[i] == 7 && out[1024 + bytes + i] == 7;
    if (h.pin) free(h.pin);
    h.pin = nullptr;
    transfer_drop_user(&h);
    g_last = hipSuccess;
    return r;
}

}  // namespace

int main() {
    int n = 0;
    const size_t sizes[] = {0, 32, 4096, 65472, 65504, 700000 / 32 * 32, (size_t(5) << 20) + 96};
    const hipMemoryType types[] = {hipMemoryTypeUnregistered, hipMemoryTypeHost, hipMemoryTypeDevice};
    for (int mode = 0; mode < 24; mode++) {
        const bool rows = mode & 1, pin = mode & 2, ring = mode & 4;
        g_type = types[mode >> 3];
        for (size_t bytes : sizes) {
            g_fail_at = -1;
            g_calls = 0;
            Run r = transfer(bytes, rows, pin, ring, kNone_);
            expect(r.s == AMR_OK && r.right && r.guards, "plain transfer", bytes, -1);
            const int calls = g_calls, chunks = r.chunks;
            expect(calls > 0, "synchronises", bytes, -1);
            for (int k = 0; k < calls; k++) {
                g_fail_at = k;
                g_calls = 0;
                r = transfer(bytes, rows, pin, ring, kNone_);
                expect(r.s == AMR_ERR_DEVICE && r.guards, "failed call", bytes, k);
                n++;
            }
            g_fail_at = -1;
            r = transfer(bytes, rows, pin, ring, kEarlier);
            expect(r.s == AMR_ERR_DEVICE && r.guards, "earlier launch refused", bytes, -1);
            for (Fault f : {kRefused, kHeadHigh, kHeadNegative}) {
                // the head is not used where there is one chunk
                if (!rows || bytes == 0 || (chunks == 1 && f != kRefused)) continue;
                r = transfer(bytes, rows, pin, ring, f);
                expect(r.s == AMR_ERR_DEVICE && r.guards, "refused launch or wrong head", bytes, -1);
                n++;
            }
        }
    }
    printf("%d failures tried, %d not reported\n", n, g_bad);
    return g_bad ? 1 : 0;
}
