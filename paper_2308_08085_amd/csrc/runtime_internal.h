// runtime_internal.h -- state shared by the host runtime files (single
// simulations in runtime.hip, batches in batch.hip): the handle behind amr_t,
// its arena layout, error reporting.
#pragma once

#include <functional>
#include <string>
#include <vector>

#include "../../include/amr_lbm.h"
#include "kernels.h"

namespace amr {

// record a message for amr_last_error() and return `code`
amr_status fail(amr_status code, const char *fmt, ...);

#define HIP_TRY(expr)                                                                          \
    do {                                                                                       \
        hipError_t e_ = (expr);                                                                \
        if (e_ != hipSuccess) return fail(AMR_ERR_DEVICE, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

// Coarse steps under AMR_USE_GRAPH: launched, or replayed from a captured step.
//
// A replay costs the host 13 to 16 us per coarse step whatever it holds, a
// launch 2.5 us, but the GPU takes launches faster and a mesh change costs
// another capture (0.25 ms).  For one simulation the GPU is what bounds the
// steps, and they are launched (D2Q9 cavity 64 x 64, three levels, us per step:
// 51 against 59).  A thread that steps several simulations in turn, each on its
// own stream, is bound by its own launches: eight such cavities 28 us per step
// launched, 20 replayed.  So a step of at least kReplayFrom launches is replayed
// if this thread has enqueued another simulation's steps on another stream since
// it last waited for one, and has twice in a row found this one's stream out of work.
// Results do not depend on it.
class StepReplay {
  public:
    // At the start of a call; true: replay its steps.  launches: of the last
    // coarse step launched.
    bool begin(hipStream_t st, int launches);
    bool captured() const { return exec_[0] && exec_[1]; }
    // Captures what `step` enqueues on st as the coarse step of level-0 parity `par`.
    hipError_t capture(hipStream_t st, int par, const std::function<bool()> &step);
    hipError_t launch(hipStream_t st, int par) const { return hipGraphLaunch(exec_[par], st); }
    // At the end of a call that enqueued steps on st.
    void enqueued(hipStream_t st) const;
    // The captured steps are out of date (or the simulation ends).
    void drop(hipStream_t st);
    // This thread has waited for the GPU.
    static void waited();

  private:
    static constexpr int kReplayFrom = 8, kDry = 2;
    static uint64_t next_id();
    const uint64_t id_ = next_id();
    hipGraphExec_t exec_[2] = {nullptr, nullptr};
    int dry_ = 0;  // calls in a row that found the stream out of work
};

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

struct Layout {
    size_t f[2], nbr, nbrc, X, level, status, tag, ldes, viol, bflag, gmask, imask;
    size_t ids, ids_tmp, iface, refl, sweep, order, force, solidl, gap, first, rlist, outl, off, scan_part;
    size_t crit, part4, solid, solid_list, ctr, staging, staging_bytes, total, hid, U, parent, fresh, desc;
};

}  // namespace amr

using namespace amr;

struct amr_handle {
    amr_config cfg;
    Ctx c;
    Layout lay;
    int lmax;
    int device;  // the GPU current at creation
    int nids[kMaxLevels], niface[kMaxLevels], nsolid[kMaxLevels], nref[kMaxLevels], nsweep[kMaxLevels];
    double ghost_w[kMaxLevels], avg_w[kMaxLevels];  // cells the grid communication of each level moves
    int gtop;
    int n_out, n_outb;  // output cells of the mesh, blocks that hold them
    int par[kMaxLevels];
    double force_sweeps[kMaxLevels] = {0};  // collide-stream sweeps per level since the force reset
    bool force_on = true;                   // accumulate the momentum exchange every sweep
    bool sync_velocity = true;              // criterion velocities from the synchronisation's averaging
    amr::StepReplay replay;                 // coarse steps under AMR_USE_GRAPH
    int launches = 0;                       // kernels launched by the coarse step under way, or the last
    bool skip_parents = false;              // sweeps leave out refined blocks without N_SKIP children
    int batches = 0;                        // batches this handle is a member of
    char *pin = nullptr;                    // pinned memory for small transfers (kPinBytes), may be null
    uint64_t read_total = 0;                // bytes transferred to the host so far
    int reads = 0;                          // transfers made without `pin`
    double tau[kMaxLevels];
    BCParams bc;
    std::vector<uint8_t> solid;
    // AMR_PROFILE: events around each solver launch (kind, start, stop, blocks, bytes)
    bool profiling = false;
    struct Timed { int kind; hipEvent_t a, b; double blocks, bytes; };
    std::vector<Timed> timed;
    std::vector<hipEvent_t> event_pool;
    double kstats[3][4] = {{0}};
    // device times of the adaptation steps (amr_adapt_step order): events at
    // the step boundaries, read after the stream synchronisations the calls
    // make anyway; the first three are those of the last amr_tag
    hipEvent_t step_ev[11] = {nullptr};  // tag: 0-3; adapt: 4-5 (prep), 6-10 (S2 ... S7)
    double step_ms[AMR_T_STEPS] = {0};
};

namespace amr {

// relaxation and rescaling of every level, with the current buffer parities
LevelParams level_params(const amr_handle *h);

// ---- device to host (transfer.hip) ----
constexpr size_t kPinBytes = size_t(64) << 10, kSlotBytes = size_t(4) << 20, kHeadBytes = 64;

// where a filled chunk goes: `bytes` from `offset` in the chunk to byte `at` of
// the destination
struct Piece {
    uint64_t at;
    size_t offset, bytes;
};

void transfer_add_user(amr_handle *h);   // with the handle's creation
void transfer_drop_user(amr_handle *h);  // with its end
// What a transfer moves, in chunks whose size depends on the way it takes.
struct Source {
    // chunks of at most `chunk` bytes from now on; how many
    std::function<int(size_t chunk)> split;
    // enqueues what writes chunk i to `to` (pinned host or device memory) on the
    // handle's stream; whether that was accepted
    std::function<hipError_t(int i, char *to)> fill;
    // where chunk i goes, given its first kHeadBytes (null if it is the only one)
    std::function<Piece(int i, const int64_t *head)> piece;
    // for a plain copy: enqueues all of it, without chunks
    std::function<hipError_t()> plain;
};
// The `total` bytes of src to dst.  Synchronises the stream.  Fails, with
// nothing moved, if an earlier launch was refused, and never writes outside dst.
amr_status transfer_out(amr_handle *h, void *dst, uint64_t total, const Source &src);
// whether memory of the caller is the host's (else the GPU's)
bool host_memory(const void *p);
// a range of device memory to the caller's memory, as transfer_out
amr_status copy_out(amr_handle *h, void *dst, const void *dev, size_t bytes);


}  // namespace amr
