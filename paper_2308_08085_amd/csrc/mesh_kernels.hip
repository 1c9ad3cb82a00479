// mesh_kernels.hip -- on-device mesh management of the AMR-LBM library:
// root-grid construction, refinement criteria to tags, the refine/coarsen
// routine (Sec. "Refinement and Coarsening": gap assignment, 2:1 reversion,
// child construction, ID-set updates, connectivity rebuild) and the ordered
// scans it is built on.  Order-dependent results come from ballot/popcount
// scans, never from atomics, so tables are deterministic.
#include "kernels.h"

#include <tuple>

namespace amr {

namespace {

constexpr int kScanTPB = 256;
constexpr int kScanPer = 4;
constexpr int kScanItems = kScanTPB * kScanPer;

inline int grid_for(int64_t n, int tpb = 256) { return (int)((n + tpb - 1) / tpb); }

// ---------------------------------------------------------------------------
// Ordered lists.  A job gives every index of its range a bin (-1: none); its
// rank is the number of earlier indexes (in order) with the same bin, and the
// job's put() places it by that rank.  A job with kSum gives a value instead,
// and the rank is the sum of the earlier values.
//   K        bins
//   n(m)     indexes
//   bin(m, ctr, i)
//   put(m, ctr, i, bin, rank, tot)   tot: all K totals; called for every index
//   done(m, ctr, tot)                one thread, beside the puts: may write
//                                    only what no bin() or put() of the launch reads
// Two launches: the counts of every 1024 indexes, then ranks and puts, for which
// every workgroup adds up the counts before its own.  Independent jobs share
// both (grid y).  Small meshes are bound by the number of launches (6 to 7 us
// each, gap included): bins, counts, their scan, ranks, compaction and copy were
// six per list and 87 for a mesh change with three levels, now 31.  64 x 64 2-D
// cavity with four changes 10.5 -> 9.6 ms, eight steps and one change of a 52^3
// cavity 4.8 -> 4.5 ms.
// Above kScanDirect workgroups a single one scans the counts in between, since
// the counts that every workgroup reads grow with the square.
constexpr int kScanDirect = 1024;

inline __host__ __device__ int scan_groups(int64_t n) { return (int)((n + kScanItems - 1) / kScanItems); }

template <typename J>
__device__ __forceinline__ void scan_count(const J &j, const DevMesh &m, const DevCounters *ctr, int32_t *part) {
    const int64_t n = j.n(m);
    const int wg = blockIdx.x, lane = threadIdx.x & 63;
    __shared__ int32_t s_cnt[kMaxLevels];
    if (wg >= scan_groups(n)) return;
    if ((int)threadIdx.x < kMaxLevels) s_cnt[threadIdx.x] = 0;
    __syncthreads();
    if constexpr (J::kSum) {
        int sum = 0;
        for (int r = 0; r < kScanPer; r++) {
            const int64_t i = (int64_t)wg * kScanItems + r * kScanTPB + threadIdx.x;
            if (i < n) sum += j.bin(m, ctr, i);
        }
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
        if (lane == 0) atomicAdd(&s_cnt[0], sum);
    } else {
        for (int r = 0; r < kScanPer; r++) {
            const int64_t i = (int64_t)wg * kScanItems + r * kScanTPB + threadIdx.x;
            const int b = i < n ? j.bin(m, ctr, i) : -1;
            for (int k = 0; k < j.K; k++) {
                const uint64_t msk = __ballot(b == k);
                if (lane == 0 && msk) atomicAdd(&s_cnt[k], (int)__popcll(msk));
            }
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < j.K) part[(int64_t)wg * j.K + threadIdx.x] = s_cnt[threadIdx.x];
}

// exclusive scan of the counts of one job in place, the totals behind them
template <typename J>
__device__ __forceinline__ void scan_part(const J &j, const DevMesh &m, int32_t *part) {
    __shared__ int32_t s[256];
    const int t = threadIdx.x, K = j.K, nwg = scan_groups(j.n(m));
    const int chunk = (nwg + 255) / 256;
    for (int k = 0; k < K; k++) {
        const int lo = min(nwg, t * chunk), hi = min(nwg, lo + chunk);
        int sum = 0;
        for (int i = lo; i < hi; i++) sum += part[(int64_t)i * K + k];
        s[t] = sum;
        __syncthreads();
        for (int off = 1; off < 256; off <<= 1) {
            const int v = t >= off ? s[t - off] : 0;
            __syncthreads();
            s[t] += v;
            __syncthreads();
        }
        int run = s[t] - sum;
        for (int i = lo; i < hi; i++) {
            const int v = part[(int64_t)i * K + k];
            part[(int64_t)i * K + k] = run;
            run += v;
        }
        if (t == 255) part[(int64_t)nwg * K + k] = s[255];
        __syncthreads();
    }
}

template <typename J>
__device__ __forceinline__ void scan_put(const J &j, const DevMesh &m, DevCounters *ctr, const int32_t *part,
                                         bool scanned) {
    const int64_t n = j.n(m);
    const int K = j.K, nwg = scan_groups(n), wg = blockIdx.x, t = threadIdx.x;
    __shared__ int32_t s_run[kMaxLevels], s_tot[kMaxLevels];
    __shared__ int32_t s_wt[4][kMaxLevels];
    if (wg >= nwg) return;
    if (t < kMaxLevels) {
        s_run[t] = scanned && t < K ? part[(int64_t)wg * K + t] : 0;
        s_tot[t] = scanned && t < K ? part[(int64_t)nwg * K + t] : 0;
    }
    __syncthreads();
    if (!scanned) {
        // a thread's entries all have the same bin
        const int step = 256 / K * K, all = nwg * K, mine = wg * K;
        int run = 0, tot = 0;
        if (t < step)
            for (int e = t; e < all; e += step) {
                const int v = part[e];
                tot += v;
                run += e < mine ? v : 0;
            }
        if (tot) atomicAdd(&s_tot[t % K], tot);
        if (run) atomicAdd(&s_run[t % K], run);
        __syncthreads();
    }
    const int lane = t & 63, wave = t >> 6;
    const uint64_t below = (1ull << lane) - 1ull;
    for (int r = 0; r < kScanPer; r++) {
        const int64_t i = (int64_t)wg * kScanItems + r * kScanTPB + t;
        int b = J::kSum ? 0 : -1;
        if (i < n) b = j.bin(m, ctr, i);
        int my = 0;
        if constexpr (J::kSum) {
            int x = b;
            for (int off = 1; off < 64; off <<= 1) {
                const int y = __shfl_up(x, off, 64);
                if (lane >= off) x += y;
            }
            my = x - b;
            if (lane == 63) s_wt[wave][0] = x;
        } else {
            for (int k = 0; k < K; k++) {
                const uint64_t msk = __ballot(b == k);
                if (b == k) my = (int)__popcll(msk & below);
                if (lane == 0) s_wt[wave][k] = (int)__popcll(msk);
            }
        }
        __syncthreads();
        if (i < n) {
            int rank = 0;
            if (J::kSum || b >= 0) {
                const int k = J::kSum ? 0 : b;
                rank = s_run[k] + my;
                for (int w = 0; w < wave; w++) rank += s_wt[w][k];
            }
            j.put(m, ctr, i, b, rank, s_tot);
        }
        __syncthreads();
        if (t < K) s_run[t] += s_wt[0][t] + s_wt[1][t] + s_wt[2][t] + s_wt[3][t];
        __syncthreads();
    }
    if (wg == 0 && t == 0) j.done(m, ctr, s_tot);
}

template <typename J>
struct Scan {
    J j;
    int32_t *part;
};

template <typename... Js>
__global__ __launch_bounds__(256) void k_scan_count(DevMesh m, const DevCounters *ctr, Scan<Js>... s) {
    int y = 0;
    ((blockIdx.y == y++ ? scan_count(s.j, m, ctr, s.part) : void()), ...);
}

template <typename... Js>
__global__ __launch_bounds__(256) void k_scan_part(DevMesh m, Scan<Js>... s) {
    int y = 0;
    ((blockIdx.y == y++ ? scan_part(s.j, m, s.part) : void()), ...);
}

template <typename... Js>
__global__ __launch_bounds__(256) void k_scan_put(DevMesh m, DevCounters *ctr, bool scanned, Scan<Js>... s) {
    int y = 0;
    ((blockIdx.y == y++ ? scan_put(s.j, m, ctr, s.part, scanned) : void()), ...);
}

template <typename... Js>
void run_lists(const Ctx &c, Js... js) {
    int nwg = 0;
    int32_t *part = c.scan_part;
    const auto place = [&](auto j) {
        const int g = scan_groups(j.n(c.m));
        Scan<decltype(j)> s{j, part};
        part += (int64_t)(g + 1) * j.K;
        nwg = g > nwg ? g : nwg;
        return s;
    };
    const auto go = [&](auto... s) {
        const dim3 grid(nwg, sizeof...(s));
        const bool scanned = nwg > kScanDirect;
        k_scan_count<<<grid, kScanTPB, 0, c.stream>>>(c.m, c.ctr, s...);
        if (scanned) k_scan_part<<<dim3(1, sizeof...(s)), 256, 0, c.stream>>>(c.m, s...);
        k_scan_put<<<grid, kScanTPB, 0, c.stream>>>(c.m, c.ctr, scanned, s...);
    };
    std::apply(go, std::tuple{place(js)...});  // braces: left to right
}

// jobs over all block IDs
struct BlockJob {
    static constexpr bool kSum = false;
    int K = 1;
    __host__ __device__ int64_t n(const DevMesh &m) const { return m.cap; }
    __device__ void done(const DevMesh &, DevCounters *, const int32_t *) const {}
};

// jobs over the virtual concatenation of per-level lists: index = L * cap + i
struct LevelJob {
    static constexpr bool kSum = false;
    int K;  // = lmax
    __host__ __device__ int64_t n(const DevMesh &m) const { return (int64_t)m.lmax * m.cap; }
};

// ---------------------------------------------------------------------------
struct RootParams {
    int dim, nroot, lmax;
    int root[3];
    int periodic[3];
    int prio[6];
};

template <typename Dd>
__device__ int32_t root_link(const RootParams &rp, const uint8_t *solid, int bi, int bj, int bk, int p) {
    int r[3] = {bi + Dd::cx(p), bj + Dd::cy(p), bk + Dd::cz(p)};
    bool crossed[6] = {false, false, false, false, false, false};
    bool out = false;
    for (int a = 0; a < rp.dim; a++) {
        if (r[a] < 0) {
            if (rp.periodic[a]) r[a] += rp.root[a];
            else { crossed[2 * a] = true; out = true; }
        } else if (r[a] >= rp.root[a]) {
            if (rp.periodic[a]) r[a] -= rp.root[a];
            else { crossed[2 * a + 1] = true; out = true; }
        }
    }
    if (out) {
        int best = -1;
        for (int fc = 0; fc < 6; fc++)
            if (crossed[fc] && (best < 0 || rp.prio[fc] > rp.prio[best])) best = fc;
        return -3 - best;
    }
    const int id = r[0] + rp.root[0] * (r[1] + rp.root[1] * r[2]);
    if (solid && solid[id]) return kSolid;
    return id;
}

template <typename Dd>
__global__ void k_init_blocks(DevMesh m, RootParams rp, const uint8_t *solid) {
    const int B = blockIdx.x * blockDim.x + threadIdx.x;
    if (B >= m.cap) return;
    m.tag[B] = 0;
    m.ldes[B] = 0;
    m.viol[B] = 0;
    m.bflag[B] = 0;
    m.gmask[B] = 0;
    m.imask[B] = 0;
    m.level[B] = 0;
    m.parent[B] = -1;
    m.fresh[B] = 0;
    if (B >= rp.nroot) {
        m.status[B] = ST_INACTIVE;
        for (int a = 0; a < 3; a++) m.X[(int64_t)a * m.cap + B] = 0;
        return;
    }
    const int bi = B % rp.root[0], bj = (B / rp.root[0]) % rp.root[1], bk = B / (rp.root[0] * rp.root[1]);
    const int W0 = 4 << (rp.lmax - 1);
    m.X[B] = bi * W0;
    m.X[(int64_t)m.cap + B] = bj * W0;
    m.X[(int64_t)2 * m.cap + B] = bk * W0;
    const bool sol = solid && solid[B];
    m.status[B] = sol ? ST_INACTIVE : ST_UNREF;
    for (int p = 0; p < Dd::NB; p++) {
        const int32_t n = sol ? 0 : root_link<Dd>(rp, solid, bi, bj, bk, p);
        m.nbr[(int64_t)p * m.cap + B] = n;
        m.nbrc[(int64_t)p * m.cap + B] = n >= 0 ? kNone : n;
    }
}

__global__ void k_init_gap(int32_t *gap, int cap, int nroot) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g < cap - nroot) gap[g] = cap - 1 - g;
}

// the root blocks that are not solid, and the counters of a new mesh
struct InitJob : BlockJob {
    int32_t *ids;
    int nroot;
    __device__ int bin(const DevMesh &m, const DevCounters *, int64_t B) const { return m.status[B] == ST_UNREF ? 0 : -1; }
    __device__ void put(const DevMesh &, DevCounters *, int64_t B, int b, int r, const int32_t *) const {
        if (b == 0) ids[r] = (int32_t)B;
    }
    __device__ void done(const DevMesh &m, DevCounters *ctr, const int32_t *tot) const {
        ctr->nids[0] = tot[0];
        for (int L = 1; L < kMaxLevels; L++) ctr->nids[L] = 0;
        for (int L = 0; L < kMaxLevels; L++) ctr->niface[L] = ctr->nref[L] = ctr->nsweep[L] = ctr->nsolid[L] = 0;
        ctr->gtop = m.cap - nroot;
        ctr->n_ref = ctr->n_coa = ctr->n_rev = ctr->nfreed = 0;
        ctr->wmax_bits = 0;
    }
};

// ---------------------------------------------------------------------------
// Cell classes (Sec. "Grid Communication"): a cell of a block on level > 0 is a
// ghost if its Chebyshev distance (adjacent = 1) to some N_SKIP neighbour
// region is at most 2, an interface cell at 3 or 4.  Also the per-block flags
// used by the solver kernels.
template <typename Dd>
__global__ void k_block_masks(DevMesh m, DevCounters *ctr) {
    const int B = blockIdx.x * blockDim.x + threadIdx.x;
    if (B < kMaxLevels) ctr->ghost_w[B] = ctr->avg_w[B] = 0;  // for k_target_cells (lbm_kernels.hip)
    if (B >= m.cap) return;
    if (m.status[B] == ST_INACTIVE) {
        m.bflag[B] = 0;
        m.gmask[B] = 0;
        m.imask[B] = 0;
        return;
    }
    uint8_t fl = 0;
    uint32_t skipset = 0;
    for (int p = 1; p < Dd::NB; p++) {
        const int32_t n = m.nbr[(int64_t)p * m.cap + B];
        if (n == kNSkip) { fl |= BF_NSKIP; skipset |= 1u << p; }
        else if (n < 0) fl |= n == kSolid ? (BF_BOUNDARY | BF_SOLID) : BF_BOUNDARY;
    }
    uint64_t gm = 0, im = 0;
    if (m.level[B] > 0 && skipset) {
        for (int l = 0; l < Dd::MB; l++) {
            const int ci[3] = {l & 3, (l >> 2) & 3, l >> 4};
            int d = 1 << 20;
            for (int p = 1; p < Dd::NB; p++) {
                if (!((skipset >> p) & 1u)) continue;
                const int v[3] = {Dd::cx(p), Dd::cy(p), Dd::cz(p)};
                int dist = 0;
                for (int a = 0; a < Dd::D; a++) {
                    const int da = v[a] == 1 ? 4 - ci[a] : (v[a] == -1 ? ci[a] + 1 : 0);
                    dist = da > dist ? da : dist;
                }
                d = dist < d ? dist : d;
            }
            if (d <= 2) gm |= 1ull << l;
            else if (d <= 4) im |= 1ull << l;
        }
    }
    m.bflag[B] = fl;
    m.gmask[B] = gm;
    m.imask[B] = im;
}

template <typename Dd>
__global__ void k_parent_mask(DevMesh m) {
    const int B = blockIdx.x * blockDim.x + threadIdx.x;
    if (B >= m.cap || !is_refined(m.status[B])) return;
    const int c0 = m.nbrc[B];
    bool any = false;
    for (int c = 0; c < Dd::NC; c++) any = any || (m.bflag[c0 + c] & BF_NSKIP);
    if (any) m.bflag[B] = m.bflag[B] | BF_PARENT_MASK;
}

// ---------------------------------------------------------------------------
// Tagging.
__global__ void k_crit_reset(double *crit, int cap, DevCounters *ctr) {
    const int B = blockIdx.x * blockDim.x + threadIdx.x;
    if (B < cap) crit[B] = -1.0;
    if (B == 0) ctr->wmax_bits = 0ull;
}

// leaves: desired level L_max-1 above theta * max, else 0; refine when above the own level
// Desired level of each leaf (Sec. "Adaptive Mesh Refinement" of the
// solver).  Relative threshold: the finest level where the block maximum
// exceeds theta times the maximum over all leaves, else level 0.  Ladder
// (Alg. 3): with eps = min(1, log2 |w|), the level L_max-1 is lowered to
// (L_max-1) - p for every p with eps < n_start - p n_inc; evaluated as
// |w| < 2^(n_start - p n_inc) against thresholds made on the host (a
// threshold above 2 always holds, as eps <= 1).
__global__ void k_tag_vort_leaf(DevMesh m, const double *crit, const DevCounters *ctr, double theta, int ladder,
                                LadderParams lad) {
    const int B = blockIdx.x * blockDim.x + threadIdx.x;
    if (B >= m.cap) return;
    if (m.status[B] != ST_UNREF) {
        m.tag[B] = 0;
        return;
    }
    int ldes;
    if (ladder) {
        const double w = crit[B] * lad.scale;
        ldes = m.lmax - 1;
        for (int p = 1; p <= m.lmax - 1; p++)
            if (w < lad.thr[p]) ldes = (m.lmax - 1) - p;
    } else {
        const double wmax = __longlong_as_double((long long)ctr->wmax_bits);
        ldes = crit[B] > theta * wmax ? m.lmax - 1 : 0;
    }
    m.ldes[B] = (int8_t)ldes;
    m.tag[B] = ldes > m.level[B] ? 1 : 0;
}

// refined blocks whose children are all leaves: coarsen when no child wants to
// be finer than the parent's level
template <typename Dd>
__global__ void k_tag_vort_parent(DevMesh m) {
    const int B = blockIdx.x * blockDim.x + threadIdx.x;
    if (B >= m.cap || m.status[B] != ST_REF) return;
    const int c0 = m.nbrc[B];
    int mx = 0;
    for (int c = 0; c < Dd::NC; c++) mx = m.ldes[c0 + c] > mx ? m.ldes[c0 + c] : mx;
    if (mx <= m.level[B]) m.tag[B] = -1;
}

struct DistParams {
    int dim, lmax, n_solid;
    int dom[3];
    int face_kind[6];
    double dspec_f;
    int freeze;
};

__global__ void k_tag_distance(DevMesh m, const int32_t *solid_list, DistParams dp) {
    const int B = blockIdx.x * blockDim.x + threadIdx.x;
    if (B >= m.cap) return;
    if (m.status[B] != ST_UNREF) {
        m.tag[B] = 0;
        return;
    }
    const int L = m.level[B];
    const int W = 4 << (dp.lmax - 1 - L), W0 = 4 << (dp.lmax - 1);
    int lo[3], hi[3];
    for (int a = 0; a < 3; a++) {
        lo[a] = m.X[(int64_t)a * m.cap + B];
        hi[a] = lo[a] + (a < dp.dim ? W : 0);
    }
    double best = -1.0;
    for (int s = 0; s < dp.n_solid; s++) {
        const int S = solid_list[s];
        long long d2 = 0;
        for (int a = 0; a < dp.dim; a++) {
            const int slo = m.X[(int64_t)a * m.cap + S], shi = slo + W0;
            long long g = 0;
            if (hi[a] < slo) g = slo - hi[a];
            else if (shi < lo[a]) g = lo[a] - shi;
            d2 += g * g;
        }
        if (best < 0 || (double)d2 < best) best = (double)d2;
    }
    for (int fc = 0; fc < 2 * dp.dim; fc++) {
        if (dp.face_kind[fc] != AMR_FACE_OUTFLOW) continue;
        const int a = fc / 2;
        const long long g = (fc & 1) ? (long long)(dp.dom[a] - hi[a]) : (long long)lo[a];
        const double d2 = (double)(g * g);
        if (best < 0 || d2 < best) best = d2;
    }
    const double thr = dp.dspec_f / (double)(1 << L);
    m.tag[B] = (best >= 0.0 && best < thr * thr) ? (dp.freeze ? 2 : 1) : 0;
}

// eligibility and the 2:1 refine-cancel; counts of refine / coarsen marks
__global__ void k_effective_tags(DevMesh m, DevCounters *ctr) {
    const int B = blockIdx.x * blockDim.x + threadIdx.x;
    int out = 0;
    if (B < m.cap) {
        const int t = m.tag[B], st = m.status[B];
        if (st != ST_INACTIVE) {
            if (t == 1 || t == 2) {
                if (st == ST_UNREF && m.level[B] < m.lmax - 1 && !(m.bflag[B] & BF_NSKIP)) out = t;
            } else if (t == -1) {
                if (st == ST_REF) out = -1;
            }
        }
        m.tag[B] = (int8_t)out;
    }
    const uint64_t r = __ballot(out > 0), c = __ballot(out < 0);
    if ((threadIdx.x & 63) == 0) {
        if (r) atomicAdd(&ctr->n_ref, (int)__popcll(r));
        if (c) atomicAdd(&ctr->n_coa, (int)__popcll(c));
    }
}

// ---------------------------------------------------------------------------
// Adaptation.
// S2: the r-th refine-marked block (ascending ID) takes the N_c gaps below
// the top of the gap stack; its first child is gap[top - 1 - N_c r]
struct RefineJob : BlockJob {
    const int32_t *gap;
    int32_t *first, *rlist;
    int nc;
    __device__ int bin(const DevMesh &m, const DevCounters *, int64_t B) const {
        const int t = m.tag[B];
        return t == 1 || t == 2 ? 0 : -1;
    }
    __device__ void put(const DevMesh &, DevCounters *ctr, int64_t B, int b, int r, const int32_t *) const {
        first[B] = b == 0 ? gap[ctr->gtop - 1 - nc * r] : -1;
        if (b == 0) rlist[r] = (int32_t)B;
    }
};

// S3: a leaf is violating if any provisional neighbour-child (this call's new
// children included, and its own at p = 0) is a valid ID
template <typename Dd>
__global__ void k_violating(DevMesh m, const int32_t *first, DevCounters *ctr, int taken) {
    const int B = blockIdx.x * blockDim.x + threadIdx.x;
    if (B == 0) ctr->gtop -= taken;
    if (B >= m.cap) return;
    int8_t v = 0;
    if (m.status[B] == ST_UNREF) {
        for (int p = 0; p < Dd::NB && !v; p++) {
            int32_t pc;
            if (p == 0) {
                pc = first[B] >= 0 ? first[B] : m.nbrc[B];
            } else {
                const int32_t n = m.nbr[(int64_t)p * m.cap + B];
                pc = (n >= 0 && first[n] >= 0) ? first[n] : m.nbrc[(int64_t)p * m.cap + B];
            }
            if (pc >= 0) v = 1;
        }
    }
    m.viol[B] = v;
}

template <typename Dd>
__global__ void k_revert(DevMesh m, DevCounters *ctr) {
    const int B = blockIdx.x * blockDim.x + threadIdx.x;
    bool rev = false;
    if (B < m.cap && m.tag[B] == -1) {
        const int c0 = m.nbrc[B];
        for (int c = 0; c < Dd::NC && c0 >= 0; c++) rev = rev || m.viol[c0 + c];
        if (rev) m.tag[B] = 0;
    }
    const uint64_t msk = __ballot(rev);
    if ((threadIdx.x & 63) == 0 && msk) atomicAdd(&ctr->n_rev, (int)__popcll(msk));
}

// S4: new children get level + 1, status NEW and their origin; the parent's
// neighbour-child p = 0 becomes its first child
template <typename Dd>
__global__ void k_build_children(DevMesh m, const int32_t *rlist, const int32_t *first, int n_ref) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_ref * Dd::NC) return;
    const int r = e / Dd::NC, c = e - r * Dd::NC;
    const int P = rlist[r];
    const int ch = first[P] + c;
    const int L = m.level[P] + 1;
    const int W = 4 << (m.lmax - 1 - L);
    m.level[ch] = (int8_t)L;
    m.status[ch] = ST_NEW;
    m.tag[ch] = 0;
    const int cv[3] = {c & 1, (c >> 1) & 1, (c >> 2) & 1};
    for (int a = 0; a < 3; a++) m.X[(int64_t)a * m.cap + ch] = m.X[(int64_t)a * m.cap + P] + cv[a] * W;
    m.nbrc[ch] = kNone;
    m.parent[ch] = P;
    m.fresh[ch] = 1;
    if (c == 0) m.nbrc[P] = first[P];
}

// S5: freed children in (parent level, parent ID, child) order F; the gap
// stack receives reverse(F) on top
struct CoarsenJob : BlockJob {
    int32_t *gap;
    int nc;
    __device__ int bin(const DevMesh &m, const DevCounters *, int64_t B) const { return m.tag[B] == -1 ? m.level[B] : -1; }
    __device__ void put(const DevMesh &m, DevCounters *ctr, int64_t B, int b, int r, const int32_t *tot) const {
        if (b < 0) return;
        int nF = 0, pos = r;
        for (int k = 0; k < K; k++) {
            nF += tot[k];
            if (k < b) pos += tot[k];
        }
        nF *= nc;
        const int c0 = m.nbrc[B];
        for (int c = 0; c < nc; c++) {
            gap[ctr->gtop + nF - 1 - (pos * nc + c)] = c0 + c;
            m.status[c0 + c] = ST_REMOVE;
        }
        m.nbrc[B] = kNone;
    }
    // the stack's new top: once every put has read the old one (k_copy_kept)
    __device__ void done(const DevMesh &, DevCounters *ctr, const int32_t *tot) const {
        int n = 0;
        for (int k = 0; k < K; k++) n += tot[k];
        ctr->nfreed = nc * n;
        ctr->n_coa = n;
    }
};

// the blocks of each ID set that are not freed
struct KeepJob : LevelJob {
    const int32_t *ids;
    int32_t *kept;
    __device__ int bin(const DevMesh &m, const DevCounters *ctr, int64_t e) const {
        const int L = (int)(e / m.cap), i = (int)(e - (int64_t)L * m.cap);
        return i < ctr->nids[L] && m.status[ids[e]] != ST_REMOVE ? L : -1;
    }
    __device__ void put(const DevMesh &m, DevCounters *, int64_t e, int b, int r, const int32_t *) const {
        if (b >= 0) kept[(int64_t)b * m.cap + r] = ids[e];
    }
    __device__ void done(const DevMesh &, DevCounters *ctr, const int32_t *tot) const {
        for (int k = 0; k < kMaxLevels; k++) ctr->totals[k] = k < K ? tot[k] : 0;
    }
};

// ... copied back (other workgroups were reading the ID sets)
__global__ void k_copy_kept(const int32_t *src, int32_t *dst, int cap, int lmax, DevCounters *ctr) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < (int64_t)lmax * cap) {
        const int L = (int)(e / cap), i = (int)(e - (int64_t)L * cap);
        if (i < ctr->totals[L]) dst[e] = src[e];
    }
    if (e == 0) {
        for (int L = 0; L < lmax; L++) ctr->nids[L] = ctr->totals[L];
        ctr->gtop += ctr->nfreed;
    }
}

// S6: append new children to id_set_{L+1} in (parent ID, child) order; the
// counts follow in k_finalize_status
struct AppendJob : BlockJob {
    const int32_t *first;
    int32_t *ids;
    int nc;
    __device__ int bin(const DevMesh &m, const DevCounters *, int64_t B) const {
        const int t = m.tag[B];
        return t == 1 || t == 2 ? m.level[B] : -1;
    }
    __device__ void put(const DevMesh &m, DevCounters *ctr, int64_t B, int b, int r, const int32_t *) const {
        if (b < 0) return;
        const int base = ctr->nids[b + 1] + nc * r;
        for (int c = 0; c < nc; c++) ids[(int64_t)(b + 1) * m.cap + base + c] = first[B] + c;
    }
    __device__ void done(const DevMesh &, DevCounters *ctr, const int32_t *tot) const {
        for (int k = 0; k < kMaxLevels; k++) ctr->totals[k] = k < K ? tot[k] : 0;
    }
};

// S7: finalise statuses, then branch / leaf
__global__ void k_finalize_status(DevMesh m, DevCounters *ctr, int appended) {  // appended: children per block of totals
    const int B = blockIdx.x * blockDim.x + threadIdx.x;
    if (B == 0)
        for (int L = 0; L + 1 < m.lmax; L++) ctr->nids[L + 1] += appended * ctr->totals[L];
    if (B >= m.cap) return;
    const int t = m.tag[B];
    int st = m.status[B];
    if (t == 1) st = ST_REF;
    else if (t == 2) st = ST_REF_PERM;
    else if (t == -1) st = ST_UNREF;
    if (st == ST_NEW) st = ST_UNREF;
    else if (st == ST_REMOVE) st = ST_INACTIVE;
    m.status[B] = (int8_t)st;
    m.tag[B] = 0;
}

template <typename Dd>
__global__ void k_branch_leaf(DevMesh m) {
    const int B = blockIdx.x * blockDim.x + threadIdx.x;
    if (B >= m.cap) return;
    const int st = m.status[B];
    if (st != ST_REF && st != ST_REF_CHILD) return;
    const int c0 = m.nbrc[B];
    bool any = false;
    for (int c = 0; c < Dd::NC; c++) any = any || is_refined(m.status[c0 + c]);
    m.status[B] = any ? ST_REF_CHILD : ST_REF;
}

// S8: neighbour-children of level L from its links ...
template <typename Dd>
__global__ void k_nbrc_level(DevMesh m, const int32_t *ids, const DevCounters *ctr, int L) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ctr->nids[L]) return;
    const int B = ids[(int64_t)L * m.cap + i];
    for (int p = 1; p < Dd::NB; p++) {
        const int32_t n = m.nbr[(int64_t)p * m.cap + B];
        m.nbrc[(int64_t)p * m.cap + B] = n >= 0 ? m.nbrc[n] : n;
    }
}

// ... and links of the children of level L from their parent's
// neighbour-children (Alg. 2 in closed form): for child c and direction p,
// t = c + p in {-1..2}^d, parent region q = floor(t/2), child index t mod 2
template <typename Dd>
__global__ void k_child_links(DevMesh m, const int32_t *ids, const DevCounters *ctr, int L) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    const int i = e / Dd::NC, c = e - i * Dd::NC;
    if (i >= ctr->nids[L]) return;
    const int P = ids[(int64_t)L * m.cap + i];
    if (!is_refined(m.status[P])) return;
    const int ch = m.nbrc[P] + c;
    const int cv[3] = {c & 1, (c >> 1) & 1, (c >> 2) & 1};
    int32_t pn[27];
    for (int p = 0; p < Dd::NB; p++) pn[p] = m.nbrc[(int64_t)p * m.cap + P];
    for (int p = 0; p < Dd::NB; p++) {
        const int v[3] = {Dd::cx(p), Dd::cy(p), Dd::cz(p)};
        int qv[3] = {0, 0, 0}, cc[3] = {0, 0, 0};
        for (int a = 0; a < Dd::D; a++) {
            const int t = cv[a] + v[a];
            qv[a] = t < 0 ? -1 : t / 2;
            cc[a] = t - 2 * qv[a];
        }
        // direction index of the parent region
        int qd = 0;
        for (int r = 0; r < Dd::NB; r++)
            if (Dd::cx(r) == qv[0] && Dd::cy(r) == qv[1] && Dd::cz(r) == qv[2]) qd = r;
        const int32_t X = pn[qd];
        int32_t link;
        if (X >= 0) link = X + cc[0] + 2 * cc[1] + 4 * cc[2];
        else if (X == kNone || X == kNSkip) link = kNSkip;
        else link = X;
        m.nbr[(int64_t)p * m.cap + ch] = link;
    }
}

RootParams root_params(const Ctx &c) {
    RootParams rp;
    rp.dim = c.dim;
    rp.nroot = c.nroot;
    rp.lmax = c.m.lmax;
    for (int a = 0; a < 3; a++) {
        rp.root[a] = c.root[a];
        rp.periodic[a] = c.periodic[a];
    }
    for (int f = 0; f < 6; f++) rp.prio[f] = c.face_prio[f];
    return rp;
}

// halo records: one per active block with an N_SKIP link, numbered in block-ID
// order; the numbers before go to `old`
struct HaloJob : BlockJob {
    int32_t *old;
    __device__ int bin(const DevMesh &m, const DevCounters *, int64_t B) const {
        return m.status[B] != ST_INACTIVE && (m.bflag[B] & BF_NSKIP) ? 0 : -1;
    }
    __device__ void put(const DevMesh &m, DevCounters *, int64_t B, int b, int r, const int32_t *) const {
        old[B] = m.hid[B];
        m.hid[B] = b == 0 ? r : -1;
    }
};

// leaf blocks with a link into a solid block, per level in ID order (the
// blocks whose momentum exchange is summed after each sweep)
struct SolidJob : BlockJob {
    int32_t *list;
    __device__ int bin(const DevMesh &m, const DevCounters *, int64_t B) const {
        return m.status[B] == ST_UNREF && (m.bflag[B] & BF_SOLID) ? m.level[B] : -1;
    }
    __device__ void put(const DevMesh &m, DevCounters *, int64_t B, int b, int r, const int32_t *) const {
        if (b >= 0) list[(int64_t)b * m.cap + r] = (int32_t)B;
    }
    __device__ void done(const DevMesh &, DevCounters *ctr, const int32_t *tot) const {
        for (int L = 0; L < kMaxLevels; L++) ctr->nsolid[L] = L < K ? tot[L] : 0;
    }
};

// output cells of each block: the list of the blocks that have any and their
// exclusive offsets; with them a field read needs no pass over the mesh
__device__ __forceinline__ int output_cells(const DevMesh &m, int64_t B, int mb) {
    const uint64_t full = mb == 64 ? ~0ull : ((1ull << mb) - 1);
    return m.status[B] == ST_UNREF ? (int)__popcll(~m.gmask[B] & full) : 0;
}

struct OutListJob : BlockJob {
    int32_t *list;
    int mb;
    __device__ int bin(const DevMesh &m, const DevCounters *, int64_t B) const { return output_cells(m, B, mb) > 0 ? 0 : -1; }
    __device__ void put(const DevMesh &, DevCounters *, int64_t B, int b, int r, const int32_t *) const {
        if (b == 0) list[r] = (int32_t)B;
    }
    __device__ void done(const DevMesh &, DevCounters *ctr, const int32_t *tot) const { ctr->n_outb = tot[0]; }
};

struct OutOffsetJob : BlockJob {
    static constexpr bool kSum = true;
    int32_t *off;
    int mb;
    __device__ int bin(const DevMesh &m, const DevCounters *, int64_t B) const { return output_cells(m, B, mb); }
    __device__ void put(const DevMesh &, DevCounters *, int64_t B, int, int r, const int32_t *) const { off[B] = r; }
    __device__ void done(const DevMesh &, DevCounters *ctr, const int32_t *tot) const { ctr->n_out = tot[0]; }
};

// the refined blocks of each ID set, and those of them that are interface parents
template <bool IFACE>
struct RefinedJob : LevelJob {
    const int32_t *ids;
    int32_t *list;
    __device__ int bin(const DevMesh &m, const DevCounters *ctr, int64_t e) const {
        const int L = (int)(e / m.cap), i = (int)(e - (int64_t)L * m.cap);
        if (i >= ctr->nids[L]) return -1;
        const int B = ids[e];
        return (IFACE ? (m.bflag[B] & BF_PARENT_MASK) != 0 : is_refined(m.status[B])) ? L : -1;
    }
    __device__ void put(const DevMesh &m, DevCounters *, int64_t e, int b, int r, const int32_t *) const {
        if (b >= 0) list[(int64_t)b * m.cap + r] = ids[e];
    }
    __device__ void done(const DevMesh &, DevCounters *ctr, const int32_t *tot) const {
        for (int L = 0; L < K; L++) (IFACE ? ctr->niface : ctr->nref)[L] = tot[L];
    }
};

// Launch order of level L+1 from that of level L: the children of every
// refined block, in its order (children are numbered as Morton digits).
struct OrderJob : BlockJob {
    const int32_t *order;
    int32_t *next;
    int L, nc;
    __device__ int bin(const DevMesh &m, const DevCounters *ctr, int64_t n) const {
        if (n >= ctr->nids[L]) return -1;
        const int32_t first = m.nbrc[order[n]];
        return first >= 0 && first < m.cap ? 0 : -1;
    }
    __device__ void put(const DevMesh &m, DevCounters *, int64_t n, int b, int r, const int32_t *) const {
        if (b < 0) return;
        const int32_t first = m.nbrc[order[n]];
        for (int c = 0; c < nc; c++)
            if ((int64_t)r * nc + c < m.cap) next[(int64_t)r * nc + c] = first + c;
    }
};

// sweep list of level L: its launch order without the refined blocks none of
// whose children has an N_SKIP link
struct SweepJob : BlockJob {
    const int32_t *order;
    int32_t *list;
    int L;
    __device__ int bin(const DevMesh &m, const DevCounters *ctr, int64_t n) const {
        if (n >= ctr->nids[L]) return -1;
        const int B = order[n];
        return is_refined(m.status[B]) && !(m.bflag[B] & BF_PARENT_MASK) ? -1 : 0;
    }
    __device__ void put(const DevMesh &, DevCounters *, int64_t n, int b, int r, const int32_t *) const {
        if (b == 0) list[r] = order[n];
    }
    __device__ void done(const DevMesh &, DevCounters *ctr, const int32_t *tot) const { ctr->nsweep[L] = tot[0]; }
};

// changed: the mesh was another one before, whose descriptors are still there
template <typename Dd>
void masks_and_lists(const Ctx &c, bool changed) {
    const int cap = c.m.cap, lmax = c.m.lmax;
    k_block_masks<Dd><<<grid_for(cap), 256, 0, c.stream>>>(c.m, c.ctr);
    k_parent_mask<Dd><<<grid_for(cap), 256, 0, c.stream>>>(c.m);
    run_lists(c, HaloJob{{1}, c.first}, SolidJob{{lmax}, c.solidl}, OutListJob{{1}, c.outl, c.mb}, OutOffsetJob{{1}, c.off, c.mb},
              RefinedJob<true>{{lmax}, c.ids, c.iface}, RefinedJob<false>{{lmax}, c.ids, c.refl});
    launch_block_desc(c, changed ? c.first : nullptr);
    for (int L = 0; L < lmax; L++) {
        const int32_t *cur = c.order + (size_t)L * cap;
        const SweepJob sweep{{1}, cur, c.sweep + (size_t)L * cap, L};
        if (L + 1 < lmax) run_lists(c, OrderJob{{1}, cur, c.order + (size_t)(L + 1) * cap, L, Dd::NC}, sweep);
        else run_lists(c, sweep);
    }
    launch_target_cells(c, changed ? c.first : nullptr);
}

template <typename Dd>
void init_mesh_t(const Ctx &c) {
    const int cap = c.m.cap;
    k_init_blocks<Dd><<<grid_for(cap), 256, 0, c.stream>>>(c.m, root_params(c), c.solid);
    if (cap > c.nroot) k_init_gap<<<grid_for(cap - c.nroot), 256, 0, c.stream>>>(c.gap, cap, c.nroot);
    run_lists(c, InitJob{{1}, c.ids, c.nroot});
    masks_and_lists<Dd>(c, false);
}

template <typename Dd>
void adapt_assign_t(const Ctx &c, int n_ref) {
    const int cap = c.m.cap;
    run_lists(c, RefineJob{{1}, c.gap, c.first, c.rlist, Dd::NC});
    k_violating<Dd><<<grid_for(cap), 256, 0, c.stream>>>(c.m, c.first, c.ctr, Dd::NC * n_ref);
    k_revert<Dd><<<grid_for(cap), 256, 0, c.stream>>>(c.m, c.ctr);
}

template <typename Dd>
void adapt_build_t(const Ctx &c, int n_ref) {
    const int cap = c.m.cap, lmax = c.m.lmax;
    // S4
    if (n_ref > 0) k_build_children<Dd><<<grid_for((int64_t)n_ref * Dd::NC), 256, 0, c.stream>>>(c.m, c.rlist, c.first, n_ref);
    // S5
    run_lists(c, CoarsenJob{{lmax}, c.gap, Dd::NC});
    run_lists(c, KeepJob{{lmax}, c.ids, c.ids_tmp});
    k_copy_kept<<<grid_for((int64_t)lmax * cap), 256, 0, c.stream>>>(c.ids_tmp, c.ids, cap, lmax, c.ctr);
    // S6
    if (n_ref > 0) run_lists(c, AppendJob{{lmax}, c.first, c.ids, Dd::NC});
    k_finalize_status<<<grid_for(cap), 256, 0, c.stream>>>(c.m, c.ctr, n_ref > 0 ? Dd::NC : 0);
    k_branch_leaf<Dd><<<grid_for(cap), 256, 0, c.stream>>>(c.m);
}

template <typename Dd>
void connectivity_t(const Ctx &c) {
    const int cap = c.m.cap;
    for (int L = 0; L < c.m.lmax; L++) {
        k_nbrc_level<Dd><<<grid_for(cap), 256, 0, c.stream>>>(c.m, c.ids, c.ctr, L);
        if (L < c.m.lmax - 1)
            k_child_links<Dd><<<grid_for((int64_t)cap * Dd::NC), 256, 0, c.stream>>>(c.m, c.ids, c.ctr, L);
    }
    masks_and_lists<Dd>(c, true);
}

template <typename Dd>
void tag_vorticity_t(const Ctx &c, double theta, const LadderParams *ladder) {
    const int cap = c.m.cap;
    LadderParams lad{};
    if (ladder) lad = *ladder;
    k_tag_vort_leaf<<<grid_for(cap), 256, 0, c.stream>>>(c.m, c.crit, c.ctr, theta, ladder ? 1 : 0, lad);
    k_tag_vort_parent<Dd><<<grid_for(cap), 256, 0, c.stream>>>(c.m);
}

}  // namespace

#define AMR_DIM_DISPATCH(dim, CALL) \
    do {                            \
        if ((dim) == 2) { using Dd = D2; CALL; } else { using Dd = D3; CALL; } \
    } while (0)

void launch_init_mesh(const Ctx &c) { AMR_DIM_DISPATCH(c.dim, init_mesh_t<Dd>(c)); }

void launch_crit_reset(const Ctx &c) {
    k_crit_reset<<<grid_for(c.m.cap), 256, 0, c.stream>>>(c.crit, c.m.cap, c.ctr);
}

void launch_tag_vorticity(const Ctx &c, double theta, const LadderParams *ladder) {
    AMR_DIM_DISPATCH(c.dim, tag_vorticity_t<Dd>(c, theta, ladder));
}

void launch_tag_distance(const Ctx &c, double d_spec, int freeze) {
    DistParams dp;
    dp.dim = c.dim;
    dp.lmax = c.m.lmax;
    dp.n_solid = c.n_solid;
    const int W0 = 4 << (c.m.lmax - 1);
    for (int a = 0; a < 3; a++) dp.dom[a] = c.root[a] * W0;
    for (int f = 0; f < 6; f++) dp.face_kind[f] = c.periodic[f / 2] ? -1 : c.face_kind[f];
    dp.dspec_f = d_spec * (double)(1 << (c.m.lmax - 1));
    dp.freeze = freeze;
    k_tag_distance<<<grid_for(c.m.cap), 256, 0, c.stream>>>(c.m, c.solid_list, dp);
}

__global__ void k_zero_counts(DevCounters *ctr) {
    if (threadIdx.x == 0 && blockIdx.x == 0) ctr->n_ref = ctr->n_coa = ctr->n_rev = 0;
}

void launch_effective_tags(const Ctx &c) {
    k_zero_counts<<<1, 64, 0, c.stream>>>(c.ctr);
    k_effective_tags<<<grid_for(c.m.cap), 256, 0, c.stream>>>(c.m, c.ctr);
}

void launch_adapt_assign(const Ctx &c, int n_ref) { AMR_DIM_DISPATCH(c.dim, adapt_assign_t<Dd>(c, n_ref)); }

void launch_adapt_build(const Ctx &c, int n_ref) { AMR_DIM_DISPATCH(c.dim, adapt_build_t<Dd>(c, n_ref)); }

void launch_connectivity(const Ctx &c, int) { AMR_DIM_DISPATCH(c.dim, connectivity_t<Dd>(c)); }

}  // namespace amr
