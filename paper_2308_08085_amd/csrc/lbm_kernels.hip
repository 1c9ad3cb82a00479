// lbm_kernels.hip -- lattice Boltzmann kernels of the AMR-LBM library for
// gfx950: fused BGK collide + stream per level sweep, coarse-to-fine linear
// interpolation, fine-to-coarse averaging, the vorticity criterion and field
// gathers.  Arithmetic is written in the shifted variables g = f - w for every
// storage format (FP64 storage computes in FP64, the rest in FP32).
//
// Distributions are stored source-indexed in block-major rows (see common.h):
// every kernel finds population p of a cell with entry_slot().
#include <algorithm>
#include <mutex>
#include <utility>

#include "kernels.h"

namespace amr {

template <typename Lt>
__device__ __forceinline__ int64_t mslot(int B, int p, int l) {
    return ((int64_t)B * Lt::Q + p) * Lt::MB + l;
}

template <typename Lt>
__device__ __forceinline__ int dir_region(int p) {
    return offset_slot(Lt::cx(p), Lt::cy(p), Lt::cz(p)) - (Lt::D == 2 ? 9 : 0);
}

// slot holding population p of cell l of block B (h = its halo record); link
// is the block's link table in region-slot order
template <typename Lt>
__device__ __forceinline__ int64_t entry_slot(const DevMesh &m, const int32_t *link, int B, int h, int p, int l) {
    const int sx = (l & 3) - Lt::cx(p), sy = ((l >> 2) & 3) - Lt::cy(p), sz = (l >> 4) - Lt::cz(p);
    const int32_t code = link[region_of<Lt>(sx, sy, sz)];
    if (code >= 0 && code < m.cap) return mslot<Lt>(code, p, (sx & 3) + 4 * (sy & 3) + 16 * (sz & 3));
    if (code == kNSkip && h >= 0) return m.halo_base + (int64_t)h * m.nh + kHalo<Lt>.idx[p][l];
    return mslot<Lt>(B, Lt::opp(p), l);
}

template <typename Lt, typename R>
__device__ inline void moments_g(const R *g, R &drho, R &ux, R &uy, R &uz) {
    R d = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
    for (int p = 0; p < Lt::Q; p++) {
        d += g[p];
        if (Lt::cx(p) > 0) jx += g[p]; else if (Lt::cx(p) < 0) jx -= g[p];
        if (Lt::cy(p) > 0) jy += g[p]; else if (Lt::cy(p) < 0) jy -= g[p];
        if (Lt::cz(p) > 0) jz += g[p]; else if (Lt::cz(p) < 0) jz -= g[p];
    }
    const R rho = R(1) + d;
    drho = d;
    ux = jx / rho;
    uy = jy / rho;
    uz = jz / rho;
}

// a b + c, rounded once
__device__ __forceinline__ float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }

// deviation of the second-order equilibrium from the rest state over the
// weight: (rho - 1) + rho (3 c.u + 4.5 (c.u)^2 - 1.5 u.u), so g_eq = w y.
// Callers fuse the weight into the difference with g (one rounding fewer).
template <typename Lt, typename R>
__device__ inline R geq_y(int p, R drho, R ux, R uy, R uz, R uu) {
    const R cu = R(Lt::cx(p)) * ux + R(Lt::cy(p)) * uy + R(Lt::cz(p)) * uz;
    const R rho = R(1) + drho;
    return drho + rho * (R(3) * cu + R(4.5) * cu * cu - R(1.5) * uu);
}

// g_eq + r (g - g_eq): the non-equilibrium part rescaled by r
template <typename Lt, typename R>
__device__ __forceinline__ R rescale_neq(int p, R g, R r, R drho, R ux, R uy, R uz, R uu) {
    const R w = R(Lt::w(p)), y = geq_y<Lt, R>(p, drho, ux, uy, uz, uu);
    return fmadd(w, y, r * fmadd(-w, y, g));
}

// RAW: the stored value itself, also for unshifted storage
template <typename Lt, typename ST, bool RAW = false>
__device__ __forceinline__ typename ST::R load_g(const typename ST::T *f, int64_t slot, int p) {
    using R = typename ST::R;
    const R v = ST::ld(f + slot);
    return (ST::shift || RAW) ? v : v - R(Lt::w(p));
}

template <typename Lt, typename ST, bool NT = false>
__device__ __forceinline__ void store_g(typename ST::T *f, int64_t slot, int p, typename ST::R g) {
    using R = typename ST::R;
    if constexpr (NT)
        ST::stnt(f + slot, ST::shift ? g : g + R(Lt::w(p)));
    else
        ST::st(f + slot, ST::shift ? g : g + R(Lt::w(p)));
}

// gather / scatter all populations of one cell
template <typename Lt, typename ST, bool RAW = false>
__device__ __forceinline__ void gather_cell(const DevMesh &m, const int32_t *link, int B, int h, int l,
                                            const typename ST::T *f, typename ST::R *g) {
#pragma unroll
    for (int p = 0; p < Lt::Q; p++) g[p] = load_g<Lt, ST, RAW>(f, entry_slot<Lt>(m, link, B, h, p, l), p);
}

// Gather of an interior 3-D block (every region link a same-level block; one
// block per wave) through a per-wave LDS table of its 27 region rows.
//
// Population p of cell (i, j, k) comes from cell s = (i, j, k) - c_p, which
// lies in region r = floor(s / 4) (per axis -1, 0 or +1) at local cell s - 4 r.
// Its address is row(r) + p Mb + (s - 4 r) . (1, 4, 16), i.e.
//     tab[r] + own + (p Mb - c_p . (1, 4, 16))   (in elements)
// with tab[r] = row(r) - 4 r . (1, 4, 16) stored per region, own = the
// lane's cell index, and the last term a constant of p.  The region offset
// along x is -1 only for c_x = +1 on the face i = 0 and +1 only for c_x = -1 on
// i = 3, so each lane keeps one table offset per axis and sign of c.  Per
// population that is one three-way add for the table entry, one LDS read and
// one 64-bit add, with no selects and no 64-bit multiplies.
struct InteriorLane {
    uint32_t xm, x0, xp;  // LDS byte address of tab[13 + r_x] for c_x = -1 / 0 / +1
    uint32_t ym, yp;      // byte offset of the y part of the region for c_y = -1 / +1
    uint32_t zm, zp;      // the same along z
    uint32_t own;         // byte offset of the lane's own cell in a row
};

template <typename T, typename Lt = D3>
__device__ __forceinline__ InteriorLane interior_lane(const uint64_t *tab, int i, int j, int k) {
    InteriorLane u;
    // LDS byte offset of the table's centre entry (the pointer cast to the local address space)
    const uint32_t t = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint64_t *)tab +
                       (uint32_t)kCenterSlot<Lt> * 8u;
    u.x0 = t;
    u.xm = t + (i == 3 ? 8u : 0u);
    u.xp = t - (i == 0 ? 8u : 0u);
    u.ym = j == 3 ? 24u : 0u;
    u.yp = j == 0 ? uint32_t(-24) : 0u;
    u.zm = k == 3 ? 72u : 0u;
    u.zp = k == 0 ? uint32_t(-72) : 0u;
    u.own = (uint32_t)(i + 4 * j + 16 * k) * (uint32_t)sizeof(T);
    return u;
}

// f(std::integral_constant<int, 0>()) .. f(<N - 1>): an unrolled loop whose
// index is a constant expression
template <typename F, int... P>
__device__ __forceinline__ void static_for_seq(F &&f, std::integer_sequence<int, P...>) {
    (f(std::integral_constant<int, P>()), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_seq(f, std::make_integer_sequence<int, N>());
}

// row-table entry of the region that population P of the lane's cell streams
// from (for opp(P): the region that its population P leaves to)
template <typename Lt, int P>
__device__ __forceinline__ uint64_t row_entry(const InteriorLane &u) {
    constexpr int cx = Lt::cx(P), cy = Lt::cy(P), cz = Lt::cz(P);
    const uint32_t ex = cx < 0 ? u.xm : (cx > 0 ? u.xp : u.x0);
    const uint32_t ey = cy < 0 ? u.ym : (cy > 0 ? u.yp : 0u);
    const uint32_t ez = cz < 0 ? u.zm : (cz > 0 ? u.zp : 0u);
    return *(const __attribute__((address_space(3))) uint64_t *)(uintptr_t)(ex + ey + ez);
}

// that region's slot
template <typename Lt, int P>
__device__ __forceinline__ int region_slot(const InteriorLane &u) {
    constexpr int cx = Lt::cx(P), cy = Lt::cy(P), cz = Lt::cz(P);
    const uint32_t ex = cx < 0 ? u.xm : (cx > 0 ? u.xp : u.x0);
    const uint32_t ey = cy < 0 ? u.ym : (cy > 0 ? u.yp : 0u);
    const uint32_t ez = cz < 0 ? u.zm : (cz > 0 ? u.zp : 0u);
    return (int)(ex + ey + ez - u.x0) / 8 + kCenterSlot<Lt>;
}

// byte offset of population P from a row-table entry plus the lane's own offset
template <typename Lt, typename T, int P>
constexpr int64_t row_offset() {
    return ((int64_t)P * Lt::MB - (Lt::cx(P) + 4 * Lt::cy(P) + 16 * Lt::cz(P))) * (int64_t)sizeof(T);
}

// a global-memory pointer, so that a load is a global (not flat) load and does
// not hold up the waits on the LDS table reads
template <typename T>
__device__ __forceinline__ T *global_ptr(uint64_t a) {
    return (T *)(__attribute__((address_space(1))) T *)a;
}

// out[p] = conv(stored value of population p, p) for every population
template <typename Lt, typename ST, typename Out, typename Conv>
__device__ __forceinline__ void gather_interior_by(const InteriorLane &u, Out *out, Conv conv) {
    using T = typename ST::T;
    static_for<Lt::Q>([&](auto pc) {
        constexpr int P = decltype(pc)::value;
        const uint64_t row = row_entry<Lt, P>(u);
        out[P] = conv(ST::ld(global_ptr<const T>(row + u.own + row_offset<Lt, T, P>())), P);
    });
}

// the shifted populations g (as load_g; RAW: the stored values)
template <typename Lt, typename ST, bool RAW = false>
__device__ __forceinline__ void gather_interior(const InteriorLane &u, typename ST::R *g) {
    using R = typename ST::R;
    gather_interior_by<Lt, ST>(u, g, [](R v, int p) { return (ST::shift || RAW) ? v : v - R(Lt::w(p)); });
}

// ---------------------------------------------------------------------------
// A block's descriptor and row table, handled by the lanes of the block alone:
// a wave in 3-D, 16 lanes in 2-D.  Nothing is shared between waves, so no wave
// waits for another: list entry, descriptor, populations are the only
// dependent loads.  With the links staged from the 27 link arrays by the whole
// workgroup (three barriers, one cache line per link and block) and a branch
// per population for blocks with walls or coarser neighbours, a D3Q27 sweep of
// the cylinder (4.2e5 blocks) took 1,360 us with FP32 and 871 us with FP16
// storage, now 1,297 and 744 us (1,250 and 739 with the wave limit of
// collide_waves); a D3Q19 FP32 sweep of 16,384 blocks 33.0,
// now 30.2 us; a D2Q9 FP64 sweep of 64 blocks 7.2, now 5.3 us; a coarse step of
// 32 mixed cavities in a batch 870, now 700 us.  An entry whose link is not a
// block holds the link code, sign extended, so it is negative as an int64.
template <typename Lt> constexpr int kTab = Desc<Lt::D>::kWords;  // table entries per block

// orders the LDS writes of a wave before its later LDS reads
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// word `lane` of the descriptor of block B (0 past its end; B < 0: zeros)
template <typename Lt>
__device__ __forceinline__ int32_t desc_word(const int32_t *__restrict__ desc, int B, int lane) {
    constexpr int NW = Desc<Lt::D>::kWords;
    return lane < NW && B >= 0 ? desc[(int64_t)B * NW + lane] : 0;
}

// word k of the descriptor whose words the block's lanes hold
template <typename Lt>
__device__ __forceinline__ int32_t desc_get(int32_t w, int k) {
    if constexpr (Lt::D == 3) return __builtin_amdgcn_readlane(w, k);
    else return __shfl(w, k, 16);
}

// the row table of a block from its descriptor words (`base`: a distribution buffer)
template <typename Lt, typename T>
__device__ __forceinline__ void put_rows(uint64_t *tab, int32_t w, int lane, const T *base) {
    if (lane < Desc<Lt::D>::kLinks) {
        const int rx = lane % 3 - 1, ry = (lane / 3) % 3 - 1, rz = Lt::D == 3 ? lane / 9 - 1 : 0;
        const int64_t el = (int64_t)w * (Lt::Q * Lt::MB) - 4 * (rx + 4 * ry + 16 * rz);
        tab[lane] = w >= 0 ? (uint64_t)(uintptr_t)base + (uint64_t)(el * (int64_t)sizeof(T)) : (uint64_t)(int64_t)w;
    }
}

// The regions whose links are walls (domain faces, solid blocks) and coarser
// neighbours, as bits in region-slot order: of a wave's block, or of any of the
// four blocks of a 2-D wave.  They are the same for the whole wave, so a
// direction none of whose regions is among them costs one scalar test.
struct LinkMask {
    uint32_t wall, skip;
};

// from the descriptor words of the wave's blocks (lane: of the block)
template <typename Lt>
__device__ __forceinline__ LinkMask wave_links(int32_t w, int lane) {
    const bool link = lane < Desc<Lt::D>::kLinks;
    uint64_t wall = __ballot(link && w < 0 && w != kNSkip), skip = __ballot(link && w == kNSkip);
    if constexpr (Lt::D == 2) {
        wall |= wall >> 32;
        wall = (wall | wall >> 16) & 0x1ff;
        skip |= skip >> 32;
        skip = (skip | skip >> 16) & 0x1ff;
    }
    return {(uint32_t)wall, (uint32_t)skip};
}

// regions outside the block that population P of some cell streams from
template <typename Lt, int P>
constexpr uint32_t source_regions() {
    uint32_t m = 0;
    for (int k = 1; k < 8; k++) {
        const int rx = k & 1 ? -Lt::cx(P) : 0, ry = k & 2 ? -Lt::cy(P) : 0, rz = k & 4 ? -Lt::cz(P) : 0;
        if (rx || ry || rz) m |= 1u << (offset_slot(rx, ry, rz) - (Lt::D == 2 ? 9 : 0));
    }
    return m;
}

// Addresses of the populations of one cell of a block with any links.
template <typename T>
struct CellRows {
    InteriorLane u;
    LinkMask any;    // over the wave
    uint64_t own;    // the cell's own slot of population 0
    uint64_t halo;   // the block's halo record
    uint64_t below;  // bits of the cells below the lane's cell
};

template <typename Lt, typename T>
__device__ __forceinline__ CellRows<T> cell_rows(const uint64_t *tab, LinkMask any, int B, int h, int l,
                                                 const T *base, const DevMesh &m) {
    CellRows<T> r;
    r.any = any;
    r.u = interior_lane<T, Lt>(tab, l & 3, (l >> 2) & 3, l >> 4);
    r.own = (uint64_t)(uintptr_t)(base + (int64_t)B * (Lt::Q * Lt::MB)) + r.u.own;
    r.halo = (uint64_t)(uintptr_t)(base + (m.halo_base + (int64_t)h * m.nh));
    r.below = (uint64_t(1) << l) - 1;
    return r;
}

// entry of population P of a cell in the block's halo record
template <typename Lt, int P>
__device__ __forceinline__ uint32_t halo_entry(uint64_t below) {
    constexpr uint64_t out = kHaloMask<Lt>.out[P];
    uint32_t n = kHaloMask<Lt>.base[P] + __popc((uint32_t)out & (uint32_t)below);
    if constexpr (Lt::MB == 64) n += __popc((uint32_t)(out >> 32) & (uint32_t)(below >> 32));
    return n;
}

// address of population P: its source's slot on the same level, the halo
// record (HALO: some source lies under a coarser neighbour), or the cell's own
// opposite slot
template <typename Lt, typename T, int P, bool HALO>
__device__ __forceinline__ uint64_t slot_address(const CellRows<T> &r) {
    if constexpr (P == 0) {
        return r.own;
    } else {
        const uint64_t e = row_entry<Lt, P>(r.u);
        uint64_t a = e + r.u.own + row_offset<Lt, T, P>();
        a = (int64_t)e >= 0 ? a : r.own + (uint64_t)Lt::opp(P) * (Lt::MB * sizeof(T));
        if constexpr (HALO) {
            const uint64_t ha = r.halo + halo_entry<Lt, P>(r.below) * (uint32_t)sizeof(T);
            a = e == (uint64_t)(int64_t)kNSkip ? ha : a;
        }
        return a;
    }
}

// The same for a population known only at run time (uniform over the wave).
template <typename Lt>
struct DirTable {
    int32_t c[Lt::Q][3], opp[Lt::Q];
    constexpr DirTable() : c(), opp() {
        for (int p = 0; p < Lt::Q; p++) {
            c[p][0] = Lt::cx(p);
            c[p][1] = Lt::cy(p);
            c[p][2] = Lt::cz(p);
            opp[p] = Lt::opp(p);
        }
    }
};
template <typename Lt> constexpr DirTable<Lt> kDir{};

template <typename Lt, typename T>
__device__ __forceinline__ uint64_t slot_address_any(const CellRows<T> &r, const uint64_t *tab, int l, int p) {
    const int cx = kDir<Lt>.c[p][0], cy = kDir<Lt>.c[p][1], cz = kDir<Lt>.c[p][2];
    const uint64_t e = tab[region_of<Lt>((l & 3) - cx, ((l >> 2) & 3) - cy, (l >> 4) - cz)];
    if ((int64_t)e >= 0) return e + r.u.own + (int64_t)(p * Lt::MB - (cx + 4 * cy + 16 * cz)) * (int64_t)sizeof(T);
    if (e != (uint64_t)(int64_t)kNSkip) return r.own + (uint32_t)(kDir<Lt>.opp[p] * Lt::MB) * (uint32_t)sizeof(T);
    return r.halo + (uint32_t)(kHaloMask<Lt>.base[p] + __popcll(kHaloMask<Lt>.out[p] & r.below)) * (uint32_t)sizeof(T);
}

// gather of a cell of a block with any links: every population's address by
// selects, so all loads are in flight together
template <typename Lt, typename ST, bool HALO, typename Out, typename Conv>
__device__ __forceinline__ void gather_rows_by_(const CellRows<typename ST::T> &r, Out *out, Conv conv) {
    using T = typename ST::T;
    static_for<Lt::Q>([&](auto pc) {
        constexpr int P = decltype(pc)::value;
        out[P] = conv(ST::ld(global_ptr<const T>(slot_address<Lt, T, P, HALO>(r))), P);
    });
}

template <typename Lt, typename ST, typename Out, typename Conv>
__device__ __forceinline__ void gather_rows_by(const CellRows<typename ST::T> &r, Out *out, Conv conv) {
    if (r.any.skip) gather_rows_by_<Lt, ST, true>(r, out, conv);
    else gather_rows_by_<Lt, ST, false>(r, out, conv);
}

// The shifted populations of a cell (RAW: the stored values); `r` from cell_rows.
template <typename Lt, typename ST, bool RAW = false>
__device__ __forceinline__ void gather_rows(const CellRows<typename ST::T> &r, typename ST::R *g) {
    using R = typename ST::R;
    if (!(r.any.wall | r.any.skip))
        gather_interior<Lt, ST, RAW>(r.u, g);
    else
        gather_rows_by<Lt, ST>(r, g, [](R v, int p) { return (ST::shift || RAW) ? v : v - R(Lt::w(p)); });
}

// BGK relaxation of one cell in the shifted variables: moments, then
// g <- g + omega (g_eq - g).  (A form with 1/rho taken once and the
// equilibrium grouped by weight saved no time here, and the reciprocal's
// rounding moved FP32 runs measurably further from FP64.)
template <typename Lt, typename R>
__device__ __forceinline__ void bgk_relax(R *g, R om, R &drho, R &ux, R &uy, R &uz, R &uu) {
    moments_g<Lt, R>(g, drho, ux, uy, uz);
    uu = ux * ux + uy * uy + uz * uz;
#pragma unroll
    for (int p = 0; p < Lt::Q; p++)
        g[p] = fmadd(om, fmadd(R(Lt::w(p)), geq_y<Lt, R>(p, drho, ux, uy, uz, uu), -g[p]), g[p]);
}

// ---------------------------------------------------------------------------
// Moment-space (multiple-relaxation-time) collision for D3Q27, optional: the
// paper's method is BGK and it names moment-space operators only as the
// alternative (Sec. "Lattice Boltzmann Method").  Moment k = a + 3 b + 9 c is
// sum_p phi_a(c_x) phi_b(c_y) phi_c(c_z) f_p with phi_0 = 1, phi_1 = c,
// phi_2 = 3 c^2 - 1; the rows are orthogonal under the lattice weights with
// norms N_k = n_a n_b n_c (n = 1, 1/3, 2), so M^-1 = diag(w) M^T diag(1/N).
// Moments of order <= 2 relax at omega, the 17 others at s_high.  With the
// non-equilibrium part n = g - g_eq this is BGK plus a correction in the high
// moments only:
//     g* = g - omega n - w_p sum_{k high} M_kp ((s_high - omega) / N_k) (M n)_k
// so s_high = omega gives the BGK arithmetic exactly.
struct Mrt27 {
    static constexpr int NH = 17;
    int hk[NH];  // the moments of order > 2, ascending
    static constexpr int order(int k) { return k % 3 + k / 3 % 3 + k / 9; }
    static constexpr int phi(int a, int c) { return a == 0 ? 1 : (a == 1 ? c : 3 * c * c - 1); }
    static constexpr int m(int k, int p) { return phi(k % 3, D3::cx(p)) * phi(k / 3 % 3, D3::cy(p)) * phi(k / 9, D3::cz(p)); }
    static constexpr double norm(int k) {
        return (k % 3 == 0 ? 1.0 : (k % 3 == 1 ? 1.0 / 3.0 : 2.0)) *
               (k / 3 % 3 == 0 ? 1.0 : (k / 3 % 3 == 1 ? 1.0 / 3.0 : 2.0)) *
               (k / 9 == 0 ? 1.0 : (k / 9 == 1 ? 1.0 / 3.0 : 2.0));
    }
    constexpr Mrt27() : hk() {
        int n = 0;
        for (int k = 0; k < 27; k++)
            if (order(k) > 2) hk[n++] = k;
    }
};
constexpr Mrt27 kMrt27{};

// g -= w_p sum_k M_kp fac h_k / N_k with h = M n over the high moments, on the
// vector ALU (every coefficient a compile-time constant)
template <typename R, int S = 0>
__device__ __forceinline__ void mrt27_high(const R *n, R fac, R *g) {
    if constexpr (S < Mrt27::NH) {
        constexpr int k = kMrt27.hk[S];
        R h = R(0);
#pragma unroll
        for (int p = 0; p < 27; p++)
            if constexpr (true) {
                const int c = Mrt27::m(k, p);
                if (c == 1) h += n[p];
                else if (c == -1) h -= n[p];
                else if (c != 0) h += R(c) * n[p];
            }
        h *= fac * R(1.0 / Mrt27::norm(k));
#pragma unroll
        for (int p = 0; p < 27; p++) {
            const int c = Mrt27::m(k, p);
            if (c != 0) g[p] -= R(Lat<27>::w(p) * c) * h;
        }
        mrt27_high<R, S + 1>(n, fac, g);
    }
}

// The same correction with both transforms on the matrix cores
// (v_mfma_f32_16x16x32_f16; FP16 operands, FP32 accumulation).  One wave, 64
// cells = four tiles of 16.  Lane layout of the instruction: A[i][k] at lane l
// for i = l % 16, k = 8 (l / 16) + e (e = 0..7); B[k][j] for j = l % 16, the same
// k; D[i][j] in register r of lane l for i = 4 (l / 16) + r, j = l % 16.
//   forward:  H = M_high N   (rows: 32 slots, the 17 high moments first;
//                             K: the 27 populations; columns: cells)
//   scale:    slot s by (s_high - omega) / N_k, to FP16
//   back:     C = M_high^T H' (rows: populations; K in the order in which each
//             lane already holds the forward result: k = 8 g + e is slot
//             4 g + e for e < 4 and 16 + 4 g + e - 4 otherwise, g = l / 16)
// N is scaled by 2^8 before rounding to FP16 (non-equilibrium parts are small)
// and C by 2^-8 after.  The cell-major transposes go through LDS.
typedef _Float16 mf_h8 __attribute__((ext_vector_type(8)));
typedef float mf_f4 __attribute__((ext_vector_type(4)));

struct MrtMfmaOps {
    _Float16 af[2][64][8];  // forward A, row blocks 0 / 1, per lane
    _Float16 ab[2][64][8];  // back A, population blocks 0 / 1, per lane
    float invn[32];         // 1 / N of the slot's moment; 0 past the 17
    static constexpr int slot_of_back_k(int k) { return (k % 8) < 4 ? 4 * (k / 8) + k % 8 : 16 + 4 * (k / 8) + k % 8 - 4; }
    constexpr MrtMfmaOps() : af(), ab(), invn() {
        for (int s = 0; s < 32; s++) invn[s] = s < Mrt27::NH ? float(1.0 / Mrt27::norm(kMrt27.hk[s])) : 0.0f;
        for (int b = 0; b < 2; b++)
            for (int l = 0; l < 64; l++)
                for (int e = 0; e < 8; e++) {
                    const int i = l % 16, k = 8 * (l / 16) + e;
                    const int sf = 16 * b + i;  // forward: row = slot, K = population
                    af[b][l][e] = (_Float16)((sf < Mrt27::NH && k < 27) ? Mrt27::m(kMrt27.hk[sf], k) : 0);
                    const int p = 16 * b + i, sb = slot_of_back_k(k);  // back: row = population
                    ab[b][l][e] = (_Float16)((sb < Mrt27::NH && p < 27) ? Mrt27::m(kMrt27.hk[sb], p) : 0);
                }
    }
};
constexpr MrtMfmaOps kMrtMfma{};

__device__ __forceinline__ void mrt27_high_mfma(const float *n, float fac, float *g) {
    constexpr float kScale = 256.0f;
    // per wave: 64 cells x 36 words (FP16 rows of 32 for the forward pass, FP32 rows of 32 for the back pass)
    __shared__ __attribute__((aligned(16))) float buf[4][64 * 36];
    const int l = threadIdx.x & 63, grp = l >> 4, col = l & 15;
    float *wb = buf[threadIdx.x >> 6];
    _Float16 *hb = (_Float16 *)wb;
    // cell-major FP16 rows of the scaled non-equilibrium parts: [cell][32]
#pragma unroll
    for (int c = 0; c < 4; c++) {
        mf_h8 v;
#pragma unroll
        for (int e = 0; e < 8; e++) v[e] = (_Float16)(8 * c + e < 27 ? n[8 * c + e] * kScale : 0.0f);
        *(mf_h8 *)(hb + l * 72 + 8 * c) = v;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    mf_h8 af0, af1, ab0, ab1;
#pragma unroll
    for (int e = 0; e < 8; e++) {
        af0[e] = kMrtMfma.af[0][l][e];
        af1[e] = kMrtMfma.af[1][l][e];
        ab0[e] = kMrtMfma.ab[0][l][e];
        ab1[e] = kMrtMfma.ab[1][l][e];
    }
    float fs[8];
#pragma unroll
    for (int e = 0; e < 8; e++) fs[e] = fac * kMrtMfma.invn[e < 4 ? 4 * grp + e : 16 + 4 * grp + e - 4];
    const mf_f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    mf_h8 bb[4];
#pragma unroll
    for (int t = 0; t < 4; t++) {
        const mf_h8 b = *(const mf_h8 *)(hb + (16 * t + col) * 72 + 8 * grp);
        const mf_f4 d0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(af0, b, zero, 0, 0, 0);
        const mf_f4 d1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(af1, b, zero, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 8; e++) bb[t][e] = (_Float16)((e < 4 ? d0[e] : d1[e - 4]) * fs[e]);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int t = 0; t < 4; t++) {
        const mf_f4 c0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(ab0, bb[t], zero, 0, 0, 0);
        const mf_f4 c1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(ab1, bb[t], zero, 0, 0, 0);
        // populations 4 grp + r and 16 + 4 grp + r of cell 16 t + col
        *(mf_f4 *)(wb + (16 * t + col) * 36 + 4 * grp) = c0;
        *(mf_f4 *)(wb + (16 * t + col) * 36 + 16 + 4 * grp) = c1;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int p = 0; p < 27; p++) g[p] -= float(Lat<27>::w(p) / 256.0) * wb[l * 36 + p];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// Collision of one cell: COLL 0 = BGK, 1 = moment-space on the vector ALU,
// 2 = moment-space with the high-moment transforms on the matrix cores (a
// whole wave, every lane active; mrt27_high_mfma).
template <typename Lt, typename R, int COLL>
__device__ __forceinline__ void relax(R *g, R om, R sh, R &drho, R &ux, R &uy, R &uz, R &uu) {
    if constexpr (COLL == 0 || Lt::Q != 27) {
        bgk_relax<Lt, R>(g, om, drho, ux, uy, uz, uu);
    } else {
        moments_g<Lt, R>(g, drho, ux, uy, uz);
        uu = ux * ux + uy * uy + uz * uz;
        R n[27];
#pragma unroll
        for (int p = 0; p < 27; p++) {
            n[p] = fmadd(-R(Lt::w(p)), geq_y<Lt, R>(p, drho, ux, uy, uz, uu), g[p]);
            g[p] -= om * n[p];
        }
        if constexpr (COLL == 1)
            mrt27_high<R>(n, sh - om, g);
        else if constexpr (sizeof(R) == 4)
            mrt27_high_mfma(n, sh - om, g);
    }
}

// Per-workgroup staging of NBLK block descriptors; links by region slot.
// sim[] names the simulation of each entry in the batched kernels.
template <typename Lt, int NBLK>
struct BlockStage {
    static constexpr int NS = Lt::D == 2 ? 9 : 27;
    int32_t link[NBLK][NS];
    int32_t id[NBLK];
    int32_t hid[NBLK];
    int32_t sim[NBLK];
};

// st.id[] (-1 = none) must be written and synchronised before the call;
// mesh_of(s) gives the mesh of entry s
template <typename Lt, int NBLK, typename MeshOf>
__device__ void stage_blocks_by(MeshOf mesh_of, BlockStage<Lt, NBLK> &st) {
    for (int e = threadIdx.x; e < NBLK * Lt::NB; e += blockDim.x) {
        const int s = e / Lt::NB, p = e - s * Lt::NB;
        const int B = st.id[s];
        int32_t v = 0, h = -1;
        if (B >= 0) {
            const DevMesh &m = mesh_of(s);
            v = m.nbr[(int64_t)p * m.cap + B];
            if (p == 0) h = m.hid[B];
        }
        st.link[s][dir_region<Lt>(p)] = v;
        if (p == 0) st.hid[s] = h;
    }
    __syncthreads();
}

template <typename Lt, int NBLK>
__device__ void stage_blocks(const DevMesh &m, BlockStage<Lt, NBLK> &st) {
    stage_blocks_by<Lt, NBLK>([&](int) -> const DevMesh & { return m; }, st);
}

// Contiguous range of work units [u0, u1) of a persistent workgroup: the
// count is read on the device, so one launch shape serves every mesh.  With
// fewer units than workgroups only the first `units` workgroups work, which
// dispatch spreads over the XCDs, and shares differ by one unit at most.  When
// the ranges were numbered over the whole grid, the units of a small level
// went to the first XCDs only: D2Q9 sweeps of the 16 cavities of a batch 9.4,
// now 6.6 us, their interpolation 7.3 and 5.4, averaging 6.9 and 5.0; a batch
// of 32 mixed cavities, 50 coarse steps, 30.0 and 26.3 ms.
__device__ inline void persistent_range(int units, int &u0, int &u1) {
    const int G = min((int)gridDim.x, units);
    u0 = u1 = 0;
    if ((int)blockIdx.x >= G) return;
    const int wg = xcd_remap(blockIdx.x, G);
    const int per = units / G, more = units - per * G;
    u0 = wg * per + min(wg, more);
    u1 = u0 + per + (wg < more ? 1 : 0);
}

// Read-only view of the batch descriptors in the constant address space: with
// a wave-uniform index their fields come in through scalar loads.
typedef const __attribute__((address_space(4))) SimDesc CSimDesc;
__device__ inline CSimDesc *const_view(const SimDesc *p) { return (CSimDesc *)p; }

__device__ inline DevMesh load_mesh(CSimDesc *cs) {
    DevMesh m;
    m.cap = cs->m.cap;
    m.capc = cs->m.capc;
    m.lmax = cs->m.lmax;
    m.halo_base = cs->m.halo_base;
    m.nh = cs->m.nh;
    m.interp = cs->m.interp;
    m.force = cs->m.force;
    m.hid = cs->m.hid;
    m.parent = cs->m.parent;
    m.fresh = cs->m.fresh;
    m.desc = cs->m.desc;
    m.nbr = cs->m.nbr;
    m.nbrc = cs->m.nbrc;
    m.X = cs->m.X;
    m.level = cs->m.level;
    m.status = cs->m.status;
    m.tag = cs->m.tag;
    m.ldes = cs->m.ldes;
    m.viol = cs->m.viol;
    m.bflag = cs->m.bflag;
    m.gmask = cs->m.gmask;
    m.imask = cs->m.imask;
    return m;
}

// Thread index hidden from loop-invariant code motion: inside a persistent
// loop the per-cell index arithmetic is then redone per work unit instead of
// being hoisted and kept live across the loop.
__device__ __forceinline__ int opaque_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// decode a batch work item into (simulation, block)
__device__ inline void decode_item(uint32_t it, int &sim, int &B) {
    sim = (int)(it >> kItemSimShift);
    B = (int)(it & kItemBlockMask);
}

// ---------------------------------------------------------------------------
// Fused collide + stream of one level (Secs. "Streaming", "Collision").  One
// 4^d block per 64-lane group (3-D: one block per wave; 2-D: four blocks per
// wave).  Each cell gathers its populations, collides, and writes its
// outgoing populations to its own slots; an outgoing population that would
// leave the fluid is replaced there by its bounce-back.  A population arriving
// from a region covered only by a coarser block keeps the cell's own
// post-collision value (halo record).  NTS: write with non-temporal stores
// (for levels whose output is too large to stay cached until the next sweep).
// EX: a leaf block next to a solid also adds its momentum exchange of this
// sweep to its total, exactly as the separate pass (exchange_block) would from
// the values just stored.
//
// Kind and wall velocity of the domain's faces, as the lanes of a block read them.
template <typename Lt, typename R>
struct FaceTable {
    static constexpr int NF = 2 * Lt::D;
    R u[NF][3];
    int32_t kind[NF];
    // by the block's lanes: NF * D <= 18 of 64, 8 of 16
    __device__ void put(const BCParams &bc, int lane) {
        if (lane < NF * Lt::D) u[lane / Lt::D][lane % Lt::D] = R(bc.u[lane / Lt::D][lane % Lt::D]);
        if (lane < NF) {
            kind[lane] = bc.kind[lane];
            if (Lt::D == 2) u[lane][2] = R(0);
        }
    }
};

// LDS of one wave: row table and faces of each of its blocks (the blocks of a
// wave of a 2-D batch may belong to different simulations)
template <typename Lt, typename R>
struct CollideSmem {
    uint64_t tab[64 / Lt::MB][kTab<Lt>];
    FaceTable<Lt, R> face[64 / Lt::MB];
};

// Keeps a result in FP32 until it is stored: the conversion to FP16 may fuse
// with the multiply-add before it and then rounds once instead of twice.  Used
// where that must not depend on the code around it: for every population of a
// block with walls or coarser neighbours, and in 2-D for every block, since which
// path a 2-D block takes depends on the three that share its wave.
template <int S, typename R>
__device__ __forceinline__ void pin_result(R &g) {
    if constexpr (S == AMR_F16S) asm volatile("" : "+v"(g));
}

// Body: cell l of block B (B < 0: none), whole wave; `glane` = the lane's
// index among the block's lanes (= l).
template <int Q, int S, bool NTS, int COLL = 0, bool EX = false>
__device__ __forceinline__ void collide_block(const DevMesh &m, int B, int l, const typename Store<S>::T *__restrict__ src,
                                              typename Store<S>::T *__restrict__ dst, typename Store<S>::R om,
                                              const BCParams &bc, CollideSmem<Lat<Q>, typename Store<S>::R> &sm,
                                              typename Store<S>::R sh = typename Store<S>::R(0)) {
    using Lt = Lat<Q>;
    using ST = Store<S>;
    using R = typename ST::R;
    using T = typename ST::T;
    using De = Desc<Lt::D>;
    const int lane = threadIdx.x & 63;
    uint64_t *tab = sm.tab[Lt::D == 3 ? 0 : lane >> 4];
    const int32_t w = desc_word<Lt>(m.desc, B, l);
    put_rows<Lt>(tab, w, l, src);
    wave_lds_sync();
    const uint32_t flag = (uint32_t)desc_get<Lt>(w, De::kFlags);
    const int h = desc_get<Lt>(w, De::kHid);
    const LinkMask any = wave_links<Lt>(w, l);
    if (B < 0) return;

    R g[Q];
    R drho, ux, uy, uz, uu;
    // Interior blocks (every region link a same-level block; 2-D: all four of the wave)
    if (!(any.wall | any.skip)) {
        gather_interior<Lt, ST>(interior_lane<T, Lt>(tab, l & 3, (l >> 2) & 3, l >> 4), g);
        relax<Lt, R, COLL>(g, om, sh, drho, ux, uy, uz, uu);
#pragma unroll
        for (int p = 0; p < Q; p++) {
            if constexpr (Lt::D == 2) pin_result<S>(g[p]);
            store_g<Lt, ST, NTS>(dst, mslot<Lt>(B, p, l), p, g[p]);
        }
        return;
    }
    // Walls.  Most blocks meet one face or solid only: `code`, whose data then
    // sit in registers; where some block of the wave meets several, each link
    // looks its own up in LDS.  A small level is bound by this serial path of its
    // wall blocks: with a look-up per link and direction a sweep took, us, D3Q27
    // of 64 blocks FP32 10.0 (now 9.1), of 4096 blocks FP16 12.4 (11.8), D3Q19 of
    // 64 blocks 7.8 (7.1), D2Q9 of 16384 blocks FP64 8.7 (8.2).
    FaceTable<Lt, R> &face = sm.face[Lt::D == 3 ? 0 : lane >> 4];
    uint32_t wall = any.wall;  // of the block
    int code = kSolid, kind = 0;
    bool one = true;
    R wx = R(0), wy = R(0), wz = R(0);
    if (any.wall) {
        const bool is_wall = l < De::kLinks && w < 0 && w != kNSkip;
        if constexpr (Lt::D == 2) wall = (uint32_t)(__ballot(is_wall) >> (lane & 48)) & 0x1ff;
        code = desc_get<Lt>(w, wall ? __builtin_ctz(wall) : 0);
        one = !__any(is_wall && w != code);
        if (!one) face.put(bc, l);
        const int f = code >= -8 && code <= -3 ? -3 - code : 0;
        kind = bc.kind[f];
        wx = R(bc.u[f][0]);
        wy = R(bc.u[f][1]);
        if constexpr (Lt::D == 3) wz = R(bc.u[f][2]);
    }
    const CellRows<T> r = cell_rows<Lt, T>(tab, any, B, h, l, src, m);
    gather_rows_by<Lt, ST>(r, g, [](R v, int p) { return ST::shift ? v : v - R(Lt::w(p)); });
    relax<Lt, R, COLL>(g, om, sh, drho, ux, uy, uz, uu);
    wave_lds_sync();
    // index, links and velocity hidden from common subexpressions: what the
    // gather and the relaxation computed per population is not kept for the
    // stores
    int lf = l;
    asm volatile("" : "+v"(lf));
    const InteriorLane u = interior_lane<T, Lt>(tab, lf & 3, (lf >> 2) & 3, lf >> 4);
    uint32_t walls = any.wall, skips = any.skip;
    asm volatile("" : "+s"(walls), "+s"(skips));
    asm volatile("" : "+v"(ux), "+v"(uy), "+v"(uz), "+v"(uu));

    [[maybe_unused]] double fx = 0.0, fy = 0.0, fz = 0.0;
    static_for<Q>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        R val = g[q];
        if (walls & source_regions<Lt, Lt::opp(q)>()) {  // regions that population q leaves to
            bool hit;
            int c = code, kd = kind;
            R vx = wx, vy = wy, vz = wz;
            if (one) {
                hit = (wall >> region_slot<Lt, Lt::opp(q)>(u)) & 1u;
            } else {
                const int64_t e = (int64_t)row_entry<Lt, Lt::opp(q)>(u);
                hit = e < 0 && e != kNSkip;
                c = (int)e;
                if (hit && c != kSolid) {
                    const int f = -3 - c;
                    kd = face.kind[f];
                    vx = face.u[f][0];
                    vy = face.u[f][1];
                    vz = face.u[f][2];
                }
            }
            if (hit) {
                if (c == kSolid) {
                    if constexpr (EX) {
                        // 2 f*_q c_q from the value as stored (rounded to the storage type)
                        T t;
                        ST::st(&t, ST::shift ? val : val + R(Lt::w(q)));
                        const double two_f = 2.0 * double(ST::ld(&t) + (ST::shift ? Lt::w(q) : 0.0));
                        fx += two_f * Lt::cx(q);
                        fy += two_f * Lt::cy(q);
                        fz += two_f * Lt::cz(q);
                    }
                } else {
                    const R cx = R(Lt::cx(q)), cy = R(Lt::cy(q)), cz = R(Lt::cz(q));
                    if (kd == AMR_FACE_VELOCITY) {
                        const R cuw = cx * vx + cy * vy + cz * vz;
                        val = g[q] - R(6) * R(Lt::w(q)) * cuw;
                    } else {
                        const R cu = cx * ux + cy * uy + cz * uz;
                        val = -g[q] + R(2) * R(Lt::w(q)) * (R(4.5) * cu * cu - R(1.5) * uu);
                    }
                }
            }
        }
        // outside the fluid the slot now holds population opposite(q) of this cell
        pin_result<S>(val);
        store_g<Lt, ST, NTS>(dst, mslot<Lt>(B, q, l), q, val);
        __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (EX) {
        // uniform over the block's lanes: sum over the block, one lane adds
        if ((flag & BF_SOLID) && (flag & DF_LEAF)) {
#pragma unroll
            for (int mask = 1; mask < Lt::MB; mask <<= 1) {
                fx += __shfl_xor(fx, mask, 64);
                fy += __shfl_xor(fy, mask, 64);
                fz += __shfl_xor(fz, mask, 64);
            }
            if (l == 0) {
                m.force[(int64_t)B * 3 + 0] += fx;
                m.force[(int64_t)B * 3 + 1] += fy;
                m.force[(int64_t)B * 3 + 2] += fz;
            }
        }
    }
    if (skips) {
        const int64_t rec = m.halo_base + (int64_t)h * m.nh;
        static_for<Q>([&](auto pc) {
            constexpr int p = decltype(pc)::value;
            if (skips & source_regions<Lt, p>()) {
                if (row_entry<Lt, p>(u) == (uint64_t)(int64_t)kNSkip)
                    store_g<Lt, ST, NTS>(dst, rec + halo_entry<Lt, p>((uint64_t(1) << lf) - 1), p, g[p]);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    }
}

// Workgroup size: 256 threads (3-D: four blocks of the Morton launch order)
// for every storage.  Boundary and interface blocks take the slower generic
// path, and a CU can start a new workgroup only when all of its waves fit: with
// 512 threads a slow wave held back seven others (16-bit storage on the
// cylinder set-up: 968 us per launch against 915 us with 256), while 128
// threads lose the neighbour reuse between the blocks of a workgroup.
template <int S>
constexpr int collide_threads() { return 256; }

// Waves per SIMD of the large 3-D sweeps (those stored past the caches): more
// waves keep more loads in flight but also more blocks, and the rows that
// neighbouring blocks share have to stay in the XCD's 4 MB L2 until the last of
// them has read its part.  D3Q27 cylinder, us per sweep with 2, 3, 4, 5, 6, 7
// waves: FP32 1398, 1264, 1250, 1289, 1306, 1364; FP16 (half the bytes per block)
// 1140, 876, 760, 742, 739, 779.  Uniform D3Q19 FP32 level of 256^3 cells with
// 3, 4, 5, 6, 7: 531, 510, 517, 520, 526.  FP64 is left to the compiler (2256 to
// 2386 over runs; 2 to 4 waves 2298 to 2462, 4 with spills).  Smaller levels do
// not depend on it; k_collide_stream and BGK only, the joined kernel and the
// other collisions were not swept.
template <int Q, int S, bool NTS, int COLL>
constexpr int collide_waves(bool most) {
    if (!(NTS && COLL == 0 && Lat<Q>::D == 3) || S == AMR_F64) return most ? 8 : 1;  // the compiler's choice
    return sizeof(typename Store<S>::T) == 2 ? 6 : 4;
}

// blocks per workgroup of k_collide_stream (one per 64-lane group)
template <int Q, int S>
constexpr int collide_blocks_per_wg() { return collide_threads<S>() / Lat<Q>::MB; }

// COLL: 0 = BGK, 1 / 2 = moment-space collision (D3Q27) on the vector ALU /
// with the matrix-core transforms; s_high = its rate above second order
// One workgroup's share of a level sweep: blocks wg * BPW .. of the list
template <int Q, int S, bool NTS, int COLL, bool EX = false>
__device__ __forceinline__ void collide_wg(const int32_t *__restrict__ list, int n, const DevMesh &m,
                                           const typename Store<S>::T *__restrict__ src,
                                           typename Store<S>::T *__restrict__ dst, double omega_d, const BCParams &bc,
                                           double s_high, int wg) {
    using Lt = Lat<Q>;
    using R = typename Store<S>::R;
    constexpr int MB = Lt::MB, BPW = collide_blocks_per_wg<Q, S>();
    __shared__ CollideSmem<Lt, R> sm[collide_threads<S>() / 64];
    int pos = wg * BPW + (int)threadIdx.x / MB;
    if constexpr (Lt::D == 3) {
        pos = __builtin_amdgcn_readfirstlane(pos);  // one block per wave
        if (pos >= n) return;
    }
    const int B = pos < n ? list[pos] : -1;
    collide_block<Q, S, NTS, COLL, EX>(m, B, threadIdx.x % MB, src, dst, R(omega_d), bc, sm[threadIdx.x >> 6],
                                       R(s_high));
}

template <int Q, int S, bool NTS, int COLL = 0, bool EX = false>
__global__ __launch_bounds__(collide_threads<S>())
    __attribute__((amdgpu_waves_per_eu(collide_waves<Q, S, NTS, COLL>(false), collide_waves<Q, S, NTS, COLL>(true)))) void k_collide_stream(
    const int32_t *__restrict__ list, int n, DevMesh m, const typename Store<S>::T *__restrict__ src,
    typename Store<S>::T *__restrict__ dst, double omega_d, BCParams bc, double s_high) {
    collide_wg<Q, S, NTS, COLL, EX>(list, n, m, src, dst, omega_d, bc, s_high, xcd_remap(blockIdx.x, gridDim.x));
}

// Batched form: level L of every simulation of a batch in one persistent
// launch of NT-thread workgroups (NT / Mb blocks each); all simulations share
// the buffer parity `par` of level L.
template <int Q, int S, int NT>
__global__ __launch_bounds__(NT) void k_collide_stream_batch(const SimDesc *__restrict__ sims,
                                                             const uint32_t *__restrict__ items,
                                                             const int32_t *__restrict__ count, int L, int par) {
    using Lt = Lat<Q>;
    using ST = Store<S>;
    using R = typename ST::R;
    using T = typename ST::T;
    constexpr int MB = Lt::MB, BPW = NT / MB;
    __shared__ CollideSmem<Lt, R> sm[NT / 64];
    const int n = *count;
    int u0, u1;
    persistent_range((n + BPW - 1) / BPW, u0, u1);
    for (int u = u0; u < u1; u++) {
        const int tid = opaque_tid();
        int idx = u * BPW + tid / MB;
        if (MB == 64) {
            idx = __builtin_amdgcn_readfirstlane(idx);  // one block per wave
            if (idx >= n) break;
        }
        int sim = 0, B = -1;
        if (idx < n) decode_item(items[idx], sim, B);
        if (MB == 64) sim = __builtin_amdgcn_readfirstlane(sim);
        CSimDesc *cs = const_view(sims) + sim;
        const DevMesh m = load_mesh(cs);
        collide_block<Q, S, false>(m, B, tid % MB, (const T *)cs->f[par], (T *)cs->f[1 - par], R(cs->lp.omega[L]),
                                   sims[sim].bc, sm[tid >> 6]);
        wave_lds_sync();
    }
}

// ---------------------------------------------------------------------------
// Coarse-to-fine linear interpolation with Dupuis-Chopard rescaling (Sec.
// "Linear Interpolation").  One parent block per team (3-D: a 256-thread
// workgroup, 2-D: a wave): its cells are rescaled into LDS, the coefficients of
// the (bi/tri)linear polynomial through the 2^d parent cells of each quadrant
// are formed once per quadrant and population, and every targeted fine cell
// evaluates them at (-1/4 + I/2, -1/4 + J/2, -1/4 + K/2).
template <int D>
constexpr int kLinCoef = D == 2 ? 4 : 8;

template <typename Lt, typename R>
__device__ __forceinline__ void lin_coef(const R *P, int c, R *a) {
    const R *F = P + 2 * (c & 1) + 8 * ((c >> 1) & 1) + (Lt::D == 3 ? 32 * (c >> 2) : 0);
    if constexpr (Lt::D == 2) {
        const R F0 = F[0], F1 = F[1], F2 = F[4], F3 = F[5];
        a[0] = F0;
        a[1] = F1 - F0;
        a[2] = F2 - F0;
        a[3] = F3 - F2 - F1 + F0;
    } else {
        R G[8];
#pragma unroll
        for (int n = 0; n < 8; n++) G[n] = F[(n & 1) + 4 * ((n >> 1) & 1) + 16 * (n >> 2)];
        a[0] = G[0];
        a[1] = G[1] - G[0];
        a[2] = G[2] - G[0];
        a[3] = G[4] - G[0];
        a[4] = G[3] - G[1] - G[2] + G[0];
        a[5] = G[6] - G[2] - G[4] + G[0];
        a[6] = G[5] - G[1] - G[4] + G[0];
        a[7] = G[7] - G[3] - G[5] - G[6] + G[1] + G[2] + G[4] - G[0];
    }
}

template <typename Lt, typename R>
__device__ __forceinline__ R lin_value(const R *a, int lf) {
    const int I = lf & 3, J = (lf >> 2) & 3, K = lf >> 4;
    const R x = R(-0.25) + R(0.5) * R(I), y = R(-0.25) + R(0.5) * R(J), z = R(-0.25) + R(0.5) * R(K);
    if constexpr (Lt::D == 2) return a[0] + a[1] * x + a[2] * y + a[3] * x * y;
    else return a[0] + a[1] * x + a[2] * y + a[3] * z + a[4] * x * y + a[5] * y * z + a[6] * x * z + a[7] * x * y * z;
}

// Weights of the cubic Lagrange polynomials through the nodes u = 0, 1, 2, 3 at u.
template <typename R>
__device__ __forceinline__ void lagrange4(R u, R *w) {
    const R a = u, b = u - R(1), c = u - R(2), d = u - R(3);
    w[0] = -(b * c * d) / R(6);
    w[1] = (a * c * d) / R(2);
    w[2] = -(a * b * d) / R(2);
    w[3] = (a * b * c) / R(6);
}

// Interpolated value of fine cell lf of child c from one population of the
// parent's rescaled cells F[Mb].  Linear: the polynomial through the 2^d
// parent cells of the quadrant at (-1/4 + I/2, ...).  Cubic (Sec. "Cubic
// Interpolation"): the tensor product through all 4^d parent cells, nodes at
// parent cell centres u = 0 .. 3, evaluated at u = 3 (-1/12 + I/6 + 2 c/3)
// one axis at a time.
template <typename Lt, typename R>
__device__ __forceinline__ R interp_value(const R *F, int c, int lf, int cubic) {
    const int cx = c & 1, cy = (c >> 1) & 1, cz = (c >> 2) & 1;
    const int I = lf & 3, J = (lf >> 2) & 3, K = lf >> 4;
    if (!cubic) {
        R a[kLinCoef<Lt::D>];
        lin_coef<Lt, R>(F, c, a);
        return lin_value<Lt, R>(a, lf);
    }
    R wx[4], wy[4], wz[4];
    lagrange4<R>(R(-0.25) + R(0.5) * R(I) + R(2 * cx), wx);
    lagrange4<R>(R(-0.25) + R(0.5) * R(J) + R(2 * cy), wy);
    lagrange4<R>(R(-0.25) + R(0.5) * R(K) + R(2 * cz), wz);
    R v = R(0);
#pragma unroll
    for (int e = 0; e < (Lt::D == 3 ? 4 : 1); e++) {
        R plane = R(0);
#pragma unroll
        for (int n = 0; n < 4; n++) {
            R row = R(0);
#pragma unroll
            for (int mm = 0; mm < 4; mm++) row += wx[mm] * F[mm + 4 * n + 16 * e];
            plane += wy[n] * row;
        }
        v += (Lt::D == 3 ? wz[e] : R(1)) * plane;
    }
    return v;
}

// Children that one lane group of a team handles, and the teams of a
// 256-thread workgroup.
template <typename Lt> constexpr int kTeamThreads = Lt::D == 3 ? 256 : 64;
template <typename Lt> constexpr int kTeamTurns = Lt::NC * Lt::MB / kTeamThreads<Lt>;  // children per lane group

template <typename Lt, typename R>
struct InterpSmem {
    R g[Lt::Q][Lt::MB];                         // the parent's rescaled cells
    R coef[Lt::NC][Lt::Q][kLinCoef<Lt::D>];     // linear: per quadrant and population
    uint64_t ptab[kTab<Lt>];                    // rows of the parent and of the children
    uint64_t tab[Lt::NC][kTab<Lt>];
};

template <typename Lt>
__device__ __forceinline__ void team_sync() {
    if constexpr (Lt::D == 3) __syncthreads();
    else wave_lds_sync();
}

// Body (whole team, thread t of it): targeted cells of the children of parent P
// (a block that is not a refined parent is skipped).  CUB: 0 linear, 1 cubic,
// 2 the mesh's choice at run time.  src_of(L) / dst_of(L): current buffers of
// the parent's and the children's level, r_of(L): the rescaling.
// Two team barriers: parent's cells, coefficients.  Bound by its chain of
// dependent loads (list, parent's descriptor, its cells and the children's
// descriptors) and by the address work of the ghost cells' scattered stores.
// D3Q27 cylinder, per launch: 174 us with FP32 and 120 us with FP16 storage when
// links were staged for the workgroup, each cell formed its polynomial from
// eight LDS reads per population and stores branched on their link; now 167
// and 95 us.
template <int Q, int S, int CUB, typename SrcOf, typename DstOf, typename ROf>
__device__ __forceinline__ void interp_parent(const DevMesh &m, int P, SrcOf src_of, DstOf dst_of, ROf r_of,
                                              int all_cells, InterpSmem<Lat<Q>, typename Store<S>::R> &sm, int t) {
    using Lt = Lat<Q>;
    using ST = Store<S>;
    using R = typename ST::R;
    using T = typename ST::T;
    using De = Desc<Lt::D>;
    constexpr int MB = Lt::MB, NC = Lt::NC, TT = kTeamThreads<Lt>, NT = kTeamTurns<Lt>;
    const int l = t % MB, grp = t / MB;  // lane among the MB of a block; child grp + k TT / MB in turn k
    const int32_t pw = desc_word<Lt>(m.desc, P, l);
    const int first = desc_get<Lt>(pw, De::kFirst);
    const uint32_t pflag = (uint32_t)desc_get<Lt>(pw, De::kFlags);
    const int L = (int)(pflag >> 16);
    if (first < 0 || first > m.cap - NC || L + 1 >= m.lmax) return;  // uniform over the team
    const T *src = src_of(L);
    T *dst = dst_of(L);
    int32_t w[NT];
#pragma unroll
    for (int k = 0; k < NT; k++) w[k] = desc_word<Lt>(m.desc, first + grp + k * (TT / MB), l);
    if (grp == 0) {
        put_rows<Lt>(sm.ptab, pw, l, src);
        wave_lds_sync();
        const CellRows<T> r = cell_rows<Lt, T>(sm.ptab, wave_links<Lt>(pw, l), P, desc_get<Lt>(pw, De::kHid), l, src, m);
        R g[Q];
        gather_rows<Lt, ST>(r, g);
        R drho, ux, uy, uz;
        moments_g<Lt, R>(g, drho, ux, uy, uz);
        const R uu = ux * ux + uy * uy + uz * uz, sc = r_of(L);
#pragma unroll
        for (int p = 0; p < Q; p++) sm.g[p][l] = rescale_neq<Lt, R>(p, g[p], sc, drho, ux, uy, uz, uu);
    }
#pragma unroll
    for (int k = 0; k < NT; k++) put_rows<Lt>(sm.tab[grp + k * (TT / MB)], w[k], l, dst);
    team_sync<Lt>();
    const int cubic = CUB == 2 ? m.interp : CUB;
    if (!cubic) {
        for (int e = t; e < NC * Q; e += TT) lin_coef<Lt, R>(sm.g[e % Q], e / Q, sm.coef[e / Q][e % Q]);
        team_sync<Lt>();
    }
#pragma unroll 1
    for (int k = 0; k < NT; k++) {
        const int c = grp + k * (TT / MB);
        const int32_t wk = NT == 1 || k == 0 ? w[0] : w[NT - 1];
        uint64_t gm = (uint32_t)desc_get<Lt>(wk, De::kGhost);
        if constexpr (Lt::D == 3) gm |= (uint64_t)(uint32_t)desc_get<Lt>(wk, De::kGhost + 1) << 32;
        else gm &= 0xffff;
        if (all_cells) gm = ~0ull;
        const int h = desc_get<Lt>(wk, De::kHid);
        const LinkMask any = wave_links<Lt>(wk, l);
        if (!((gm >> l) & 1ull)) continue;
        // the cell's index hidden from loop-invariant code motion: per
        // population offsets kept across the two turns would take 50 VGPRs
        int lf = l;
        asm volatile("" : "+v"(lf));
        const CellRows<T> r = cell_rows<Lt, T>(sm.tab[c], any, first + c, h, lf, dst, m);
        const auto put = [&](auto pc, auto halo, R v) {
            constexpr int p = decltype(pc)::value;
            T *a = global_ptr<T>(slot_address<Lt, T, p, decltype(halo)::value>(r));
            ST::st(a, ST::shift ? v : v + R(Lt::w(p)));
            // one population at a time: reading all coefficients ahead would take 160 VGPRs
            __builtin_amdgcn_sched_barrier(0);
        };
        if (cubic) {
            // 4^d terms per population: not unrolled over the populations
#pragma unroll 1
            for (int p = 0; p < Q; p++) {
                const R v = interp_value<Lt, R>(sm.g[p], c, lf, 1);
                T *a = global_ptr<T>(slot_address_any<Lt, T>(r, sm.tab[c], lf, p));
                ST::st(a, ST::shift ? v : v + R(Lt::w(p)));
            }
        } else if (any.skip) {
            static_for<Q>([&](auto pc) {
                put(pc, std::true_type(), lin_value<Lt, R>(sm.coef[c][decltype(pc)::value], lf));
            });
        } else {
            static_for<Q>([&](auto pc) {
                put(pc, std::false_type(), lin_value<Lt, R>(sm.coef[c][decltype(pc)::value], lf));
            });
        }
    }
}

// parents per 256-thread workgroup
template <typename Lt> constexpr int kInterpPerWg = 256 / kTeamThreads<Lt>;

template <int Q, int S, int CUB>
__device__ __forceinline__ void interp_wg(const int32_t *__restrict__ list, int n, const DevMesh &m,
                                          typename Store<S>::T *f0, typename Store<S>::T *f1, const LevelParams &lp,
                                          int all_cells, int wg) {
    using Lt = Lat<Q>;
    using R = typename Store<S>::R;
    __shared__ InterpSmem<Lt, R> sm[kInterpPerWg<Lt>];
    const int team = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kTeamThreads<Lt>);
    const int item = wg * kInterpPerWg<Lt> + team;
    if (item >= n) return;
    interp_parent<Q, S, CUB>(
        m, list[item], [&](int L) { return lp.par[L] ? f1 : f0; }, [&](int L) { return lp.par[L + 1] ? f1 : f0; },
        [&](int L) { return R(lp.r_cf[L]); }, all_cells, sm[team], threadIdx.x % kTeamThreads<Lt>);
}

template <int Q, int S, int CUB>
__global__ __launch_bounds__(256) void k_interp(const int32_t *__restrict__ list, int n, DevMesh m,
                                                typename Store<S>::T *f0, typename Store<S>::T *f1, LevelParams lp,
                                                int all_cells) {
    interp_wg<Q, S, CUB>(list, n, m, f0, f1, lp, all_cells, blockIdx.x);
}

// The ghost interpolation into level L+1 and the collide-stream sweep of level
// L in one 256-thread launch: the first workgroups interpolate one parent each
// (2-D: four), the rest sweep the level.  Both read level L's current buffer; one
// writes ghost cells of level L+1, the other level L's other buffer, so they
// need no order, and small levels save a launch gap.  EX: the sweep adds the
// momentum exchange too (collide_block).
template <int Q, int S, bool NTS, int CUB, bool EX = false>
__global__ __launch_bounds__(256) void k_interp_collide(const int32_t *__restrict__ ilist, int ni,
                                                        const int32_t *__restrict__ clist, int nblk, DevMesh m,
                                                        typename Store<S>::T *f0, typename Store<S>::T *f1,
                                                        LevelParams lp, int L, BCParams bc) {
    const int b = blockIdx.x;
    const int iwg = (ni + kInterpPerWg<Lat<Q>> - 1) / kInterpPerWg<Lat<Q>>;
    if (b < iwg) {
        interp_wg<Q, S, CUB>(ilist, ni, m, f0, f1, lp, 0, b);
    } else {
        const typename Store<S>::T *src = lp.par[L] ? f1 : f0;
        typename Store<S>::T *dst = lp.par[L] ? f0 : f1;
        collide_wg<Q, S, NTS, 0, EX>(clist, nblk, m, src, dst, lp.omega[L], bc, lp.omega[L],
                                     xcd_remap(b - iwg, (int)gridDim.x - iwg));
    }
}

// Batched ghost fill of level L+1 from level L (interface parents of every
// simulation), persistent teams; par0/par1 = buffers of levels L, L+1.
// CUB: 0 every member linear, 2 the member's choice (131 instead of 77 VGPRs for
// D3Q19 at 16 bits, so groups without a cubic member do not carry it).
template <int Q, int S, int CUB>
__global__ __launch_bounds__(256) void k_interp_batch(const SimDesc *__restrict__ sims,
                                                      const uint32_t *__restrict__ items,
                                                      const int32_t *__restrict__ count, int L, int par0, int par1) {
    using Lt = Lat<Q>;
    using R = typename Store<S>::R;
    using T = typename Store<S>::T;
    __shared__ InterpSmem<Lt, R> sm[kInterpPerWg<Lt>];
    const int team = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kTeamThreads<Lt>);
    const int n = *count;
    int u0, u1;
    persistent_range((n + kInterpPerWg<Lt> - 1) / kInterpPerWg<Lt>, u0, u1);
    for (int u = u0; u < u1; u++) {
        const int item = u * kInterpPerWg<Lt> + team;
        if (item >= n) break;  // 3-D: never
        int sim, P;
        decode_item(items[item], sim, P);
        sim = __builtin_amdgcn_readfirstlane(sim);  // one item per team
        P = __builtin_amdgcn_readfirstlane(P);
        CSimDesc *cs = const_view(sims) + sim;
        const DevMesh m = load_mesh(cs);
        interp_parent<Q, S, CUB>(
            m, P, [&](int) { return (const T *)cs->f[par0]; }, [&](int) { return (T *)cs->f[par1]; },
            [&](int) { return R(cs->lp.r_cf[L]); }, 0, sm[team], opaque_tid() % kTeamThreads<Lt>);
        team_sync<Lt>();
    }
}

// Refresh after refinement.  A cell x of an existing block N next to a new
// same-level block C now receives the populations that stream from C's cells;
// they are stored in C's rows, which the interpolation of C's own cells does
// not write.  Their values are those x already had: the ghost interpolation
// from N's parent (x was adjacent to the region C now covers, which was
// covered only by a coarser block).  One workgroup per refined parent.
template <int Q, int S>
__global__ __launch_bounds__(256) void k_refresh_neighbours(const int32_t *__restrict__ list, int n, DevMesh m,
                                                            typename Store<S>::T *f0, typename Store<S>::T *f1,
                                                            LevelParams lp) {
    using Lt = Lat<Q>;
    using ST = Store<S>;
    using R = typename ST::R;
    using T = typename ST::T;
    constexpr int MB = Lt::MB, NC = Lt::NC, NS = Lt::D == 2 ? 9 : 27;
    __shared__ R s_g[Q][MB];
    __shared__ BlockStage<Lt, NC + 1> st;  // the new children, then the neighbour's parent
    __shared__ int s_nb[NC][NS];           // existing same-level neighbour per child and region, -1 none
    if ((int)blockIdx.x >= n) return;
    const int P = list[blockIdx.x];
    const int L = m.level[P];
    const int first = m.nbrc[P];
    if (first < 0 || first > m.cap - NC || L + 1 >= m.lmax) return;
    const T *psrc = lp.par[L] ? f1 : f0;
    T *dst = lp.par[L + 1] ? f1 : f0;
    const R r = R(lp.r_cf[L]);
    const int t = threadIdx.x;
    if (t < NC) st.id[t] = first + t;
    if (t == NC) st.id[NC] = -1;
    __syncthreads();
    stage_blocks<Lt, NC + 1>(m, st);
    for (int e = t; e < NC * NS; e += blockDim.x) {
        const int c = e / NS, rg = e - c * NS;
        const int N = st.link[c][rg];
        s_nb[c][rg] = (rg != kCenterSlot<Lt> && N >= 0 && N < m.cap && !m.fresh[N] && m.parent[N] >= 0) ? N : -1;
    }
    __syncthreads();
    for (int c = 0; c < NC; c++) {
        for (int rg = 0; rg < NS; rg++) {
            const int N = s_nb[c][rg];  // uniform over the workgroup
            if (N < 0) continue;
            const int PN = m.parent[N];
            const int cN = N - m.nbrc[PN];
            if (t == 0) st.id[NC] = PN;
            __syncthreads();
            for (int e = t; e < Lt::NB; e += blockDim.x)
                st.link[NC][dir_region<Lt>(e)] = m.nbr[(int64_t)e * m.cap + PN];
            if (t == 0) st.hid[NC] = m.hid[PN];
            __syncthreads();
            if (t < MB) {
                R g[Q];
                gather_cell<Lt, ST>(m, st.link[NC], PN, st.hid[NC], t, psrc, g);
                R drho, ux, uy, uz;
                moments_g<Lt, R>(g, drho, ux, uy, uz);
                const R uu = ux * ux + uy * uy + uz * uz;
#pragma unroll
                for (int p = 0; p < Q; p++) s_g[p][t] = rescale_neq<Lt, R>(p, g[p], r, drho, ux, uy, uz, uu);
            }
            __syncthreads();
            if (t < MB) {
                const int si = t & 3, sj = (t >> 2) & 3, sk = t >> 4;
#pragma unroll
                for (int p = 1; p < Q; p++) {
                    const int tx = si + Lt::cx(p), ty = sj + Lt::cy(p), tz = sk + Lt::cz(p);
                    if (region_of<Lt>(tx, ty, tz) != rg) continue;
                    // cell x of N (quadrant cN of N's parent): its ghost-fill value
                    const int lx = (tx & 3) + 4 * (ty & 3) + 16 * (tz & 3);
                    const R v = interp_value<Lt, R>(s_g[p], cN, lx, m.interp);
                    store_g<Lt, ST>(dst, mslot<Lt>(first + c, p, t), p, v);
                }
            }
            __syncthreads();
        }
    }
}

// Halo records across a mesh change.  Records are numbered in block order, so
// a block that stays (not new) may have another number than before; and where
// its neighbour C was removed, the populations that streamed from C's cells are
// in C's rows and belong to the record from now on.  The next step's ghost
// fill rewrites all of it, but a synchronisation may come first, and its
// averaging reads it.  So what a block needs goes to its new number in the
// buffer that is free between steps (records_out), and back from there once
// all have (records_back).  (Not moved, records held another block's values or
// zeros after a change that no step followed.  Records at the block's own ID
// would not have to move, but so spread out they cost the steps of the 64^3
// D3Q19 cavity 2 to 4 %.)
//
// 64 block IDs per 256-thread workgroup: their numbers in one coalesced read,
// then each block that has something to move by one wave.  Both halves ride on
// launches that a mesh change makes anyway: 6 us more of a change of a small 2-D
// mesh (210 us), chains of dependent loads; as launches of their own 10 to 15 us.

// populations of every cell of a block that come from a region whose entry in
// `links` is not kNone, by its MB lanes: at(p, record entry, region's entry,
// source cell)
template <typename Lt, typename F>
__device__ __forceinline__ void for_record_entries(const int32_t *links, int l, F &&at) {
    static_for<Lt::Q>([&](auto pc) {
        constexpr int p = decltype(pc)::value;
        const int sx = (l & 3) - Lt::cx(p), sy = ((l >> 2) & 3) - Lt::cy(p), sz = (l >> 4) - Lt::cz(p);
        const int rg = region_of<Lt>(sx, sy, sz);
        const int32_t code = rg == kCenterSlot<Lt> ? kNone : links[rg];
        if (code != kNone)
            at(pc, halo_entry<Lt, p>((uint64_t(1) << l) - 1), code, (sx & 3) + 4 * (sy & 3) + 16 * (sz & 3));
    });
}

// `old`: the records' numbers before the change; on return whether they move.
// Descriptors, and the rows of removed blocks, are those before the change.
template <int Q, typename T>
__device__ __forceinline__ void records_out(const DevMesh &m, const DevCounters *ctr, int32_t *old,
                                            const T *__restrict__ src, T *__restrict__ dst, int32_t *links) {
    using Lt = Lat<Q>;
    using De = Desc<Lt::D>;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int B0 = blockIdx.x * 64;
    // a number that stays may still gain entries from a removed block
    const bool removed = ctr->nfreed > 0;
    int now = -1, was = -1;
    if (B0 + lane < m.cap) {
        now = m.hid[B0 + lane];
        was = old[B0 + lane];
    }
    const uint64_t look = __ballot(now >= 0 && (removed || now != was) && !m.fresh[min(B0 + lane, m.cap - 1)]);
    __syncthreads();  // every wave has read `old`
    if (wave == 0 && B0 + lane < m.cap && !((look >> lane) & 1ull)) old[B0 + lane] = 0;
    int k = 0;
    for (uint64_t todo = look; todo; todo &= todo - 1) {
        if ((k++ & 3) != wave) continue;
        const int i = __builtin_ctzll(todo), B = B0 + i;
        const int nw = __shfl(now, i, 64), wa = __shfl(was, i, 64);
        // the links before the change: N_SKIP, a block that was removed, or nothing to move
        int32_t w = kNone;
        if (lane < De::kLinks) {
            w = m.desc[(int64_t)B * De::kWords + lane];
            if (w >= 0 ? m.status[w] != ST_INACTIVE : w != kNSkip) w = kNone;
            links[lane] = w;
        }
        const bool moves = wa != nw || __any(w >= 0);
        if (lane == 0) old[B] = moves;
        if (!moves) continue;
        wave_lds_sync();
        T *rec = dst + (m.halo_base + (int64_t)nw * m.nh);
        const T *from = src + (m.halo_base + (int64_t)wa * m.nh);
        if (lane < Lt::MB)
            for_record_entries<Lt>(links, lane, [&](auto pc, uint32_t e, int32_t code, int s) {
                rec[e] = code < 0 ? from[e] : src[mslot<Lt>(code, decltype(pc)::value, s)];
            });
        wave_lds_sync();
    }
}

// moved: as records_out left it; the descriptors are the new ones
template <int Q, typename T>
__device__ __forceinline__ void records_back(const DevMesh &m, const int32_t *__restrict__ moved, int wg,
                                             const T *__restrict__ src, T *__restrict__ dst, int32_t *links) {
    using Lt = Lat<Q>;
    using De = Desc<Lt::D>;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int B0 = wg * 64;
    int k = 0;
    for (uint64_t todo = __ballot(B0 + lane < m.cap && moved[B0 + lane] != 0); todo; todo &= todo - 1) {
        if ((k++ & 3) != wave) continue;
        const int B = B0 + __builtin_ctzll(todo);
        const int32_t w = lane < De::kWords ? m.desc[(int64_t)B * De::kWords + lane] : 0;
        if (lane < De::kLinks) links[lane] = w == kNSkip ? w : kNone;
        const int64_t rec = m.halo_base + (int64_t)__shfl(w, De::kHid, 64) * m.nh;
        wave_lds_sync();
        if (lane < Lt::MB)
            for_record_entries<Lt>(links, lane, [&](auto, uint32_t e, int32_t, int) { dst[rec + e] = src[rec + e]; });
        wave_lds_sync();
    }
}

// Packed block descriptors (Desc): one workgroup turns the links of 64
// consecutive blocks, read along each link array, into 64 rows through LDS.
// Before it overwrites the descriptors of the mesh before, it moves what their
// halo records need (old: null for a new mesh).
template <int Q, int S>
__global__ __launch_bounds__(256) void k_block_desc(DevMesh m, const DevCounters *ctr, int32_t *old,
                                                    const typename Store<S>::T *__restrict__ f0,
                                                    typename Store<S>::T *__restrict__ f1) {
    using Dd = Lat<Q>;
    using De = Desc<Dd::D>;
    constexpr int NW = De::kWords;
    __shared__ int32_t row[64][NW + 1];
    if (old) {
        records_out<Q>(m, ctr, old, f0, f1, row[threadIdx.x >> 6]);
        __syncthreads();
    }
    const int B0 = blockIdx.x * 64;
    const int b = threadIdx.x & 63, B = B0 + b;
    const bool act = B < m.cap && m.status[B] != ST_INACTIVE;
    for (int p = threadIdx.x >> 6; p < NW; p += 4) {
        int32_t v = 0;
        if (act) {
            if (p < Dd::NB) v = m.nbr[(int64_t)p * m.cap + B];
            else if (p == De::kHid) v = m.hid[B];
            else if (p == De::kFlags)
                v = (int32_t)(m.bflag[B] | (m.status[B] == ST_UNREF ? DF_LEAF : 0u) | ((uint32_t)m.level[B] << 16));
            else if (p == De::kFirst) v = m.nbrc[B];
            else if (p == De::kGhost)
                v = Dd::D == 3 ? (int32_t)m.gmask[B] : (int32_t)(m.gmask[B] | m.imask[B] << 16);
            else if (Dd::D == 3) v = (int32_t)(m.gmask[B] >> 32);
        }
        const int at = p < Dd::NB ? dir_region<Dd>(p) : p;
        row[b][at] = v;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 64 * NW; e += 256)
        if (B0 + e / NW < m.cap) m.desc[(int64_t)B0 * NW + e] = row[e / NW][e % NW];
}

// Cells the interpolation and the averaging of each level move (for the
// byte counts of the solver's kernel statistics): over the interface parents
// of level L, the ghost cells of their children and the parent cells whose
// first fine cell (even i, j, k) is an interface cell.
// One thread per interface parent of one level; the sums are reduced over the
// wave before one atomic per wave.
template <typename Lt>
__device__ __forceinline__ void target_cells(const DevMesh &m, const int32_t *__restrict__ iface, DevCounters *ctr,
                                             int L, int i) {
    unsigned long long g = 0, a = 0;
    if (i < ctr->niface[L]) {
        const int P = iface[(int64_t)L * m.cap + i];
        const int first = m.nbrc[P];
        // fine cells with even coordinates: the first of each parent cell's 2^d
        const uint64_t lead = Lt::D == 3 ? 0x0000050500000505ull : 0x0505ull;
        if (first >= 0 && first <= m.cap - Lt::NC)
            for (int c = 0; c < Lt::NC; c++) {
                g += __popcll(m.gmask[first + c]);
                a += __popcll(m.imask[first + c] & lead);
            }
    }
    for (int off = 32; off > 0; off >>= 1) {
        g += __shfl_xor(g, off, 64);
        a += __shfl_xor(a, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        if (g) atomicAdd(&ctr->ghost_w[L], g);
        if (a) atomicAdd(&ctr->avg_w[L], a);
    }
}

// The first workgroups take the records that moved, 64 block IDs each (none for
// a new mesh), the others the levels, `per` each.
template <int Q, int S>
__global__ __launch_bounds__(256) void k_target_cells(DevMesh m, const int32_t *__restrict__ iface, DevCounters *ctr,
                                                      const int32_t *__restrict__ moved, int nrec, int per,
                                                      typename Store<S>::T *__restrict__ f0,
                                                      const typename Store<S>::T *__restrict__ f1) {
    __shared__ int32_t links[4][Desc<Lat<Q>::D>::kLinks];
    const int wg = (int)blockIdx.x - nrec;
    if (wg < 0) records_back<Q>(m, moved, blockIdx.x, f1, f0, links[threadIdx.x >> 6]);
    else target_cells<Lat<Q>>(m, iface, ctr, wg / per, wg % per * 256 + (int)threadIdx.x);
}

static __global__ void k_clear_fresh(const int32_t *__restrict__ list, int n, DevMesh m, int nc) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * nc) return;
    const int P = list[e / nc];
    const int first = m.nbrc[P];
    if (first >= 0 && first + e % nc < m.cap) m.fresh[first + e % nc] = 0;
}

// ---------------------------------------------------------------------------
// Fine-to-coarse averaging with rescaling (Sec. "Averaging"): parent cell
// (i,j,k) takes the mean of the 2^d rescaled cells of child octant
// (i/2, j/2, k/2) starting at fine cell (2(i mod 2), 2(j mod 2), 2(k mod 2)).
// One lane per fine cell of the children (3-D: a wave per child, on its own, so
// that children that end early hold back no other): every lane gathers and
// rescales its cell, the 2^d cells of a parent cell (lanes differing in bits 0, 2, 4 of the
// cell index, all in one wave) are summed with xor shuffles, and the lane of
// the first one writes the parent cell.  Children without a targeted cell are
// skipped whole.

// The vorticity criterion reads velocities of leaf blocks and, across the six
// faces of a leaf, of its same-level neighbours: a refined block none of whose
// face neighbours is a leaf is never read.
// w, flag: the block's descriptor words and its flags.
template <typename Lt>
__device__ __forceinline__ bool velocity_read(const DevMesh &m, int32_t w, uint32_t flag) {
    if (flag & DF_LEAF) return true;
    bool read = false;
#pragma unroll
    for (int a = 0; a < Lt::D; a++)
#pragma unroll
        for (int sg = -1; sg <= 1; sg += 2) {
            const int32_t code = desc_get<Lt>(w, kCenterSlot<Lt> + sg * (a == 0 ? 1 : (a == 1 ? 3 : 9)));
            if (code >= 0 && m.status[code] == ST_UNREF) read = true;
        }
    return read;
}

// FP64 velocity j / rho of cell `cell` from its populations fv, into U[3][capc]
template <typename Lt>
__device__ __forceinline__ void cell_velocity(const double *fv, double *U, int64_t capc, int64_t cell) {
    double rho = 0.0, j[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int p = 0; p < Lt::Q; p++) {
        rho += fv[p];
        j[0] += fv[p] * Lt::cx(p);
        j[1] += fv[p] * Lt::cy(p);
        j[2] += fv[p] * Lt::cz(p);
    }
    for (int a = 0; a < 3; a++) U[a * capc + cell] = j[a] / rho;
}

// The value of the lane whose index differs in bit MASK (1, 4 or 16).
template <int MASK>
__device__ __forceinline__ int xor_lane32(int v) {
    if constexpr (MASK == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true);  // quad_perm 1, 0, 3, 2
    else return __builtin_amdgcn_ds_swizzle(v, 0x1f | (MASK << 10));
}
template <int MASK>
__device__ __forceinline__ float xor_sum(float v) {
    return v + __builtin_bit_cast(float, xor_lane32<MASK>(__builtin_bit_cast(int, v)));
}
template <int MASK>
__device__ __forceinline__ double xor_sum(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)xor_lane32<MASK>((int)(uint32_t)b), hi = (uint32_t)xor_lane32<MASK>((int)(b >> 32));
    return v + __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// child c of refined parent P, by the lanes of the child (3-D: a wave, 2-D: 16
// lanes), with nothing shared beyond them: ctab, ptab are their own row tables.
// The chain of dependent loads (parent's descriptor, child's descriptor and
// mask, cells) and the gather's address work bound it.  D3Q27 cylinder, per
// launch of interface averaging: 143 us with FP32 and 134 us with FP16 storage
// in workgroups of four children that shared staged links, now 117 and 95 us;
// every cell of every parent before an adaptation: 2.9 and 2.4, now 2.6 and 1.9 ms.  VEL (every cell
// averaged): also the criterion's FP64 velocity of each child cell that it
// reads (velocity_read) and that the ghost interpolation after the averaging
// does not rewrite (no N_SKIP link), from the values as stored, into U: the
// same values and arithmetic as k_velocity, so that pass can skip those blocks.
template <int Q, int S, bool VEL = false>
__device__ __forceinline__ void average_child(const DevMesh &m, int P, int c, const typename Store<S>::T *src,
                                              typename Store<S>::T *dst, typename Store<S>::R r, int all_cells,
                                              uint64_t *ctab, uint64_t *ptab, int lf, double *U = nullptr) {
    using Lt = Lat<Q>;
    using ST = Store<S>;
    using R = typename ST::R;
    using T = typename ST::T;
    using De = Desc<Lt::D>;
    // with unshifted storage the velocities need the stored values: gather
    // those, then form g exactly as load_g does
    constexpr bool RAW = VEL && !ST::shift;
    constexpr int MB = Lt::MB, NC = Lt::NC;
    const int32_t pw = desc_word<Lt>(m.desc, P, lf);
    const int first = desc_get<Lt>(pw, De::kFirst);
    if (first < 0 || first > m.cap - NC) return;
    const int child = first + c;
    const int32_t w = desc_word<Lt>(m.desc, child, lf);
    const uint64_t im = all_cells ? ~0ull : m.imask[child];
    if (im == 0) return;  // the whole child
    put_rows<Lt>(ptab, pw, lf, dst);
    put_rows<Lt>(ctab, w, lf, src);
    wave_lds_sync();
    const uint32_t flag = (uint32_t)desc_get<Lt>(w, De::kFlags);
    const int h = desc_get<Lt>(w, De::kHid);
    const int ph = desc_get<Lt>(pw, De::kHid);
    const LinkMask any = wave_links<Lt>(w, lf), pany = wave_links<Lt>(pw, lf);
    // the 2^d lanes of one parent cell (cell-index bits 0, 2 and, in 3-D, 4)
    // are exactly the partners of the sums below: a group whose parent cell
    // is not written loads nothing
    const int lead = lf & ~(Lt::D == 3 ? 0x15 : 0x5);
    [[maybe_unused]] bool read = false;
    if constexpr (VEL) read = !(flag & BF_NSKIP) && velocity_read<Lt>(m, w, flag);
    R g[Q];
    if ((im >> lead) & 1ull) {
        gather_rows<Lt, ST, RAW>(cell_rows<Lt, T>(ctab, any, child, h, lf, src, m), g);
    } else {
#pragma unroll
        for (int p = 0; p < Q; p++) g[p] = R(0);
    }
    if constexpr (VEL) {
        if (read) {
            double fv[Q];
#pragma unroll
            for (int p = 0; p < Q; p++) fv[p] = double(g[p]) + (ST::shift ? Lt::w(p) : 0.0);
            cell_velocity<Lt>(fv, U, m.capc, (int64_t)child * MB + lf);
        }
        if constexpr (RAW) {
            if ((im >> lead) & 1ull) {
#pragma unroll
                for (int p = 0; p < Q; p++) g[p] = g[p] - R(Lt::w(p));
            }
        }
    }
    R drho, ux, uy, uz;
    moments_g<Lt, R>(g, drho, ux, uy, uz);
    const R uu = ux * ux + uy * uy + uz * uz;
#pragma unroll
    for (int p = 0; p < Q; p++) {
        R v = rescale_neq<Lt, R>(p, g[p], r, drho, ux, uy, uz, uu);
        v = xor_sum<1>(v);
        v = xor_sum<4>(v);
        if constexpr (Lt::D == 3) v = xor_sum<16>(v);
        g[p] = v;
    }
    const int i = lf & 3, j = (lf >> 2) & 3, k = lf >> 4;
    if (lf != lead || !((im >> lf) & 1ull)) return;
    const int l = ((c & 1) * 2 + (i >> 1)) + 4 * (((c >> 1) & 1) * 2 + (j >> 1)) + 16 * ((c >> 2) * 2 + (k >> 1));
    const CellRows<T> pr = cell_rows<Lt, T>(ptab, pany, P, ph, l, dst, m);
    const auto put = [&](auto pc, auto halo) {
        constexpr int p = decltype(pc)::value;
        const R v = g[p] / R(NC);
        ST::st(global_ptr<T>(slot_address<Lt, T, p, decltype(halo)::value>(pr)), ST::shift ? v : v + R(Lt::w(p)));
    };
    if (pany.skip) static_for<Q>([&](auto pc) { put(pc, std::true_type()); });
    else static_for<Q>([&](auto pc) { put(pc, std::false_type()); });
}

// children per 256-thread workgroup: one per wave in 3-D, four per wave in 2-D
template <typename Lt> constexpr int kAvgPerWg = 256 / Lt::MB;

template <typename Lt>
struct AvgSmem {
    uint64_t ctab[kAvgPerWg<Lt>][kTab<Lt>], ptab[kAvgPerWg<Lt>][kTab<Lt>];
};

// list: refined blocks of level L; a workgroup takes kAvgPerWg of their children.
// At least 6 waves per SIMD: left alone the compiler takes more than 80 VGPRs
// (5 waves) for D3Q27 FP32, 9 % slower on the cylinder set-up.
template <int Q, int S, bool VEL = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(S == AMR_F64 ? 1 : 6))) void k_average(
    const int32_t *__restrict__ list, int n, DevMesh m, const typename Store<S>::T *src, typename Store<S>::T *dst,
    double r_fc, int all_cells, double *U) {
    using Lt = Lat<Q>;
    using R = typename Store<S>::R;
    __shared__ AvgSmem<Lt> sm;
    const int slot = threadIdx.x / Lt::MB;
    int64_t unit = (int64_t)blockIdx.x * kAvgPerWg<Lt> + slot;
    const int item = __builtin_amdgcn_readfirstlane((int)(unit / Lt::NC));  // one parent per wave
    if (item >= n) return;
    average_child<Q, S, VEL>(m, list[item], (int)(unit % Lt::NC), src, dst, R(r_fc), all_cells, sm.ctab[slot],
                             sm.ptab[slot], threadIdx.x % Lt::MB, U);
}

// Batched interface averaging of level L+1 into level L, persistent
// workgroups; par0/par1 = buffers of levels L, L+1.
template <int Q, int S>
__global__ __launch_bounds__(256) void k_average_batch(const SimDesc *__restrict__ sims,
                                                       const uint32_t *__restrict__ items,
                                                       const int32_t *__restrict__ count, int L, int par0, int par1) {
    using Lt = Lat<Q>;
    using R = typename Store<S>::R;
    using T = typename Store<S>::T;
    __shared__ AvgSmem<Lt> sm;
    const int n = *count;
    int u0, u1;
    persistent_range((n * Lt::NC + kAvgPerWg<Lt> - 1) / kAvgPerWg<Lt>, u0, u1);
    for (int u = u0; u < u1; u++) {
        const int tid = opaque_tid(), slot = tid / Lt::MB;
        const int unit = u * kAvgPerWg<Lt> + slot;
        const int item = __builtin_amdgcn_readfirstlane(unit / Lt::NC);  // one parent per wave
        if (item >= n) break;
        int sim, P;
        decode_item(items[item], sim, P);
        sim = __builtin_amdgcn_readfirstlane(sim);
        P = __builtin_amdgcn_readfirstlane(P);
        CSimDesc *cs = const_view(sims) + sim;
        const DevMesh m = load_mesh(cs);
        average_child<Q, S>(m, P, unit % Lt::NC, (const T *)cs->f[par1], (T *)cs->f[par0], R(cs->lp.r_fc[L]), 0,
                            sm.ctab[slot], sm.ptab[slot], tid % Lt::MB);
        wave_lds_sync();
    }
}

// Work items of a batch for every level: kind 0 = launch order of the level,
// kind 1 = its interface parents, kind 2 = its leaf blocks next to a solid
// block; simulations in batch order.  Grid: x chunks of a list, y =
// simulation, z = 3 * level + kind.  counts[3 L + kind].
__device__ inline int item_count(const SimDesc &d, int L, int kind) {
    if (L >= d.m.lmax) return 0;
    return kind == 0 ? d.nids[L] : (kind == 1 ? d.niface[L] : (d.force_on ? d.nsolid[L] : 0));
}

static __global__ void k_batch_items(const SimDesc *__restrict__ sims, int nsims, uint32_t *__restrict__ items,
                              int64_t stride, int32_t *__restrict__ counts) {
    const int s = blockIdx.y, L = blockIdx.z / 3, kind = blockIdx.z % 3;
    __shared__ int s_part[4], s_n;
    // items of the simulations before this one: their counts loaded side by side
    int off = 0;
    for (int t = threadIdx.x; t < s; t += blockDim.x) off += item_count(sims[t], L, kind);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) off += __shfl_xor(off, o, 64);
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = off;
    if (threadIdx.x == 0) s_n = item_count(sims[s], L, kind);
    __syncthreads();
    const int s_off = s_part[0] + s_part[1] + s_part[2] + s_part[3];
    if (threadIdx.x == 0 && s == nsims - 1 && blockIdx.x == 0) counts[blockIdx.z] = s_off + s_n;
    const SimDesc &sd = sims[s];
    const int32_t *src = (kind == 0 ? sd.order : (kind == 1 ? sd.iface : sd.solid)) + (int64_t)L * sd.m.cap;
    uint32_t *dst = items + (int64_t)blockIdx.z * stride + s_off;
    const uint32_t tag = (uint32_t)s << kItemSimShift;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < s_n; i += gridDim.x * blockDim.x)
        dst[i] = tag | (uint32_t)src[i];
}

// ---------------------------------------------------------------------------
// Momentum exchange with solid blocks (Sec. "Flow Past a Square Cylinder"),
// after a collide-stream sweep: a leaf cell's post-collision population f*_q
// whose link ends in a solid block was reflected into the cell's own slot
// (x, q) of the buffer just written; it passes 2 f*_q c_q to the solid.  One
// block per 64 lanes (2-D: 16), summed over the block, added to its FP64 total
// (each block's total is written by one lane only).
template <int Q, int S>
__device__ __forceinline__ void exchange_block(const DevMesh &m, const BlockStage<Lat<Q>, 256 / Lat<Q>::MB> &st,
                                               int s, int l, const typename Store<S>::T *f) {
    using Lt = Lat<Q>;
    using ST = Store<S>;
    const int B = st.id[s];
    if (B < 0) return;
    const int32_t *link = st.link[s];
    const int i = l & 3, j = (l >> 2) & 3, k = l >> 4;
    double fx = 0.0, fy = 0.0, fz = 0.0;
#pragma unroll
    for (int q = 1; q < Q; q++) {
        if (link[region_of<Lt>(i + Lt::cx(q), j + Lt::cy(q), k + Lt::cz(q))] != kSolid) continue;
        const double two_f = 2.0 * double(ST::ld(f + mslot<Lt>(B, q, l)) + (ST::shift ? Lt::w(q) : 0.0));
        fx += two_f * Lt::cx(q);
        fy += two_f * Lt::cy(q);
        fz += two_f * Lt::cz(q);
    }
#pragma unroll
    for (int mask = 1; mask < Lt::MB; mask <<= 1) {
        fx += __shfl_xor(fx, mask, 64);
        fy += __shfl_xor(fy, mask, 64);
        fz += __shfl_xor(fz, mask, 64);
    }
    if (l == 0) {
        m.force[(int64_t)B * 3 + 0] += fx;
        m.force[(int64_t)B * 3 + 1] += fy;
        m.force[(int64_t)B * 3 + 2] += fz;
    }
}

template <int Q, int S>
__global__ __launch_bounds__(256) void k_exchange(const int32_t *__restrict__ list, int n, DevMesh m,
                                                  const typename Store<S>::T *__restrict__ f) {
    using Lt = Lat<Q>;
    constexpr int MB = Lt::MB, BPW = 256 / MB;
    __shared__ BlockStage<Lt, BPW> st;
    const int base = blockIdx.x * BPW;
    if ((int)threadIdx.x < BPW) st.id[threadIdx.x] = base + (int)threadIdx.x < n ? list[base + threadIdx.x] : -1;
    __syncthreads();
    stage_blocks<Lt, BPW>(m, st);
    exchange_block<Q, S>(m, st, threadIdx.x / MB, threadIdx.x % MB, f);
}

template <int Q, int S>
__global__ __launch_bounds__(256) void k_exchange_batch(const SimDesc *__restrict__ sims,
                                                        const uint32_t *__restrict__ items,
                                                        const int32_t *__restrict__ count, int par) {
    using Lt = Lat<Q>;
    using T = typename Store<S>::T;
    constexpr int MB = Lt::MB, BPW = 256 / MB;
    __shared__ BlockStage<Lt, BPW> st;
    const int n = *count;
    int u0, u1;
    persistent_range((n + BPW - 1) / BPW, u0, u1);
    for (int u = u0; u < u1; u++) {
        if ((int)threadIdx.x < BPW) {
            const int idx = u * BPW + (int)threadIdx.x;
            int sim = 0, B = -1;
            if (idx < n) decode_item(items[idx], sim, B);
            st.id[threadIdx.x] = B;
            st.sim[threadIdx.x] = sim;
        }
        __syncthreads();
        stage_blocks_by<Lt, BPW>([&](int e) -> const DevMesh & { return sims[st.sim[e]].m; }, st);
        const int tid = opaque_tid();
        const int s = tid / MB;
        int sim = st.sim[s];
        if (MB == 64) sim = __builtin_amdgcn_readfirstlane(sim);
        CSimDesc *cs = const_view(sims) + sim;
        const DevMesh m = load_mesh(cs);
        exchange_block<Q, S>(m, st, s, tid % MB, (const T *)cs->f[par]);
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Per-level totals of the momentum exchange (one workgroup per level, fixed
// summation order): out[L][0..2].  Only leaf blocks next to a solid block, the
// level's list, hold any; reading every block of the capacity instead took
// 440 us for 3.9e5 blocks (3 levels), the lists 4 us.
static __global__ __launch_bounds__(1024) void k_force_sum(const double *force, const int32_t *__restrict__ lists,
                                                           int cap, const DevCounters *ctr, double *out) {
    __shared__ double s[3][16];
    const int L = blockIdx.x, t = threadIdx.x, n = ctr->nsolid[L];
    double a[3] = {0.0, 0.0, 0.0};
    for (int i = t; i < n; i += 1024) {
        const int64_t B = lists[(int64_t)L * cap + i];
        for (int c = 0; c < 3; c++) a[c] += force[B * 3 + c];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        for (int c = 0; c < 3; c++) a[c] += __shfl_xor(a[c], off, 64);
    if ((t & 63) == 0)
        for (int c = 0; c < 3; c++) s[c][t >> 6] = a[c];
    __syncthreads();
    if (t < 3) {
        double v = 0.0;
        for (int w = 0; w < 16; w++) v += s[t][w];
        out[L * 3 + t] = v;
    }
}

static __global__ void k_force_reset(DevMesh m) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < (int64_t)m.cap * 3) m.force[e] = 0.0;
}

// ---------------------------------------------------------------------------
// initial states: every slot at rest (g = 0, f = w)
template <int Q, int S>
__global__ void k_fill_rest(DevMesh m, typename Store<S>::T *f0, typename Store<S>::T *f1, int64_t total) {
    using Lt = Lat<Q>;
    using ST = Store<S>;
    using R = typename ST::R;
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    R v = R(0);
    if (!ST::shift && e < m.halo_base) {
        const int p = (int)((e / Lt::MB) % Q);
        v = R(Lt::w(p));
    }
    ST::st(f0 + e, v);
    ST::st(f1 + e, v);
}

// Block-parallel kernels below run 256/Mb blocks per 256-thread workgroup
// over a contiguous block-ID range [b0, b1).

// f = feq(rho, u) of root cells from (rho, ux, uy, uz), ru[((B - b0) Mb + l) 4]
template <int Q, int S>
__global__ __launch_bounds__(256) void k_set_rho_u(DevMesh m, typename Store<S>::T *f, const double *__restrict__ ru,
                                                   int b0, int b1) {
    using Lt = Lat<Q>;
    using ST = Store<S>;
    using R = typename ST::R;
    constexpr int MB = Lt::MB, BPW = 256 / MB;
    __shared__ BlockStage<Lt, BPW> st;
    if ((int)threadIdx.x < BPW) {
        const int B = b0 + blockIdx.x * BPW + threadIdx.x;
        st.id[threadIdx.x] = (B < b1 && m.status[B] != ST_INACTIVE) ? B : -1;
    }
    __syncthreads();
    stage_blocks<Lt, BPW>(m, st);
    const int s = threadIdx.x / MB, l = threadIdx.x % MB;
    const int B = st.id[s];
    if (B < 0) return;
    const double *v = ru + ((int64_t)(B - b0) * MB + l) * 4;
    const double rho = v[0], ux = v[1], uy = v[2], uz = v[3];
    const double uu = ux * ux + uy * uy + uz * uz;
#pragma unroll
    for (int p = 0; p < Q; p++) {
        const double cu = Lt::cx(p) * ux + Lt::cy(p) * uy + Lt::cz(p) * uz;
        const double val = ST::shift ? Lt::w(p) * ((rho - 1.0) + rho * (3.0 * cu + 4.5 * cu * cu - 1.5 * uu))
                                     : Lt::w(p) * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu);
        ST::st(f + entry_slot<Lt>(m, st.link[s], B, st.hid[s], p, l), R(val));
    }
}

// ---------------------------------------------------------------------------
// Vorticity criterion, FP64 (Sec. "Adaptive Mesh Refinement" of the solver).
// First the FP64 velocity of every cell of a level, then central differences
// over same-level neighbour cells (one-sided where a neighbour is missing),
// scaled to root-cell units; block maximum per leaf and the global maximum
// (atomic max on the bit pattern of a non-negative double).
template <typename Lt, typename ST>
__device__ __forceinline__ void cell_f64_desc(const DevMesh &m, uint64_t *tab, int32_t w, int B, int l,
                                              const typename ST::T *f, double *fv) {
    using T = typename ST::T;
    using De = Desc<Lt::D>;
    put_rows<Lt>(tab, w, l, f);
    wave_lds_sync();
    const CellRows<T> r = cell_rows<Lt, T>(tab, wave_links<Lt>(w, l), B, desc_get<Lt>(w, De::kHid), l, f, m);
    const auto conv = [](typename ST::R v, int p) { return double(v) + (ST::shift ? Lt::w(p) : 0.0); };
    if (!(r.any.wall | r.any.skip))
        gather_interior_by<Lt, ST>(r.u, fv, conv);
    else
        gather_rows_by<Lt, ST>(r, fv, conv);
}

// ghost cells of a block from its descriptor words
template <typename Lt>
__device__ __forceinline__ uint64_t desc_ghost(int32_t w) {
    using De = Desc<Lt::D>;
    const uint64_t lo = (uint32_t)desc_get<Lt>(w, De::kGhost);
    if constexpr (Lt::D == 3) return lo | (uint64_t)(uint32_t)desc_get<Lt>(w, De::kGhost + 1) << 32;
    else return lo & 0xffff;
}

template <typename Lt, typename ST>
__device__ inline void cell_f64(const DevMesh &m, const int32_t *link, int B, int h, int l,
                                const typename ST::T *f, double *fv) {
#pragma unroll
    for (int p = 0; p < Lt::Q; p++)
        fv[p] = double(ST::ld(f + entry_slot<Lt>(m, link, B, h, p, l))) + (ST::shift ? Lt::w(p) : 0.0);
}

// children = 0: `list` holds the blocks.  children = 1: `list` holds parents
// (the interface parents of the level above) and the kernel takes those of
// their children that have an N_SKIP link: after k_average with VEL, the only
// blocks below level 0 whose velocities are still missing.
template <int Q, int S>
__global__ __launch_bounds__(256) void k_velocity(const int32_t *__restrict__ list, int n, DevMesh m,
                                                  const typename Store<S>::T *__restrict__ f, double *U,
                                                  int children) {
    using Lt = Lat<Q>;
    using ST = Store<S>;
    using De = Desc<Lt::D>;
    constexpr int MB = Lt::MB, BPW = 256 / MB;
    __shared__ uint64_t tabs[BPW][kTab<Lt>];
    const int slot = threadIdx.x / MB, l = threadIdx.x % MB;
    const int64_t i = (int64_t)blockIdx.x * BPW + slot;
    int B = -1;
    if (!children) {
        if (i < n) B = list[i];
    } else if (i < (int64_t)n * Lt::NC) {
        const int c0 = m.nbrc[list[i / Lt::NC]];
        const int C = c0 + (int)(i % Lt::NC);
        if (c0 >= 0 && (m.bflag[C] & BF_NSKIP)) B = C;
    }
    if constexpr (Lt::D == 3) B = __builtin_amdgcn_readfirstlane(B);  // one block per wave
    if (B < 0) return;  // the block's lanes together
    const int32_t w = desc_word<Lt>(m.desc, B, l);
    if (!velocity_read<Lt>(m, w, (uint32_t)desc_get<Lt>(w, De::kFlags))) return;
    double fv[Q];
    cell_f64_desc<Lt, ST>(m, tabs[slot], w, B, l, f, fv);
    cell_velocity<Lt>(fv, U, m.capc, (int64_t)B * MB + l);
}

template <int Q>
__global__ __launch_bounds__(256) void k_vorticity(const int32_t *__restrict__ list, int n, DevMesh m,
                                                   const double *__restrict__ U, double scale, double *crit,
                                                   unsigned long long *wmax_bits) {
    using Lt = Lat<Q>;
    constexpr int MB = Lt::MB, BPW = 256 / MB;
    __shared__ BlockStage<Lt, BPW> st;
    const int base = blockIdx.x * BPW;
    if ((int)threadIdx.x < BPW) st.id[threadIdx.x] = base + (int)threadIdx.x < n ? list[base + threadIdx.x] : -1;
    __syncthreads();
    stage_blocks<Lt, BPW>(m, st);
    const int s = threadIdx.x / MB, l = threadIdx.x % MB;
    const int B = st.id[s];
    const bool leaf = B >= 0 && m.status[B] == ST_UNREF;
    const int ci[3] = {l & 3, (l >> 2) & 3, l >> 4};
    // the neighbour cells along +-x, +-y (+-z): those in other blocks are read
    // here, all loads at once and before the barrier; those inside the block
    // come from the block's own velocities in LDS below
    double nv[3][2][3] = {};
    int nlc[3][2];
    bool nhas[3][2], nin[3][2];
#pragma unroll
    for (int a = 0; a < Lt::D; a++)
#pragma unroll
        for (int sg = 0; sg < 2; sg++) {
            int t[3] = {ci[0], ci[1], ci[2]};
            t[a] += sg == 0 ? 1 : -1;
            const int rg = region_of<Lt>(t[0], t[1], t[2]);
            const int32_t code = leaf ? st.link[s][rg] : -1;
            nhas[a][sg] = code >= 0 && code < m.cap;
            nin[a][sg] = rg == kCenterSlot<Lt>;
            nlc[a][sg] = (t[0] & 3) + 4 * (t[1] & 3) + 16 * (t[2] & 3);
            if (nhas[a][sg] && !nin[a][sg]) {
                const int64_t nc = (int64_t)code * MB + nlc[a][sg];
#pragma unroll
                for (int b = 0; b < 3; b++) nv[a][sg][b] = U[b * m.capc + nc];
            }
        }
    // the velocities of the block's own cells, for the neighbours inside it
    __shared__ double us[BPW][3][MB];
    if (leaf)
        for (int b = 0; b < 3; b++) us[s][b][l] = U[b * m.capc + (int64_t)B * MB + l];
    __syncthreads();
    double w = 0.0;
    if (leaf) {
        double u0[3];
        for (int b = 0; b < 3; b++) u0[b] = us[s][b][l];
        double gr[3][3];
        for (int a = 0; a < 3; a++)
            for (int b = 0; b < 3; b++) gr[a][b] = 0.0;
#pragma unroll
        for (int a = 0; a < Lt::D; a++) {
            double up[3], um[3];
            bool hp = false, hm = false;
#pragma unroll
            for (int sg = 0; sg < 2; sg++) {
                if (!nhas[a][sg]) continue;
                double *dstv = sg == 0 ? up : um;
#pragma unroll
                for (int b = 0; b < 3; b++) dstv[b] = nin[a][sg] ? us[s][b][nlc[a][sg]] : nv[a][sg][b];
                if (sg == 0) hp = true; else hm = true;
            }
#pragma unroll
            for (int b = 0; b < 3; b++) {
                if (hp && hm) gr[a][b] = (up[b] - um[b]) / 2.0;
                else if (hp) gr[a][b] = up[b] - u0[b];
                else if (hm) gr[a][b] = u0[b] - um[b];
            }
        }
        if (Lt::D == 2) {
            w = fabs(gr[0][1] - gr[1][0]) * scale;
        } else {
            const double wx = gr[1][2] - gr[2][1], wy = gr[2][0] - gr[0][2], wz = gr[0][1] - gr[1][0];
            w = sqrt(wx * wx + wy * wy + wz * wz) * scale;
        }
    }
    // block maximum over the MB lanes of the block
#pragma unroll
    for (int off = MB / 2; off > 0; off >>= 1) w = fmax(w, __shfl_xor(w, off, 64));
    if (leaf && l == 0) {
        crit[B] = w;
        // the running maximum rarely grows: compare first, so that most blocks
        // skip the atomic on the one shared address
        const unsigned long long bits = (unsigned long long)__double_as_longlong(w);
        if (bits > __hip_atomic_load(wmax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(wmax_bits, bits);
    }
}

// ---------------------------------------------------------------------------
// Gathers / scatters of unshifted FP64 data through the staging buffer.
// Every cell of every active block, [B - b0][l][q]; inactive blocks read 0.
template <int Q, int S>
__global__ __launch_bounds__(256) void k_block_f(DevMesh m, typename Store<S>::T *f0, typename Store<S>::T *f1,
                                                 LevelParams lp, int set, int b0, int b1, double *stage) {
    using Lt = Lat<Q>;
    using ST = Store<S>;
    using R = typename ST::R;
    constexpr int MB = Lt::MB, BPW = 256 / MB;
    __shared__ BlockStage<Lt, BPW> st;
    if ((int)threadIdx.x < BPW) {
        const int B = b0 + blockIdx.x * BPW + threadIdx.x;
        st.id[threadIdx.x] = (B < b1 && m.status[B] != ST_INACTIVE) ? B : -1;
    }
    __syncthreads();
    stage_blocks<Lt, BPW>(m, st);
    const int s = threadIdx.x / MB, l = threadIdx.x % MB;
    const int Braw = b0 + blockIdx.x * BPW + s;
    if (Braw >= b1) return;
    double *row = stage + ((int64_t)(Braw - b0) * MB + l) * Q;
    const int B = st.id[s];
    if (B < 0) {
        if (!set)
            for (int p = 0; p < Q; p++) row[p] = 0.0;
        return;
    }
    typename ST::T *f = lp.par[m.level[B]] ? f1 : f0;
    if (set) {
#pragma unroll
        for (int p = 0; p < Q; p++)
            ST::st(f + entry_slot<Lt>(m, st.link[s], B, st.hid[s], p, l), R(row[p] - (ST::shift ? Lt::w(p) : 0.0)));
    } else {
        cell_f64<Lt, ST>(m, st.link[s], B, st.hid[s], l, f, row);
    }
}

// output cells: leaf, non-ghost cells in (block ID, cell) order; kind: cells,
// rho/u, or f.  Entries [k0, k1) of the list of blocks with output cells, one
// block per 64 (2-D: 16) lanes; head receives the first row's number and the
// rows written.  n_list, n_out: the list's length and the rows of all of it.
template <int Q, int S>
__global__ __launch_bounds__(256) void k_out_gather(DevMesh m, const typename Store<S>::T *f0,
                                                    const typename Store<S>::T *f1, LevelParams lp, int kind,
                                                    const int32_t *__restrict__ list, int k0, int k1, int n_list,
                                                    const int32_t *__restrict__ off, int32_t n_out, int64_t *head,
                                                    void *stage) {
    using Lt = Lat<Q>;
    using ST = Store<S>;
    using De = Desc<Lt::D>;
    constexpr int MB = Lt::MB, BPW = 256 / MB;
    __shared__ uint64_t tabs[BPW][kTab<Lt>];
    const int slot = threadIdx.x / MB, l = threadIdx.x % MB;
    int k = k0 + blockIdx.x * BPW + slot;
    if constexpr (Lt::D == 3) k = __builtin_amdgcn_readfirstlane(k);  // one block per wave
    const int32_t off0 = off[list[k0]];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        head[0] = off0;
        head[1] = (k1 < n_list ? off[list[k1]] : n_out) - off0;
    }
    if (k >= k1) return;
    const int B = list[k];
    const int32_t w = desc_word<Lt>(m.desc, B, l);
    const uint64_t full = MB == 64 ? ~0ull : ((1ull << MB) - 1);
    const uint64_t outm = ~desc_ghost<Lt>(w) & full;
    const int64_t pos = (int64_t)off[B] - off0 + __popcll(outm & ((1ull << l) - 1));
    const bool out = (outm >> l) & 1ull;
    if (kind == AMR_FIELD_CELLS) {
        int32_t *o = (int32_t *)stage + 2 * pos;
        if (out) {
            o[0] = B;
            o[1] = l;
        }
        return;
    }
    const int L = (int)((uint32_t)desc_get<Lt>(w, De::kFlags) >> 16);
    double fv[Q];
    cell_f64_desc<Lt, ST>(m, tabs[slot], w, B, l, lp.par[L] ? f1 : f0, fv);
    if (!out) return;
    if (kind == AMR_FIELD_RHO_U) {
        double rho = 0.0, j[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int p = 0; p < Q; p++) {
            rho += fv[p];
            j[0] += fv[p] * Lt::cx(p);
            j[1] += fv[p] * Lt::cy(p);
            j[2] += fv[p] * Lt::cz(p);
        }
        double *o = (double *)stage + 4 * pos;
        o[0] = rho;
        o[1] = j[0] / rho;
        o[2] = j[1] / rho;
        o[3] = j[2] / rho;
    } else {
        double *o = (double *)stage + Q * pos;
#pragma unroll
        for (int p = 0; p < Q; p++) o[p] = fv[p];
    }
}

// FP64 mass and momentum of the output cells: fixed-order per-block partials,
// then a single-workgroup fixed-order sum.
//
// Body: the partial of block b + thread / Mb, by its Mb lanes; lane 0 of them
// returns it in v.  A workgroup of 256 threads has no barrier here, and blocks
// that are not leaves (most of the capacity of a mesh that may still grow) cost
// their status only: 41 to 17 us for a 2-D capacity of 3.9e5 blocks.
template <int Q, int S>
__device__ __forceinline__ void mass_block_partial(const DevMesh &m, typename Store<S>::T *f0,
                                                   typename Store<S>::T *f1, const LevelParams &lp,
                                                   uint64_t (*tabs)[kTab<Lat<Q>>], int64_t b, double *v) {
    using Lt = Lat<Q>;
    using ST = Store<S>;
    using De = Desc<Lt::D>;
    constexpr int MB = Lt::MB;
    const int tid = opaque_tid();  // called in a loop: nothing of a cell's addressing is kept across it
    const int slot = tid / MB, l = tid % MB;
    int64_t Bw = b + slot;
    if (Bw >= m.cap || m.status[Bw] != ST_UNREF) Bw = -1;
    int B = (int)Bw;
    if constexpr (Lt::D == 3) B = __builtin_amdgcn_readfirstlane(B);  // one block per wave
    for (int a = 0; a < 4; a++) v[a] = 0.0;
    if (B < 0) return;  // the block's lanes together
    const int32_t w = desc_word<Lt>(m.desc, B, l);
    const int L = (int)((uint32_t)desc_get<Lt>(w, De::kFlags) >> 16);
    double fv[Q];
    cell_f64_desc<Lt, ST>(m, tabs[slot], w, B, l, lp.par[L] ? f1 : f0, fv);
    if (!((desc_ghost<Lt>(w) >> l) & 1ull)) {
        double rho = 0.0, j[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int p = 0; p < Q; p++) {
            rho += fv[p];
            j[0] += fv[p] * Lt::cx(p);
            j[1] += fv[p] * Lt::cy(p);
            j[2] += fv[p] * Lt::cz(p);
        }
        const double vol = 1.0 / double(1 << (Lt::D * L));
        v[0] = vol * rho;
        for (int a = 0; a < 3; a++) v[1 + a] = vol * rho * (j[a] / rho);
    }
#pragma unroll
    for (int off = MB / 2; off > 0; off >>= 1)
        for (int a = 0; a < 4; a++) v[a] += __shfl_xor(v[a], off, 64);
}

template <int Q, int S>
__global__ __launch_bounds__(256) void k_mass_blocks(DevMesh m, typename Store<S>::T *f0, typename Store<S>::T *f1,
                                                     LevelParams lp, double *part4) {
    constexpr int MB = Lat<Q>::MB, BPW = 256 / MB;
    __shared__ uint64_t tabs[BPW][kTab<Lat<Q>>];
    double v[4];
    mass_block_partial<Q, S>(m, f0, f1, lp, tabs, (int64_t)blockIdx.x * BPW, v);
    const int64_t Braw = (int64_t)blockIdx.x * BPW + threadIdx.x / MB;
    if (Braw < m.cap && threadIdx.x % MB == 0)
        for (int a = 0; a < 4; a++) part4[Braw * 4 + a] = v[a];
}

// Fixed-order sums of the per-block partials: each workgroup reduces one chunk
// of kMassChunk blocks and leaves the result in the chunk's first entry (which
// no other workgroup reads); one workgroup then reduces the chunk results.
constexpr int kMassChunk = 4096;

__device__ inline void tree_sum4(double (*s)[256], double *v) {
    for (int a = 0; a < 4; a++) s[a][threadIdx.x] = v[a];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int a = 0; a < 4; a++) s[a][threadIdx.x] += s[a][threadIdx.x + w];
        __syncthreads();
    }
}

static __global__ __launch_bounds__(256) void k_mass_chunks(double *part4, int cap) {
    __shared__ double s[4][256];
    const int64_t b0 = (int64_t)blockIdx.x * kMassChunk;
    const int64_t b1 = b0 + kMassChunk < cap ? b0 + kMassChunk : cap;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t B = b0 + threadIdx.x; B < b1; B += 256)
        for (int a = 0; a < 4; a++) v[a] += part4[B * 4 + a];
    tree_sum4(s, v);  // ends with a barrier: every read of the chunk is done
    if (threadIdx.x < 4) part4[b0 * 4 + threadIdx.x] = s[threadIdx.x][0];
}

static __global__ __launch_bounds__(256) void k_mass_final(const double *part4, int cap, double *out) {
    __shared__ double s[4][256];
    const int nchunk = (cap + kMassChunk - 1) / kMassChunk;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int c = threadIdx.x; c < nchunk; c += 256)
        for (int a = 0; a < 4; a++) v[a] += part4[(int64_t)c * kMassChunk * 4 + a];
    tree_sum4(s, v);
    if (threadIdx.x < 4) out[threadIdx.x] = s[threadIdx.x][0];
}

// The same sums without the arena's per-block partials, for callers that cannot
// allocate: one workgroup per chunk of kMassChunk blocks forms the block
// partials itself, BPW blocks at a time, and adds them in the order the
// per-chunk pass above does (thread t: blocks b0 + t, b0 + t + 256, ...); the
// chunk sums go to `chunks` (kMassStaticChunks entries at most), and the final
// pass is the same as above.  The result equals the arena form bit for bit.
constexpr int kMassStaticChunks = 1024;  // blocks up to 1024 * kMassChunk = 4,194,304

template <int Q, int S>
__global__ __launch_bounds__(256) void k_mass_chunks_direct(DevMesh m, typename Store<S>::T *f0,
                                                            typename Store<S>::T *f1, LevelParams lp,
                                                            double *chunks) {
    constexpr int MB = Lat<Q>::MB, BPW = 256 / MB;
    __shared__ uint64_t tabs[BPW][kTab<Lat<Q>>];
    __shared__ double s_part[256][4];
    __shared__ double s[4][256];
    const int64_t b0 = (int64_t)blockIdx.x * kMassChunk;
    const int t = threadIdx.x;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int r = 0; r < kMassChunk / 256; r++) {
        for (int i = 0; i < 256 / BPW; i++) {
            double v[4];
            mass_block_partial<Q, S>(m, f0, f1, lp, tabs, b0 + 256 * r + BPW * i, v);
            if (t % MB == 0)
                for (int a = 0; a < 4; a++) s_part[BPW * i + t / MB][a] = v[a];
            wave_lds_sync();
        }
        __syncthreads();
        if (b0 + 256 * r + t < m.cap)
            for (int a = 0; a < 4; a++) acc[a] += s_part[t][a];
        __syncthreads();
    }
    tree_sum4(s, acc);
    if (t < 4) chunks[(int64_t)blockIdx.x * 4 + t] = s[t][0];
}

static __global__ __launch_bounds__(256) void k_mass_final_direct(const double *chunks, int cap, double *out) {
    __shared__ double s[4][256];
    const int nchunk = (cap + kMassChunk - 1) / kMassChunk;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int c = threadIdx.x; c < nchunk; c += 256)
        for (int a = 0; a < 4; a++) v[a] += chunks[(int64_t)c * 4 + a];
    tree_sum4(s, v);
    if (threadIdx.x < 4) out[threadIdx.x] = s[threadIdx.x][0];
}

// ---------------------------------------------------------------------------
// Launchers of one (lattice, storage).  Each pair is compiled in a unit of its
// own (AMR_TU_Q, AMR_TU_S; the build lists them), side by side; the unit
// without them holds the dispatch and what depends on neither.
template <int Q, int S>
struct Launch {
    static bool collide_stream(const Ctx &c, const int32_t *list, int n, int L, const LevelParams &lp,
                               const BCParams &bc, bool exchange);
    static bool interp_collide(const Ctx &c, const int32_t *ilist, int ni, const int32_t *clist, int nblk, int L,
                               const LevelParams &lp, const BCParams &bc, bool exchange);
    static void interp(const Ctx &c, const int32_t *list, int n, const LevelParams &lp, int all_cells);
    static void exchange(const Ctx &c, const int32_t *list, int n, int L, const LevelParams &lp);
    static void exchange_batch(hipStream_t stream, const SimDesc *sims, const uint32_t *items, const int32_t *count,
                               int par, int grid);
    static void collide_batch(hipStream_t stream, const SimDesc *sims, const uint32_t *items, const int32_t *count,
                              int L, int par, const BatchShape &s);
    static void interp_batch(hipStream_t stream, const SimDesc *sims, const uint32_t *items, const int32_t *count,
                             int L, int par0, int par1, const BatchShape &s);
    static void average_batch(hipStream_t stream, const SimDesc *sims, const uint32_t *items, const int32_t *count,
                              int L, int par0, int par1, const BatchShape &s);
    static void refresh_neighbours(const Ctx &c, const int32_t *list, int n, const LevelParams &lp);
    static void block_desc(const Ctx &c, int32_t *old);
    static void target_cells(const Ctx &c, const int32_t *moved);
    static void average(const Ctx &c, const int32_t *list, int n, int L, const LevelParams &lp, int all_cells,
                        double *U);
    static void fill_rest(const Ctx &c);
    static void set_rho_u_root(const Ctx &c, const double *ru, int b0, int b1);
    static void velocity(const Ctx &c, const int32_t *list, int n, int L, const LevelParams &lp, bool children);
    static void block_f(const Ctx &c, int set, int b0, int b1, double *stage, const LevelParams &lp);
    static void out_gather(const Ctx &c, int kind, int k0, int k1, int n_list, int32_t n_out, int64_t *head,
                           void *stage, const LevelParams &lp);
    static void mass_blocks(const Ctx &c, const LevelParams &lp);
    static void mass_chunks_direct(const Ctx &c, const LevelParams &lp, double *chunks);
};

static inline int grid_blocks(int64_t nblocks, int mb) {
    const int bpw = 256 / mb;
    return (int)((nblocks + bpw - 1) / bpw);
}

#ifdef AMR_TU_Q

template <int S>
static typename Store<S>::T *buf(const Ctx &c, int k) {
    return (typename Store<S>::T *)c.f[k];
}

// A level sweep whose output exceeds c.stream_bytes (by default half the 256 MB
// Infinity Cache) stores with non-temporal writes.  Smaller levels are still
// cached when the next sweep (or the interpolation and averaging) reads them.
template <int Q, int S>
bool Launch<Q, S>::collide_stream(const Ctx &c, const int32_t *list, int n, int L, const LevelParams &lp,
                                  const BCParams &bc, bool exchange) {
    const int sp = lp.par[L];
    constexpr int bpw = collide_blocks_per_wg<Q, S>();
    const int grid = (n + bpw - 1) / bpw;
    const typename Store<S>::T *src = buf<S>(c, sp);
    typename Store<S>::T *dst = buf<S>(c, 1 - sp);
    const bool nts = (int64_t)n * Q * c.mb * (int64_t)sizeof(typename Store<S>::T) > c.stream_bytes;
    const int tpb = collide_threads<S>();
    const double om = lp.omega[L];
    if constexpr (Q == 27) {
        if (c.coll == AMR_COLLIDE_MRT) {
            if (nts) k_collide_stream<Q, S, true, 1><<<grid, tpb, 0, c.stream>>>(list, n, c.m, src, dst, om, bc, c.s_high);
            else k_collide_stream<Q, S, false, 1><<<grid, tpb, 0, c.stream>>>(list, n, c.m, src, dst, om, bc, c.s_high);
            return false;
        }
        if constexpr (S != AMR_F64) {
            if (c.coll == AMR_COLLIDE_MRT_MFMA) {
                if (nts) k_collide_stream<Q, S, true, 2><<<grid, tpb, 0, c.stream>>>(list, n, c.m, src, dst, om, bc, c.s_high);
                else k_collide_stream<Q, S, false, 2><<<grid, tpb, 0, c.stream>>>(list, n, c.m, src, dst, om, bc, c.s_high);
                return false;
            }
        }
    }
    // The sweep that adds the momentum exchange itself costs no wave per SIMD with
    // streaming stores, and saves a pass over the solid neighbours per sweep: half-size
    // D3Q27 channel, FP16, 36.6 -> 35.4 ms for 32 coarse steps, full size FP32 663 -> 658 for 64.
    if (exchange) {
        if (nts) k_collide_stream<Q, S, true, 0, true><<<grid, tpb, 0, c.stream>>>(list, n, c.m, src, dst, om, bc, om);
        else k_collide_stream<Q, S, false, 0, true><<<grid, tpb, 0, c.stream>>>(list, n, c.m, src, dst, om, bc, om);
        return true;
    }
    if (nts) k_collide_stream<Q, S, true><<<grid, tpb, 0, c.stream>>>(list, n, c.m, src, dst, om, bc, om);
    else k_collide_stream<Q, S, false><<<grid, tpb, 0, c.stream>>>(list, n, c.m, src, dst, om, bc, om);
    return false;
}

template <int Q, int S>
bool Launch<Q, S>::interp_collide(const Ctx &c, const int32_t *ilist, int ni, const int32_t *clist, int nblk, int L,
                                  const LevelParams &lp, const BCParams &bc, bool exchange) {
    constexpr int bpw = collide_blocks_per_wg<Q, S>();
    const int grid = (ni + kInterpPerWg<Lat<Q>> - 1) / kInterpPerWg<Lat<Q>> + (nblk + bpw - 1) / bpw;
    const bool nts = (int64_t)nblk * Q * c.mb * (int64_t)sizeof(typename Store<S>::T) > c.stream_bytes;
    typename Store<S>::T *f0 = buf<S>(c, 0), *f1 = buf<S>(c, 1);
    if (exchange && !nts) {
        if (c.m.interp == AMR_INTERP_CUBIC)
            k_interp_collide<Q, S, false, 1, true><<<grid, 256, 0, c.stream>>>(ilist, ni, clist, nblk, c.m, f0, f1, lp, L, bc);
        else
            k_interp_collide<Q, S, false, 0, true><<<grid, 256, 0, c.stream>>>(ilist, ni, clist, nblk, c.m, f0, f1, lp, L, bc);
        return true;
    }
    if (c.m.interp == AMR_INTERP_CUBIC) {
        if (nts) k_interp_collide<Q, S, true, 1><<<grid, 256, 0, c.stream>>>(ilist, ni, clist, nblk, c.m, f0, f1, lp, L, bc);
        else k_interp_collide<Q, S, false, 1><<<grid, 256, 0, c.stream>>>(ilist, ni, clist, nblk, c.m, f0, f1, lp, L, bc);
    } else {
        if (nts) k_interp_collide<Q, S, true, 0><<<grid, 256, 0, c.stream>>>(ilist, ni, clist, nblk, c.m, f0, f1, lp, L, bc);
        else k_interp_collide<Q, S, false, 0><<<grid, 256, 0, c.stream>>>(ilist, ni, clist, nblk, c.m, f0, f1, lp, L, bc);
    }
    return false;
}

template <int Q, int S>
void Launch<Q, S>::interp(const Ctx &c, const int32_t *list, int n, const LevelParams &lp, int all_cells) {
    const int grid = (n + kInterpPerWg<Lat<Q>> - 1) / kInterpPerWg<Lat<Q>>;
    if (c.m.interp == AMR_INTERP_CUBIC)
        k_interp<Q, S, 1><<<grid, 256, 0, c.stream>>>(list, n, c.m, buf<S>(c, 0), buf<S>(c, 1), lp, all_cells);
    else
        k_interp<Q, S, 0><<<grid, 256, 0, c.stream>>>(list, n, c.m, buf<S>(c, 0), buf<S>(c, 1), lp, all_cells);
}

template <int Q, int S>
void Launch<Q, S>::exchange(const Ctx &c, const int32_t *list, int n, int L, const LevelParams &lp) {
    k_exchange<Q, S><<<grid_blocks(n, c.mb), 256, 0, c.stream>>>(list, n, c.m, buf<S>(c, lp.par[L]));
}

template <int Q, int S>
void Launch<Q, S>::exchange_batch(hipStream_t stream, const SimDesc *sims, const uint32_t *items, const int32_t *count,
                                  int par, int grid) {
    k_exchange_batch<Q, S><<<grid, 256, 0, stream>>>(sims, items, count, par);
}

// Workgroups of a persistent launch: wg_per_cu per compute unit, but no more
// than fit at a time.  The workgroups share the items evenly, so those that
// start only when others have ended would double the launch.
template <typename K>
static int resident(K kernel, int threads) {
    int fit = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&fit, kernel, threads, 0) != hipSuccess || fit < 1) fit = 64;
    return fit;
}
static int persistent_grid(const BatchShape &s, int fit) { return std::max(1, s.n_cu * std::min(s.wg_per_cu, fit)); }

template <int Q, int S, int NT>
static void collide_batch_nt(hipStream_t stream, const SimDesc *sims, const uint32_t *items, const int32_t *count,
                             int L, int par, const BatchShape &s) {
    static const int fit = resident(k_collide_stream_batch<Q, S, NT>, NT);
    const int grid = persistent_grid(s, fit);
    k_collide_stream_batch<Q, S, NT><<<grid, NT, 0, stream>>>(sims, items, count, L, par);
}

template <int Q, int S>
void Launch<Q, S>::collide_batch(hipStream_t stream, const SimDesc *sims, const uint32_t *items, const int32_t *count,
                                 int L, int par, const BatchShape &s) {
    if (s.threads == 64) collide_batch_nt<Q, S, 64>(stream, sims, items, count, L, par, s);
    else if (s.threads == 128) collide_batch_nt<Q, S, 128>(stream, sims, items, count, L, par, s);
    else collide_batch_nt<Q, S, 256>(stream, sims, items, count, L, par, s);
}

template <int Q, int S>
void Launch<Q, S>::interp_batch(hipStream_t stream, const SimDesc *sims, const uint32_t *items, const int32_t *count,
                                int L, int par0, int par1, const BatchShape &s) {
    static const int fit[2] = {resident(k_interp_batch<Q, S, 0>, 256),
                               resident(k_interp_batch<Q, S, 2>, 256)};
    const int grid = persistent_grid(s, fit[s.cubic ? 1 : 0]);
    if (s.cubic) k_interp_batch<Q, S, 2><<<grid, 256, 0, stream>>>(sims, items, count, L, par0, par1);
    else k_interp_batch<Q, S, 0><<<grid, 256, 0, stream>>>(sims, items, count, L, par0, par1);
}

template <int Q, int S>
void Launch<Q, S>::average_batch(hipStream_t stream, const SimDesc *sims, const uint32_t *items, const int32_t *count,
                                 int L, int par0, int par1, const BatchShape &s) {
    static const int fit = resident(k_average_batch<Q, S>, 256);
    const int grid = persistent_grid(s, fit);
    k_average_batch<Q, S><<<grid, 256, 0, stream>>>(sims, items, count, L, par0, par1);
}

template <int Q, int S>
void Launch<Q, S>::refresh_neighbours(const Ctx &c, const int32_t *list, int n, const LevelParams &lp) {
    const int threads = c.dim == 2 ? 64 : 256;
    k_refresh_neighbours<Q, S><<<n, threads, 0, c.stream>>>(list, n, c.m, buf<S>(c, 0), buf<S>(c, 1), lp);
}

// Buffers: mesh changes come between coarse steps, when every level above 0 is
// back in buffer 0; level 0 has no records.
template <int Q, int S>
void Launch<Q, S>::block_desc(const Ctx &c, int32_t *old) {
    k_block_desc<Q, S><<<(c.m.cap + 63) / 64, 256, 0, c.stream>>>(c.m, c.ctr, old, buf<S>(c, 0), buf<S>(c, 1));
}

template <int Q, int S>
void Launch<Q, S>::target_cells(const Ctx &c, const int32_t *moved) {
    const int nrec = moved ? (c.m.cap + 63) / 64 : 0, per = (c.m.cap + 255) / 256;
    k_target_cells<Q, S><<<nrec + per * c.m.lmax, 256, 0, c.stream>>>(c.m, c.iface, c.ctr, moved, nrec, per,
                                                                    buf<S>(c, 0), buf<S>(c, 1));
}

template <int Q, int S>
void Launch<Q, S>::average(const Ctx &c, const int32_t *list, int n, int L, const LevelParams &lp, int all_cells,
                           double *U) {
    const int grid = (int)(((int64_t)n * c.nc + kAvgPerWg<Lat<Q>> - 1) / kAvgPerWg<Lat<Q>>);
    const typename Store<S>::T *src = buf<S>(c, lp.par[L + 1]);
    typename Store<S>::T *dst = buf<S>(c, lp.par[L]);
    if (U) k_average<Q, S, true><<<grid, 256, 0, c.stream>>>(list, n, c.m, src, dst, lp.r_fc[L], 1, U);
    else k_average<Q, S><<<grid, 256, 0, c.stream>>>(list, n, c.m, src, dst, lp.r_fc[L], all_cells, nullptr);
}

template <int Q, int S>
void Launch<Q, S>::fill_rest(const Ctx &c) {
    const int64_t total = c.m.halo_base + (int64_t)c.m.cap * c.m.nh;
    k_fill_rest<Q, S><<<(int)((total + 255) / 256), 256, 0, c.stream>>>(c.m, buf<S>(c, 0), buf<S>(c, 1), total);
}

template <int Q, int S>
void Launch<Q, S>::set_rho_u_root(const Ctx &c, const double *ru, int b0, int b1) {
    k_set_rho_u<Q, S><<<grid_blocks(b1 - b0, c.mb), 256, 0, c.stream>>>(c.m, buf<S>(c, 0), ru, b0, b1);
}

template <int Q, int S>
void Launch<Q, S>::velocity(const Ctx &c, const int32_t *list, int n, int L, const LevelParams &lp, bool children) {
    const int64_t items = children ? (int64_t)n * c.nc : n;
    k_velocity<Q, S><<<grid_blocks(items, c.mb), 256, 0, c.stream>>>(list, n, c.m, buf<S>(c, lp.par[L]), c.U,
                                                                     children ? 1 : 0);
}

template <int Q, int S>
void Launch<Q, S>::block_f(const Ctx &c, int set, int b0, int b1, double *stage, const LevelParams &lp) {
    k_block_f<Q, S><<<grid_blocks(b1 - b0, c.mb), 256, 0, c.stream>>>(c.m, buf<S>(c, 0), buf<S>(c, 1), lp, set, b0, b1,
                                                                      stage);
}

template <int Q, int S>
void Launch<Q, S>::out_gather(const Ctx &c, int kind, int k0, int k1, int n_list, int32_t n_out, int64_t *head,
                              void *stage, const LevelParams &lp) {
    k_out_gather<Q, S><<<grid_blocks(k1 - k0, c.mb), 256, 0, c.stream>>>(
        c.m, buf<S>(c, 0), buf<S>(c, 1), lp, kind, c.outl, k0, k1, n_list, c.off, n_out, head, stage);
}

template <int Q, int S>
void Launch<Q, S>::mass_blocks(const Ctx &c, const LevelParams &lp) {
    k_mass_blocks<Q, S><<<grid_blocks(c.m.cap, c.mb), 256, 0, c.stream>>>(c.m, buf<S>(c, 0), buf<S>(c, 1), lp, c.part4);
}

template <int Q, int S>
void Launch<Q, S>::mass_chunks_direct(const Ctx &c, const LevelParams &lp, double *chunks) {
    const int nchunk = (c.m.cap + kMassChunk - 1) / kMassChunk;
    k_mass_chunks_direct<Q, S><<<nchunk, 256, 0, c.stream>>>(c.m, buf<S>(c, 0), buf<S>(c, 1), lp, chunks);
}

template struct Launch<AMR_TU_Q, AMR_TU_S>;
#else

// X(Q, S) for every lattice and storage
#define AMR_STORAGES(X, Q) X(Q, AMR_F64) X(Q, AMR_F32) X(Q, AMR_F32S) X(Q, AMR_F16S) X(Q, AMR_BF16S)
#define AMR_PAIRS(X) AMR_STORAGES(X, 9) AMR_STORAGES(X, 19) AMR_STORAGES(X, 27)

#define AMR_EXTERN(Qc, Sc) extern template struct Launch<Qc, Sc>;
AMR_PAIRS(AMR_EXTERN)

// calls fn(Launch<Q, S>()) of the run-time lattice and storage
template <typename F>
static void dispatch(int q, int storage, F &&fn) {
    switch (q * 8 + storage) {
#define AMR_CASE(Qc, Sc) case Qc * 8 + Sc: fn(Launch<Qc, Sc>()); break;
        AMR_PAIRS(AMR_CASE)
    default: break;
    }
}

bool launch_collide_stream(const Ctx &c, const int32_t *list, int n, int L, const LevelParams &lp, const BCParams &bc,
                           bool exchange) {
    if (n <= 0) return false;
    bool done = false;
    dispatch(c.q, c.storage, [&](auto l) { done = l.collide_stream(c, list, n, L, lp, bc, exchange); });
    return done;
}

bool launch_interp_collide(const Ctx &c, const int32_t *ilist, int ni, const int32_t *clist, int nblk, int L,
                           const LevelParams &lp, const BCParams &bc, bool exchange) {
    bool done = false;
    dispatch(c.q, c.storage, [&](auto l) { done = l.interp_collide(c, ilist, ni, clist, nblk, L, lp, bc, exchange); });
    return done;
}

void launch_interp(const Ctx &c, const int32_t *list, int n, const LevelParams &lp, int all_cells) {
    if (n <= 0) return;
    dispatch(c.q, c.storage, [&](auto l) { l.interp(c, list, n, lp, all_cells); });
}

void launch_exchange(const Ctx &c, const int32_t *list, int n, int L, const LevelParams &lp) {
    if (n <= 0) return;
    dispatch(c.q, c.storage, [&](auto l) { l.exchange(c, list, n, L, lp); });
}

void launch_exchange_batch(hipStream_t stream, int q, int storage, const SimDesc *sims, const uint32_t *items,
                           const int32_t *count, int par, int grid) {
    dispatch(q, storage, [&](auto l) { l.exchange_batch(stream, sims, items, count, par, grid); });
}

void launch_collide_batch(hipStream_t stream, int q, int storage, const SimDesc *sims, const uint32_t *items,
                          const int32_t *count, int L, int par, const BatchShape &s) {
    dispatch(q, storage, [&](auto l) { l.collide_batch(stream, sims, items, count, L, par, s); });
}

void launch_interp_batch(hipStream_t stream, int q, int storage, const SimDesc *sims, const uint32_t *items,
                         const int32_t *count, int L, int par0, int par1, const BatchShape &s) {
    dispatch(q, storage, [&](auto l) { l.interp_batch(stream, sims, items, count, L, par0, par1, s); });
}

void launch_average_batch(hipStream_t stream, int q, int storage, const SimDesc *sims, const uint32_t *items,
                          const int32_t *count, int L, int par0, int par1, const BatchShape &s) {
    dispatch(q, storage, [&](auto l) { l.average_batch(stream, sims, items, count, L, par0, par1, s); });
}

void launch_batch_items(hipStream_t stream, const SimDesc *sims, int nsims, int lmax, int cap_max, uint32_t *items,
                        int64_t stride, int32_t *counts) {
    if (nsims <= 0 || lmax <= 0) return;
    const int chunks = std::min(64, (cap_max + 255) / 256);
    k_batch_items<<<dim3(chunks, nsims, 3 * lmax), 256, 0, stream>>>(sims, nsims, items, stride, counts);
}

void launch_refresh_neighbours(const Ctx &c, const int32_t *list, int n, const LevelParams &lp) {
    if (n <= 0) return;
    dispatch(c.q, c.storage, [&](auto l) { l.refresh_neighbours(c, list, n, lp); });
    k_clear_fresh<<<(n * c.nc + 255) / 256, 256, 0, c.stream>>>(list, n, c.m, c.nc);
}

void launch_block_desc(const Ctx &c, int32_t *old) {
    dispatch(c.q, c.storage, [&](auto l) { l.block_desc(c, old); });
}

void launch_target_cells(const Ctx &c, const int32_t *moved) {
    dispatch(c.q, c.storage, [&](auto l) { l.target_cells(c, moved); });
}

void launch_average(const Ctx &c, const int32_t *list, int n, int L, const LevelParams &lp, int all_cells, double *U) {
    if (n <= 0) return;
    dispatch(c.q, c.storage, [&](auto l) { l.average(c, list, n, L, lp, all_cells, U); });
}

void launch_fill_rest(const Ctx &c) {
    dispatch(c.q, c.storage, [&](auto l) { l.fill_rest(c); });
}

void launch_set_rho_u_root(const Ctx &c, const double *ru, int b0, int b1) {
    if (b1 <= b0) return;
    dispatch(c.q, c.storage, [&](auto l) { l.set_rho_u_root(c, ru, b0, b1); });
}

void launch_velocity(const Ctx &c, const int32_t *list, int n, int L, const LevelParams &lp, bool children) {
    if (n <= 0) return;
    dispatch(c.q, c.storage, [&](auto l) { l.velocity(c, list, n, L, lp, children); });
}

void launch_vorticity(const Ctx &c, const int32_t *list, int n, int L, const LevelParams &) {
    if (n <= 0) return;
    const double scale = double(1 << L);
    const int grid = grid_blocks(n, c.mb);
    if (c.q == 9) k_vorticity<9><<<grid, 256, 0, c.stream>>>(list, n, c.m, c.U, scale, c.crit, &c.ctr->wmax_bits);
    else if (c.q == 19) k_vorticity<19><<<grid, 256, 0, c.stream>>>(list, n, c.m, c.U, scale, c.crit, &c.ctr->wmax_bits);
    else k_vorticity<27><<<grid, 256, 0, c.stream>>>(list, n, c.m, c.U, scale, c.crit, &c.ctr->wmax_bits);
}

void launch_block_f(const Ctx &c, int set, int b0, int b1, double *stage, const LevelParams &lp) {
    if (b1 <= b0) return;
    dispatch(c.q, c.storage, [&](auto l) { l.block_f(c, set, b0, b1, stage, lp); });
}

void launch_out_gather(const Ctx &c, int kind, int k0, int k1, int n_list, int32_t n_out, int64_t *head, void *stage,
                       const LevelParams &lp) {
    if (k1 <= k0) return;
    dispatch(c.q, c.storage, [&](auto l) { l.out_gather(c, kind, k0, k1, n_list, n_out, head, stage, lp); });
}

void launch_force_sum(const Ctx &c, double *out) { 
    k_force_sum<<<c.m.lmax, 1024, 0, c.stream>>>(c.m.force, c.solidl, c.m.cap, c.ctr, out);
 }

void launch_force_reset(const Ctx &c) {
    const int64_t n = (int64_t)c.m.cap * 3;
    k_force_reset<<<(int)((n + 255) / 256), 256, 0, c.stream>>>(c.m);
}

// The chunk sums' storage: a fixed array in device memory, one copy per GPU
// for the life of the process.  Host code uses the address resolved once per
// device with hipGetSymbolAddress (mass_scratch), never the array's name.
static __device__ __align__(256) double scratch[kMassStaticChunks * 4];

int64_t mass_static_max_blocks() { return (int64_t)kMassStaticChunks * kMassChunk; }

hipError_t mass_scratch(int device, double **ptr) {
    static std::mutex mu;
    static double *addr[kMaxDevices] = {nullptr};
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device) return hipErrorInvalidDevice;  // resolved with its device current
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[device] = (double *)p;
    }
    *ptr = addr[device];
    return hipSuccess;
}

void launch_mass_static(const Ctx &c, const LevelParams &lp, double *chunks, double *out_dev) {
    dispatch(c.q, c.storage, [&](auto l) { l.mass_chunks_direct(c, lp, chunks); });
    k_mass_final_direct<<<1, 256, 0, c.stream>>>(chunks, c.m.cap, out_dev);
}

void launch_mass(const Ctx &c, const LevelParams &lp) {
    dispatch(c.q, c.storage, [&](auto l) { l.mass_blocks(c, lp); });
    k_mass_chunks<<<(c.m.cap + kMassChunk - 1) / kMassChunk, 256, 0, c.stream>>>(c.part4, c.m.cap);
    k_mass_final<<<1, 256, 0, c.stream>>>(c.part4, c.m.cap, c.ctr->mass);
}

#endif  // AMR_TU_Q

}  // namespace amr
