// gfx950 kernels of the layered-stencil PCG.
//
// Stencil mapping.  A workgroup is `by` wavefronts; wavefront row w owns grid
// row j of a tile, and lane q owns `vx` consecutive cells along x, so a
// wavefront covers 64*vx cells of one row with one 16-byte load per lane for
// FP32 vx = 4 and FP64 vx = 2.  Each lane marches up through a chunk of zc
// layers with the values of the layers below, at and above in registers; x
// neighbours come from the adjacent lanes (cross-lane shuffles), y neighbours
// from the rows above and below (cache hits: the same lines the neighbouring
// rows load).
//
// XCD-aware order.  Workgroups are dispatched round-robin over the eight XCDs
// (workgroup b runs on XCD b mod 8), each XCD with its own L2.  Workgroup b is
// given slot s of a banded order: the slots are split into eight contiguous
// bands, one per XCD, and slots are laid out problem by problem, tile row by
// tile row, with the layer chunks of one lateral tile adjacent.  The tiles above
// and below a tile (whose rows it reads as halo) and the chunks sharing its
// boundary layers thus run on the same XCD at about the same time and their
// shared lines hit that XCD's L2.
//
// Batches.  The inner-PCG kernels take an array of problem descriptors (one per
// system and right-hand side); a workgroup finds its problem by binary search
// over the problems' first slots.  A single solve is a batch of one.  Kernel
// arguments depend on the iteration only through its parity, so a chunk of an
// even number of CG iterations can be captured once into a graph and replayed.
//
// Reductions.  Each workgroup reduces its values with wavefront butterflies and
// a fixed-order pass over its wavefronts, and writes one partial per value.
// The next kernel in the stream (or the host) sums a problem's partials in a
// fixed order; every workgroup of the consuming kernel computes the same sum,
// so no grid-wide synchronisation, fence or atomic is needed, and results are
// run-to-run deterministic.
#include "device_util.hpp"

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <mutex>

namespace cuth {
namespace {

template <typename D>
__device__ __forceinline__ int find_prob(const D *probs, int nprob, int slot) {
    int lo = 0, hi = nprob - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (probs[mid].tile0 <= slot) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

struct Lane {
    int lane, i0, j, l0, l1;
    bool act;
};

// Lane coordinates for tile `local` of an operator tiled ntx wide, ntz deep.
template <int VX, typename T>
__device__ __forceinline__ Lane lane_at(const OpView<T> &op, int local, int ntx, int ntz) {
    const int tz = local % ntz;
    const int t = local / ntz;
    const int tx = t % ntx, ty = t / ntx;
    Lane L;
    L.lane = threadIdx.x;
    L.i0 = (tx * kWave + L.lane) * VX;
    L.j = ty * blockDim.y + threadIdx.y;
    L.l0 = tz * op.zc;
    L.l1 = min(op.nz, L.l0 + op.zc);
    L.act = L.i0 < op.nx && L.j < op.ny;
    return L;
}

template <int VX, typename T>
__device__ __forceinline__ Lane lane_of(const OpView<T> &op) {
    return lane_at<VX>(op, xcd_slot(), (op.nx + kWave * VX - 1) / (kWave * VX),
                       (op.nz + op.zc - 1) / op.zc);
}

template <typename T, int VX>
__device__ __forceinline__ Vec<T, VX> f32load(const float *p) {
    const Vec<float, VX> b = vload<float, VX>(p);
    Vec<T, VX> v;
#pragma unroll
    for (int e = 0; e < VX; ++e) v.a[e] = (T)b.a[e];
    return v;
}

// Lateral conductances of a per-cell operator at cell c of layer L for one
// lane: gxp, gyp (to +x, +y), gym (from -y) and gxl (from -x, via the lane to the
// left or a load on lane 0), from the source CS.  Split in two so that a kernel
// can issue the loads (lateral_load) a layer ahead of their use
// (lateral_finish); lateral_coefs does both at once.
//
// Raw loads of one lane: the +x, +y and -y values and the west value.
template <typename T, int VX, int CS>
struct LatRaw {
    Vec<T, VX> xp, yp, ym;
    T xw;
};
template <typename T, int VX>
struct LatRaw<T, VX, CS_F16> {
    Vec<uint16_t, VX> xp, yp, ym;
    uint16_t xw;
};
template <typename T, int VX>
struct LatRaw<T, VX, CS_F32> {
    Vec<float, VX> xp, yp, ym;
    float xw;
};

template <typename T, int VX, int CS>
__device__ __forceinline__ LatRaw<T, VX, CS> lateral_load(const OpView<T> &op, int64_t c, int lane,
                                                          bool act, bool has_l, bool has_s) {
    const int nx = op.nx;
    LatRaw<T, VX, CS> q;
    if constexpr (CS == CS_F16) {
        // FP16-stored lateral conductances.  Every lane loads from an
        // in-bounds cell (inactive lanes sit at cell 0, a missing south or
        // west neighbour falls back to the cell itself) and selects after the
        // promotion: a guarded load with the promotion inside made the
        // compiler wait for each load in turn.
        q.xp = vload<uint16_t, VX>(op.hx + c);
        q.yp = vload<uint16_t, VX>(op.hy + c);
        q.ym = vload<uint16_t, VX>(op.hy + (has_s ? c - nx : c));
        q.xw = gld(op.hx + (has_l ? c - 1 : c));
    } else if constexpr (CS == CS_F32) {
        // FP32-stored lateral conductances, promoted (loads as above)
        q.xp = vload<float, VX>(op.fx + c);
        q.yp = vload<float, VX>(op.fy + c);
        q.ym = vload<float, VX>(op.fy + (has_s ? c - nx : c));
        q.xw = gld(op.fx + (has_l ? c - 1 : c));
    } else {
        // vector loads unguarded as in the column walker (callers discard the
        // terms of a missing neighbour); lane 0's west value guarded
        q.xp = vload<T, VX>(op.gx + c);
        q.yp = vload<T, VX>(op.gy + c);
        q.ym = vload<T, VX>(op.gy + (has_s ? c - nx : c));
        q.xw = (lane == 0 && has_l) ? gld(op.gx + c - 1) : T(0);
    }
    return q;
}

template <typename T, int VX, int CS>
__device__ __forceinline__ void lateral_finish(const LatRaw<T, VX, CS> &q, const LayerCoef<T> &L,
                                               int lane, bool act, bool has_l, bool has_s,
                                               Vec<T, VX> &gxp, Vec<T, VX> &gyp, Vec<T, VX> &gym,
                                               T &gxl) {
    if constexpr (CS == CS_F16 || CS == CS_F32) {
        T west;
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            if constexpr (CS == CS_F16) {
                gxp.a[e] = act ? (T)h16one(q.xp.a[e]) * L.hs : T(0);
                gyp.a[e] = act ? (T)h16one(q.yp.a[e]) * L.hs : T(0);
                gym.a[e] = has_s ? (T)h16one(q.ym.a[e]) * L.hs : T(0);
            } else {
                gxp.a[e] = act ? (T)q.xp.a[e] : T(0);
                gyp.a[e] = act ? (T)q.yp.a[e] : T(0);
                gym.a[e] = has_s ? (T)q.ym.a[e] : T(0);
            }
        }
        // every lane promotes its west value; lane 0 selects it (a branch
        // around the promotion would wait for the load)
        if constexpr (CS == CS_F16) west = has_l ? (T)h16one(q.xw) * L.hs : T(0);
        else west = has_l ? (T)q.xw : T(0);
        gxl = lane_left(gxp.a[VX - 1]);
        gxl = lane == 0 ? west : gxl;
    } else {
        gxp = q.xp;
        gyp = q.yp;
        gym = q.ym;
        gxl = lane_left(gxp.a[VX - 1]);
        if (lane == 0) gxl = q.xw;
    }
}

template <typename T, int VX, int CS>
__device__ __forceinline__ void lateral_coefs(const OpView<T> &op, const LayerCoef<T> &L, int64_t c,
                                              int lane, bool act, bool has_l, bool has_s,
                                              Vec<T, VX> &gxp, Vec<T, VX> &gyp, Vec<T, VX> &gym,
                                              T &gxl) {
    lateral_finish<T, VX, CS>(lateral_load<T, VX, CS>(op, c, lane, act, has_l, has_s), L, lane, act,
                              has_l, has_s, gxp, gyp, gym, gxl);
}

// diag(A) at cell (i, jr, l) from the face conductances of the stencil: the
// sink plus every face that exists (the Jacobi-scaled sweeps).
template <typename T>
__device__ __forceinline__ T jac_diag(const LayerCoef<T> &L, T gm, T gp, T gs, T gn, int i, int nx,
                                      int jr, int ny, int l, int nz) {
    T d = L.sink;
    if (i > 0) d += gm;
    if (i < nx - 1) d += gp;
    if (jr > 0) d += gs;
    if (jr < ny - 1) d += gn;
    if (l > 0) d += L.gzd;
    if (l < nz - 1) d += L.gzu;
    return d;
}

// March the VX cells of one lane through its layers; emit(l, c, x, A x, ex) per
// layer (active lanes only).  XV(q) fetches the raw loads of VX consecutive
// values of the operand starting at cell q and fin(raw) forms the values (by
// default XV returns them and fin is the identity: an operand formed from
// several streams keeps its arithmetic out of XV, so that the loads of the next
// layer can fly while the current one is computed), XS(q) one value, PRE(c)
// whatever else emit needs at cell c (fetched with the layer's loads).  Every lane of the wavefront must call this (the
// x halo comes through cross-lane shuffles), except with CS_CSR.  Two variants
// measured slower on gfx950 and are not used: issuing the next layer's loads
// before computing the current one (more registers, no gain in overlap), and
// guarding the loads with branches instead of selects (about 15 % slower sweeps).
// EDGE_ALL: every lane loads the west and east values (see issue below), for
// an XS with arithmetic, which would otherwise wait for its loads inside the
// branch.  EMIT_ALL: inactive lanes call emit too (emit tests Lane::act
// itself), for an emit whose inputs would otherwise be loaded under the
// branch around it.  XS may likewise return raw loads, which fins forms into
// the value (default: the identity).  pro() runs after the first layer's loads
// are issued and before any is used: the kernel's own prologue (a sum of the
// previous kernel's partials, say) then overlaps them; the march stops at once
// if it returns false.  A pro that the loads depend on cannot be passed here.
struct IdentFin {
    template <typename V>
    __device__ __forceinline__ const V &operator()(const V &v) const { return v; }
};
struct NoPro {
    __device__ __forceinline__ bool operator()() const { return true; }
};

template <typename T, bool PC, int VX, int CS, bool EDGE_ALL = false, bool EMIT_ALL = false,
          typename FV, typename FS,
          typename FP, typename E, typename FX = IdentFin, typename FXS = IdentFin,
          typename PRO = NoPro>
__device__ __forceinline__ void column_pre(const OpView<T> &op, const Lane &ln, FV &&XV, FS &&XS,
                                           FP &&PRE, E &&emit, FX &&fin = FX{},
                                           FXS &&fins = FXS{}, PRO &&pro = PRO{}) {
    const int nx = op.nx, ny = op.ny, nz = op.nz;
    const int64_t plane = (int64_t)nx * ny;
    const bool act = ln.act;
    if constexpr (CS == CS_CSR) {
        // the CSR baseline: each of the lane's rows walks its own entries and
        // gathers the operand at their columns (no neighbour exchange between
        // lanes, so inactive lanes may leave at once)
        if (!pro() || !act) return;
        int64_t c = ln.i0 + (int64_t)nx * ln.j + plane * ln.l0;
        for (int l = ln.l0; l < ln.l1; ++l, c += plane) {
            const Vec<T, VX> xc = fin(XV(c));
            Vec<T, VX> ax;
#pragma unroll
            for (int e = 0; e < VX; ++e) {
                const int k1 = gld(op.csr_ptr + c + e + 1);
                T a = T(0);
                for (int k = gld(op.csr_ptr + c + e); k < k1; ++k)
                    a += (T)gld(op.csr_val + k) * fins(XS(gld(op.csr_col + k)));
                ax.a[e] = a;
            }
            emit(l, c, xc, ax, PRE(c), vzero<T, VX>());
        }
        return;
    }
    const bool has_l = act && ln.i0 > 0, has_r = act && ln.i0 + VX < nx;
    const bool has_s = act && ln.j > 0, has_n = act && ln.j < ny - 1;
    int64_t c = act ? ln.i0 + (int64_t)nx * ln.j + plane * ln.l0 : 0;
    const Vec<T, VX> zero = vzero<T, VX>();
    // All loads of a layer are gathered in one Loads set, issued before any
    // of them is used.  The vector loads are not guarded: a missing neighbour
    // is read at the cell itself and an inactive lane at its own in-bounds
    // cell, and every such value only feeds a term the boundary tests below
    // discard (or a result that is not emitted); a guard costs a branch per
    // load and makes the compiler wait for every load in flight where the
    // branches meet.  Only the edge lanes' west and east values stay guarded
    // (unguarded, they would be 64-lane gathers for two lanes' values).  FP32 operators issue layer l + 1's set while layer l is
    // computed (one layer of software pipelining; measured 2-4 % faster FP32
    // sweeps); FP64 ones issue each set in its own layer (the second set's
    // registers cost FP64 kernels occupancy: 5-16 % slower).  Inactive lanes
    // sit at cells (l - l0) * plane, and a missing neighbour is not loaded,
    // so every address is in bounds.
    using Pre = decltype(PRE(int64_t(0)));
    using Raw = std::decay_t<decltype(XV(int64_t(0)))>;
    using RawS = std::decay_t<decltype(XS(int64_t(0)))>;
    struct Loads {
        Raw xup, xso, xno;
        RawS west, east;
        LatRaw<T, VX, CS> lat;
        Pre pre;
    };
    auto issue = [&](int l, int64_t cc) {
        Loads q;
        q.xup = XV((act && l + 1 < nz) ? cc + plane : cc);
        q.xso = XV(has_s ? cc - nx : cc);
        q.xno = XV(has_n ? cc + nx : cc);
        if constexpr (EDGE_ALL) {
            // every lane loads (at its own cell where it has no such
            // neighbour): XS's arithmetic then waits outside any branch
            q.west = XS((ln.lane == 0 && has_l) ? cc - 1 : cc);
            q.east = XS((ln.lane == kWave - 1 && has_r) ? cc + VX : cc);
        } else {
            q.west = (ln.lane == 0 && has_l) ? XS(cc - 1) : RawS{};
            q.east = (ln.lane == kWave - 1 && has_r) ? XS(cc + VX) : RawS{};
        }
        if constexpr (PC) q.lat = lateral_load<T, VX, CS>(op, cc, ln.lane, act, has_l, has_s);
        q.pre = PRE(cc);
        return q;
    };
    // the column's first two operand values, formed after pro()
    const Raw xdn0 = XV((act && ln.l0 > 0) ? c - plane : c);
    const Raw xc0 = XV(c);
    Vec<T, VX> xdn, xc;
    // layer l's body with its loads already in registers (cur)
    auto layer = [&](int l, int64_t c, const Loads &cur) {
        const LayerCoef<T> L = gldc(op.lc + l);
        const Vec<T, VX> xup = fin(cur.xup), xso = fin(cur.xso), xno = fin(cur.xno);
        const auto &pre = cur.pre;
        T left = lane_left(xc.a[VX - 1]);
        T right = lane_right(xc.a[0]);
        if (ln.lane == 0) left = fins(cur.west);
        if (ln.lane == kWave - 1) right = fins(cur.east);
        Vec<T, VX> gxp, gyp, gym;
        T gxl = T(0);
        if constexpr (PC)
            lateral_finish<T, VX, CS>(cur.lat, L, ln.lane, act, has_l, has_s, gxp, gyp, gym, gxl);
        Vec<T, VX> ax, dg;
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            const int i = ln.i0 + e;
            const T x = xc.a[e];
            const T xl = (e == 0) ? left : xc.a[e > 0 ? e - 1 : 0];
            const T xr = (e == VX - 1) ? right : xc.a[e + 1 < VX ? e + 1 : 0];
            T gm, gp, gs, gn;
            if constexpr (PC) {
                gm = (e == 0) ? gxl : gxp.a[e > 0 ? e - 1 : 0];
                gp = gxp.a[e];
                gs = gym.a[e];
                gn = gyp.a[e];
            } else {
                gm = gp = L.gx;
                gs = gn = L.gy;
            }
            // A x in difference form and the diagonal of A (sink plus the
            // conductances of the faces that exist), for the Jacobi scaling.
            // Terms of missing neighbours add exactly zero without a test:
            // per-cell conductances, the +x one is 0 on the last column and
            // lane 0's west conductance and value are 0 on the first; a
            // missing y or z neighbour was loaded at the cell itself.  With
            // per-layer conductances only a lane's edge cells can miss an x
            // neighbour (vx divides nx), so the test is the lane's has_l /
            // has_r, one select per side instead of one per cell.
            T a = L.sink * x;
            if (PC || e > 0 || has_l) a += gm * (x - xl);
            if (PC || e < VX - 1 || has_r) a += gp * (x - xr);
            a += gs * (x - xso.a[e]);
            a += gn * (x - xno.a[e]);
            a += L.gzd * (x - xdn.a[e]);
            a += L.gzu * (x - xup.a[e]);
            ax.a[e] = a;
            dg.a[e] = jac_diag(L, gm, gp, gs, gn, i, nx, ln.j, ny, l, nz);
        }
        if (EMIT_ALL || act) emit(l, c, xc, ax, pre, dg);
        xdn = xc;
        xc = xup;
    };
    if constexpr (sizeof(T) == 4) {
        // two sets alternate (unrolled by hand: a copy from one set to the
        // other would make the wavefront wait for the loads in flight), and
        // the last layer is peeled, so that no prefetch sits under a branch
        // (where the two paths meet, the compiler would wait for it)
        Loads qa, qb;
        int l = ln.l0;
        if (l < ln.l1) qa = issue(l, c);
        if (!pro()) return;
        xdn = fin(xdn0);
        xc = fin(xc0);
        while (l < ln.l1) {
            if (l + 1 >= ln.l1) {
                layer(l, c, qa);
                break;
            }
            qb = issue(l + 1, c + plane);
            layer(l, c, qa);
            ++l;
            c += plane;
            if (l + 1 >= ln.l1) {
                layer(l, c, qb);
                break;
            }
            qa = issue(l + 1, c + plane);
            layer(l, c, qb);
            ++l;
            c += plane;
        }
    } else {
        if (!pro()) return;
        xdn = fin(xdn0);
        xc = fin(xc0);
        for (int l = ln.l0; l < ln.l1; ++l, c += plane) layer(l, c, issue(l, c));
    }
}

struct NoEx {};

template <typename T, bool PC, int VX, typename FV, typename FS, typename E>
__device__ __forceinline__ void column(const OpView<T> &op, const Lane &ln, FV &&XV, FS &&XS,
                                       E &&emit) {
    column_pre<T, PC, VX, CS_OWN>(
        op, ln, XV, XS, [](int64_t) { return NoEx{}; },
        [&](int l, int64_t c, const Vec<T, VX> &x, const Vec<T, VX> &ax, const NoEx &,
            const Vec<T, VX> &) { emit(l, c, x, ax); });
}

// Elementwise march over the cells of one lane (no stencil).
template <typename T, int VX, typename E>
__device__ __forceinline__ void cells(const OpView<T> &op, const Lane &ln, E &&emit) {
    if (!ln.act) return;
    const int64_t plane = (int64_t)op.nx * op.ny;
    int64_t c = ln.i0 + (int64_t)op.nx * ln.j + plane * ln.l0;
    for (int l = ln.l0; l < ln.l1; ++l, c += plane) emit(l, c);
}

// ------------------------------------------------------------------ apply
template <typename T, bool PC, int VX, bool H16>
__global__ __launch_bounds__(512) void k_apply(OpView<T> op, const T *__restrict__ x,
                                               T *__restrict__ y) {
    const Lane ln = lane_of<VX>(op);
    column_pre<T, PC, VX, H16 ? CS_F16 : CS_OWN>(
        op, ln, [&](int64_t q) { return vload<T, VX>(x + q); }, [&](int64_t q) { return gld(x + q); },
        [](int64_t) { return NoEx{}; },
        [&](int, int64_t c, const Vec<T, VX> &, const Vec<T, VX> &ax, const NoEx &,
            const Vec<T, VX> &) { vstore<T, VX>(y + c, ax); });
}

// ---------------------------------------------------- batched Chebyshev sweep
// MODE 1: z_1 = r/theta and z_0 = 0 implicit; 2: z_{j-1} = r/theta implicit;
// 0: z_{j-1} read; 3: z_1 read (written by the scale pass) and z_0 = 0.  JAC:
// the sweep of the Jacobi-scaled operator (beyond the paper): the residual term
// is multiplied by 1/diag(A), z_{j+1} = z_j + c1 (z_j - z_{j-1}) + c2 D^{-1} (r - A z_j)
// (modes 0 and 3 only: its z_1 = D^{-1} r/theta needs the neighbours' diagonal).
template <typename T, bool PC, int VX, int MODE, bool LAST, bool CHK, int CS, bool JAC>
__global__ __launch_bounds__(512) void k_cheb_b(const InnerProb<T> *__restrict__ probs, int nprob,
                                                int j, int zsel, const T *__restrict__ part_in,
                                                int red, T *__restrict__ part_out) {
    const int slot = xcd_slot();
    const int pidx = find_prob(probs, nprob, slot);
    const InnerProb<T> &P = probs[pidx];
    CgState<T> *st = P.st;
    // the sweep's constants are fetched together with the stop flag
    const T inv_th = P.cheb[0], c1 = P.cheb[1 + j], c2 = P.cheb[1 + P.kcap + j];
    const int done = st->done;
    if constexpr (!CHK) {
        if (done) return;
    }
    // the convergence test after a CG update (CHK) runs inside the march, once
    // the first layer's loads are in flight; its partial sums are fetched while
    // the stop flag is in flight too
    bool go = true;
    auto prologue = [&]() {
        if constexpr (CHK) {
            const bool stop = conv_test(st, part_in, red, pidx, P, !done && slot == P.tile0);
            go = !(done || stop);
        }
        return go;
    };
    const OpView<T> op = P.op;
    const Lane ln = lane_at<VX>(op, slot - P.tile0, P.ntx, P.ntz);
    const T *__restrict__ r = P.r;
    const T *__restrict__ z = P.z[zsel & 3];
    T *zo = P.z[zsel >> 2];
    T acc[1] = {T(0)};
    // (mode 1 scales r by 1/theta where the values are used, not at the load)
    auto XV = [&](int64_t q) -> Vec<T, VX> { return vload<T, VX>((MODE == 1 ? r : z) + q); };
    auto fin = [&](const Vec<T, VX> &v) -> Vec<T, VX> {
        if constexpr (MODE == 1) {
            Vec<T, VX> w;
#pragma unroll
            for (int e = 0; e < VX; ++e) w.a[e] = v.a[e] * inv_th;
            return w;
        } else {
            return v;
        }
    };
    auto XS = [&](int64_t q) -> T { return gld((MODE == 1 ? r : z) + q); };
    auto fins = [&](T v) -> T {
        if constexpr (MODE == 1) return v * inv_th;
        else return v;
    };
    struct Ex {
        Vec<T, VX> r, zm;
    };
    auto PRE = [&](int64_t c) {
        Ex e;
        e.r = vload<T, VX>(r + c);
        if constexpr (MODE == 0) e.zm = vload<T, VX>(zo + c);
        else e.zm = vzero<T, VX>();
        return e;
    };
    column_pre<T, PC, VX, CS>(op, ln, XV, XS, PRE,
                      [&](int, int64_t c, const Vec<T, VX> &zj, const Vec<T, VX> &az, const Ex &ex,
                          const Vec<T, VX> &dg) {
                          const Vec<T, VX> &rc = ex.r;
                          const Vec<T, VX> &zm = ex.zm;
                          Vec<T, VX> zn;
#pragma unroll
                          for (int e = 0; e < VX; ++e) {
                              T m;
                              if constexpr (MODE == 0) m = zm.a[e];
                              else if constexpr (MODE == 2) m = rc.a[e] * inv_th;
                              else m = T(0);
                              T res = rc.a[e] - az.a[e];
                              if constexpr (JAC) res *= recip(dg.a[e]);
                              zn.a[e] = zj.a[e] + c1 * (zj.a[e] - m) + c2 * res;
                              if constexpr (LAST) acc[0] += rc.a[e] * zn.a[e];
                          }
                          vstore<T, VX>(zo + c, zn);
                      },
                      fin, fins, prologue);
    if (!go) return;   // the same for every wavefront of the workgroup
    if constexpr (LAST) block_partials<T, 1>(acc, 0u, part_out, gridDim.x, slot);
}

// ------------------------------------------- fused pair of Chebyshev sweeps
// Sweeps j and j+1 of the two-term recurrence in one pass over HBM (temporal
// blocking, possible because every sweep's constants are fixed in advance):
//   z_{j+1} = z_j + c1_j (z_j - z_{j-1}) + c2_j (r - A z_j)
//   z_{j+2} = z_{j+1} + c1_{j+1} (z_{j+1} - z_j) + c2_{j+1} (r - A z_{j+1})
// A workgroup owns R whole grid rows (wavefront w holds row slot w / wpr and x
// segment w % wpr) and a chunk of layers.  Stage A marches up through the chunk
// plus one halo layer below and above, computing z_{j+1} on the R rows plus one
// halo row on each side into a ring of three layers in LDS; stage B, one layer
// behind, computes z_{j+2} on the R rows with every neighbour of z_{j+1} from the
// ring (x and y) or from registers (z).  Halo rows and layers are recomputed by
// the neighbouring workgroups with the same arithmetic.  One barrier per layer:
// stage A of layer l writes ring slot l % 3 while stage B of layer l - 1 (other
// wavefronts) reads slot (l - 1) % 3, and slot (l + 1) % 3 was last read before
// the previous barrier.  JAC: both sweeps of the Jacobi-scaled operator (the
// residual terms times 1/diag(A), as k_cheb_b).
template <typename T, bool PC, int VX, int CS, bool JAC>
__global__ __launch_bounds__(1024) void k_cheb2_b(const InnerProb<T> *__restrict__ probs, int nprob,
                                                  int j, int zsel, int R, int zcf, int wpr) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    T *ring = reinterpret_cast<T *>(lds_raw);
    const int slot = xcd_slot();
    int lo = 0, hi = nprob - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (probs[mid].f_tile0 <= slot) lo = mid;
        else hi = mid - 1;
    }
    const InnerProb<T> &P = probs[lo];
    if (P.st->done) return;   // the same for every wavefront of the workgroup
    const OpView<T> op = P.op;
    const int nx = op.nx, ny = op.ny, nz = op.nz;
    const int64_t plane = (int64_t)nx * ny;
    const int ntzf = (nz + zcf - 1) / zcf;
    const int W = wpr * kWave * VX;            // ring row length (cells)
    const int nwx = fused_windows(nx, VX, wpr, 2);
    const int hc = nwx > 1 ? fused_halo_lanes(VX, 2) * VX : 0;   // halo cells per side
    const int local = slot - P.f_tile0;
    const int tz = local % ntzf, tx = (local / ntzf) % nwx, ty = local / ntzf / nwx;
    // a wavefront is one threadIdx.y (64 lanes along x): its row slot and x
    // segment are wave-uniform, so the ring row addresses stay scalar
    const int lane = threadIdx.x, w = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int rs = w / wpr, sg = w % wpr;
    const int RR = R + 2;                      // ring rows
    const int xo = (sg * kWave + lane) * VX;   // this lane's first cell in the window (ring row)
    const int xg = tx * (W - 2 * hc) - hc + xo;   // ... and in the grid row
    const int jr = ty * R - 1 + rs;            // grid row of this wavefront
    const bool act = jr >= 0 && jr < ny && xg >= 0 && xg < nx;
    const bool own = act && xo >= hc && xo < W - hc;   // cells this window writes
    const bool inner = act && rs >= 1 && rs <= R;
    const int l0 = tz * zcf, l1 = min(nz, l0 + zcf);
    const int la0 = max(0, l0 - 1), la1 = min(nz, l1 + 1);
    const bool has_l = act && xg > 0, has_r = act && xg + VX < nx;
    const bool has_s = act && jr > 0, has_n = act && jr < ny - 1;
    // x neighbours of the stage-B input in the ring: a halo lane at the
    // window's edge has none there (its stage-B values are not written, and no
    // written value depends on them)
    const bool ring_l = has_l && xo > 0, ring_r = has_r && xo + VX < W;
    const T c1a = P.cheb[1 + j], c2a = P.cheb[1 + P.kcap + j];
    const T c1b = P.cheb[2 + j], c2b = P.cheb[2 + P.kcap + j];
    const T *__restrict__ zN = P.z[zsel & 3];
    const T *__restrict__ zP = P.z[(zsel >> 2) & 3];
    T *__restrict__ zX = P.z[(zsel >> 4) & 3];
    T *__restrict__ zY = P.z[(zsel >> 6) & 3];
    const T *__restrict__ r = P.r;
    const Vec<T, VX> zero = vzero<T, VX>();
    auto ring_at = [&](int l, int row) -> T * { return ring + ((size_t)((l % 3) * RR + row)) * W; };

    int64_t c = act ? xg + (int64_t)nx * jr + plane * la0 : 0;
    Vec<T, VX> xdn = vload<T, VX>(zN + ((act && la0 > 0) ? c - plane : c));
    Vec<T, VX> xc = vload<T, VX>(zN + c);
    // previous layer's values kept for stage B
    Vec<T, VX> zA_m1 = zero, zA_m2 = zero, r_m1 = zero, gxp_m1 = zero, gyp_m1 = zero,
               gym_m1 = zero;
    T gxl_m1 = T(0);
    // stage B: z_{j+2} at layer lb = l - 1 of this lane's cell (cl is its cell
    // at layer l), from the ring (x and y neighbours), the registers of the
    // layers below and the stage-A result `up` of layer l
    auto stage_b = [&](int l, int64_t cl, const Vec<T, VX> &up) {
        const int lb = l - 1;
        if (!(inner && lb >= l0 && lb < l1)) return;
        const LayerCoef<T> L = gldc(op.lc + lb);
        const T *rowc = ring_at(lb, rs);
        // a y neighbour outside the grid is read at the row itself, so its
        // term vanishes (the ring rows beyond the grid hold no values)
        const Vec<T, VX> so = lds_load<T, VX>(ring_at(lb, jr > 0 ? rs - 1 : rs) + xo);
        const Vec<T, VX> no = lds_load<T, VX>(ring_at(lb, jr < ny - 1 ? rs + 1 : rs) + xo);
        const T left = ring_l ? rowc[xo - 1] : T(0);
        const T right = ring_r ? rowc[xo + VX] : T(0);
        const Vec<T, VX> &y = zA_m1;
        Vec<T, VX> z2;
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            const int i = xg + e;
            const T x = y.a[e];
            const T xl = (e == 0) ? left : y.a[e > 0 ? e - 1 : 0];
            const T xr = (e == VX - 1) ? right : y.a[e + 1 < VX ? e + 1 : 0];
            T gm, gp, gs, gn;
            if constexpr (PC) {
                gm = (e == 0) ? gxl_m1 : gxp_m1.a[e > 0 ? e - 1 : 0];
                gp = gxp_m1.a[e];
                gs = gym_m1.a[e];
                gn = gyp_m1.a[e];
            } else {
                gm = gp = L.gx;
                gs = gn = L.gy;
            }
            // y terms: see the loads above; z terms: gzd is zero on the
            // bottom layer and gzu on the top one, where the neighbour
            // registers hold zeros
            T a = L.sink * x;
            if (PC || e > 0 || has_l) a += gm * (x - xl);   // (see the column walker)
            if (PC || e < VX - 1 || has_r) a += gp * (x - xr);
            a += gs * (x - so.a[e]);
            a += gn * (x - no.a[e]);
            a += L.gzd * (x - zA_m2.a[e]);
            a += L.gzu * (x - up.a[e]);
            T res = r_m1.a[e] - a;
            if constexpr (JAC) res *= recip(jac_diag(L, gm, gp, gs, gn, i, nx, jr, ny, lb, nz));
            z2.a[e] = x + c1b * (x - xdn.a[e]) + c2b * res;   // xdn: z_j at layer lb
        }
        if (own) vstore<T, VX>(zY + cl - plane, z2);
    };
    // the loop holds every stage A (the last layer, with stage B only, is
    // peeled below, so no value needs a placeholder)
    for (int l = la0; l < la1; ++l, c += plane) {
        Vec<T, VX> zn, rv, gxp = zero, gyp = zero, gym = zero, xup;
        T gxl = T(0);
        // ---- stage A: z_{j+1} at layer l
        const LayerCoef<T> L = gldc(op.lc + l);
        // every load of the layer is issued before the first use
        // (unguarded, at in-bounds cells: see the column walker)
        xup = vload<T, VX>(zN + ((act && l + 1 < nz) ? c + plane : c));
        const Vec<T, VX> xso = vload<T, VX>(zN + (has_s ? c - nx : c));
        const Vec<T, VX> xno = vload<T, VX>(zN + (has_n ? c + nx : c));
        const T west = (lane == 0 && has_l) ? gld(zN + c - 1) : T(0);
        const T east = (lane == kWave - 1 && has_r) ? gld(zN + c + VX) : T(0);
        [[maybe_unused]] LatRaw<T, VX, CS> lat;
        if constexpr (PC) lat = lateral_load<T, VX, CS>(op, c, lane, act, has_l, has_s);
        rv = vload<T, VX>(r + c);
        const Vec<T, VX> zm = vload<T, VX>(zP + c);
        T left = lane_left(xc.a[VX - 1]);
        T right = lane_right(xc.a[0]);
        if (lane == 0) left = west;
        if (lane == kWave - 1) right = east;
        if constexpr (PC) {
            lateral_finish<T, VX, CS>(lat, L, lane, act, has_l, has_s, gxp, gyp, gym, gxl);
            // in an x window the lane at x = 0 need not be lane 0: its west
            // conductance came from an inactive lane and must vanish
            if (nwx > 1 && !has_l) gxl = T(0);
        }
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            const int i = xg + e;
            const T x = xc.a[e];
            const T xl = (e == 0) ? left : xc.a[e > 0 ? e - 1 : 0];
            const T xr = (e == VX - 1) ? right : xc.a[e + 1 < VX ? e + 1 : 0];
            T gm, gp, gs, gn;
            if constexpr (PC) {
                gm = (e == 0) ? gxl : gxp.a[e > 0 ? e - 1 : 0];
                gp = gxp.a[e];
                gs = gym.a[e];
                gn = gyp.a[e];
            } else {
                gm = gp = L.gx;
                gs = gn = L.gy;
            }
            // a missing y or z neighbour was loaded at the cell itself, so
            // its term vanishes without a test
            T a = L.sink * x;
            if (PC || e > 0 || has_l) a += gm * (x - xl);   // (see the column walker)
            if (PC || e < VX - 1 || has_r) a += gp * (x - xr);
            a += gs * (x - xso.a[e]);
            a += gn * (x - xno.a[e]);
            a += L.gzd * (x - xdn.a[e]);
            a += L.gzu * (x - xup.a[e]);
            T res = rv.a[e] - a;
            if constexpr (JAC) res *= recip(jac_diag(L, gm, gp, gs, gn, i, nx, jr, ny, l, nz));
            // lanes outside the grid compute finite values from in-bounds
            // loads; no stage B reads them (see its loads)
            zn.a[e] = x + c1a * (x - zm.a[e]) + c2a * res;
        }
        lds_store<T, VX>(ring_at(l, rs) + xo, zn);
        if (inner && own && l >= l0 && l < l1) vstore<T, VX>(zX + c, zn);
        __syncthreads();
        stage_b(l, c, zn);
        // shift the layer registers
        zA_m2 = zA_m1;
        zA_m1 = zn;
        r_m1 = rv;
        gxp_m1 = gxp;
        gyp_m1 = gyp;
        gym_m1 = gym;
        gxl_m1 = gxl;
        xdn = xc;
        xc = xup;
    }
    // stage B of layer la1 - 1: it runs only when la1 = nz, where its
    // up-neighbour term does not exist
    __syncthreads();
    stage_b(la1, c, zero);
}

// ----------------------------------------- fused triple of Chebyshev sweeps
// Sweeps j, j+1 and j+2 in one pass over HBM, the pair's scheme with a third
// stage.  A workgroup owns R whole grid rows (wavefront w holds row slot
// w / wpr, grid row ty R - 2 + slot) and a chunk of layers.  Stage A computes
// z_{j+1} on all R + 4 row slots, over the chunk plus two halo layers below
// and above, into ring A (three layers); stage B, one layer behind, computes
// z_{j+2} on slots 1 .. R + 2 into ring B (three layers); stage C, two layers
// behind, computes z_{j+3} on the R owned slots 2 .. R + 1.  B and C take the
// x and y neighbours of their input from the ring and the z neighbours from
// registers.  z_{j+1} never reaches HBM: the launch reads z_j, z_{j-1}, r (and
// the conductances) and writes z_{j+2} (zX) and z_{j+3} (zY), the two iterates
// the next sweep reads.  One barrier per layer: before it, stage A of layer l
// writes ring A slot l % 3; after it, stage B of layer l - 1 reads ring A slot
// (l - 1) % 3 and writes ring B slot (l - 1) % 3, and stage C of layer l - 2
// reads ring B slot (l - 2) % 3 (written before the barrier).  Every slot is
// written again only after a barrier that follows its last read.  A y neighbour outside
// the grid is read at the cell's own slot, so its term vanishes; ring rows
// outside the grid are never read.  JAC: the sweeps of the Jacobi-scaled
// operator (the residual terms times 1/diag(A), as k_cheb_b).  M2: the triple
// starts at j = 2 of the plain polynomial, whose z_1 = r / theta is formed from
// r instead of read (as k_cheb_b mode 2).
template <typename T, bool PC, int VX, int CS, bool JAC, bool M2>
__global__ __launch_bounds__(1024) void k_cheb3_b(const InnerProb<T> *__restrict__ probs, int nprob,
                                                  int j, int zsel, int R, int zcf, int wpr) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int slot = xcd_slot();
    int lo = 0, hi = nprob - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (probs[mid].t_tile0 <= slot) lo = mid;
        else hi = mid - 1;
    }
    const InnerProb<T> &P = probs[lo];
    if (P.st->done) return;   // the same for every wavefront of the workgroup
    const OpView<T> op = P.op;
    const int nx = op.nx, ny = op.ny, nz = op.nz;
    const int64_t plane = (int64_t)nx * ny;
    const int ntzf = (nz + zcf - 1) / zcf;
    const int W = wpr * kWave * VX;            // ring row length (cells)
    const int nwx = fused_windows(nx, VX, wpr, 3);
    const int hc = nwx > 1 ? fused_halo_lanes(VX, 3) * VX : 0;   // halo cells per side
    const int local = slot - P.t_tile0;
    const int tz = local % ntzf, tx = (local / ntzf) % nwx, ty = local / ntzf / nwx;
    // a wavefront is one threadIdx.y (64 lanes along x): its row slot and x
    // segment are wave-uniform, so the ring row addresses stay scalar
    const int lane = threadIdx.x, w = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int rs = w / wpr, sg = w % wpr;
    const int RA = R + 4, RB = R + 2;          // ring rows
    T *ringA = reinterpret_cast<T *>(lds_raw);
    T *ringB = ringA + (size_t)3 * RA * W;
    const int xo = (sg * kWave + lane) * VX;   // this lane's first cell in the window (ring row)
    const int xg = tx * (W - 2 * hc) - hc + xo;   // ... and in the grid row
    const int jr = ty * R - 2 + rs;            // grid row of this wavefront
    const bool act = jr >= 0 && jr < ny && xg >= 0 && xg < nx;
    const bool own = act && xo >= hc && xo < W - hc;   // cells this window writes
    const bool rowB = act && rs >= 1 && rs <= R + 2;
    const bool rowC = act && rs >= 2 && rs <= R + 1;
    const int l0 = tz * zcf, l1 = min(nz, l0 + zcf);
    const int la0 = max(0, l0 - 2), la1 = min(nz, l1 + 2);
    const int lb0 = max(0, l0 - 1), lb1 = min(nz, l1 + 1);
    const bool has_l = act && xg > 0, has_r = act && xg + VX < nx;
    const bool has_s = act && jr > 0, has_n = act && jr < ny - 1;
    // x neighbours of the stage-B and stage-C inputs in the rings: a halo lane
    // at the window's edge has none there (see the pair)
    const bool ring_l = has_l && xo > 0, ring_r = has_r && xo + VX < W;
    const T c1a = P.cheb[1 + j], c2a = P.cheb[1 + P.kcap + j];
    const T c1b = P.cheb[2 + j], c2b = P.cheb[2 + P.kcap + j];
    const T c1c = P.cheb[3 + j], c2c = P.cheb[3 + P.kcap + j];
    [[maybe_unused]] const T inv_th = P.cheb[0];
    const T *__restrict__ zN = P.z[zsel & 3];
    const T *__restrict__ zP = P.z[(zsel >> 2) & 3];
    T *__restrict__ zX = P.z[(zsel >> 4) & 3];
    T *__restrict__ zY = P.z[(zsel >> 6) & 3];
    const T *__restrict__ r = P.r;
    const Vec<T, VX> zero = vzero<T, VX>();
    // ring rows of the y neighbours (the own slot outside the grid)
    const int sA = jr > 0 ? rs - 1 : rs, nA = jr < ny - 1 ? rs + 1 : rs;
    auto ringA_at = [&](int l, int row) -> T * { return ringA + ((size_t)((l % 3) * RA + row)) * W; };
    auto ringB_at = [&](int l, int row) -> T * { return ringB + ((size_t)((l % 3) * RB + row - 1)) * W; };

    int64_t c = act ? xg + (int64_t)nx * jr + plane * la0 : 0;
    Vec<T, VX> xdn = vload<T, VX>(zN + ((act && la0 > 0) ? c - plane : c));
    Vec<T, VX> xc = vload<T, VX>(zN + c);
    // stage A results of the two layers below, stage B results of the two
    // layers below its current one, and the inputs the later stages reuse
    Vec<T, VX> zA_m1 = zero, zA_m2 = zero, zB_m1 = zero, zB_m2 = zero;
    Vec<T, VX> r_m1 = zero, r_m2 = zero;
    [[maybe_unused]] Vec<T, VX> gxp_m1 = zero, gyp_m1 = zero, gym_m1 = zero;
    [[maybe_unused]] Vec<T, VX> gxp_m2 = zero, gyp_m2 = zero, gym_m2 = zero;
    [[maybe_unused]] T gxl_m1 = T(0), gxl_m2 = T(0);

    // one stencil sweep at layer ls of this lane's cells: input y (own cells),
    // its x neighbours from ring row `row`, y neighbours from rows so/no,
    // z neighbours dn/up, previous iterate pv, residual input rr
    auto sweep = [&](const T *row, const T *so_row, const T *no_row, int ls, const Vec<T, VX> &y,
                     const Vec<T, VX> &dn, const Vec<T, VX> &up, const Vec<T, VX> &pv,
                     const Vec<T, VX> &rr, const Vec<T, VX> &gxp, const Vec<T, VX> &gyp,
                     const Vec<T, VX> &gym, T gxl, T c1, T c2) {
        const LayerCoef<T> L = gldc(op.lc + ls);
        const Vec<T, VX> so = lds_load<T, VX>(so_row + xo);
        const Vec<T, VX> no = lds_load<T, VX>(no_row + xo);
        const T left = ring_l ? row[xo - 1] : T(0);
        const T right = ring_r ? row[xo + VX] : T(0);
        Vec<T, VX> out;
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            const int i = xg + e;
            const T x = y.a[e];
            const T xl = (e == 0) ? left : y.a[e > 0 ? e - 1 : 0];
            const T xr = (e == VX - 1) ? right : y.a[e + 1 < VX ? e + 1 : 0];
            T gm, gp, gs, gn;
            if constexpr (PC) {
                gm = (e == 0) ? gxl : gxp.a[e > 0 ? e - 1 : 0];
                gp = gxp.a[e];
                gs = gym.a[e];
                gn = gyp.a[e];
            } else {
                gm = gp = L.gx;
                gs = gn = L.gy;
            }
            // the z conductances are zero where dn / up do not exist
            T a = L.sink * x;
            if (PC || e > 0 || has_l) a += gm * (x - xl);   // (see the column walker)
            if (PC || e < VX - 1 || has_r) a += gp * (x - xr);
            a += gs * (x - so.a[e]);
            a += gn * (x - no.a[e]);
            a += L.gzd * (x - dn.a[e]);
            a += L.gzu * (x - up.a[e]);
            T res = rr.a[e] - a;
            if constexpr (JAC) res *= recip(jac_diag(L, gm, gp, gs, gn, i, nx, jr, ny, ls, nz));
            out.a[e] = x + c1 * (x - pv.a[e]) + c2 * res;
        }
        return out;
    };

    // stages B and C after the barrier of iteration l (zn: stage A's layer l,
    // zero in the two closing iterations), then the register shifts
    auto stage_bc = [&](int l, int64_t cl, const Vec<T, VX> &zn, const Vec<T, VX> &rv,
                        const Vec<T, VX> &gxp, const Vec<T, VX> &gyp, const Vec<T, VX> &gym, T gxl,
                        const Vec<T, VX> &xup) {
        // ---- stage B: z_{j+2} at layer l - 1 (zn: stage A's layer above)
        const int lb = l - 1;
        Vec<T, VX> z2 = zero;
        if (rowB && lb >= lb0 && lb < lb1) {
            z2 = sweep(ringA_at(lb, rs), ringA_at(lb, sA), ringA_at(lb, nA), lb, zA_m1, zA_m2, zn, xdn,
                       r_m1, gxp_m1, gyp_m1, gym_m1, gxl_m1, c1b, c2b);
            lds_store<T, VX>(ringB_at(lb, rs) + xo, z2);
            if (rowC && own && lb >= l0 && lb < l1) vstore<T, VX>(zX + cl - plane, z2);
        }
        // ---- stage C: z_{j+3} at layer l - 2 (z2: stage B's layer above)
        const int lc = l - 2;
        if (rowC && lc >= l0 && lc < l1) {
            const Vec<T, VX> z3 =
                sweep(ringB_at(lc, rs), ringB_at(lc, sA), ringB_at(lc, nA), lc, zB_m1, zB_m2, z2,
                      zA_m2, r_m2, gxp_m2, gyp_m2, gym_m2, gxl_m2, c1c, c2c);
            if (own) vstore<T, VX>(zY + cl - 2 * plane, z3);
        }
        // shift the layer registers
        zA_m2 = zA_m1;
        zA_m1 = zn;
        zB_m2 = zB_m1;
        zB_m1 = z2;
        r_m2 = r_m1;
        r_m1 = rv;
        if constexpr (PC) {
            gxp_m2 = gxp_m1;
            gyp_m2 = gyp_m1;
            gym_m2 = gym_m1;
            gxl_m2 = gxl_m1;
            gxp_m1 = gxp;
            gyp_m1 = gyp;
            gym_m1 = gym;
            gxl_m1 = gxl;
        }
        xdn = xc;
        xc = xup;
    };

    // stage A's loads of layer l (at in-bounds cells: see the column walker)
    struct LoadsA {
        Vec<T, VX> xup, xso, xno, rv, zm;
        T west, east;
        LatRaw<T, VX, CS> lat;
    };
    auto issue_a = [&](int l, int64_t cc) {
        LoadsA q;
        q.xup = vload<T, VX>(zN + ((act && l + 1 < nz) ? cc + plane : cc));
        q.xso = vload<T, VX>(zN + (has_s ? cc - nx : cc));
        q.xno = vload<T, VX>(zN + (has_n ? cc + nx : cc));
        // the edge lanes' x neighbours, loaded by every lane at an in-bounds
        // cell (a load under a branch makes the waits at the join conservative,
        // which would hold the prefetched loads)
        const bool wl = lane == 0 && has_l, er = lane == kWave - 1 && has_r;
        q.west = gld(zN + (wl ? cc - 1 : cc));
        q.east = gld(zN + (er ? cc + VX : cc));
        if (!wl) q.west = T(0);
        if (!er) q.east = T(0);
        if constexpr (PC) q.lat = lateral_load<T, VX, CS>(op, cc, lane, act, has_l, has_s);
        q.rv = vload<T, VX>(r + cc);
        if constexpr (M2) {
#pragma unroll
            for (int e = 0; e < VX; ++e) q.zm.a[e] = q.rv.a[e] * inv_th;
        } else {
            q.zm = vload<T, VX>(zP + cc);
        }
        return q;
    };
    // one layer: stage A of layer l from its loads q, then (after the barrier)
    // stages B and C; `next` (when given) receives layer l + 1's loads, issued
    // before the barrier so that they fly during stages B and C
    auto layer = [&](int l, int64_t cc, const LoadsA &q, LoadsA *next) {
        Vec<T, VX> zn, gxp = zero, gyp = zero, gym = zero;
        T gxl = T(0);
        // ---- stage A: z_{j+1} at layer l
        const LayerCoef<T> L = gldc(op.lc + l);
        T left = lane_left(xc.a[VX - 1]);
        T right = lane_right(xc.a[0]);
        if (lane == 0) left = q.west;
        if (lane == kWave - 1) right = q.east;
        if constexpr (PC) {
            lateral_finish<T, VX, CS>(q.lat, L, lane, act, has_l, has_s, gxp, gyp, gym, gxl);
            // in an x window the lane at x = 0 need not be lane 0: its west
            // conductance came from an inactive lane and must vanish
            if (nwx > 1 && !has_l) gxl = T(0);
        }
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            const int i = xg + e;
            const T x = xc.a[e];
            const T xl = (e == 0) ? left : xc.a[e > 0 ? e - 1 : 0];
            const T xr = (e == VX - 1) ? right : xc.a[e + 1 < VX ? e + 1 : 0];
            T gm, gp, gs, gn;
            if constexpr (PC) {
                gm = (e == 0) ? gxl : gxp.a[e > 0 ? e - 1 : 0];
                gp = gxp.a[e];
                gs = gym.a[e];
                gn = gyp.a[e];
            } else {
                gm = gp = L.gx;
                gs = gn = L.gy;
            }
            // missing y and z neighbours were loaded at the cell itself
            T a = L.sink * x;
            if (PC || e > 0 || has_l) a += gm * (x - xl);
            if (PC || e < VX - 1 || has_r) a += gp * (x - xr);
            a += gs * (x - q.xso.a[e]);
            a += gn * (x - q.xno.a[e]);
            a += L.gzd * (x - xdn.a[e]);
            a += L.gzu * (x - q.xup.a[e]);
            T res = q.rv.a[e] - a;
            if constexpr (JAC) res *= recip(jac_diag(L, gm, gp, gs, gn, i, nx, jr, ny, l, nz));
            zn.a[e] = x + c1a * (x - q.zm.a[e]) + c2a * res;
        }
        lds_store<T, VX>(ringA_at(l, rs) + xo, zn);
        if (next) {
            const bool more = l + 1 < la1;
            *next = issue_a(more ? l + 1 : l, more ? cc + plane : cc);
        }
        __syncthreads();
        stage_bc(l, cc, zn, q.rv, gxp, gyp, gym, gxl, q.xup);
    };
    // every iteration of the loop holds a stage A; the two closing layers of
    // stages B and C follow it.  Matrix-free (the per-layer conductances leave
    // registers for a second set of loads): layer l + 1's loads are issued
    // right after layer l's stage A, before the barrier, so that they fly
    // during stages B and C; they are issued unconditionally (the last layer
    // loads its own cells again), since a load under a branch makes the waits
    // where the paths join conservative.  With per-cell conductances a second
    // set would pass the register budget of a 16-wavefront workgroup: each
    // layer issues its own loads, the edge lanes' x neighbours under their
    // lane test (written out in the loop: folding this path into the lambdas
    // above made the compiler reorder its loads and waits, 2-13 % slower)
    int l = la0;
    if constexpr (!PC) {
        LoadsA q = issue_a(l, c);
        for (; l < la1; ++l, c += plane) {
            LoadsA nq;
            layer(l, c, q, &nq);
            q = nq;
        }
    } else {
        for (; l < la1; ++l, c += plane) {
            Vec<T, VX> zn, rv, gxp = zero, gyp = zero, gym = zero;
            T gxl = T(0);
            // ---- stage A: z_{j+1} at layer l
            const LayerCoef<T> L = gldc(op.lc + l);
            const Vec<T, VX> xup = vload<T, VX>(zN + ((act && l + 1 < nz) ? c + plane : c));
            const Vec<T, VX> xso = vload<T, VX>(zN + (has_s ? c - nx : c));
            const Vec<T, VX> xno = vload<T, VX>(zN + (has_n ? c + nx : c));
            const T west = (lane == 0 && has_l) ? gld(zN + c - 1) : T(0);
            const T east = (lane == kWave - 1 && has_r) ? gld(zN + c + VX) : T(0);
            const LatRaw<T, VX, CS> lat = lateral_load<T, VX, CS>(op, c, lane, act, has_l, has_s);
            rv = vload<T, VX>(r + c);
            Vec<T, VX> zm;
            if constexpr (M2) {
#pragma unroll
                for (int e = 0; e < VX; ++e) zm.a[e] = rv.a[e] * inv_th;
            } else {
                zm = vload<T, VX>(zP + c);
            }
            T left = lane_left(xc.a[VX - 1]);
            T right = lane_right(xc.a[0]);
            if (lane == 0) left = west;
            if (lane == kWave - 1) right = east;
            lateral_finish<T, VX, CS>(lat, L, lane, act, has_l, has_s, gxp, gyp, gym, gxl);
            // in an x window the lane at x = 0 need not be lane 0: its west
            // conductance came from an inactive lane and must vanish
            if (nwx > 1 && !has_l) gxl = T(0);
#pragma unroll
            for (int e = 0; e < VX; ++e) {
                const int i = xg + e;
                const T x = xc.a[e];
                const T xl = (e == 0) ? left : xc.a[e > 0 ? e - 1 : 0];
                const T xr = (e == VX - 1) ? right : xc.a[e + 1 < VX ? e + 1 : 0];
                const T gm = (e == 0) ? gxl : gxp.a[e > 0 ? e - 1 : 0];
                const T gp = gxp.a[e], gs = gym.a[e], gn = gyp.a[e];
                // per-cell conductances: the terms of missing neighbours vanish
                T a = L.sink * x;
                a += gm * (x - xl);
                a += gp * (x - xr);
                a += gs * (x - xso.a[e]);
                a += gn * (x - xno.a[e]);
                a += L.gzd * (x - xdn.a[e]);
                a += L.gzu * (x - xup.a[e]);
                T res = rv.a[e] - a;
                if constexpr (JAC) res *= recip(jac_diag(L, gm, gp, gs, gn, i, nx, jr, ny, l, nz));
                zn.a[e] = x + c1a * (x - zm.a[e]) + c2a * res;
            }
            lds_store<T, VX>(ringA_at(l, rs) + xo, zn);
            __syncthreads();
            stage_bc(l, c, zn, rv, gxp, gyp, gym, gxl, xup);
        }
    }
    for (int q = 0; q < 2; ++q, ++l, c += plane) {
        __syncthreads();
        stage_bc(l, c, zero, zero, zero, zero, zero, T(0), zero);
    }
}

// Single-pass preconditioners, partials of r^T z:
//   PM_SCALE   z = r / theta (the Chebyshev polynomial of degree 1);
//   PM_JACOBI  z = r / diag(A), diag = sink + the sum of the cell's face
//              conductances (the Jacobi-PCG baseline of Section 5, Ablation III);
//   PM_NONE    z = r (plain CG);
//   PM_JCHEB   z = D^{-1} r / theta, the first iterate of the Jacobi-scaled
//              Chebyshev preconditioner (beyond the paper; D as for PM_JACOBI,
//              the reciprocal as in its sweeps).
enum PrecMode : int { PM_SCALE = 0, PM_JACOBI = 1, PM_NONE = 2, PM_JCHEB = 3 };

template <typename T, bool PC, int VX, bool CHK, int PM>
__global__ __launch_bounds__(512) void k_scale_b(const InnerProb<T> *__restrict__ probs, int nprob,
                                                 const T *__restrict__ part_in, int red,
                                                 T *__restrict__ part_out) {
    const int slot = xcd_slot();
    const int pidx = find_prob(probs, nprob, slot);
    const InnerProb<T> &P = probs[pidx];
    CgState<T> *st = P.st;
    const int done = st->done;
    if constexpr (CHK) {
        const bool stop = conv_test(st, part_in, red, pidx, P, !done && slot == P.tile0);
        if (done || stop) return;
    } else {
        if (done) return;
    }
    const OpView<T> op = P.op;
    const Lane ln = lane_at<VX>(op, slot - P.tile0, P.ntx, P.ntz);
    const T inv_th = P.cheb[0];
    const T *__restrict__ r = P.r;
    T *__restrict__ z0 = P.z[0];
    T acc[1] = {T(0)};
    const int nx = op.nx, ny = op.ny, nz = op.nz;
    cells<T, VX>(op, ln, [&](int l, int64_t c) {
        const Vec<T, VX> rv = vload<T, VX>(r + c);
        Vec<T, VX> zv;
        [[maybe_unused]] LayerCoef<T> L;
        if constexpr (PM == PM_JACOBI || PM == PM_JCHEB) L = gldc(op.lc + l);
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            if constexpr (PM == PM_SCALE) {
                zv.a[e] = rv.a[e] * inv_th;
            } else if constexpr (PM == PM_JACOBI || PM == PM_JCHEB) {
                const int i = ln.i0 + e;
                T d = L.sink + (l > 0 ? L.gzd : T(0)) + (l < nz - 1 ? L.gzu : T(0));
                if constexpr (PC) {
                    const int64_t q = c + e;
                    d += gld(op.gx + q) + gld(op.gy + q) + (i > 0 ? gld(op.gx + q - 1) : T(0)) +
                         (ln.j > 0 ? gld(op.gy + q - nx) : T(0));
                } else {
                    d += L.gx * (T)((i > 0) + (i < nx - 1)) + L.gy * (T)((ln.j > 0) + (ln.j < ny - 1));
                }
                if constexpr (PM == PM_JACOBI) zv.a[e] = rv.a[e] / d;
                else zv.a[e] = rv.a[e] * inv_th * recip(d);
            } else {
                zv.a[e] = rv.a[e];
            }
            acc[0] += rv.a[e] * zv.a[e];
        }
        vstore<T, VX>(z0 + c, zv);
    });
    block_partials<T, 1>(acc, 0u, part_out, gridDim.x, slot);
}

// ---------------------------------------------- CG: direction + SpMV + p^T A p
template <typename T, bool PC, int VX, int CS>
__global__ __launch_bounds__(512) void k_dir_b(const InnerProb<T> *__restrict__ probs, int nprob,
                                               int par, int zfin, const T *__restrict__ part_in,
                                               int red, T *__restrict__ part_out) {
    const int slot = xcd_slot();
    const int pidx = find_prob(probs, nprob, slot);
    const InnerProb<T> &P = probs[pidx];
    CgState<T> *st = P.st;
    const int done = st->done, gave_up = st->gave_up;
    const T rz_prev = st->rz[1 - par];
    const T rz = prev_sum(part_in, red, pidx, P);
    if (done) return;
    const bool bad = !(rz > T(0)) || !finite_val(rz);
    const bool lead = (slot == P.tile0) && tid_lin() == 0;
    // an on-chip preconditioner that gave up left no z: stop this problem here
    if (gave_up) {
        if (lead) st->done = kResAbort;
        return;
    }
    if (lead) {
        st->rz[par] = rz;
        if (bad) st->done = 4;
    }
    if (bad) return;
    const T beta = isinf(rz_prev) ? T(0) : rz / rz_prev;
    const bool has_p = beta != T(0);
    const T *__restrict__ z = P.z[zfin];
    const T *__restrict__ pold = P.p[1 - par];
    T *__restrict__ pnew = P.p[par];
    T *__restrict__ mu = P.mu;
    const OpView<T> op = P.op;
    const Lane ln = lane_at<VX>(op, slot - P.tile0, P.ntx, P.ntz);
    T acc[1] = {T(0)};
    // With per-cell conductances the operand p = z + beta p_old is formed
    // where the values are used, from the raw loads of z and p_old (p_old read
    // also on the first iteration, where it is not used: no load under a
    // branch), so that the next layer's loads fly during the current one
    // (512x512x16: 21.5 -> 19.2 us).  Matrix-free, the extra registers of the
    // raw set cost more occupancy than the overlap gains (1024x1024x20: 74.6
    // -> 83.8 us), and XV forms p at the load.
    struct Raw {
        Vec<T, VX> z, p;
    };
    auto XV = [&](int64_t q) {
        if constexpr (PC) {
            return Raw{vload<T, VX>(z + q), vload<T, VX>(pold + q)};
        } else {
            Vec<T, VX> v = vload<T, VX>(z + q);
            if (has_p) {
                const Vec<T, VX> p = vload<T, VX>(pold + q);
#pragma unroll
                for (int e = 0; e < VX; ++e) v.a[e] += beta * p.a[e];
            }
            return v;
        }
    };
    auto fin = [&](const auto &w) -> Vec<T, VX> {
        if constexpr (PC) {
            Vec<T, VX> v = w.z;
            if (has_p) {
#pragma unroll
                for (int e = 0; e < VX; ++e) v.a[e] += beta * w.p.a[e];
            }
            return v;
        } else {
            return w;
        }
    };
    auto XS = [&](int64_t q) -> T { return has_p ? gld(z + q) + beta * gld(pold + q) : gld(z + q); };
    column_pre<T, PC, VX, CS>(op, ln, XV, XS, [](int64_t) { return NoEx{}; },
                      [&](int, int64_t c, const Vec<T, VX> &p, const Vec<T, VX> &ap, const NoEx &,
                          const Vec<T, VX> &) {
                          vstore<T, VX>(pnew + c, p);
                          vstore<T, VX>(mu + c, ap);
#pragma unroll
                          for (int e = 0; e < VX; ++e) acc[0] += p.a[e] * ap.a[e];
                      },
                      fin);
    block_partials<T, 1>(acc, 0u, part_out, gridDim.x, slot);
}

// ------------------------------------------------- CG: x += a p, r -= a mu, r^T r
template <typename T, int VX>
__global__ __launch_bounds__(512) void k_update_b(const InnerProb<T> *__restrict__ probs,
                                                  int nprob, int par,
                                                  const T *__restrict__ part_in, int red,
                                                  T *__restrict__ part_out) {
    const int slot = xcd_slot();
    const int pidx = find_prob(probs, nprob, slot);
    const InnerProb<T> &P = probs[pidx];
    CgState<T> *st = P.st;
    const int done = st->done;
    const T rz = st->rz[par], rz_prev = st->rz[1 - par];
    const bool first = isinf(rz_prev);
    const T *__restrict__ p = P.p[par];
    const T *__restrict__ mu = P.mu;
    T *__restrict__ x = P.x;
    T *__restrict__ r = P.r;
    float *__restrict__ r_lo = P.r_lo;
    const OpView<T> op = P.op;
    const Lane ln = lane_at<VX>(op, slot - P.tile0, P.ntx, P.ntz);
    const int64_t plane = (int64_t)op.nx * op.ny;
    // The lane's layers stream through two alternating load sets, the first
    // issued before the partial sums of p^T A p are fetched, so that the
    // stream starts at once and two layers are in flight.  x is read at p on
    // the first iteration, where it is scaled by 0 (x starts at 0): no load
    // depends on a test.  The layer count is the workgroup's, so the loop's
    // branches are uniform; inactive lanes load at in-bounds cells (k planes
    // from cell 0), add nothing and store nothing.
    const T *__restrict__ xsrc = first ? p : x;
    const T keep = first ? T(0) : T(1);
    struct Set {
        Vec<T, VX> p, m, r, x;
    };
    auto issue = [&](int64_t c) {
        Set q;
        q.p = vload<T, VX>(p + c);
        q.m = vload<T, VX>(mu + c);
        q.r = vload<T, VX>(r + c);
        q.x = vload<T, VX>(xsrc + c);
        return q;
    };
    int64_t c = ln.act ? ln.i0 + (int64_t)op.nx * ln.j + plane * ln.l0 : 0;
    const int nl = ln.l1 - ln.l0;
    Set qa = issue(c), qb;
    const T pmu = prev_sum(part_in, red, pidx, P);
    if (done) return;
    const bool bad = !(pmu > T(0)) || !finite_val(pmu);
    if (bad) {
        if (slot == P.tile0 && tid_lin() == 0) st->done = 4;
        return;
    }
    const T alpha = rz / pmu;
    T acc[1] = {T(0)};
    // ALL: every lane of the wavefront is active (every wavefront of a tile
    // inside the grid), so the stores need no test: a store under a branch
    // leaves the loads before it unwaited on the other path, and the compiler
    // then waits for them before reusing their registers
    auto march = [&](auto all_tag) {
        constexpr bool ALL = decltype(all_tag)::value;
        auto layer = [&](int64_t cc, const Set &q) {
            Vec<T, VX> xv, rv;
            Vec<float, VX> rl;
#pragma unroll
            for (int e = 0; e < VX; ++e) {
                // the same contractions as an unmasked x += a p, r -= a mu,
                // acc += r r (one rounding each): the mask scales a factor
                xv.a[e] = keep * q.x.a[e];
                xv.a[e] += alpha * q.p.a[e];
                rv.a[e] = q.r.a[e] - alpha * q.m.a[e];
                const T rm = (ALL || ln.act) ? rv.a[e] : T(0);
                acc[0] += rm * rv.a[e];
                rl.a[e] = (float)rv.a[e];
            }
            if (ALL || ln.act) {
                vstore<T, VX>(x + cc, xv);
                vstore<T, VX>(r + cc, rv);
                if (r_lo) vstore<float, VX>(r_lo + cc, rl);
            }
        };
        // unrolled by hand as in the column walker (a copy between the sets
        // would make the wavefront wait for the loads in flight); every set
        // is issued, the one after the last layer at the current layer (an
        // L2 hit), since a load under a branch makes the compiler wait for
        // all loads where the paths meet
        for (int k = 0; k < nl; k += 2, c += 2 * plane) {
            if (k + 1 >= nl) {
                layer(c, qa);
                break;
            }
            qb = issue(c + plane);
            layer(c, qa);
            qa = issue(k + 2 < nl ? c + 2 * plane : c);
            layer(c + plane, qb);
        }
    };
    if (__all(ln.act)) march(std::true_type{});
    else march(std::false_type{});
    block_partials<T, 1>(acc, 0u, part_out, gridDim.x, slot);
}

// z = (T) z_lo (the FP32 preconditioner's result promoted) into z[0], with
// partials of r^T z in T (the inner products of the FP64 CG stay FP64).
template <typename T, int VX>
__global__ __launch_bounds__(512) void k_promote_dot(const InnerProb<T> *__restrict__ probs,
                                                     int nprob, T *__restrict__ part_out) {
    const int slot = xcd_slot();
    const int pidx = find_prob(probs, nprob, slot);
    const InnerProb<T> &P = probs[pidx];
    if (P.st->done) return;
    // (as in k_dir_b)
    if (P.gave_up_lo && *P.gave_up_lo) {
        if (slot == P.tile0 && tid_lin() == 0) P.st->done = kResAbort;
        return;
    }
    const float *__restrict__ zl = P.z_lo;
    const T *__restrict__ r = P.r;
    T *__restrict__ z = P.z[0];
    const OpView<T> op = P.op;
    const Lane ln = lane_at<VX>(op, slot - P.tile0, P.ntx, P.ntz);
    T acc[1] = {T(0)};
    cells<T, VX>(op, ln, [&](int, int64_t c) {
        const Vec<T, VX> zv = f32load<T, VX>(zl + c);
        const Vec<T, VX> rv = vload<T, VX>(r + c);
#pragma unroll
        for (int e = 0; e < VX; ++e) acc[0] += rv.a[e] * zv.a[e];
        vstore<T, VX>(z + c, zv);
    });
    block_partials<T, 1>(acc, 0u, part_out, gridDim.x, slot);
}

// One workgroup per problem: r^T r from the update's partials, the convergence
// test (rr <= tol2), and the stop flag mirrored to the FP32 preconditioner's
// state (*done_lo) so its sweeps exit early too.
template <typename T>
__global__ __launch_bounds__(256) void k_reduce_conv(const InnerProb<T> *__restrict__ probs,
                                                     const T *__restrict__ part_in) {
    const InnerProb<T> &P = probs[blockIdx.x];
    CgState<T> *st = P.st;
    const int done = st->done;
    const T tol2 = st->tol2;
    const T rr = reduce_prev(part_in + P.tile0, P.ntiles);
    if (tid_lin() != 0) return;
    if (done) {
        if (P.done_lo) *P.done_lo = done;
        return;
    }
    const bool stop = !(rr > tol2) || !finite_val(rr);
    st->rr = rr;
    st->iter = st->iter + 1;
    if (stop) {
        st->done = finite_val(rr) ? 1 : 4;
        if (P.done_lo) *P.done_lo = st->done;
    }
}

// Per-problem fixed-order sum of the previous kernel's partials (one workgroup
// per problem), for launches with many workgroups per problem: the consumer
// then reads one value instead of every workgroup summing every partial.
template <typename T>
__global__ __launch_bounds__(256) void k_reduce_b(const InnerProb<T> *__restrict__ probs,
                                                  const T *__restrict__ part_in,
                                                  T *__restrict__ red_out) {
    const InnerProb<T> &P = probs[blockIdx.x];
    const T s = reduce_prev(part_in + P.tile0, P.ntiles);
    if (tid_lin() == 0) red_out[blockIdx.x] = s;
}

// Per-problem totals of the FP64 outer residual's partials (sums of ||r||^2,
// ||b||^2 and the non-finite count, maxima of |delta| and |theta|), one
// workgroup per problem in a fixed order: the host reads five values per
// problem instead of every workgroup's (about 1 MB at 21 M unknowns, summed on
// the host while the device waited).
constexpr int kReduceOuterWaves = 16;   // wavefronts of a k_reduce_outer workgroup

template <typename TD, typename TI>
__global__ __launch_bounds__(1024) void k_reduce_outer(const OuterProb<TD, TI> *__restrict__ probs,
                                                       const double *__restrict__ part, int ntot,
                                                       double *__restrict__ out) {
    const OuterProb<TD, TI> &P = probs[blockIdx.x];
    constexpr int NV = kResidualValues, U = 4;
    // value v is a maximum (non-negative: exact in any order) for |delta| and
    // |theta|, else a sum (fixed order: per thread, then across lanes and
    // wavefronts)
    auto is_max = [](int v) { return v == 2 || v == 3; };
    const int n = nthreads(), np = P.ntiles;
    const double *base = part + P.tile0;
    double acc[NV][U];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int u = 0; u < U; ++u) acc[v][u] = 0.0;
    // U x NV independent loads in flight per thread and round
    int q = tid_lin();
    for (; q + (U - 1) * n < np; q += U * n) {
        double x[NV][U];
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int u = 0; u < U; ++u) x[v][u] = base[(size_t)v * ntot + q + u * n];
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int u = 0; u < U; ++u)
                acc[v][u] = is_max(v) ? fmax(acc[v][u], x[v][u]) : acc[v][u] + x[v][u];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool in = q + u * n < np;
        const int qq = in ? q + u * n : 0;   // in-bounds load, discarded when out
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const double x = np > 0 ? base[(size_t)v * ntot + qq] : 0.0;
            if (in) acc[v][u] = is_max(v) ? fmax(acc[v][u], x) : acc[v][u] + x;
        }
    }
    __shared__ double sh[NV][kReduceOuterWaves];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        double a = acc[v][0];
#pragma unroll
        for (int u = 1; u < U; ++u) a = is_max(v) ? fmax(a, acc[v][u]) : a + acc[v][u];
        a = is_max(v) ? wave_max(a) : wave_sum(a);
        if (threadIdx.x == 0) sh[v][threadIdx.y] = a;
    }
    __syncthreads();
    if (tid_lin() < NV) {
        const int v = tid_lin();
        double s = sh[v][0];
        for (int w = 1; w < (int)blockDim.y; ++w) s = is_max(v) ? fmax(s, sh[v][w]) : s + sh[v][w];
        out[(size_t)blockIdx.x * NV + v] = s;
    }
}

// ----------------------------------------------------- CG: true residual check
template <typename T, bool PC, int VX, int CS>
__global__ __launch_bounds__(512) void k_check_b(const InnerProb<T> *__restrict__ probs, int nprob,
                                                 T *__restrict__ part_out) {
    const int slot = xcd_slot();
    const InnerProb<T> &P = probs[find_prob(probs, nprob, slot)];
    const bool have_x = P.st->iter > 0;
    const OpView<T> op = P.op;
    const Lane ln = lane_at<VX>(op, slot - P.tile0, P.ntx, P.ntz);
    const T *__restrict__ x = P.x;
    const T *__restrict__ rhat = P.rhat;
    const T *__restrict__ rlow = P.r;
    T acc[2] = {T(0), T(0)};
    struct Ex {
        Vec<T, VX> rh, rr;
    };
    column_pre<T, PC, VX, CS>(
        op, ln,
        [&](int64_t q) { return have_x ? vload<T, VX>(x + q) : vzero<T, VX>(); },
        [&](int64_t q) { return have_x ? gld(x + q) : T(0); },
        [&](int64_t c) { return Ex{vload<T, VX>(rhat + c), vload<T, VX>(rlow + c)}; },
        [&](int, int64_t c, const Vec<T, VX> &, const Vec<T, VX> &ax, const Ex &ex,
            const Vec<T, VX> &) {
            const Vec<T, VX> &rh = ex.rh, &rr = ex.rr;
#pragma unroll
            for (int e = 0; e < VX; ++e) {
                const T rt = rh.a[e] - ax.a[e];
                const T d = rt - rr.a[e];
                acc[0] += rt * rt;
                acc[1] += d * d;
            }
        });
    block_partials<T, 2>(acc, 0u, part_out, gridDim.x, slot);
}

// ------------------------------------------------------- FP64 outer residual
// FL fixes at compile time which streams exist, so that no load sits under a
// branch (the compiler would wait for each such load in turn): bit 0 theta_in,
// bit 1 delta, bit 2 T_n, bit 3 r64 is the only output (else theta_out, r_in
// and rhat are).  FL = -1 tests the pointers at run time (a launch whose
// problems differ).
template <bool PC, int VX, typename TD, typename TI, int FL>
__global__ __launch_bounds__(512) void k_residual_b(const OuterProb<TD, TI> *__restrict__ probs,
                                                    int nprob, double *__restrict__ part_out) {
    const int slot = xcd_slot();
    const OuterProb<TD, TI> &P = probs[find_prob(probs, nprob, slot)];
    const OpView<double> op = P.op;
    const Lane ln = lane_at<VX>(op, slot - P.tile0, P.ntx, P.ntz);
    const double *__restrict__ th_in = P.th_in;
    const TD *__restrict__ delta = P.delta;
    const double *__restrict__ pw = P.P;
    const double *__restrict__ tn = P.Tn;
    double *__restrict__ th_out = P.th_out;
    double *__restrict__ r64 = P.r64;
    TI *__restrict__ r_in = P.r_in;
    TI *__restrict__ rhat = P.rhat;
    const double in_off = P.in_off, tn_off = P.tn_off;
    constexpr bool RT = FL < 0;
    const bool has_th = RT ? th_in != nullptr : (FL & 1) != 0;
    const bool has_d = RT ? delta != nullptr : (FL & 2) != 0;
    const bool has_tn = RT ? tn != nullptr : (FL & 4) != 0;
    const bool w_th = RT ? th_out != nullptr : (FL & 8) == 0;
    const bool w_r64 = RT ? r64 != nullptr : (FL & 8) != 0;
    const bool w_rin = RT ? r_in != nullptr : (FL & 8) == 0;
    double acc[kResidualValues] = {0.0, 0.0, 0.0, 0.0, 0.0};
    // theta = theta_in - in_off + delta: the loads (XV) and the sum (fin)
    // apart, so that a layer's loads are all in flight before the first sum
    struct RawX {
        Vec<double, VX> th;
        Vec<TD, VX> d;
    };
    auto XV = [&](int64_t q) {
        RawX v;
        v.th = has_th ? vload<double, VX>(th_in + q) : vzero<double, VX>();
        v.d = has_d ? vload<TD, VX>(delta + q) : vzero<TD, VX>();
        return v;
    };
    auto fin = [&](const RawX &v) {
        Vec<double, VX> x;
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            x.a[e] = has_th ? v.th.a[e] - in_off : 0.0;
            if (has_d) x.a[e] += (double)v.d.a[e];
        }
        return x;
    };
    auto XS = [&](int64_t q) -> double {
        const double t = has_th ? gld(th_in + q) : 0.0;
        const double d = has_d ? (double)gld(delta + q) : 0.0;
        double v = has_th ? t - in_off : 0.0;
        if (has_d) v += d;
        return v;
    };
    // the cell's own streams, fetched with the layer's stencil loads
    struct PreR {
        Vec<double, VX> pv, tv;
        Vec<TD, VX> dv;
    };
    auto PRE = [&](int64_t c) {
        PreR q;
        q.pv = vload<double, VX>(pw + c);
        q.tv = has_tn ? vload<double, VX>(tn + c) : vzero<double, VX>();
        q.dv = has_d ? vload<TD, VX>(delta + c) : vzero<TD, VX>();
        return q;
    };
    column_pre<double, PC, VX, CS_OWN, !RT, !RT>(
        op, ln, XV, XS, PRE,
        [&](int l, int64_t c, const Vec<double, VX> &th, const Vec<double, VX> &ath, const PreR &pr,
            const Vec<double, VX> &) {
            // with FL >= 0 every lane comes here (inactive ones at in-bounds
            // cells) and adds zeros, so that the layer's loads stay unguarded
            const bool act = ln.act;
            const double cap = gldc(op.lc + l).cap;
            Vec<double, VX> rv;
            Vec<TI, VX> rl;
#pragma unroll
            for (int e = 0; e < VX; ++e) {
                double b = pr.pv.a[e];
                if (has_tn) b += cap * (pr.tv.a[e] - tn_off);
                const double rc = b - ath.a[e];
                rv.a[e] = rc;
                rl.a[e] = (TI)rc;
                // masked factors keep the sums' contractions (one rounding
                // per term, as unmasked)
                acc[0] += (act ? rc : 0.0) * rc;
                acc[1] += (act ? b : 0.0) * b;
                if (has_d) acc[2] = fmax(acc[2], act ? fabs((double)pr.dv.a[e]) : 0.0);
                acc[3] = fmax(acc[3], act ? fabs(th.a[e]) : 0.0);
                acc[4] += (act && !isfinite(rc)) ? 1.0 : 0.0;
            }
            if (act) {
                if (w_th) vstore<double, VX>(th_out + c, th);
                if (w_r64) vstore<double, VX>(r64 + c, rv);
                if (w_rin) {
                    vstore<TI, VX>(r_in + c, rl);
                    vstore<TI, VX>(rhat + c, rl);
                }
            }
        },
        fin);
    block_partials<double, kResidualValues>(acc, (1u << 2) | (1u << 3), part_out, gridDim.x, slot);
}

// CSR fill: one thread per cell writes its row (neighbours below, south, west,
// the cell, east, north, above: ascending columns); off-diagonals -g, the
// diagonal sink + the sum of the face conductances (as the stencil's rows).
__global__ __launch_bounds__(256) void k_csr_fill(OpView<double> op, const int *__restrict__ ptr,
                                                  int *__restrict__ col, double *__restrict__ val) {
    const int nx = op.nx, ny = op.ny, nz = op.nz;
    const int64_t plane = (int64_t)nx * ny, n = plane * nz;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += stride) {
        const int i = (int)(c % nx), j = (int)((c / nx) % ny), l = (int)(c / plane);
        const LayerCoef<double> L = op.lc[l];
        const bool pc = op.gx != nullptr;
        const double gw = i > 0 ? (pc ? op.gx[c - 1] : L.gx) : 0.0;
        const double ge = i < nx - 1 ? (pc ? op.gx[c] : L.gx) : 0.0;
        const double gs = j > 0 ? (pc ? op.gy[c - nx] : L.gy) : 0.0;
        const double gn = j < ny - 1 ? (pc ? op.gy[c] : L.gy) : 0.0;
        const double gd = l > 0 ? L.gzd : 0.0, gu = l < nz - 1 ? L.gzu : 0.0;
        int k = ptr[c];
        if (l > 0) { col[k] = (int)(c - plane); val[k++] = -gd; }
        if (j > 0) { col[k] = (int)(c - nx); val[k++] = -gs; }
        if (i > 0) { col[k] = (int)(c - 1); val[k++] = -gw; }
        col[k] = (int)c;
        val[k++] = L.sink + gd + gs + gw + ge + gn + gu;
        if (i < nx - 1) { col[k] = (int)(c + 1); val[k++] = -ge; }
        if (j < ny - 1) { col[k] = (int)(c + nx); val[k++] = -gn; }
        if (l < nz - 1) { col[k] = (int)(c + plane); val[k++] = -gu; }
    }
}

// Row-wise CSR product, one thread per row (the Ablation I baseline).
__global__ __launch_bounds__(256) void k_csr_spmv(int64_t n, const int *__restrict__ ptr,
                                                  const int *__restrict__ col,
                                                  const double *__restrict__ val,
                                                  const double *__restrict__ x,
                                                  double *__restrict__ y) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    double a = 0.0;
    for (int k = ptr[r]; k < ptr[r + 1]; ++k) a += val[k] * x[col[k]];
    y[r] = a;
}

__global__ __launch_bounds__(256) void k_to_f32(int64_t n, const double *__restrict__ x,
                                                float *__restrict__ y) {
    const int64_t stride = (int64_t)gridDim.x * nthreads();
    for (int64_t q = (int64_t)blockIdx.x * nthreads() + tid_lin(); q < n; q += stride)
        y[q] = (float)x[q];
}

__global__ __launch_bounds__(256) void k_add_scalar(int64_t n, const double *__restrict__ x,
                                                    double a, double *__restrict__ y) {
    const int64_t stride = (int64_t)gridDim.x * nthreads();
    for (int64_t q = (int64_t)blockIdx.x * nthreads() + tid_lin(); q < n; q += stride)
        y[q] = x[q] + a;
}

// ------------------------------------------------------ coefficient build
__global__ __launch_bounds__(256) void k_build_lateral(
    int nx, int ny, int nz, double dx, double dy, const double *__restrict__ dz,
    const double *__restrict__ k_lat, const double *__restrict__ mult, double *__restrict__ gx64,
    double *__restrict__ gy64, float *__restrict__ gx32, float *__restrict__ gy32,
    unsigned int *bad) {
    const int i = blockIdx.x * kWave + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    if (i >= nx || j >= ny) return;
    const int64_t plane = (int64_t)nx * ny;
    int64_t c = i + (int64_t)nx * j;
    for (int l = 0; l < nz; ++l, c += plane) {
        const double kl = k_lat[l], d = dz[l];
        const double m = mult[c];
        if (!(m > 0.0) || !isfinite(m)) atomicAdd(bad, 1u);
        const double ka = kl * m;
        double gx = 0.0, gy = 0.0;
        // series half-cell conductance across the +x and +y faces
        if (i < nx - 1) gx = (dy * d) / (dx / (2.0 * ka) + dx / (2.0 * (kl * mult[c + 1])));
        if (j < ny - 1) gy = (dx * d) / (dy / (2.0 * ka) + dy / (2.0 * (kl * mult[c + nx])));
        gx64[c] = gx;
        gy64[c] = gy;
        gx32[c] = (float)gx;
        gy32[c] = (float)gy;
    }
}

// Per-layer max over cells of the lateral off-diagonal row sum and of a single
// lateral conductance (after the planes exist).  Positive doubles order like
// their bit patterns, so an integer max of the patterns is the max.
__global__ __launch_bounds__(256) void k_lateral_rowmax(int nx, int ny, int nz,
                                                        const double *__restrict__ gx,
                                                        const double *__restrict__ gy,
                                                        unsigned long long *maxrow,
                                                        unsigned long long *maxg) {
    const int i = blockIdx.x * kWave + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const bool act = (i < nx && j < ny);
    const int64_t plane = (int64_t)nx * ny;
    for (int l = 0; l < nz; ++l) {
        double s = 0.0, m = 0.0;
        if (act) {
            const int64_t c = i + (int64_t)nx * j + plane * l;
            s = gx[c] + gy[c] + (i > 0 ? gx[c - 1] : 0.0) + (j > 0 ? gy[c - nx] : 0.0);
            m = fmax(gx[c], gy[c]);
        }
        s = wave_max(s);
        m = wave_max(m);
        if (threadIdx.x == 0) {
            atomicMax(&maxrow[l], (unsigned long long)__double_as_longlong(s));
            atomicMax(&maxg[l], (unsigned long long)__double_as_longlong(m));
        }
    }
}

// FP16 copies of the lateral planes at the per-layer power-of-two scale.
__global__ __launch_bounds__(256) void k_build_fp16(int nx, int ny, int nz,
                                                    const double *__restrict__ gx,
                                                    const double *__restrict__ gy,
                                                    const double *__restrict__ scale,
                                                    uint16_t *__restrict__ hx,
                                                    uint16_t *__restrict__ hy) {
    const int i = blockIdx.x * kWave + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    if (i >= nx || j >= ny) return;
    const int64_t plane = (int64_t)nx * ny;
    int64_t c = i + (int64_t)nx * j;
    for (int l = 0; l < nz; ++l, c += plane) {
        const double sc = scale[l];
        const _Float16 a = (_Float16)(float)(gx[c] * sc);
        const _Float16 b = (_Float16)(float)(gy[c] * sc);
        hx[c] = __builtin_bit_cast(uint16_t, a);
        hy[c] = __builtin_bit_cast(uint16_t, b);
    }
}

// --------------------------------------------------------------- Lanczos
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    // SplitMix64 (Steele, Lea, Flood 2014): counter-based, one output per index.
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

__global__ __launch_bounds__(256) void k_fill_random(int64_t n, uint64_t seed,
                                                     float *__restrict__ v) {
    const int64_t stride = (int64_t)gridDim.x * nthreads();
    for (int64_t q = (int64_t)blockIdx.x * nthreads() + tid_lin(); q < n; q += stride) {
        const uint64_t h = splitmix64(seed ^ (uint64_t)q * 0xD1B54A32D192ED03ull);
        // uniform in [-1, 1) from the top 24 bits
        v[q] = (float)((double)(h >> 40) * (2.0 / 16777216.0) - 1.0);
    }
}

__global__ __launch_bounds__(256) void k_norm2(int64_t n, const float *__restrict__ v,
                                               float *__restrict__ part_out) {
    float acc[1] = {0.f};
    const int64_t stride = (int64_t)gridDim.x * nthreads();
    for (int64_t q = (int64_t)blockIdx.x * nthreads() + tid_lin(); q < n; q += stride)
        acc[0] += v[q] * v[q];
    block_partials<float, 1>(acc, 0u, part_out, gridDim.x, blockIdx.x);
}

__global__ __launch_bounds__(256) void k_scale_rsqrt(int64_t n, const float *__restrict__ v,
                                                     const float *__restrict__ part_in,
                                                     int np_in, float *__restrict__ out) {
    const float s = 1.0f / sqrtf(reduce_prev(part_in, np_in));
    const int64_t stride = (int64_t)gridDim.x * nthreads();
    for (int64_t q = (int64_t)blockIdx.x * nthreads() + tid_lin(); q < n; q += stride)
        out[q] = v[q] * s;
}

// dis = D^{-1/2}, D = diag(A) = sink + the conductances of the faces that
// exist, per cell of an FP64 operator (one thread per cell).
__global__ __launch_bounds__(256) void k_jacobi_dis(OpView<double> op, float *__restrict__ dis) {
    const int nx = op.nx, ny = op.ny, nz = op.nz;
    const int64_t plane = (int64_t)nx * ny, n = plane * nz;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n;
         q += (int64_t)gridDim.x * blockDim.x) {
        const int l = (int)(q / plane);
        const int64_t rem = q - (int64_t)l * plane;
        const int j = (int)(rem / nx), i = (int)(rem - (int64_t)j * nx);
        const LayerCoef<double> L = op.lc[l];
        const bool pc = op.gx != nullptr;
        double d = L.sink;
        if (l > 0) d += L.gzd;
        if (l < nz - 1) d += L.gzu;
        if (i > 0) d += pc ? op.gx[q - 1] : L.gx;
        if (i < nx - 1) d += pc ? op.gx[q] : L.gx;
        if (j > 0) d += pc ? op.gy[q - nx] : L.gy;
        if (j < ny - 1) d += pc ? op.gy[q] : L.gy;
        dis[q] = (float)(1.0 / sqrt(d));
    }
}

template <bool PC, int VX, bool SC>
__global__ __launch_bounds__(512) void k_lanczos_av(OpView<float> op, int j,
                                                    const float *__restrict__ v,
                                                    const float *__restrict__ vprev,
                                                    const float *__restrict__ lz,
                                                    const float *__restrict__ dis,
                                                    float *__restrict__ w,
                                                    float *__restrict__ part_out) {
    // SC: the operator is D^{-1/2} A D^{-1/2} (dis = D^{-1/2} per cell; the
    // interval of the Jacobi-scaled preconditioner)
    const float bp = j > 0 ? lz[256 + j - 1] : 0.f;
    const Lane ln = lane_of<VX>(op);
    float acc[1] = {0.f};
    column<float, PC, VX>(
        op, ln,
        [&](int64_t q) {
            Vec<float, VX> x = vload<float, VX>(v + q);
            if constexpr (SC) {
                const Vec<float, VX> s = vload<float, VX>(dis + q);
#pragma unroll
                for (int e = 0; e < VX; ++e) x.a[e] *= s.a[e];
            }
            return x;
        },
        [&](int64_t q) {
            if constexpr (SC) return gld(v + q) * gld(dis + q);
            else return gld(v + q);
        },
        [&](int, int64_t c, const Vec<float, VX> &xv, const Vec<float, VX> &av) {
            Vec<float, VX> wc;
            Vec<float, VX> pv = vzero<float, VX>();
            if (j > 0) pv = vload<float, VX>(vprev + c);
            Vec<float, VX> vc = xv, s;
            if constexpr (SC) {
                vc = vload<float, VX>(v + c);
                s = vload<float, VX>(dis + c);
            }
#pragma unroll
            for (int e = 0; e < VX; ++e) {
                const float a = SC ? s.a[e] * av.a[e] : av.a[e];
                wc.a[e] = a - bp * pv.a[e];
                acc[0] += vc.a[e] * wc.a[e];
            }
            vstore<float, VX>(w + c, wc);
        });
    block_partials<float, 1>(acc, 0u, part_out, gridDim.x, xcd_slot());
}

__global__ __launch_bounds__(256) void k_lanczos_orth(int64_t n, int j, float *__restrict__ w,
                                                      const float *__restrict__ v,
                                                      float *__restrict__ lz,
                                                      const float *__restrict__ part_in,
                                                      int np_in, float *__restrict__ part_out) {
    const float a = reduce_prev(part_in, np_in);
    if (blockIdx.x == 0 && tid_lin() == 0) lz[j] = a;
    float acc[1] = {0.f};
    const int64_t stride = (int64_t)gridDim.x * nthreads();
    for (int64_t q = (int64_t)blockIdx.x * nthreads() + tid_lin(); q < n; q += stride) {
        const float wc = w[q] - a * v[q];
        w[q] = wc;
        acc[0] += wc * wc;
    }
    block_partials<float, 1>(acc, 0u, part_out, gridDim.x, blockIdx.x);
}

__global__ __launch_bounds__(256) void k_lanczos_div(int64_t n, int j, float *__restrict__ w,
                                                     float *__restrict__ lz,
                                                     const float *__restrict__ part_in,
                                                     int np_in) {
    const float b = sqrtf(reduce_prev(part_in, np_in));
    if (blockIdx.x == 0 && tid_lin() == 0) lz[256 + j] = b;
    const float s = 1.0f / b;
    const int64_t stride = (int64_t)gridDim.x * nthreads();
    for (int64_t q = (int64_t)blockIdx.x * nthreads() + tid_lin(); q < n; q += stride) w[q] *= s;
}

// --------------------------------------------------------------- adjoint
template <bool PC>
__global__ __launch_bounds__(256) void k_adjoint_sums(OpView<double> op,
                                                      const double *__restrict__ lam,
                                                      const double *__restrict__ T, double t_amb,
                                                      double *__restrict__ part) {
    __shared__ double sh[kMaxBY][2 * kMaxLayers];
    const int i = blockIdx.x % ((op.nx + kWave - 1) / kWave) * kWave + threadIdx.x;
    const int j = blockIdx.x / ((op.nx + kWave - 1) / kWave) * blockDim.y + threadIdx.y;
    const int lane = threadIdx.x, w = threadIdx.y;
    const bool act = (i < op.nx && j < op.ny);
    const int nz = op.nz, nx = op.nx, ny = op.ny;
    const int64_t plane = (int64_t)nx * ny;
    int64_t c = act ? i + (int64_t)nx * j : 0;
    for (int l = 0; l < nz; ++l, c += plane) {
        const LayerCoef<double> L = op.lc[l];
        double slat = 0.0, svert = 0.0;
        if (act) {
            const double la = lam[c], th = T[c] - t_amb;
            if (i < nx - 1) {
                const double g = PC ? op.gx[c] : L.gx;
                slat += g * (la - lam[c + 1]) * (th - (T[c + 1] - t_amb));
            }
            if (j < ny - 1) {
                const double g = PC ? op.gy[c] : L.gy;
                slat += g * (la - lam[c + nx]) * (th - (T[c + nx] - t_amb));
            }
            if (l < nz - 1) svert = (la - lam[c + plane]) * (th - (T[c + plane] - t_amb));
        }
        slat = wave_sum(slat);
        svert = wave_sum(svert);
        if (lane == 0) {
            sh[w][l] = slat;
            sh[w][kMaxLayers + l] = svert;
        }
    }
    __syncthreads();
    if (tid_lin() == 0) {
        const int nb = gridDim.x;
        for (int l = 0; l < nz; ++l) {
            double a = 0.0, v = 0.0;
            for (int q = 0; q < (int)blockDim.y; ++q) {
                a += sh[q][l];
                v += sh[q][kMaxLayers + l];
            }
            part[(size_t)l * nb + blockIdx.x] = a;
            part[(size_t)(nz + l) * nb + blockIdx.x] = v;
        }
    }
}

// One workgroup: per-layer fixed-order sums of the partials, then the gradient
// with respect to each layer's conductivity: the lateral faces of layer l
// (dg/dk = g / k_lat[l]) plus the vertical faces touching it (dg/dk_vert[l]
// from the faces above and below), summed in that order.
__global__ __launch_bounds__(256) void k_adjoint_finish(int nz, int np,
                                                        const double *__restrict__ part,
                                                        const double *__restrict__ fac,
                                                        double *__restrict__ dk) {
    __shared__ double sums[2 * kMaxLayers];
    for (int k = 0; k < 2 * nz; ++k) {
        const double s = reduce_prev(part + (size_t)k * np, np);
        if (tid_lin() == 0) sums[k] = s;
    }
    __syncthreads();
    const int l = tid_lin();
    if (l < nz) {
        const double *fac_lat = fac, *fac_up = fac + nz, *fac_dn = fac + 2 * nz;
        const double lat = fac_lat[l] * sums[l];
        double v = 0.0;
        if (l < nz - 1) v += fac_up[l] * sums[nz + l];
        if (l > 0) v += fac_dn[l] * sums[nz + l - 1];
        dk[l] = -(lat + v);
    }
}

}  // namespace

// =================================================================== launchers
// CALL is a parenthesised statement using the compile-time VX chosen from the
// runtime lane width VXV (FP32: 1, 2, 4; FP64: 1, 2).
#define CUTH_STRIP(...) __VA_ARGS__
#define CUTH_VX_DISPATCH(T, VXV, CALL)                                          \
    do {                                                                        \
        if constexpr (sizeof(T) == 4) {                                         \
            if (VXV == 4) { constexpr int VX = 4; CUTH_STRIP CALL; break; }     \
        }                                                                       \
        if (VXV == 2) { constexpr int VX = 2; CUTH_STRIP CALL; }                \
        else { constexpr int VX = 1; CUTH_STRIP CALL; }                         \
    } while (0)
#define CUTH_PC_VX_DISPATCH(T, PCV, VXV, CALL)                                  \
    do {                                                                        \
        if (PCV) { constexpr bool PC = true; CUTH_VX_DISPATCH(T, VXV, CALL); }  \
        else { constexpr bool PC = false; CUTH_VX_DISPATCH(T, VXV, CALL); }     \
    } while (0)

template <typename T>
void launch_apply(const OpView<T> &op, const T *x, T *y, hipStream_t s) {
    const dim3 g(stencil_blocks(op)), b(kWave, op.by);
    if constexpr (sizeof(T) == 4) {
        if (op.gx != nullptr && op.hx != nullptr) {
            CUTH_VX_DISPATCH(T, op.vx, (hipLaunchKernelGGL((k_apply<T, true, VX, true>), g, b, 0, s,
                                                           op, x, y)));
            return;
        }
    }
    CUTH_PC_VX_DISPATCH(T, op.gx != nullptr, op.vx,
                        (hipLaunchKernelGGL((k_apply<T, PC, VX, false>), g, b, 0, s, op, x, y)));
}

template <typename T, bool PC, int VX, int CS>
static void cheb_modes(const InnerProb<T> *probs, int nprob, int nb, int by, int mode, bool last,
                       bool chk, bool jac, int j, int zin, const T *pin, bool red, T *pout,
                       hipStream_t s) {
    const dim3 g(nb), b(kWave, by);
#define CUTH_CHEB(M, LST, CK)                                                                      \
    hipLaunchKernelGGL((k_cheb_b<T, PC, VX, M, LST, CK, CS, false>), g, b, 0, s, probs, nprob, j, \
                       zin, pin, (int)red, pout)
#define CUTH_CHEBJ(M, LST)                                                                         \
    hipLaunchKernelGGL((k_cheb_b<T, PC, VX, M, LST, false, CS, true>), g, b, 0, s, probs, nprob, j,\
                       zin, pin, (int)red, pout)
    if (jac) {
        // Jacobi-scaled sweeps: mode 3 (z_1 read, z_0 = 0) or 0; the
        // convergence test runs in the scale pass before them
        if (mode == 3) {
            if (last) CUTH_CHEBJ(3, true); else CUTH_CHEBJ(3, false);
        } else {
            if (last) CUTH_CHEBJ(0, true); else CUTH_CHEBJ(0, false);
        }
        return;
    }
    if (mode == 1) {
        if (chk) {
            if (last) CUTH_CHEB(1, true, true); else CUTH_CHEB(1, false, true);
        } else {
            if (last) CUTH_CHEB(1, true, false); else CUTH_CHEB(1, false, false);
        }
    } else if (mode == 2) {
        if (last) CUTH_CHEB(2, true, false); else CUTH_CHEB(2, false, false);
    } else {
        if (last) CUTH_CHEB(0, true, false); else CUTH_CHEB(0, false, false);
    }
#undef CUTH_CHEB
#undef CUTH_CHEBJ
}

template <typename T>
void launch_cheb_b(const InnerProb<T> *probs, int nprob, int nb, bool pc, int cs, bool jac, int vx,
                   int by, int mode, bool last, bool chk, int j, int zin, const T *part_in,
                   bool red, T *part_out, hipStream_t s) {
    if constexpr (sizeof(T) == 4) {
        if (pc && cs == CS_F16) {
            CUTH_VX_DISPATCH(T, vx, (cheb_modes<T, true, VX, CS_F16>(probs, nprob, nb, by, mode,
                                                                     last, chk, jac, j, zin,
                                                                     part_in, red, part_out, s)));
            return;
        }
    } else {
        if (cs == CS_CSR) {
            CUTH_VX_DISPATCH(T, vx, (cheb_modes<T, false, VX, CS_CSR>(probs, nprob, nb, by, mode,
                                                                      last, chk, false, j, zin,
                                                                      part_in, red, part_out, s)));
            return;
        }
    }
    CUTH_PC_VX_DISPATCH(T, pc, vx, (cheb_modes<T, PC, VX, CS_OWN>(probs, nprob, nb, by, mode, last,
                                                                  chk, jac, j, zin, part_in, red,
                                                                  part_out, s)));
}

template <typename T, bool JAC>
static void cheb2_jac(const InnerProb<T> *probs, int nprob, int nb, bool pc, bool h16, int vx, int R,
                      int zc, int wpr, int j, int zsel, hipStream_t s) {
    const dim3 g(nb), b(kWave, wpr * (R + 2));
    const size_t lds = (size_t)3 * (R + 2) * wpr * kWave * vx * sizeof(T);
    if (pc && h16) {
        CUTH_VX_DISPATCH(T, vx, (hipLaunchKernelGGL((k_cheb2_b<T, true, VX, CS_F16, JAC>), g, b, lds,
                                                    s, probs, nprob, j, zsel, R, zc, wpr)));
        return;
    }
    CUTH_PC_VX_DISPATCH(T, pc, vx, (hipLaunchKernelGGL((k_cheb2_b<T, PC, VX, CS_OWN, JAC>), g, b, lds,
                                                       s, probs, nprob, j, zsel, R, zc, wpr)));
}

template <typename T>
void launch_cheb2_b(const InnerProb<T> *probs, int nprob, int nb, bool pc, bool h16, bool jac,
                    int vx, int R, int zc, int wpr, int j, int zsel, hipStream_t s) {
    if (jac) cheb2_jac<T, true>(probs, nprob, nb, pc, h16, vx, R, zc, wpr, j, zsel, s);
    else cheb2_jac<T, false>(probs, nprob, nb, pc, h16, vx, R, zc, wpr, j, zsel, s);
}

template <typename T, bool JAC, bool M2>
static void cheb3_jac(const InnerProb<T> *probs, int nprob, int nb, bool pc, bool h16, int vx, int R,
                      int zc, int wpr, int j, int zsel, hipStream_t s) {
    const dim3 g(nb), b(kWave, wpr * (R + 4));
    const size_t lds = (size_t)3 * ((R + 4) + (R + 2)) * wpr * kWave * vx * sizeof(T);
    if (pc && h16) {
        CUTH_VX_DISPATCH(T, vx, (hipLaunchKernelGGL((k_cheb3_b<T, true, VX, CS_F16, JAC, M2>), g, b, lds,
                                                    s, probs, nprob, j, zsel, R, zc, wpr)));
        return;
    }
    CUTH_PC_VX_DISPATCH(T, pc, vx, (hipLaunchKernelGGL((k_cheb3_b<T, PC, VX, CS_OWN, JAC, M2>), g, b,
                                                       lds, s, probs, nprob, j, zsel, R, zc, wpr)));
}

template <typename T>
void launch_cheb3_b(const InnerProb<T> *probs, int nprob, int nb, bool pc, bool h16, bool jac, int vx,
                    int R, int zc, int wpr, int j, int zsel, hipStream_t s) {
    if (jac) cheb3_jac<T, true, false>(probs, nprob, nb, pc, h16, vx, R, zc, wpr, j, zsel, s);
    else if (j == 2) cheb3_jac<T, false, true>(probs, nprob, nb, pc, h16, vx, R, zc, wpr, j, zsel, s);
    else cheb3_jac<T, false, false>(probs, nprob, nb, pc, h16, vx, R, zc, wpr, j, zsel, s);
}

template <typename T, bool PC, int VX, int PM>
static void scale_chk(const InnerProb<T> *probs, int nprob, int nb, int by, bool chk,
                      const T *part_in, bool red, T *part_out, hipStream_t s) {
    const dim3 g(nb), b(kWave, by);
    if (chk)
        hipLaunchKernelGGL((k_scale_b<T, PC, VX, true, PM>), g, b, 0, s, probs, nprob, part_in,
                           (int)red, part_out);
    else
        hipLaunchKernelGGL((k_scale_b<T, PC, VX, false, PM>), g, b, 0, s, probs, nprob, part_in,
                           (int)red, part_out);
}

template <typename T>
void launch_scale_b(const InnerProb<T> *probs, int nprob, int nb, bool pc, int pm, int vx, int by,
                    bool chk, const T *part_in, bool red, T *part_out, hipStream_t s) {
    if (pm == PM_JACOBI) {
        CUTH_PC_VX_DISPATCH(T, pc, vx, (scale_chk<T, PC, VX, PM_JACOBI>(probs, nprob, nb, by, chk,
                                                                        part_in, red, part_out, s)));
    } else if (pm == PM_JCHEB) {
        CUTH_PC_VX_DISPATCH(T, pc, vx, (scale_chk<T, PC, VX, PM_JCHEB>(probs, nprob, nb, by, chk,
                                                                       part_in, red, part_out, s)));
    } else if (pm == PM_NONE) {
        CUTH_VX_DISPATCH(T, vx, (scale_chk<T, false, VX, PM_NONE>(probs, nprob, nb, by, chk, part_in,
                                                                  red, part_out, s)));
    } else {
        CUTH_VX_DISPATCH(T, vx, (scale_chk<T, false, VX, PM_SCALE>(probs, nprob, nb, by, chk, part_in,
                                                                   red, part_out, s)));
    }
}

template <typename T>
void launch_dir_b(const InnerProb<T> *probs, int nprob, int nb, bool pc, int cs, int vx,
                  int by, int par, int zfin, const T *part_in, bool red, T *part_out,
                  hipStream_t s) {
    const dim3 g(nb), b(kWave, by);
    if constexpr (sizeof(T) == 8) {
        if (cs == CS_CSR) {
            CUTH_VX_DISPATCH(T, vx, (hipLaunchKernelGGL((k_dir_b<T, false, VX, CS_CSR>), g, b, 0, s,
                                                        probs, nprob, par, zfin, part_in, (int)red,
                                                        part_out)));
            return;
        }
        if (pc && cs == CS_F32) {
            CUTH_VX_DISPATCH(T, vx, (hipLaunchKernelGGL((k_dir_b<T, true, VX, CS_F32>), g, b, 0, s,
                                                        probs, nprob, par, zfin, part_in, (int)red,
                                                        part_out)));
            return;
        }
    }
    CUTH_PC_VX_DISPATCH(T, pc, vx, (hipLaunchKernelGGL((k_dir_b<T, PC, VX, CS_OWN>), g, b, 0, s,
                                                       probs, nprob, par, zfin, part_in, (int)red,
                                                       part_out)));
}

template <typename T>
void launch_promote_dot(const InnerProb<T> *probs, int nprob, int nb, int vx, int by, T *part_out,
                        hipStream_t s) {
    const dim3 g(nb), b(kWave, by);
    CUTH_VX_DISPATCH(T, vx, (hipLaunchKernelGGL((k_promote_dot<T, VX>), g, b, 0, s, probs, nprob,
                                                part_out)));
}

template <typename T>
void launch_reduce_conv(const InnerProb<T> *probs, int nprob, const T *part_in, hipStream_t s) {
    hipLaunchKernelGGL((k_reduce_conv<T>), dim3(nprob), dim3(kWave, 4), 0, s, probs, part_in);
}

template <typename T>
void launch_update_b(const InnerProb<T> *probs, int nprob, int nb, int vx, int by, int par,
                     const T *part_in, bool red, T *part_out, hipStream_t s) {
    const dim3 g(nb), b(kWave, by);
    CUTH_VX_DISPATCH(T, vx, (hipLaunchKernelGGL((k_update_b<T, VX>), g, b, 0, s, probs, nprob, par,
                                                part_in, (int)red, part_out)));
}

template <typename T>
void launch_reduce_b(const InnerProb<T> *probs, int nprob, const T *part_in, T *red_out,
                     hipStream_t s) {
    hipLaunchKernelGGL((k_reduce_b<T>), dim3(nprob), dim3(kWave, 4), 0, s, probs, part_in, red_out);
}

template <typename T>
void launch_check_b(const InnerProb<T> *probs, int nprob, int nb, bool pc, int cs, int vx, int by,
                    T *part_out, hipStream_t s) {
    const dim3 g(nb), b(kWave, by);
    if constexpr (sizeof(T) == 8) {
        if (cs == CS_CSR) {
            CUTH_VX_DISPATCH(T, vx, (hipLaunchKernelGGL((k_check_b<T, false, VX, CS_CSR>), g, b, 0,
                                                        s, probs, nprob, part_out)));
            return;
        }
    }
    CUTH_PC_VX_DISPATCH(T, pc, vx, (hipLaunchKernelGGL((k_check_b<T, PC, VX, CS_OWN>), g, b, 0, s,
                                                       probs, nprob, part_out)));
}

template <typename TD, typename TI>
void launch_residual_b(const OuterProb<TD, TI> *probs, int nprob, int nb, bool pc, int vx, int by,
                       int flags, double *part_out, hipStream_t s) {
    const dim3 g(nb), b(kWave, by);
    // the stream sets the solver launches (see k_residual_b), at the default
    // lane width; anything else takes the run-time tests
#define CUTH_RES(FLV)                                                                               \
    do {                                                                                           \
        if (pc) hipLaunchKernelGGL((k_residual_b<true, 2, TD, TI, FLV>), g, b, 0, s, probs, nprob,  \
                                   part_out);                                                      \
        else hipLaunchKernelGGL((k_residual_b<false, 2, TD, TI, FLV>), g, b, 0, s, probs, nprob,    \
                                part_out);                                                         \
    } while (0)
    if (vx == 2) {
        switch (flags) {
        case 0: CUTH_RES(0); return;
        case 1: CUTH_RES(1); return;
        case 3: CUTH_RES(3); return;
        case 5: CUTH_RES(5); return;
        case 7: CUTH_RES(7); return;
        case 9: CUTH_RES(9); return;
        default: break;
        }
    }
#undef CUTH_RES
    CUTH_PC_VX_DISPATCH(double, pc, vx, (hipLaunchKernelGGL((k_residual_b<PC, VX, TD, TI, -1>), g, b,
                                                            0, s, probs, nprob, part_out)));
}

template <typename TD, typename TI>
void launch_reduce_outer(const OuterProb<TD, TI> *probs, int nprob, const double *part, int ntot,
                         double *out, hipStream_t s) {
    hipLaunchKernelGGL((k_reduce_outer<TD, TI>), dim3(nprob), dim3(kWave, kReduceOuterWaves), 0, s, probs, part,
                       ntot, out);
}

void launch_csr_fill(const OpView<double> &op, const int *ptr, int *col, double *val,
                     hipStream_t s) {
    const int64_t n = (int64_t)op.nx * op.ny * op.nz;
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 65536);
    hipLaunchKernelGGL(k_csr_fill, dim3((unsigned)blocks), dim3(256), 0, s, op, ptr, col, val);
}

void launch_csr_spmv(int64_t n, const int *ptr, const int *col, const double *val,
                     const double *x, double *y, hipStream_t s) {
    hipLaunchKernelGGL(k_csr_spmv, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, ptr, col,
                       val, x, y);
}

void launch_to_f32(int64_t n, const double *x, float *y, hipStream_t s) {
    hipLaunchKernelGGL(k_to_f32, dim3(red_blocks(n)), dim3(kWave, 4), 0, s, n, x, y);
}

void launch_add_scalar(int64_t n, const double *x, double a, double *y, hipStream_t s) {
    hipLaunchKernelGGL(k_add_scalar, dim3(red_blocks(n)), dim3(kWave, 4), 0, s, n, x, a, y);
}

void launch_build_lateral(int nx, int ny, int nz, double dx, double dy, const double *dz,
                          const double *k_lat, const double *mult, double *gx64, double *gy64,
                          float *gx32, float *gy32, unsigned long long *maxrow,
                          unsigned long long *maxg, unsigned int *bad, hipStream_t s) {
    const dim3 g((nx + kWave - 1) / kWave, (ny + 3) / 4), b(kWave, 4);
    hipLaunchKernelGGL(k_build_lateral, g, b, 0, s, nx, ny, nz, dx, dy, dz, k_lat, mult, gx64,
                       gy64, gx32, gy32, bad);
    hipLaunchKernelGGL(k_lateral_rowmax, g, b, 0, s, nx, ny, nz, (const double *)gx64,
                       (const double *)gy64, maxrow, maxg);
}

void launch_build_fp16(int nx, int ny, int nz, const double *gx64, const double *gy64,
                       const double *scale, uint16_t *hx, uint16_t *hy, hipStream_t s) {
    const dim3 g((nx + kWave - 1) / kWave, (ny + 3) / 4), b(kWave, 4);
    hipLaunchKernelGGL(k_build_fp16, g, b, 0, s, nx, ny, nz, gx64, gy64, scale, hx, hy);
}

void launch_fill_random(int64_t n, uint64_t seed, float *v, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_random, dim3(red_blocks(n)), dim3(kWave, 4), 0, s, n, seed, v);
}

void launch_norm2(int64_t n, const float *v, float *part_out, hipStream_t s) {
    hipLaunchKernelGGL(k_norm2, dim3(red_blocks(n)), dim3(kWave, 4), 0, s, n, v, part_out);
}

void launch_scale_rsqrt(int64_t n, const float *v, const float *part_in, int np_in, float *out,
                        hipStream_t s) {
    hipLaunchKernelGGL(k_scale_rsqrt, dim3(red_blocks(n)), dim3(kWave, 4), 0, s, n, v, part_in,
                       np_in, out);
}

void launch_lanczos_av(const OpView<float> &op, int j, const float *v, const float *vprev,
                       const float *lz, const float *dis, float *w, float *part_out,
                       hipStream_t s) {
    const dim3 g(stencil_blocks(op)), b(kWave, op.by);
    if (dis) {
        CUTH_PC_VX_DISPATCH(float, op.gx != nullptr, op.vx,
                            (hipLaunchKernelGGL((k_lanczos_av<PC, VX, true>), g, b, 0, s, op, j, v,
                                                vprev, lz, dis, w, part_out)));
        return;
    }
    CUTH_PC_VX_DISPATCH(float, op.gx != nullptr, op.vx,
                        (hipLaunchKernelGGL((k_lanczos_av<PC, VX, false>), g, b, 0, s, op, j, v,
                                            vprev, lz, dis, w, part_out)));
}

void launch_jacobi_dis(const OpView<double> &op, float *dis, hipStream_t s) {
    const int64_t n = (int64_t)op.nx * op.ny * op.nz;
    const int nb = (int)std::min<int64_t>((n + 255) / 256, 65536);
    hipLaunchKernelGGL(k_jacobi_dis, dim3(nb), dim3(256), 0, s, op, dis);
}

void launch_lanczos_orth(int64_t n, int j, float *w, const float *v, float *lz,
                         const float *part_in, int np_in, float *part_out, hipStream_t s) {
    hipLaunchKernelGGL(k_lanczos_orth, dim3(red_blocks(n)), dim3(kWave, 4), 0, s, n, j, w, v, lz,
                       part_in, np_in, part_out);
}

void launch_lanczos_div(int64_t n, int j, float *w, float *lz, const float *part_in, int np_in,
                        hipStream_t s) {
    hipLaunchKernelGGL(k_lanczos_div, dim3(red_blocks(n)), dim3(kWave, 4), 0, s, n, j, w, lz,
                       part_in, np_in);
}

void launch_adjoint(const OpView<double> &op, const double *lam, const double *T, double t_amb,
                    const double *fac, double *part, double *dL_dk, hipStream_t s) {
    const int nb = ((op.nx + kWave - 1) / kWave) * ((op.ny + 3) / 4);
    if (op.gx)
        hipLaunchKernelGGL((k_adjoint_sums<true>), dim3(nb), dim3(kWave, 4), 0, s, op, lam, T,
                           t_amb, part);
    else
        hipLaunchKernelGGL((k_adjoint_sums<false>), dim3(nb), dim3(kWave, 4), 0, s, op, lam, T,
                           t_amb, part);
    hipLaunchKernelGGL(k_adjoint_finish, dim3(1), dim3(kWave, 4), 0, s, op.nz, nb,
                       (const double *)part, fac, dL_dk);
}

#define CUTH_INST(T)                                                                              \
    template void launch_apply<T>(const OpView<T> &, const T *, T *, hipStream_t);                \
    template void launch_cheb_b<T>(const InnerProb<T> *, int, int, bool, int, bool, int, int, int,\
                                   bool, bool, int, int, const T *, bool, T *, hipStream_t);      \
    template void launch_scale_b<T>(const InnerProb<T> *, int, int, bool, int, int, int, bool,    \
                                    const T *, bool, T *, hipStream_t);                           \
    template void launch_dir_b<T>(const InnerProb<T> *, int, int, bool, int, int, int, int, int,  \
                                  const T *, bool, T *, hipStream_t);                             \
    template void launch_update_b<T>(const InnerProb<T> *, int, int, int, int, int, const T *,    \
                                     bool, T *, hipStream_t);                                     \
    template void launch_reduce_b<T>(const InnerProb<T> *, int, const T *, T *, hipStream_t);     \
    template void launch_check_b<T>(const InnerProb<T> *, int, int, bool, int, int, int, T *,     \
                                    hipStream_t);
CUTH_INST(float)
CUTH_INST(double)
#undef CUTH_INST

template void launch_cheb2_b<float>(const InnerProb<float> *, int, int, bool, bool, bool, int, int,
                                      int, int, int, int, hipStream_t);
template void launch_cheb3_b<float>(const InnerProb<float> *, int, int, bool, bool, bool, int, int,
                                      int, int, int, int, hipStream_t);
template void launch_promote_dot<double>(const InnerProb<double> *, int, int, int, int, double *,
                                         hipStream_t);
template void launch_reduce_conv<double>(const InnerProb<double> *, int, const double *,
                                         hipStream_t);

template void launch_reduce_outer<float, float>(const OuterProb<float, float> *, int, const double *,
                                                int, double *, hipStream_t);
template void launch_reduce_outer<double, double>(const OuterProb<double, double> *, int,
                                                  const double *, int, double *, hipStream_t);
template void launch_residual_b<float, float>(const OuterProb<float, float> *, int, int, bool, int,
                                              int, int, double *, hipStream_t);
template void launch_residual_b<double, double>(const OuterProb<double, double> *, int, int, bool,
                                                int, int, int, double *, hipStream_t);

// ------------------------------------------------ allocation-free scratch
// Device memory of the allocation-free preconditioner entry point: one array
// per device, held until the process ends.  On the host the array's name is a
// stand-in, not a device address, so host code never hands it to a kernel or a
// copy: it uses the address hipGetSymbolAddress returns for the device.
namespace {
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

constexpr int kPutWords = 512;   // 2 KiB of kernel arguments per launch
struct PutBlob {
    unsigned int w[kPutWords];
};

__global__ __launch_bounds__(256) void k_put(PutBlob src, unsigned int *__restrict__ dst, int nw) {
    for (int i = threadIdx.x; i < nw; i += blockDim.x) dst[i] = src.w[i];
}

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
unsigned char *g_scratch_ptr[kMaxScratchDevices] = {};
}  // namespace

hipError_t noalloc_scratch(int device, unsigned char **ptr) {
    *ptr = nullptr;
    if (device < 0 || device >= kMaxScratchDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        // the lookup runs once per device, with that device current
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device && (e = hipSetDevice(device)) != hipSuccess) return e;
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != device) {
            const hipError_t e2 = hipSetDevice(cur);
            if (e == hipSuccess) e = e2;
        }
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = static_cast<unsigned char *>(p);
    }
    *ptr = g_scratch_ptr[device];
    return hipSuccess;
}

hipError_t launch_put(const void *src, size_t n, void *dst, hipStream_t s) {
    const unsigned char *in = static_cast<const unsigned char *>(src);
    unsigned char *out = static_cast<unsigned char *>(dst);
    if (reinterpret_cast<uintptr_t>(out) % 4 != 0 || n % 4 != 0) return hipErrorInvalidValue;
    while (n > 0) {
        const size_t m = std::min(n, sizeof(PutBlob));
        PutBlob b;
        std::memset(&b, 0, sizeof b);
        std::memcpy(&b, in, m);
        hipLaunchKernelGGL(k_put, dim3(1), dim3(256), 0, s, b,
                           reinterpret_cast<unsigned int *>(out), (int)(m / 4));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        in += m;
        out += m;
        n -= m;
    }
    return hipSuccess;
}

}  // namespace cuth
