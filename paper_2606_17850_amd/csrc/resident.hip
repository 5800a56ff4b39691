// The whole Chebyshev preconditioner in one launch, for operators whose sweep
// vectors fit on the chip.
//
// What bounds it.  A launch per sweep (or per two or three) streams z_j,
// z_{j-1}, r and the conductances from memory for every sweep.  The registers
// of the 256 CUs hold 128 MB, so up to 4 M unknowns keep all of it on chip: a
// workgroup owns a tile of 64 x (VY NW) whole columns of the grid, a lane VY
// columns, and z_j, z_{j-1}, r and the conductances stay in registers from the
// first sweep to the last.  A sweep then costs its arithmetic (14.5 vector
// instructions per unknown; 19 to 23 with all around it) and one exchange of the tile's edge values with the
// four neighbouring tiles (about 1 us through memory, behind the arithmetic
// where that is long enough).  Per sweep, launches as before -> here: 512x512x16
// per cell 10.0 -> 2.9 us (256 tiles of 64 x 16 columns, two wavefronts per SIMD: a
// wavefront issues a vector instruction every 12 cycles, 5.5 being the least, and
// waits for edges, LDS and barriers 38 % of the time),
// 256x256x10 4.0 -> 1.5 us, 64x64x8 3.6 -> 1.1 us (the exchange).
//
// Tiles.  64 x 8 columns where the CUs hold all such tiles at once, one each, else
// 64 x 16 (FP32), which do twice the arithmetic per exchange (res_fit).
//
// Groups.  Several problems (a batch), or a grid of more tiles than CUs, go
// through the chip as groups of tiles: a problem is a group, and such a grid is
// cut into slabs of rows that compute k - 1 rows beyond their own on each side
// from r alone (a sweep spoils one row more) and write their own.  An
// application then reads and writes its vectors once whatever the size.  12
// stacks of 128^2 to 384^2 x 8 to 16 with 4 power maps each: 866 -> 405 ms a
// solve; one application at 1024x1024x16 (5 slabs, 25 % of the rows computed
// twice) 1190 -> 540 us with per-layer and 2080 -> 580 us with per-cell
// conductances, launches as before -> here.
//
// 17 to 20 layers (FP32) take 14 rows, which fill the LDS, where the plain
// per-layer kernel fits its registers (255), else 8: 1024x1024x20, 6 slabs, 1490 ->
// 660 us an application by itself, a backward-Euler step 9.4 -> 6.0 ms (14 slabs of 8-row
// tiles: 1070 us).
//
// FP64.  The same kernel with half the rows per tile.  A value takes two exchange
// words, and the exchange sets the time: 3 us a sweep at 192x128x12, 7 us for a
// slab of 512x216x16.  One application, launches as before -> here: 64x64x8 238
// -> 78 us, 192x128x12 250 -> 126; 512x512x16 solves (3 slabs) 175 -> 129 ms.
//
// Exchange.  Neighbouring tiles may sit on different XCDs, whose L2 caches are
// not coherent, so edge values go through memory with agent-scope accesses.
// Each FP32 word travels in one 64-bit word with a 32-bit tag (launch epoch +
// sweep): the reader polls the word itself until the tag matches, so a value
// needs neither a fence nor a separate flag, and one round trip suffices.  Two
// buffers alternate by sweep parity: a tile writes its sweep j + 2 values only
// after it has read its neighbour's sweep j + 1 values, which that neighbour
// sent after reading the sweep j ones.
//
// Within a tile, x neighbours move by DPP shifts, z neighbours are in the
// lane's registers, and y neighbours of other wavefronts come from an LDS copy
// of z_j (double-buffered, so one barrier per sweep suffices).
//
// Waiting.  Every tile of a group must be running for its neighbours to make
// progress.  The host launches at most one workgroup per CU, over all such launches
// of the process on the device (ResLease); every wait is bounded all the same
// (ResArgs::spin polls): a tile that gives up marks its problem (CgState::gave_up)
// and ends, its neighbours see the mark while they wait and end too, and the host
// repeats the application with ordinary launches, which only read r (of several
// problems: the whole solve of those marked).  Tiles that start after the mark run
// all the same: the problem's lead tile counts the iteration, whenever it starts.
#include "device_util.hpp"

namespace cuth {
namespace {

using u64 = unsigned long long;

template <typename T> struct Bits;
template <> struct Bits<float> { static constexpr int n = 1; };
template <> struct Bits<double> { static constexpr int n = 2; };

__device__ __forceinline__ void put_word(u64 *q, unsigned bits, unsigned tag) {
    __hip_atomic_store((__attribute__((address_space(1))) u64 *)q, ((u64)tag << 32) | bits,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 get_word(const u64 *q) {
    return __hip_atomic_load((const __attribute__((address_space(1))) u64 *)q, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
}

// All loads so far have returned.  Where the compiler cannot see that, it waits at
// their next possible use, after a branch or at the head of a loop, and with them
// for every store since (one counter serves both): without these, each sweep
// waited for the edges just sent to reach memory (512x512x16 3.3 us a sweep
// instead of 2.9).
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0f70); }   // vmcnt 0

// One value as Bits<T>::n consecutive tagged words.
template <typename T>
__device__ __forceinline__ void put_value(u64 *q, T v, unsigned tag) {
    unsigned w[Bits<T>::n];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (int i = 0; i < Bits<T>::n; ++i) {
        // (a copy the compiler cannot merge with v: it would keep v, and so every
        // value of a lane's columns, in one half of a register pair for the store)
        unsigned c;
        asm volatile("v_mov_b32 %0, %1" : "=v"(c) : "v"(w[i]));
        put_word(q + i, c, tag);
    }
}

// The value lane q (uniform) holds, as a scalar.
template <typename T>
__device__ __forceinline__ T lane_value(T v, int q) {
    int w[sizeof(T) / 4];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) w[i] = __builtin_amdgcn_readlane(w[i], q);
    T r;
    __builtin_memcpy(&r, w, sizeof(T));
    return r;
}
// A uniform value held in scalar registers; 0 without `keep`.
template <typename T>
__device__ __forceinline__ T uniform(T v, bool keep) {
    int w[sizeof(T) / 4];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i)
        w[i] = __builtin_amdgcn_readfirstlane(keep ? w[i] : 0);
    T r;
    __builtin_memcpy(&r, w, sizeof(T));
    return r;
}
// The value of the lane to the left / right; 0 where there is none.
template <int CTRL, typename T>
__device__ __forceinline__ T dpp_zero(T v) {
    int w[sizeof(T) / 4];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i)
        w[i] = __builtin_amdgcn_update_dpp(0, w[i], CTRL, 0xf, 0xf, true);
    T r;
    __builtin_memcpy(&r, w, sizeof(T));
    return r;
}
template <typename T>
__device__ __forceinline__ T left0(T v) { return dpp_zero<0x138>(v); }
template <typename T>
__device__ __forceinline__ T right0(T v) { return dpp_zero<0x130>(v); }

// NZ: layers a lane holds (the grid's, rounded up; the padding layers hold
// zeros and couple to nothing).  VY: rows per lane.  NW: wavefronts.  PC:
// per-cell lateral conductances (FP32 or FP16-stored, promoted once here).
// JAC: the Jacobi-scaled sweeps, from z_1 = D^-1 r / theta, formed here but for
// FP16-stored conductances, whose z_1 (by k_scale_b, D in full precision) is in
// z[0].  390x270x14 mixed solve 10.4 -> 9.5 ms without the separate pass.
//
// A sweep first forms every cell's result without the faces to other tiles
// (their values are still on their way), then adds those faces' terms to the
// tile's edge cells: c2 g (z_neighbour - z).  The first part needs nothing from
// outside, so the exchange runs behind it.
template <typename T, bool PC, bool JAC, int NZ, int VY, int NW>
__device__ __forceinline__ void res_tile(const InnerProb<T> *__restrict__ probs, int k, int zout, int chk,
                                         const T *__restrict__ part_in, int red, T *__restrict__ part_out,
                                         const ResArgs &ra, int slot) {
    constexpr int NR = VY * NW;        // rows of a tile
    constexpr int RS = kWave;          // LDS stride of a row's layers (every layer within a paired access's offsets)
    constexpr int WT = Bits<T>::n;
    constexpr int SY = NZ * kWave * WT, SX = NR * NZ * WT;   // words of a y and of an x side
    extern __shared__ __align__(16) unsigned char lds_raw[];
    // x-edge corrections [2 sides][NR][NZ], then two copies of the tile's rows [2][NR][NZ][RS]
    T *cx = reinterpret_cast<T *>(lds_raw);
    T *rows = cx + 2 * NR * NZ;
    // a wait ran out: sweep j writes entry j & 1 and reads the other, which the barrier
    // between them has closed (all wavefronts leave in the same sweep)
    __shared__ int bad_s[2];

    int gi = 0;
    {
        int hi = ra.ngroups - 1;
        while (gi < hi) {
            const int mid = (gi + hi + 1) >> 1;
            if (ra.groups[mid].tile0 <= slot) gi = mid;
            else hi = mid - 1;
        }
    }
    const ResGroup G = ra.ngroups > 1 ? ra.groups[gi] : ra.one;
    const int pidx = G.prob;
    const InnerProb<T> &P = probs[pidx];
    CgState<T> *st = P.st;
    const int local = slot - G.tile0, part = G.part0 + local;   // tile of the group, of the problem
    // The whole workgroup acts on one lane's reading of the stop flag: the problem's
    // lead tile may set it during this launch, and wavefronts that read it for
    // themselves could part here and meet different barriers.
    __shared__ int done_s;
    int done = 0;
    if (tid_lin() == 0) done_s = done = st->done;
    const bool stop = chk && conv_test(st, part_in, red, pidx, P, part == 0 && !done);
    if (!chk || red) __syncthreads();   // (otherwise the test's sum has had its barriers)
    if (stop || done_s) return;

    // (opaque: what follows from them is not kept in registers over the loop over
    // tiles, and the layers' constants come by vector loads, all in flight at once)
    int lane = threadIdx.x, w = threadIdx.y, zero = 0;
    asm volatile("" : "+v"(lane), "+v"(w), "+v"(zero));
    w = __builtin_amdgcn_readfirstlane(w);
    if (tid_lin() == 0) bad_s[0] = bad_s[1] = 0;
    const OpView<T> &op = P.op;
    const int nx = op.nx, ny = op.ny, nz = op.nz;
    const int64_t plane = (int64_t)nx * ny;
    int ntx = P.r_ntx;
    asm volatile("" : "+s"(ntx));   // (as k below)
    const int tx = local % ntx, ty = local / ntx;
    const int nty = G.nty;
    const bool nbW = tx > 0, nbE = tx + 1 < ntx, nbS = ty > 0, nbN = ty + 1 < nty;
    const int i = tx * kWave + lane, row0 = w * VY, j0 = G.y0 + ty * NR + row0;
    const int own0 = G.own0, own1 = G.own1;   // rows this group writes
    const bool act = i < nx;
    // (kernel arguments kept, not read again in every sweep)
    asm volatile("" : "+s"(k));
    const bool edgeS = w == 0 && nbS, edgeN = w == NW - 1 && nbN;   // wavefronts with a y face to another tile
    // those have the exchange to do besides, so they compute first
    if (edgeS || edgeN) __builtin_amdgcn_s_setprio(2);
    const unsigned epoch = __builtin_amdgcn_readfirstlane(gld(ra.epoch + slot));
    const T inv_th = P.cheb[0];

    // A layer's values of a vector, by a 32-bit byte offset within the layer (the
    // layer's base address stays scalar).  Loads are unguarded, at an in-bounds
    // cell (layer nz - 1 for the padding layers), and masked after.
    auto cell = [&](int j, int ii) -> unsigned {
        const bool ok = j >= 0 && j < ny && ii >= 0 && ii < nx;
        return ok ? (unsigned)(j * nx + ii) : 0u;
    };
    auto ld = [&](const auto *p, int l, unsigned c) {
        using V = std::decay_t<decltype(*p)>;
        const char *b = reinterpret_cast<const char *>(p + (int64_t)(l < nz ? l : nz - 1) * plane);
        return gld(reinterpret_cast<const V *>(b + (size_t)(c * (unsigned)sizeof(V))));
    };
    auto in_grid = [&](int j, int ii) { return j >= 0 && j < ny && ii >= 0 && ii < nx; };
    auto layer = [&](int l) { return gldc(op.lc + ((l < nz ? l : nz - 1) + zero)); };
    // one lateral conductance from (j, ii) to +x / +y, 0 where there is no such face
    auto lat_at = [&](const T *g, const uint16_t *h, int l, int j, int ii) -> T {
        const T v = h ? (T)h16one(ld(h, l, cell(j, ii))) * layer(l).hs : ld(g, l, cell(j, ii));
        return in_grid(j, ii) && l < nz ? v : T(0);
    };
    auto gx_at = [&](int l, int j, int ii) -> T {
        if constexpr (PC) return lat_at(op.gx, op.hx, l, j, ii);
        else return in_grid(j, ii) && ii + 1 < nx && l < nz ? layer(l).gx : T(0);
    };
    auto gy_at = [&](int l, int j, int ii) -> T {
        if constexpr (PC) return lat_at(op.gy, op.hy, l, j, ii);
        else return in_grid(j, ii) && j + 1 < ny && l < nz ? layer(l).gy : T(0);
    };
    auto row_at = [&](int buf, int row) -> int {
        int q = (buf * NR + row) * (NZ * RS);
        asm volatile("" : "+v"(q));
        return q;
    };

    // ---- the lane's columns
    T za[VY][NZ], zb[VY][NZ], rr[VY][NZ];
    // conductances to +x (0 at the tile's last column) and, per cell, to +y and from the row below
    T gxp[PC ? VY : 1][NZ];
    [[maybe_unused]] T gyp[VY][NZ], gs0[NZ];
    [[maybe_unused]] T di[VY][NZ];
#pragma unroll
    for (int v = 0; v < VY; ++v) {
        const unsigned c = cell(j0 + v, i);
#pragma unroll
        for (int l = 0; l < NZ; ++l) {
            rr[v][l] = ld(P.r, l, c);
            if constexpr (JAC && PC)
                if (op.hx) za[v][l] = ld(P.z[0], l, c);
        }
    }
    if constexpr (PC) {
        const unsigned cs = cell(j0 - 1, i);
        if (op.hx) {
#pragma unroll
            for (int l = 0; l < NZ; ++l) {
                const T hs = layer(l).hs;
#pragma unroll
                for (int v = 0; v < VY; ++v) {
                    const unsigned c = cell(j0 + v, i);
                    gxp[v][l] = (T)h16one(ld(op.hx, l, c)) * hs;
                    gyp[v][l] = (T)h16one(ld(op.hy, l, c)) * hs;
                }
                gs0[l] = (T)h16one(ld(op.hy, l, cs)) * hs;
            }
        } else {
#pragma unroll
            for (int l = 0; l < NZ; ++l) {
#pragma unroll
                for (int v = 0; v < VY; ++v) {
                    const unsigned c = cell(j0 + v, i);
                    gxp[v][l] = ld(op.gx, l, c);
                    gyp[v][l] = ld(op.gy, l, c);
                }
                gs0[l] = ld(op.gy, l, cs);
            }
        }
    }
    // (opaque: the padding layers' tests are not kept for the end)
    int nzq = nz;
    asm volatile("" : "+s"(nzq));
#pragma unroll
    for (int l = 0; l < NZ; ++l) {
#pragma unroll
        for (int v = 0; v < VY; ++v) {
            const bool ok = act && j0 + v < ny && l < nzq;
            rr[v][l] = ok ? rr[v][l] : T(0);
            if constexpr (!JAC) za[v][l] = rr[v][l] * inv_th;
            zb[v][l] = T(0);
            if constexpr (PC) {
                gyp[v][l] = ok ? gyp[v][l] : T(0);
                gxp[v][l] = ok ? gxp[v][l] : T(0);
            }
        }
        if constexpr (PC) {
            gs0[l] = act && j0 > 0 && j0 <= ny && l < nzq ? gs0[l] : T(0);
        } else {
            gxp[0][l] = l < nzq && i + 1 < nx ? layer(l).gx : T(0);
        }
    }
    if constexpr (JAC) {
        // 1/diag(A), 0 outside the grid (gxp still holds the faces to other tiles)
#pragma unroll
        for (int l = 0; l < NZ; ++l) {
            const LayerCoef<T> L = layer(l);
#pragma unroll
            for (int v = 0; v < VY; ++v) {
                const bool ok = act && j0 + v < ny && l < nzq;
                T gm = left0(gxp[PC ? v : 0][l]), gs, gn;
                if (lane == 0) gm = gx_at(l, j0 + v, i - 1);
                if constexpr (PC) {
                    gs = v == 0 ? gs0[l] : gyp[v > 0 ? v - 1 : 0][l];
                    gn = gyp[v][l];
                } else {
                    gs = j0 + v > 0 ? L.gy : T(0);
                    gn = j0 + v + 1 < ny ? L.gy : T(0);
                }
                const T d = L.sink + gm + gxp[PC ? v : 0][l] + gs + gn + L.gzd + L.gzu;
                di[v][l] = ok ? recip(d) : T(0);
                const T z1 = rr[v][l] * inv_th * di[v][l];
                if constexpr (PC) za[v][l] = op.hx ? (ok ? za[v][l] : T(0)) : z1;
                else za[v][l] = z1;
            }
        }
    }
#pragma unroll
    for (int l = 0; l < NZ; ++l)
#pragma unroll
        for (int v = 0; v < (PC ? VY : 1); ++v) gxp[v][l] = lane == kWave - 1 ? T(0) : gxp[v][l];
    // the lane's x-edge cell: side, row and layer, conductance of its face to the
    // neighbouring tile, value in the current iterate
    constexpr int XI = 2 * VY * NZ;   // x-edge cells of a wavefront: XN or fewer per lane
    constexpr int XN = (XI + kWave - 1) / kWave;
    const int xs = lane & 1;                                     // (sides alternate: two LDS banks at a time)
    const int xi = tx * kWave + (xs == 0 ? 0 : kWave - 1);       // its column
    bool wx[XN];
    T ge[XN], xe[XN];
    [[maybe_unused]] T de[XN];
    int x_at[XN], x_row[XN];   // its slot in cx and in LDS copy 0
    unsigned side_at[XN];
#pragma unroll
    for (int n = 0; n < XN; ++n) {
        const int xq = lane + n * kWave < XI ? lane + n * kWave : xs;
        const int xr = (xq >> 1) / NZ, xl = (xq >> 1) % NZ;
        wx[n] = lane + n * kWave < XI && (xs == 0 ? nbW : nbE);
        ge[n] = wx[n] ? gx_at(xl, j0 + xr, xs == 0 ? xi - 1 : xi) : T(0);
        if constexpr (JAC) {
            const LayerCoef<T> L = layer(xl);
            const int j = j0 + xr;
            const T d = L.sink + gx_at(xl, j, xi - 1) + gx_at(xl, j, xi) + gy_at(xl, j - 1, xi) + gy_at(xl, j, xi) +
                        L.gzd + L.gzu;
            de[n] = wx[n] && in_grid(j, xi) && xl < nz ? recip(d) : T(0);
        }
        xe[n] = T(0);
        x_at[n] = (xs * NR + row0 + xr) * NZ + xl;
        x_row[n] = ((row0 + xr) * NZ + xl) * RS + (xs == 0 ? 0 : kWave - 1);
        side_at[n] = 8u * (unsigned)((row0 * NZ + xr * NZ + xl) * WT);
    }
    const bool x_edge = (lane == 0 && nbW) || (lane == kWave - 1 && nbE);   // lanes with an x face to another tile
    const int c_at = ((lane == 0 ? 0 : NR) + row0) * NZ;                    // their corrections in cx
    // the layers' constants, uniform: one scalar register each (LDS reads of them,
    // broadcast or not, cost the LDS more than the rows' reads do)
    T sink[NZ], gzu[NZ];
    [[maybe_unused]] T gyl[NZ];
#pragma unroll
    for (int l = 0; l < NZ; ++l) {
        const LayerCoef<T> L = layer(l);
        sink[l] = uniform(L.sink, l < nz);
        gzu[l] = uniform(L.gzu, l < nz);
        if constexpr (!PC) {
            gyl[l] = l < nz ? L.gy : T(0);
            asm volatile("" : "+v"(gyl[l]));   // (in a vector register: faster to read)
        }
    }
    // the sweeps' constants: lane q holds those of sweep q + 1 of the current 64
    T vc1 = T(0), vc2 = T(0);
    // y neighbours outside the tile or the grid: the row itself (its term vanishes)
    const bool self_s = w == 0 || j0 >= ny, self_n = w == NW - 1 || j0 + VY >= ny;
    // (per-layer conductances) the lane's second row lies outside the grid
    [[maybe_unused]] const bool half = j0 + 1 >= ny;

    // the exchange words by 32-bit byte offsets from the buffer (the host keeps it below 4 GB)
    constexpr unsigned kTileBytes = 8u * 2u * (SY + SX);
    const unsigned par_bytes = kTileBytes * (unsigned)ra.tiles;
    auto word = [&](unsigned bytes) -> u64 * {
        return reinterpret_cast<u64 *>(reinterpret_cast<char *>(ra.buf) + (size_t)bytes);
    };
    const unsigned y_lane = 8u * (unsigned)(lane * WT);

    // own rows of z into LDS copy `buf`
    auto put_rows = [&](const T(&z)[VY][NZ], int buf) {
#pragma unroll
        for (int v = 0; v < VY; ++v) {
            T *q = rows + row_at(buf, row0 + v) + lane;
#pragma unroll
            for (int l = 0; l < NZ; ++l) q[l * RS] = z[v][l];
        }
    };
    // edges of z (sweep j's result; x edges: xe) to the neighbours
    auto send = [&](const T(&z)[VY][NZ], int j) {
        const unsigned tag = epoch + (unsigned)j;
        unsigned pb = (unsigned)(j & 1) * par_bytes;
        asm volatile("" : "+s"(pb));   // (as row_at)
        // the tile below reads its north side, the tile above its south side
        if (edgeS) {
            const unsigned q = pb + (unsigned)(slot - ntx) * kTileBytes + 8u * SY + y_lane;
#pragma unroll
            for (int l = 0; l < NZ; ++l) put_value(word(q) + l * kWave * WT, z[0][l], tag);
        }
        if (edgeN) {
            const unsigned q = pb + (unsigned)(slot + ntx) * kTileBytes + y_lane;
#pragma unroll
            for (int l = 0; l < NZ; ++l) put_value(word(q) + l * kWave * WT, z[VY - 1][l], tag);
        }
        // x edges, one value per lane; the west neighbour reads its east side
        // (after SX), and the reverse
#pragma unroll
        for (int n = 0; n < XN; ++n)
            if (wx[n])
                put_value(word(pb + (unsigned)(xs == 0 ? slot - 1 : slot + 1) * kTileBytes +
                               8u * (2 * SY + (xs == 0 ? SX : 0)) + side_at[n]),
                          xe[n], tag);
    };
    auto value = [&](const u64(&g)[WT]) -> T {
        unsigned wd[WT];
#pragma unroll
        for (int n = 0; n < WT; ++n) wd[n] = (unsigned)g[n];
        T v;
        __builtin_memcpy(&v, wd, sizeof(T));
        return v;
    };
    int left = 0;
    auto waited_out = [&]() -> bool {   // one more poll; true when the bound is reached
        if (--left <= 0) return true;
        if ((left & 255) == 0 &&
            __hip_atomic_load(&st->gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            left = 1;
        return false;
    };

    // ---- sweep j: out = z_{j+1} from in = z_j and out = z_{j-1}, y neighbours
    // of other wavefronts from LDS copy `buf`, then the faces to other tiles.
    // False when a wait ran out before this sweep.
    auto sweep = [&](const T(&in)[VY][NZ], T(&out)[VY][NZ], int j, int buf) -> bool {
        const int bad = bad_s[(j - 1) & 1];
        if (((j - 1) & (kWave - 1)) == 0) {
            const int jl = min(j + lane, k - 1);
            vc1 = gld(P.cheb + 1 + jl);
            vc2 = gld(P.cheb + 1 + P.kcap + jl);
            wait_loads();
        }
        const T c1 = lane_value(vc1, (j - 1) & (kWave - 1)), c2 = lane_value(vc2, (j - 1) & (kWave - 1));
        // The neighbours' edges: a wavefront polls its own x-edge words and, at the
        // tile's y edges, its row's.  First polled before layer IL: what has arrived
        // by then costs no wait.  The largest tile takes the y words LC layers at a
        // time, for want of registers (all at once spill in FP64 from 12 layers on:
        // 390x270x14 200 -> 540 us an application).
        constexpr int GL = sizeof(T) == 4 && NZ % 4 == 0 && VY == 1 ? 4 : 2, IL = NZ * 3 / 4 / GL * GL;
        constexpr int LC = sizeof(T) == 8 ? (NZ == 8 ? 8 : 4) : VY == 1 || (NZ <= 16 && NZ * (PC ? 4 : 3) * (JAC ? 4 : 3) < 16 * 4 * 3) ? NZ : NZ / 2;
        const unsigned tag = epoch + (unsigned)(j - 1);
        unsigned own = (unsigned)((j - 1) & 1) * par_bytes + (unsigned)slot * kTileBytes;
        asm volatile("" : "+s"(own));   // (as row_at)
        const unsigned qx = own + 8u * (2 * SY + (xs == 0 ? 0 : SX));
        const u64 *const qy = word(own + (w == 0 ? 0u : 8u * SY) + y_lane);
        u64 wy[LC][WT], wxv[XN][WT] = {};
        auto poll_x = [&]() {
#pragma unroll
            for (int m = 0; m < XN; ++m)
                if (wx[m]) {
#pragma unroll
                    for (int n = 0; n < WT; ++n) wxv[m][n] = get_word(word(qx + side_at[m]) + n);
                }
        };
        auto poll_y = [&](int lc) {
#pragma unroll
            for (int l = 0; l < LC; ++l)
#pragma unroll
                for (int n = 0; n < WT; ++n) wy[l][n] = get_word(qy + ((lc + l) * kWave * WT + n));
        };
        T du[VY];   // x - (value above), per row
        const T *so_row = rows + row_at(buf, self_s ? row0 : row0 - 1) + lane;
        const T *no_row = rows + row_at(buf, self_n ? row0 + VY - 1 : row0 + VY) + lane;
        // a group's values from LDS, fetched while the group before is computed
        struct Grp {
            T so[GL], no[GL];
        };
        auto fetch = [&](int lg) {
            Grp g;
#pragma unroll
            for (int q = 0; q < GL; ++q) {
                const int l = lg + q;
                g.so[q] = so_row[l * RS];
                g.no[q] = no_row[l * RS];
            }
            return g;
        };
        Grp cur = fetch(0);
        int new_row[VY];
#pragma unroll
        for (int v = 0; v < VY; ++v) new_row[v] = row_at(buf ^ 1, row0 + v) + lane;
#pragma unroll
        for (int lg = 0; lg < NZ; lg += GL) {
            Grp nxt = cur;
            if (lg + GL < NZ) nxt = fetch(lg + GL);
            // The group's cells step by step together: a wavefront issues an
            // operation that depends on the one before only after 8 cycles, one
            // that does not after 5.5, and two or fewer wavefronts share a SIMD.
            T f[VY][GL], a[VY][GL], ds[VY][GL], dn[VY][GL], dz[VY][GL], m[VY][GL];
            auto step = [&](auto &&body) {
#pragma unroll
                for (int q = 0; q < GL; ++q)
#pragma unroll
                    for (int v = 0; v < VY; ++v) body(lg + q, q, v);
                __builtin_amdgcn_sched_barrier(0);
            };
            step([&](int l, int q, int v) { f[v][q] = in[v][l] - right0(in[v][l]); });
            step([&](int l, int q, int v) { f[v][q] *= gxp[PC ? v : 0][l]; });   // flux to +x
            step([&](int l, int q, int v) { a[v][q] = sink[l] * in[v][l] + f[v][q]; });
            step([&](int l, int q, int v) { m[v][q] = in[v][l] - out[v][l]; });
            step([&](int, int q, int v) { a[v][q] -= left0(f[v][q]); });
            step([&](int l, int q, int v) {
                dn[v][q] = in[v][l] - (v == VY - 1 ? cur.no[q] : in[v + 1 < VY ? v + 1 : v][l]);
                if (!PC && v < VY - 1) dn[v][q] = half ? T(0) : dn[v][q];
                ds[v][q] = v == 0 ? in[v][l] - cur.so[q] : -dn[v > 0 ? v - 1 : 0][q];
            });
            step([&](int l, int q, int v) {
                T gs;
                if constexpr (PC) gs = v == 0 ? gs0[l] : gyp[v > 0 ? v - 1 : 0][l];
                else gs = gyl[l];
                a[v][q] += gs * ds[v][q];
            });
            step([&](int l, int q, int v) { m[v][q] = in[v][l] + c1 * m[v][q]; });
            step([&](int l, int q, int v) {
                T gn;
                if constexpr (PC) gn = gyp[v][l];
                else gn = gyl[l];
                a[v][q] += gn * dn[v][q];
            });
            step([&](int l, int q, int v) { dz[v][q] = in[v][l] - (l + 1 < NZ ? in[v][l + 1 < NZ ? l + 1 : l] : T(0)); });
            step([&](int l, int q, int v) {
                if (l > 0) a[v][q] -= gzu[l > 0 ? l - 1 : 0] * (q > 0 ? dz[v][q > 0 ? q - 1 : 0] : du[v]);
            });
            step([&](int l, int q, int v) { a[v][q] += gzu[l] * dz[v][q]; });
            step([&](int l, int q, int v) {
                a[v][q] = rr[v][l] - a[v][q];
                if constexpr (JAC) a[v][q] *= di[v][l];
            });
            step([&](int l, int q, int v) { out[v][l] = m[v][q] + c2 * a[v][q]; });
#pragma unroll
            for (int v = 0; v < VY; ++v) du[v] = dz[v][GL - 1];
            // a few layers at a time, formed here and not where they are used
            // after the wait below
#pragma unroll
            for (int q = 0; q < GL; ++q)
#pragma unroll
                for (int v = 0; v < VY; ++v) asm volatile("" : "+v"(out[v][lg + q]));
            // into the LDS copy at once (the LDS has time now); what the faces to
            // other tiles change is written again below
#pragma unroll
            for (int v = 0; v < VY; ++v)
#pragma unroll
                for (int q = 0; q < GL; ++q) rows[new_row[v] + (lg + q) * RS] = out[v][lg + q];
            if (lg + GL == IL) {
                poll_x();
                if (edgeS || edgeN) poll_y(0);
            }
            cur = nxt;
        }
        // ---- the faces to other tiles
        left = ra.spin;
        const bool edge_y = edgeS || edgeN;
        T xc[XN] = {};   // the x-edge cells' corrections
#pragma unroll
        for (int lc = 0; lc < NZ; lc += LC) {
            if (lc > 0 && edge_y) poll_y(lc);
            for (;;) {
                unsigned off = 0;   // any bit by which a word's tag differs
                if (lc == 0) {
#pragma unroll
                    for (int m = 0; m < XN; ++m)
                        if (wx[m]) {
#pragma unroll
                            for (int n = 0; n < WT; ++n) off |= (unsigned)(wxv[m][n] >> 32) ^ tag;
                        }
                }
                if (edge_y) {
#pragma unroll
                    for (int l = 0; l < LC; ++l)
#pragma unroll
                        for (int n = 0; n < WT; ++n) off |= (unsigned)(wy[l][n] >> 32) ^ tag;
                }
                if (__all(off == 0) || waited_out()) break;
                if (lc == 0) poll_x();
                if (edge_y) poll_y(lc);
            }
            if (lc == 0) {
#pragma unroll
                for (int m = 0; m < XN; ++m) {
                    xc[m] = c2 * (ge[m] * (value(wxv[m]) - xe[m]));
                    if constexpr (JAC) xc[m] *= de[m];
                }
            }
            auto y_face = [&](auto vt) {
                constexpr int v = decltype(vt)::value;
#pragma unroll
                for (int q = 0; q < LC; ++q) {
                    const int l = lc + q;
                    T g;
                    if constexpr (PC) g = w == 0 ? gs0[l] : gyp[v][l];
                    else g = gyl[l];
                    T c = c2 * (g * (value(wy[q]) - in[v][l]));
                    if constexpr (JAC) c *= di[v][l];
                    out[v][l] += c;
                    rows[new_row[v] + l * RS] = out[v][l];
                }
            };
            if (edgeS) y_face(std::integral_constant<int, 0>{});
            if (edgeN) y_face(std::integral_constant<int, VY - 1>{});
            if (!edge_y) break;
        }
        wait_loads();
        if (left <= 0) bad_s[j & 1] = 1;   // (any lane may write it: the value is the same)
#pragma unroll
        for (int m = 0; m < XN; ++m)
            if (wx[m]) {
                // the x-edge cell itself in the LDS copy, and its correction for the lane that holds it
                T *q = rows + (x_row[m] + (buf ^ 1) * (NR * NZ * RS));
                xe[m] = *q + xc[m];
                *q = xe[m];
                cx[x_at[m]] = xc[m];
            }
        if (x_edge) {
            constexpr int HV = 16 / sizeof(T);
#pragma unroll
            for (int v = 0; v < VY; ++v)
#pragma unroll
                for (int l = 0; l < NZ; l += HV) {
                    const Vec<T, HV> t = lds_load<T, HV>(cx + c_at + v * NZ + l);
#pragma unroll
                    for (int e = 0; e < HV; ++e) out[v][l + e] += t.a[e];
                }
        }
        return bad == 0;
    };

    // ---- the result and the partials of r^T z; false when a wait ran out
    auto finish = [&](const T(&z)[VY][NZ]) -> bool {
        T *zo = P.z[zout];
        T acc = T(0);
#pragma unroll
        for (int l = 0; l < NZ; ++l)
#pragma unroll
            for (int v = 0; v < VY; ++v)
                if (act && j0 + v >= own0 && j0 + v < own1 && l < nz) {
                    *as_global(zo + (int64_t)l * plane + (int64_t)(j0 + v) * nx + i) = z[v][l];
                    acc += rr[v][l] * z[v][l];
                }
        __shared__ T sh[NW];
        const T a = wave_sum(acc);
        if (lane == 0) sh[w] = a;
        __syncthreads();
        if (bad_s[0] | bad_s[1]) return false;
        // one partial per tile; the problem's other slots are zero
        for (int q = part + tid_lin() * P.r_ntiles; q < P.ntiles; q += nthreads() * P.r_ntiles) {
            T t = T(0);
            if (q == part) {
                t = sh[0];
                for (int v = 1; v < NW; ++v) t += sh[v];
            }
            part_out[P.tile0 + q] = t;
        }
        // every tile of a problem runs in the same launches, so all their epochs agree
        if (tid_lin() == 0) *as_global(ra.epoch + slot) = epoch + (unsigned)k;
        return true;
    };

    put_rows(za, 0);
#pragma unroll
    for (int n = 0; n < XN; ++n)
        if (wx[n]) xe[n] = rows[x_row[n]];
    wait_loads();
    send(za, 0);
    __syncthreads();
    bool ok = true;
    for (int j = 1;; j += 2) {
        if (!(ok = sweep(za, zb, j, 0))) break;
        if (j == k - 1) {
            ok = finish(zb);
            break;
        }
        send(zb, j);
        __syncthreads();
        if (!(ok = sweep(zb, za, j + 1, 1))) break;
        if (j + 1 == k - 1) {
            ok = finish(za);
            break;
        }
        send(za, j + 1);
        __syncthreads();
    }
    if (!ok && tid_lin() == 0)
        __hip_atomic_store(&st->gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Tiles blockIdx.x, blockIdx.x + gridDim.x, ... in turn.  All workgroups run at
// once and a group has no more tiles than there are workgroups, so a workgroup
// has at most one tile of a group, and by the time it waits in that the groups
// before are running elsewhere or done: no wait depends on a tile that cannot
// run.  (A grid of all tiles, handed out as workgroups start, is not enough: a
// workgroup stays on the XCD it was dispatched to, and one XCD can be full of
// waiting tiles whose neighbours queue for it while other XCDs idle.)
template <typename T, bool PC, bool JAC, int NZ, int VY, int NW>
__global__ __launch_bounds__(kWave *NW, 2) void k_cheb_res(const InnerProb<T> *__restrict__ probs,
                                                           int k, int zout, int chk,
                                                           const T *__restrict__ part_in, int red,
                                                           T *__restrict__ part_out, ResArgs ra) {
    for (int slot = blockIdx.x;;) {
        res_tile<T, PC, JAC, NZ, VY, NW>(probs, k, zout, chk, part_in, red, part_out, ra, slot);
        slot += gridDim.x;
        if (slot >= ra.tiles) break;
        __syncthreads();   // the next tile reuses the LDS
    }
}

// Cleared edge words (tag 0) and tile epochs of 1.
__global__ __launch_bounds__(256) void k_res_clear(u64 *buf, size_t words, size_t tiles) {
    const size_t n = (size_t)gridDim.x * blockDim.x, q0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (size_t q = q0; q < words; q += n) *as_global(buf + q) = 0;
    unsigned *epoch = reinterpret_cast<unsigned *>(buf + words);
    for (size_t q = q0; q < tiles; q += n) *as_global(epoch + q) = 1u;
}

// The launch arguments beyond the kernel's shape.
template <typename T>
struct Args {
    const InnerProb<T> *probs;
    int k, zout, chk;
    const T *part_in;
    int red;
    T *part_out;
    const ResArgs &ra;
    hipStream_t s;
};

template <typename T, bool PC, bool JAC, int NZ, int VY, int NW>
bool launch_one(const Args<T> &a) {
    if (a.probs)
        hipLaunchKernelGGL((k_cheb_res<T, PC, JAC, NZ, VY, NW>), dim3(a.ra.width), dim3(kWave, NW),
                           res_lds<T>(NZ, VY, NW), a.s, a.probs, a.k, a.zout, a.chk, a.part_in, a.red, a.part_out, a.ra);
    return true;
}
template <typename T, bool PC, bool JAC, int VY, int NW>
bool launch_nz(int nzc, const Args<T> &a) {
    switch (nzc) {
    case 8: return launch_one<T, PC, JAC, 8, VY, NW>(a);
    case 12: return launch_one<T, PC, JAC, 12, VY, NW>(a);
    case 16: return launch_one<T, PC, JAC, 16, VY, NW>(a);
    case 20:
        if constexpr (sizeof(T) == 4 && VY == 1) return launch_one<T, PC, JAC, 20, VY, NW>(a);
    }
    return false;
}
template <typename T, bool PC, bool JAC>
bool launch_tile(const ResShape &rs, const Args<T> &a) {
    if constexpr (sizeof(T) == 4)
        if (rs.vy == 2 && rs.nw == 8) return launch_nz<T, PC, JAC, 2, 8>(rs.nzc, a);
    if constexpr (sizeof(T) == 4 && !PC && !JAC)
        if (rs.vy == 2 && rs.nw == 7 && rs.nzc == 20) return launch_one<T, PC, JAC, 20, 2, 7>(a);
    if (rs.vy == 1 && rs.nw == 8) return launch_nz<T, PC, JAC, 1, 8>(rs.nzc, a);
    return false;
}

}  // namespace

void launch_res_clear(unsigned long long *buf, size_t words, size_t tiles, hipStream_t s) {
    const size_t nb = (words + 255) / 256;
    hipLaunchKernelGGL(k_res_clear, dim3((unsigned)(nb < 1024 ? (nb < 1 ? 1 : nb) : 1024)), dim3(256), 0, s,
                       reinterpret_cast<u64 *>(buf), words, tiles);
}

template <typename T>
bool launch_cheb_res(const ResShape &rs, const InnerProb<T> *probs, bool pc, bool jac, int k, int zout,
                     bool chk, const T *part_in, bool red, T *part_out, const ResArgs &ra, hipStream_t s) {
    const Args<T> a{probs, k, zout, (int)chk, part_in, (int)red, part_out, ra, s};
    if (pc) return jac ? launch_tile<T, true, true>(rs, a) : launch_tile<T, true, false>(rs, a);
    return jac ? launch_tile<T, false, true>(rs, a) : launch_tile<T, false, false>(rs, a);
}

template bool launch_cheb_res<float>(const ResShape &, const InnerProb<float> *, bool, bool, int, int, bool,
                                     const float *, bool, float *, const ResArgs &, hipStream_t);
template bool launch_cheb_res<double>(const ResShape &, const InnerProb<double> *, bool, bool, int, int, bool,
                                      const double *, bool, double *, const ResArgs &, hipStream_t);

}  // namespace cuth
