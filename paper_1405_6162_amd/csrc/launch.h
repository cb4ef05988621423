// Host side of liblb.so below the C ABI: the context, its memory layout, the
// launch policies and, per storage type, the launchers that queue kernels on
// the context's stream.  The launchers are instantiated once per storage type
// (launch_f64.hip, launch_f32.hip, launch_f16.hip), so the kernels of the
// three compile side by side.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>
#include <vector>

#include "../../include/lb.h"
#include "kernels.h"

namespace lbl {

using namespace lbk;

// Launch policy of every kernel in the library but the single-pass binary
// step (below): 64 x 4 sites per block, one site per lane, nontemporal
// stores (the next step reads the values from HBM anyway), XCD-ordered
// tiles.  Chosen by a sweep over tile shapes, sites per lane (1, 2, 4),
// nontemporal loads/stores and direction padding on 128^3 and 256^3
// lattices; the differences were within 5%.
using Pol = Tiling<64, 4, 1, false, true, true>;
// The same with ordinary stores: for states that stay in the 256 MB memory-side
// cache (kCachedBytes, both copies of every distribution), from which the next
// step then reads them.  us a step, ordinary / nontemporal stores: binary FP16
// 96^3 34 / 47, 112^3 (213 MB) 44 / 65, FP32 48^3 11.2 / 14.9, FP64 64^3 31 / 34;
// single fluid in pairs FP32 96^3 15.6 / 19.7, 112^3 22.9 / 30.0, one at a time
// FP64 64^3 12.9 / 17.0; beyond the cache they lose: FP64 128^3 261 / 247, 256^3
// 1919 / 1819.  So they do where a single fluid's state fits the eight 4 MB L2
// caches (kL2Bytes; BGK and TRT seven eighths of them), which have to write
// back what they hold after every launch: FP16 BGK 64^3 (20 MB) 5.4 / 5.2, 320 x 320
// x 2 (16 MB) 5.8 / 4.9, 64 x 53 x 96 (25 MB) 6.3 / 5.9, MRT 60^3 7.5 / 6.3, FP32 56^3
// (30 MB) MRT 6.9 / 6.2, BGK 6.1 / 6.9; 64^3 (40 MB) MRT 8.2 / 9.3.  The march gains at
// all sizes.
template <class P> using Cached = Tiling<P::TX, P::TY, P::TZ, P::nt_load, false, P::xcd>;
// The same for blocked states of 4 GiB and more a buffer, or an FP32 plane (layout_of).
template <class P> using Wide = Tiling<P::TX, P::TY, P::TZ, P::nt_load, P::nt_store, P::xcd, true>;
constexpr size_t kCachedBytes = 280000000;
constexpr size_t kL2Bytes = 32000000;
// Pol with 2 and 4 sites per lane along z (lb_params.vvl).
using Pol2 = Tiling<64, 4, 2, false, true, true>;
using Pol4 = Tiling<64, 4, 4, false, true, true>;
constexpr int kCUs = 256;
// Tiles of the single-pass binary step (k_binary_march).  A 64 x 8
// tile has 144 halo sites per 512 against 136 per 256 for 64 x 4, so
// the halo's phi gathers (mostly re-reads of neighbouring tiles' g) fall from
// 53% to 28% of the sites gathered: measured A/B on one box, 64 x 8 is 6.5%
// faster than 64 x 4 in FP64 at 256^3, 2% at 128^3, 3% in FP32 and 1% in FP16;
// 64 x 16 and 32 x 16 were slower in every storage.  In FP32 and FP16 a
// 128 x 4 tile, which has half the x-halo sites (whose gathers each hit
// a cache line of their own, 2 or 4 bytes used), is used where its rows leave
// no more lanes idle than 64-site rows (nx mod 128 is 0 or above 64): 200 x 204
// x 100 289 against 297 us in FP32, 384^3 1817 against 1840 in FP16.
using MarchTile = Tiling<64, 8, 1, false, true, true>;
using MarchTileWide = Tiling<128, 4, 1, false, true, true>;
// Blocks of the march the chip runs at once: one 512-lane block a CU where it
// is compiled for two waves per SIMD (FP64, FP32), two for four (FP16).
template <class S>
constexpr int march_slots() { return kCUs * MarchHold<S, 0>::waves * 4 * 64 / MarchTile::TPB; }
// Two single-fluid steps per launch (k_single_pair).  A CU holds one 512-lane
// block in FP64 (128 KB of LDS, up to 256 VGPRs a lane), and 1024 lanes in
// FP32 and FP16 (128 VGPRs): two blocks of 64 x 8 or, where 128-wide rows
// leave no more lanes idle, one of 128 x 8 (256^3: 490 against 559 us a pair
// in FP32, 355 against 384 in FP16).
// From kPairMinSites up a pair can beat two single steps (pair_pays).  us a step,
// in pairs / single: FP64 48^3 8.8 / 7.5, 64^3 11.1 / 12.9, 256^3 480 / 896; FP32
// 64^3 7.0 / 7.2, 256^3 250 / 450; FP16 112^3 24.5 / 18.4, 128^3 24.3 / 23.9, 256^3
// 174 / 224.
template <class S>
constexpr int64_t kPairMinSites = sizeof(S) == 8 ? 130000 : (sizeof(S) == 4 ? 200000 : 2000000);
using PairTile = Tiling<64, 8, 1, false, true, true>;
using PairTileWide = Tiling<128, 8, 1, false, true, true>;

constexpr size_t kAlign = 4096;
// Extra bytes between consecutive direction arrays, so the 19 (38) streams of
// a power-of-two lattice do not start on the same HBM channel (measured:
// 0 B padding is 5-10% slower than the best offsets; 9472 B = 37 x 256 B was
// among the best on 128^3 and 256^3).
constexpr size_t kDirPadBytes = 9472;

inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

inline size_t storage_size(int storage) { return storage == LB_F64 ? 8 : (storage == LB_F32 ? 4 : 2); }
inline size_t compute_size(int storage) { return storage == LB_F64 ? 8 : 4; }

struct Layout {
    int64_t nsite;
    int64_t dstride;        // elements between consecutive directions
    bool blocked;           // 64-site blocks holding their 19 directions together
    bool wide;              // blocked, with byte offsets beyond 32 bits
    bool wide_plane;        // blocked FP32, with byte offsets within a plane beyond 32 bits
    uint32_t zs, ys, xbs;   // site-offset strides (Geo)
    size_t dist_bytes;      // one 19-direction buffer
    size_t phi_bytes;
    int nblocks;
    size_t partial_bytes;
    size_t off_f[2], off_g[2], off_phi, off_partial, total;
};

inline int check_params(const lb_params* p) {
    if (!p) return LB_EINVAL;
    if (p->nx < 1 || p->ny < 1 || p->nz < 1) return LB_EINVAL;
    const int64_t n = (int64_t)p->nx * p->ny * p->nz;
    // Kernels form byte offsets of FP64 arrays in 32 bits: N * 8 < 2^32.
    if (n >= ((int64_t)1 << 29)) return LB_EINVAL;
    if (p->model != LB_SINGLE && p->model != LB_BINARY) return LB_EINVAL;
    if (p->storage != LB_F64 && p->storage != LB_F32 && p->storage != LB_F16) return LB_EINVAL;
    if (p->vvl != 0 && p->vvl != 1 && p->vvl != 2 && p->vvl != 4) return LB_EINVAL;
    if (p->binary_step < LB_STEP_AUTO || p->binary_step > LB_STEP_TWO_PASS) return LB_EINVAL;
    if (p->collision != LB_BGK && p->collision != LB_TRT && p->collision != LB_MRT) return LB_EINVAL;
    auto valid_tau = [](double t) { return std::isfinite(t) && t > 0.5; };
    if (p->collision != LB_BGK && !valid_tau(p->tau_minus)) return LB_EINVAL;
    if (p->collision == LB_MRT &&
        (!valid_tau(p->tau_bulk) || !valid_tau(p->tau_ghost_even) || !valid_tau(p->tau_ghost_odd)))
        return LB_EINVAL;
    if (!std::isfinite(p->tau_f) || !(p->tau_f > 0.5)) return LB_EINVAL;
    if (p->model == LB_BINARY) {
        if (!std::isfinite(p->A) || !std::isfinite(p->B) || !std::isfinite(p->kappa)) return LB_EINVAL;
        if (!(p->kappa >= 0.0)) return LB_EINVAL;
        if (!std::isfinite(p->mobility) || !(p->mobility > 0.0)) return LB_EINVAL;
        if (!std::isfinite(p->gamma) || !(p->gamma > 0.0)) return LB_EINVAL;
    }
    if (!std::isfinite(p->rho0) || !std::isfinite(p->phi0)) return LB_EINVAL;
    return LB_OK;
}

inline Layout layout_of(const lb_params* p) {
    Layout L{};
    L.nsite = (int64_t)p->nx * p->ny * p->nz;
    const size_t es = storage_size(p->storage);
    // Blocked layout (see Geo) whenever a buffer's offsets fit in 32 bits (in
    // bytes; for 4-byte elements, which are addressed by element, in elements);
    // the last x block of a row is padded to 64 sites.  Measured A/B on one
    // box against the structure-of-arrays layout: the single-fluid step
    // +4.6% (FP64) and +5.6% (FP32) at 256^3, the binary march +4.3% (FP64,
    // 256^3), +3.0% (FP64, 128^3), +3.6% (FP16, 384^3) and +2.5 to +5.6%
    // (FP32, 128^3 to 256^3); padding between the buffers changed none of
    // these.
    // From 4 GiB a buffer up, where the blocks need no more room than the
    // structure of arrays (a lattice that fitted still does), the kernels take
    // offsets by element (Wide) and the marching ones, whose bases are per
    // plane, are as below 4 GiB: FP64 320^3 us a step, blocked / structure of
    // arrays, 3652 / 3966 binary.  A state with more than one site per lane
    // keeps the arrays.  Planes of 4 GiB are blocked in FP32, whose marching
    // kernels then take element offsets, for the binary fluid (8192 x 8192 x 1
    // 4590 / 4910, x 2 8753 / 9120); the single fluid's pairs gain more from byte
    // offsets (8192 x 8192 x 2 3046 structure of arrays, 3607 blocked single steps).
    const uint64_t xblocks = (uint64_t)tiles(p->nx, 64);
    const uint64_t blocked_elems = (uint64_t)p->nz * (uint64_t)p->ny * xblocks * Q * 64;
    const size_t stride_bytes = round_up((size_t)L.nsite * es, kAlign) + kDirPadBytes;
    const size_t soa_bytes = round_up(stride_bytes * Q, kAlign);
    const uint64_t u32 = (uint64_t)1 << 32;
    const bool small_plane = blocked_elems / (uint64_t)p->nz * es < u32;   // PlaneBase's offsets
    L.blocked = (es == 4 ? blocked_elems : blocked_elems * es) < u32 && (small_plane || p->model == LB_BINARY);
    L.wide_plane = L.blocked && !small_plane;
    if (!L.blocked && small_plane && es != 4 && p->vvl <= 1)
        L.blocked = L.wide = blocked_elems < u32 && blocked_elems * es <= soa_bytes;
    if (L.blocked) {
        L.dstride = 64;
        L.xbs = Q * 64;
        L.ys = (uint32_t)(xblocks * L.xbs);
        L.zs = (uint32_t)((uint64_t)p->ny * L.ys);
        L.dist_bytes = L.wide ? soa_bytes : round_up((size_t)blocked_elems * es, kAlign);
    } else {
        L.dstride = (int64_t)(stride_bytes / es);
        L.xbs = 64;
        L.ys = (uint32_t)p->nx;
        L.zs = (uint32_t)p->nx * (uint32_t)p->ny;
        L.dist_bytes = soa_bytes;
    }
    L.phi_bytes = round_up((size_t)L.nsite * compute_size(p->storage), kAlign);
    L.nblocks = tiles(p->nx, Pol::TX) * tiles(p->ny, Pol::TY) * tiles(p->nz, Pol::TZ);
    L.partial_bytes = round_up((size_t)L.nblocks * 16 * sizeof(double), kAlign);
    size_t o = 0;
    for (int b = 0; b < 2; ++b) { L.off_f[b] = o; o += L.dist_bytes; }
    if (p->model == LB_BINARY) {
        for (int b = 0; b < 2; ++b) { L.off_g[b] = o; o += L.dist_bytes; }
        L.off_phi = o; o += L.phi_bytes;
    } else {
        L.off_g[0] = L.off_g[1] = L.off_phi = 0;
    }
    L.off_partial = o; o += L.partial_bytes;
    L.total = o;
    return L;
}

// Chunks a marching kernel cuts nz planes into, `columns` tile columns and
// `slots` blocks at a time.  A chunk of d planes costs about d + 3 (its ends take
// two planes of phi, or of step one, more): nz is cut, evenly, into the number
// of chunks (at most 128 planes each) that makes rounds x (d + 3) least.
// Measured against fixed counts, us a step, FP64: pairs 256^3 480 with 2 chunks
// (one round), 512 with 4; 128^3 69 with 8 (one round), 80 with 16.  March 96^3
// 126 with 10 chunks (240 blocks), 163 with 6; 160^3 496 with 4 (one round), 511
// with 8; 64^3 31 with 32 chunks of 2 planes, 93 with 4 of 16.
//
// This runs at every launch, so it may not take time that grows with nz (1 x 1 x
// 4e8, every count tried: 0.9 s a launch).  All counts from c to the last that
// needs no more rounds cost the least at their least depth, whose fewest
// chunks are taken; and no count from c on costs less than columns x nz / slots
// + 3 rounds(c), where the search ends: 10 to 100 counts.
inline int chunks_of(int64_t columns, int nz, int slots) {
    int64_t best = INT64_MAX;
    int chunks = 1;
    for (int64_t c = lbk::tiles(nz, 128); c <= nz;) {
        const int64_t rounds = (columns * c + slots - 1) / slots;
        if (columns * nz / slots + 3 * rounds >= best) break;
        const int64_t last = std::min<int64_t>(nz, rounds * slots / columns), depth = (nz + last - 1) / last;
        if (rounds * (depth + 3) < best) {
            best = rounds * (depth + 3);
            chunks = (int)std::max(c, (nz + depth - 1) / depth);
        }
        c = last + 1;
    }
    return chunks;
}

struct Rec { int kind; hipEvent_t start, stop; };

}  // namespace lbl

struct lb_ctx {
    lb_params p;
    lbl::Layout L;
    hipStream_t stream;
    char* ws;
    int cur;          // buffer index holding the state
    bool pending;     // true: the state is propagate(buffer[cur])
    bool profiling;
    unsigned profile_kinds;   // bit k: time launches of kernel class k
    bool launched;    // any device work queued (lb_destroy waits for it)
    std::vector<lbl::Rec> recs;
    std::vector<hipEvent_t> pool;

    lbk::Geo geo() const {
        lbk::Geo g;
        g.nx = p.nx; g.ny = p.ny; g.nz = p.nz;
        g.plane = (uint32_t)p.nx * (uint32_t)p.ny;
        g.nsite = (uint32_t)L.nsite;
        g.dstride = L.dstride;
        g.gx = lbk::tiles(p.nx, lbl::Pol::TX);
        g.gy = lbk::tiles(p.ny, lbl::Pol::TY);
        g.gz = lbk::tiles(p.nz, lbl::Pol::TZ);
        g.nblocks = g.gx * g.gy * g.gz;
        g.zs = L.zs; g.ys = L.ys; g.xbs = L.xbs;
        return g;
    }
    // g with the layout of canonical caller arrays: direction stride N, x fastest
    lbk::Geo canonical(lbk::Geo g) const {
        g.dstride = L.nsite;
        g.zs = g.plane; g.ys = (uint32_t)p.nx; g.xbs = 64;
        return g;
    }
    lbk::Geo canonical_geo() const { return canonical(geo()); }
    template <class P>
    lbk::Geo geo_for() const {
        lbk::Geo g = geo();
        g.gz = lbk::tiles(p.nz, P::TZ);
        g.nblocks = g.gx * g.gy * g.gz;
        return g;
    }
    // Tiling of a marching kernel (k_binary_march, k_single_pair) of which the
    // chip runs `slots` blocks at a time.
    template <class TP>
    lbk::Geo column_geo(int slots) const {
        lbk::Geo g = geo();
        g.gx = lbk::tiles(p.nx, TP::TX);
        g.gy = lbk::tiles(p.ny, TP::TY);
        g.gz = lbl::chunks_of((int64_t)g.gx * g.gy, p.nz, slots);
        g.nblocks = g.gx * g.gy * g.gz;
        return g;
    }
    // Whether ordinary stores keep the state where the next step reads it (see Cached).
    bool cached() const {
        if (p.model == LB_BINARY) return 4 * L.dist_bytes <= lbl::kCachedBytes;
        const size_t least = p.collision == LB_MRT ? lbl::kL2Bytes : lbl::kL2Bytes / 8 * 7;
        return 2 * L.dist_bytes > least && 2 * L.dist_bytes <= lbl::kCachedBytes;
    }
    // The same for copies from the state to the caller's arrays, which no step reads:
    // only where rows end within 64 bytes, which a nontemporal store then writes in
    // parts.  us a copy out, ordinary / nontemporal: FP32 100^3 28.7 / 37.1, binary
    // FP16 80^3 17.5 / 25.4; rows of whole 64 bytes FP32 64^3 6.1 / 5.2, 80^3 15.0 / 14.3,
    // binary FP64 48^3 12.4 / 10.7.  (Copies into the state are as its steps' stores:
    // binary FP64 64^3, a record of one step, 62.0 / 68.4.)
    bool cached_copy() const { return cached() && (size_t)p.nx * lbl::storage_size(p.storage) % 64 != 0; }
    // Whether 128-wide tiles leave no more lanes of a row idle than 64-wide ones.
    bool wide_rows() const { return lbk::tiles(p.nx, 128) * 2 == lbk::tiles(p.nx, 64); }
    dim3 grid() const { return dim3(L.nblocks); }
    static dim3 block() { return dim3(lbl::Pol::TPB); }
    void* fbuf(int b) const { return ws + L.off_f[b]; }
    void* gbuf(int b) const { return p.model == LB_BINARY ? ws + L.off_g[b] : nullptr; }
    void* phi() const { return ws + L.off_phi; }
    double* partial() const { return reinterpret_cast<double*>(ws + L.off_partial); }

    // Timing-only events.  An ordinary event record ends with a system-scope
    // fence (cache write-back and invalidation); between two dependent
    // launches of the 128^3 binary step with profiling on, the rocprofv3
    // kernel trace shows 11 us gaps with it and 8.5 us without.  Without it
    // the profiled 64^3 adjoint rollout runs 12% faster and the 128^3 binary
    // step 1%.  The events are only
    // ever read by lb_kernel_times.
    hipEvent_t take_event() {
        if (!pool.empty()) { hipEvent_t e = pool.back(); pool.pop_back(); return e; }
        hipEvent_t e = nullptr;
        if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) return nullptr;
        return e;
    }
    void release_records() {
        for (auto& r : recs) { pool.push_back(r.start); pool.push_back(r.stop); }
        recs.clear();
    }
};

namespace lbl {

// Brackets one launch with an event pair when profiling is on.
struct Timed {
    lb_ctx* c; int kind; hipEvent_t a = nullptr, b = nullptr;
    Timed(lb_ctx* c_, int kind_) : c(c_), kind(kind_) {
        if (c->profiling && ((c->profile_kinds >> kind) & 1u)) {
            a = c->take_event(); b = c->take_event();
            if (a && b) (void)hipEventRecord(a, c->stream);
        }
    }
    ~Timed() {
        if (a && b) {
            (void)hipEventRecord(b, c->stream);
            c->recs.push_back({kind, a, b});
        } else {
            if (a) c->pool.push_back(a);
            if (b) c->pool.push_back(b);
        }
    }
};

inline int launch_status() { return hipGetLastError() == hipSuccess ? LB_OK : LB_EDEVICE; }



template <class S>
CollParams<typename Compute<S>::T> coll_params(const lb_ctx* c) {
    using T = typename Compute<S>::T;
    CollParams<T> cp;
    cp.omega_f = (T)(1.0 / c->p.tau_f);
    const double tau_g = c->p.model == LB_BINARY ? c->p.mobility / c->p.gamma + 0.5 : 1.0;
    cp.omega_g = (T)(1.0 / tau_g);
    cp.A = (T)c->p.A; cp.B = (T)c->p.B; cp.kappa = (T)c->p.kappa; cp.gamma = (T)c->p.gamma;
    const bool dev = c->p.storage != LB_F64;
    cp.rho0 = dev ? (T)c->p.rho0 : T(0);
    cp.phi0 = dev ? (T)c->p.phi0 : T(0);
    cp.omega_m = c->p.collision != LB_BGK ? (T)(1.0 / c->p.tau_minus) : cp.omega_f;
    const bool mrt = c->p.collision == LB_MRT;
    cp.omega_b = mrt ? (T)(1.0 / c->p.tau_bulk) : cp.omega_f;
    cp.omega_ge = mrt ? (T)(1.0 / c->p.tau_ghost_even) : cp.omega_f;
    cp.omega_go = mrt ? (T)(1.0 / c->p.tau_ghost_odd) : cp.omega_m;
    return cp;
}

// ----- typed launchers ------------------------------------------------------

// Calls fn with the launch policy of the context's sites per lane.
template <class F>
int by_vvl(const lb_ctx* c, F&& fn) {
    switch (c->p.vvl) {
        case 0: case 1: return c->L.wide ? fn(Wide<Pol>{}) : (c->cached() ? fn(Cached<Pol>{}) : fn(Pol{}));
        case 2: return fn(Pol2{});
        case 4: return fn(Pol4{});
    }
    return LB_EINVAL;
}

// Calls fn with the policy of a kernel that has one site per lane and stores
// no distributions.
template <class F>
int by_width(const lb_ctx* c, F&& fn) {
    return c->L.wide ? fn(Wide<Pol>{}) : fn(Pol{});
}

template <class S>
int run_phi(lb_ctx* c) {
    using T = typename Compute<S>::T;
    Timed t(c, LB_K_PHI);
    const S* g = (const S*)c->gbuf(c->cur);
    const T phi0 = coll_params<S>(c).phi0;
    by_vvl(c, [&](auto pol) {
        using P = decltype(pol);
        const Geo geo = c->template geo_for<P>();
        if (c->pending) k_phi<P, S, true><<<geo.nblocks, P::TPB, 0, c->stream>>>(g, (T*)c->phi(), geo, phi0);
        else k_phi<P, S, false><<<geo.nblocks, P::TPB, 0, c->stream>>>(g, (T*)c->phi(), geo, phi0);
        return 0;
    });
    return launch_status();
}

// Whether the context's stream is being captured into a graph (the null
// stream never is).
inline bool capturing(const lb_ctx* c) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (c->stream && hipStreamIsCapturing(c->stream, &status) != hipSuccess) (void)hipGetLastError();
    return status != hipStreamCaptureStatusNone;
}

// Calls fn with the context's collision as an integral constant.
template <class F>
void by_collision(const lb_ctx* c, F&& fn) {
    if (c->p.collision == LB_TRT) fn(std::integral_constant<int, COLL_TRT>{});
    else if (c->p.collision == LB_MRT) fn(std::integral_constant<int, COLL_MRT>{});
    else fn(std::integral_constant<int, COLL_BGK>{});
}

// Grid of a marching kernel of which the chip runs `slots` blocks at once
// (tile_of_block).  Blocks that all run at once take their tiles in XCD order.  In
// several rounds each XCD's run of tiles would be swept at a place of its own in
// the lattice; in launch order the chip sweeps one place, whose neighbour lines
// then come from the memory-side cache.  us a step, launch / XCD order: several
// rounds, FP64 320^3 binary 3652 / 3808, single 1001 / 1044, 300 x 240 x 220
// binary 1927 / 2022, FP32 320^3 binary 1881 / 1960, 512 x 512 x 24 367 / 388; one
// round, FP64 256^3 binary 1864 / 1820, single 505 / 479, 128^3 256 / 245, FP32
// 256^3 932 / 907.  FP32 pairs and FP16 show no rule (-5 to +3%) and keep XCD order.
// So do the march's short chunks: they are no sweep worth the name, and what their
// ends read again comes from an XCD's own L2 (march_order).
inline unsigned march_grid(const Geo& g, int slots, bool launch_order) {
    const int n = g.nblocks;
    if (launch_order && n > slots) return (unsigned)(n % 8 != 0 ? n : n + 1);
    return (unsigned)((n + 7) / 8 * 8);
}

// Whether the march's tiles go in launch order where they need several rounds.
// us a step, launch / XCD order: chunks of 3 to 15 planes FP32 512 x 512 x 4 79.7 /
// 70.3, x 12 193.4 / 189.0, 1024 x 1024 x 4 272 / 260, FP64 512 x 512 x 4 138 / 133; two
// planes FP64 1024 x 1024 x 2 283 / 269, FP32 2048 x 2048 x 2 500 / 519; one plane FP32
// 2048 x 2048 276 / 285, FP64 560 / 559; within the cache FP32 512 x 512 x 2 35.7 / 29.0,
// 512 x 512 20.4 / 18.8.  Pairs go either way at every depth (FP64 512 x 512 x 4 40.8 /
// 42.2, x 2 24.7 / 21.2).
template <class S>
bool march_order(const lb_ctx* c, const Geo& g) {
    const int depth = tiles(g.nz, g.gz);
    return sizeof(S) > 2 && (depth > 15 || (depth < (sizeof(S) == 8 ? 2 : 3) && !c->cached()));
}

// One march from the pending state (fs, gs) to (fd, gd), all in the layout of
// geo() or canonical; phi, if not NULL, receives the order parameter of the
// state it collides.
//
// What is loaded ahead (MarchHold): the next plane's f and g, in FP16 only with
// 64 x 8 tiles (160^3 173 against 183 us, 192^3 237 against 253; with 128 x 4 ones,
// whose ring is another 264 gathers, it costs 1% at 384^3); in FP32 the ring's g
// too with 128 x 4 tiles and, with 64 x 8 ones, from 6 million sites up (192^3 419
// against 432 us, 320^3 1947 against 1996; 160^3 261 against 250).  Not in FP64 and
// FP32 chunks of 4 to 7 planes beyond the cache, taken in several rounds, where
// filling the pipeline is much of a block's work: FP32 512 x 512 x 4 66.8 against
// 70.3, 1024 x 1024 x 4 256 against 260, FP64 512 x 512 x 4 131.7 against 133.0, x 6
// 195 against 197; x 8 equal, 1024 x 1024 x 8 FP32 512 against 495.
template <class S, bool BLK, bool PHI_OUT>
int launch_march(lb_ctx* c, const S* fs, const S* gs, S* fd, S* gd, bool canonical, typename Compute<S>::T* phi) {
    const auto cp = coll_params<S>(c);
    auto with = [&](auto tiling, auto ahead) {
        using TP = decltype(tiling);
        Geo g = c->template column_geo<TP>(march_slots<S>());
        if (canonical) g = c->canonical(g);
        Timed t(c, LB_K_COLLIDE);
        by_collision(c, [&](auto coll) {
            k_binary_march<TP, S, PHI_OUT, decltype(coll)::value, BLK, decltype(ahead)::value>
                <<<march_grid(g, march_slots<S>(), march_order<S>(c, g)), TP::TPB, 0, c->stream>>>(fs, gs, fd, gd, g, cp, phi);
        });
    };
    // records and structure-of-arrays states are far larger than the cache
    auto launch = [&](auto tiling, auto ahead) {
        using TP = decltype(tiling);
        if constexpr (BLK && !PHI_OUT) {
            if constexpr (sizeof(S) == 4) {
                if (c->L.wide_plane) { with(Wide<TP>{}, ahead); return; }
            }
            if (c->cached()) { with(Cached<TP>{}, ahead); return; }
            if constexpr (sizeof(S) > 2) {
                const Geo g = c->template column_geo<TP>(march_slots<S>());
                const int depth = tiles(g.nz, g.gz);
                if (g.nblocks > march_slots<S>() && depth >= 4 && depth < 8) {
                    with(tiling, std::integral_constant<int, 0>{});
                    return;
                }
            }
        }
        with(tiling, ahead);
    };
    constexpr std::integral_constant<int, 0> nothing{};
    constexpr std::integral_constant<int, 1> own{};
    constexpr std::integral_constant<int, 2> ring{};
    if constexpr (sizeof(S) == 8) {
        launch(MarchTile{}, own);
    } else if constexpr (sizeof(S) == 4) {
        if (c->wide_rows()) launch(MarchTileWide{}, ring);
        else if (c->L.nsite >= 6000000) launch(MarchTile{}, ring);
        else launch(MarchTile{}, own);
    } else {
        if (c->wide_rows()) launch(MarchTileWide{}, nothing);
        else launch(MarchTile{}, own);
    }
    return launch_status();
}

// Single-pass binary step from a pending buffer; on return the state is direct.
template <class S>
int run_binary_march(lb_ctx* c) {
    const int src = c->cur, dst = 1 - c->cur;
    const S* fs = (const S*)c->fbuf(src);
    const S* gs = (const S*)c->gbuf(src);
    S* fd = (S*)c->fbuf(dst);
    S* gd = (S*)c->gbuf(dst);
    const int rc = c->L.blocked ? launch_march<S, true, false>(c, fs, gs, fd, gd, false, nullptr)
                                : launch_march<S, false, false>(c, fs, gs, fd, gd, false, nullptr);
    if (rc) return rc;
    c->cur = dst;
    c->pending = false;
    return LB_OK;
}

// Which binary step LB_STEP_AUTO takes.  One launch of the march beats the
// two of the two-pass step (phi pass + fused collide, every site in parallel)
// but on small FP64 lattices, whose few blocks each run a plane's gathers and
// FP64 collision in sequence.  us a step, march / two-pass:
//          24^3        32^3        40^3        48^3        56^3        64^3        80^3        96^3        112^3
//   FP64  12.0 / 9.6  13.0 / 10.4 14.3 / 14.3 19.6 / 18.3 24.7 / 27.9 31.1 / 33.1 82.1 / 87.2 125 / 135   177 / 203
//   FP32   6.6 / 8.2   6.9 / 8.5   8.5 / 10.4 11.4 / 13.4 13.4 / 16.7 15.4 / 18.9 33.2 / 38.0 59.6 / 64.9  96 / 101
//   FP16   7.1 / 8.2   7.3 / 8.2   8.1 / 9.9  11.3 / 11.8 12.3 / 13.9 12.4 / 14.6 27.9 / 29.9 34.1 / 39.8  45 / 53
// Of 60 random FP64 boxes of 200000 to 1.9 million sites the march lost on five,
// by 1 to 5%, and won by 9% on average.
// Fewer than six rows leave much of a march block idle, whose wavefronts work all
// the same: FP64 700 x 3 x 300 93 / 87, 700 x 5 x 200 102 / 97, 2048 x 1 x 256 142 /
// 80; in the other storages beyond the cache (Cached): 4 x 4 x 16384 FP32 191 / 171,
// FP16 186 / 158, 2 x 2 x 50000 FP32 411 / 325; within it 700 x 3 x 300 41 / 47.
// With more than one site per lane, which only the two-pass kernels have, the
// march runs from 256 blocks of at most 16 planes up: 512 x 512 x 4 with vvl 2 FP64
// 131 / 147, FP32 67 / 73; 128^3 247 / 300.  The two paths give the same bits.
template <class S>
bool march_pays(const lb_ctx* c) {
    if (c->p.binary_step == LB_STEP_MARCH) return true;
    if (c->p.binary_step == LB_STEP_TWO_PASS) return false;
    if (c->p.vvl > 1)
        return (int64_t)tiles(c->p.nx, MarchTile::TX) * tiles(c->p.ny, MarchTile::TY) * tiles(c->p.nz, 16) >= kCUs;
    if (c->p.ny < 6 && (sizeof(S) == 8 || !c->cached())) return false;
    return sizeof(S) != 8 || c->L.nsite >= 200000;
}

// One collision of the logical state; on return the state is direct.
template <class S>
int run_collide(lb_ctx* c) {
    using T = typename Compute<S>::T;
    const bool bin = c->p.model == LB_BINARY;
    if (bin && c->pending && march_pays<S>(c)) return run_binary_march<S>(c);
    if (bin) { int rc = run_phi<S>(c); if (rc) return rc; }
    const auto cp = coll_params<S>(c);
    const int src = c->cur, dst = c->pending ? 1 - c->cur : c->cur;
    const S* fs = (const S*)c->fbuf(src); S* fd = (S*)c->fbuf(dst);
    const S* gs = (const S*)c->gbuf(src); S* gd = (S*)c->gbuf(dst);
    const T* phi = (const T*)c->phi();
    {
        Timed t(c, LB_K_COLLIDE);
        by_vvl(c, [&](auto pol) {
            using P = decltype(pol);
            const Geo geo = c->template geo_for<P>();
            const dim3 grid(geo.nblocks), block(P::TPB);
            if (bin && c->p.collision == LB_TRT) {
                if (c->pending) k_collide<P, MODEL_BINARY, S, true, COLL_TRT><<<grid, block, 0, c->stream>>>(fs, gs, fd, gd, phi, geo, cp);
                else k_collide<P, MODEL_BINARY, S, false, COLL_TRT><<<grid, block, 0, c->stream>>>(fs, gs, fd, gd, phi, geo, cp);
            } else if (bin && c->p.collision == LB_MRT) {
                if (c->pending) k_collide<P, MODEL_BINARY, S, true, COLL_MRT><<<grid, block, 0, c->stream>>>(fs, gs, fd, gd, phi, geo, cp);
                else k_collide<P, MODEL_BINARY, S, false, COLL_MRT><<<grid, block, 0, c->stream>>>(fs, gs, fd, gd, phi, geo, cp);
            } else if (bin) {
                if (c->pending) k_collide<P, MODEL_BINARY, S, true><<<grid, block, 0, c->stream>>>(fs, gs, fd, gd, phi, geo, cp);
                else k_collide<P, MODEL_BINARY, S, false><<<grid, block, 0, c->stream>>>(fs, gs, fd, gd, phi, geo, cp);
            } else if (c->p.collision == LB_TRT) {
                if (c->pending) k_collide<P, MODEL_SINGLE, S, true, COLL_TRT><<<grid, block, 0, c->stream>>>(fs, gs, fd, gd, phi, geo, cp);
                else k_collide<P, MODEL_SINGLE, S, false, COLL_TRT><<<grid, block, 0, c->stream>>>(fs, gs, fd, gd, phi, geo, cp);
            } else if (c->p.collision == LB_MRT) {
                if (c->pending) k_collide<P, MODEL_SINGLE, S, true, COLL_MRT><<<grid, block, 0, c->stream>>>(fs, gs, fd, gd, phi, geo, cp);
                else k_collide<P, MODEL_SINGLE, S, false, COLL_MRT><<<grid, block, 0, c->stream>>>(fs, gs, fd, gd, phi, geo, cp);
            } else {
                if (c->pending) k_collide<P, MODEL_SINGLE, S, true><<<grid, block, 0, c->stream>>>(fs, gs, fd, gd, phi, geo, cp);
                else k_collide<P, MODEL_SINGLE, S, false><<<grid, block, 0, c->stream>>>(fs, gs, fd, gd, phi, geo, cp);
            }
            return 0;
        });
    }
    int rc = launch_status();
    if (rc) return rc;
    c->cur = dst;
    c->pending = false;
    return LB_OK;
}

// Copy a state (f, and g for the binary model) from layout sgeo to layout
// dgeo, site by site (the context's layout <-> canonical caller memory, or its
// own layout to itself), pulled when GATHER; with ordinary stores if `cached`.
template <class S, bool GATHER>
int run_copy(lb_ctx* c, const S* fs, const S* gs, S* fd, S* gd, const Geo& sgeo, const Geo& dgeo, bool cached) {
    auto with = [&](auto pol) {
        using P = decltype(pol);
        if (c->p.model == LB_BINARY)
            k_stream2<P, S, GATHER><<<c->grid(), c->block(), 0, c->stream>>>(fs, gs, fd, gd, sgeo, dgeo);
        else
            k_stream<P, S, GATHER><<<c->grid(), c->block(), 0, c->stream>>>(fs, fd, sgeo, dgeo);
        return launch_status();
    };
    return c->L.wide ? with(Wide<Pol>{}) : (cached ? with(Cached<Pol>{}) : with(Pol{}));
}

// Materialise propagate(buffer[src]) into (f, g) of layout dgeo.
template <class S>
int run_stream_into(lb_ctx* c, int src, S* f, S* g, const Geo& dgeo, bool cached) {
    Timed t(c, LB_K_STREAM);
    return run_copy<S, true>(c, (const S*)c->fbuf(src), (const S*)c->gbuf(src), f, g, c->geo(), dgeo, cached);
}

template <class S>
int run_convert(lb_ctx* c, const S* fs, const S* gs, S* fd, S* gd, const Geo& sgeo, const Geo& dgeo, bool cached) {
    return run_copy<S, false>(c, fs, gs, fd, gd, sgeo, dgeo, cached);
}

template <class S>
int run_propagate(lb_ctx* c) {
    if (!c->pending) { c->pending = true; return LB_OK; }   // propagation of a direct buffer is deferred
    const int dst = 1 - c->cur;
    int rc = run_stream_into<S>(c, c->cur, (S*)c->fbuf(dst), (S*)c->gbuf(dst), c->geo(), c->cached());
    if (rc) return rc;
    c->cur = dst;
    return LB_OK;
}

// Blocks of k_single_pair the chip runs at once: FP64 one 512-lane block a CU,
// FP32 and FP16 1024 lanes.
template <class S, class TP>
constexpr int pair_slots() { return kCUs * (sizeof(S) == 8 ? 1 : 1024 / TP::TPB); }

// Two collisions, with the propagation between them, of the state in `src`
// (a pending one is pulled), into `dst`; REC: the first one's values into
// `mid`.  All three in the layout of geo().
template <class S, bool BLK, bool REC>
int launch_single_pair(lb_ctx* c, bool pending, const S* src, S* mid, S* dst, bool canonical) {
    const auto cp = coll_params<S>(c);
    auto with = [&](auto tiling) {
        using TP = decltype(tiling);
        const int slots = pair_slots<S, TP>();
        Geo g = c->template column_geo<TP>(slots);
        if (canonical) g = c->canonical(g);
        const dim3 grid(march_grid(g, slots, sizeof(S) == 8)), block(TP::TPB);
        Timed t(c, LB_K_COLLIDE);
        by_collision(c, [&](auto coll) {
            constexpr int COLL = decltype(coll)::value;
            if (pending) k_single_pair<TP, S, true, COLL, BLK, REC><<<grid, block, 0, c->stream>>>(src, mid, dst, g, cp);
            else k_single_pair<TP, S, false, COLL, BLK, REC><<<grid, block, 0, c->stream>>>(src, mid, dst, g, cp);
        });
    };
    auto launch = [&](auto tiling) {
        if constexpr (BLK && !REC) {
            if (c->cached()) { with(Cached<decltype(tiling)>{}); return; }
        }
        with(tiling);
    };
    if constexpr (sizeof(S) < 8) {
        if (c->wide_rows()) { launch(PairTileWide{}); return launch_status(); }
    }
    launch(PairTile{});
    return launch_status();
}

// Whether two single-fluid steps run as one launch.  A single step moves its bytes
// at the rate of a copy, a pair half of them, but its lanes do step one also in
// the planes a chunk leads in and out over, and do all of their work where they
// are idle.  Lanes a site, with the idle rows of a tile, which load nothing of
// their own, at three quarters: x * (1 + 3/4 (y - 1)) * z.  us a step, pair /
// single, by lanes a site at nz of 1 to 8 planes of 2048 x 2048 (1024 x 1024 x 8):
//                3           2           1.67        1.5         1.25        gain up to
//   FP64 BGK  228 / 224   378 / 444   495 / 679   598 / 885   286 / 447     2.7
//        TRT  242 / 224   391 / 442   513 / 676   616 / 881   295 / 448     2.5
//        MRT  282 / 224   424 / 443   568 / 677   708 / 882   328 / 445     2.05
//   FP32 BGK  102 / 114   170 / 226   237 / 343   300 / 445   145 / 225     3.05
//        TRT  112 / 114   177 / 226   243 / 343   310 / 445   148 / 225     2.9
//        MRT  152 / 115   222 / 226   297 / 343   373 / 443   168 / 225     2
//   FP16 BGK   93 / 56    134 / 112   179 / 168   231 / 222   103 / 110     1.4
//        TRT  116 / 56    164 / 114   216 / 169   267 / 221   118 / 111     1.15 (256^3 204 / 225)
// (few rows: FP64 BGK 2048 x 1 x 256 52 / 24, 2 rows 64 / 60, 3 71 / 88, 4 77 / 114).
// Rows shorter than a wavefront cost a single step time as well, by 0.43 a lane:
// FP64 4 x 8 x 16384 148 / 183, 16 x 16 x 2048 41 / 50, 4 x 4 x 16384 114 / 96; beyond
// the cache, rows that end within a 64-site block about another 128 bytes each:
// FP32 60 x 2 x 40000 160 / 196, FP64 MRT 65 x 130 x 70 42 / 46.
// A state in the cache whose blocks run all at once is bound by latency, and a pair
// has half the launches.  BGK pairs there from three rows up: FP64 64 x 8 x 255
// 7.4 / 8.7, 256 x 512 x 1 7.3 / 7.6, 64 x 2 x 2000 17.6 / 12.5; TRT up to 2.9 lanes:
// FP64 256 x 256 x 2 9.3 / 8.8, 64^3 11.9 / 12.7, 72^3 19.9 / 20.1; in FP32 from 550000
// sites: 80^3 14.9 / 14.0, 84^3 15.3 / 16.5; MRT in FP64 up to 1.9: 64^3 14.1 / 13.0,
// 80^3 28.3 / 24.4, 128 x 128 x 32 21.5 / 24.0; in FP32 with 64-wide tiles from 800000
// sites: 150 x 70 x 90 27.0 / 28.4, 192 x 96 x 30 14.6 / 13.8; 96^3, 128 wide, 26.2 /
// 21.7, 104^3 30.2 / 28.9; beyond the cache 128^3 44 / 59.
// FP16's pair, bound by its arithmetic, wants no lanes idle besides, and with
// 64-wide tiles a chip nine tenths full: BGK 192^3 86 / 93, TRT 93 / 92; 200 x 204 x
// 100 70.7 / 67.3.  MRT never there: 128^3 43 / 31.
template <class S>
bool pair_pays(const lb_ctx* c) {
    const lb_params& p = c->p;
    const int64_t n = c->L.nsite;
    constexpr int t = sizeof(S) == 8 ? 0 : (sizeof(S) == 4 ? 1 : 2);
    if (p.model != LB_SINGLE || p.vvl > 1 || n < kPairMinSites<S>) return false;
    if (p.collision == LB_MRT && (t == 2 || (t == 1 && n < 800000))) return false;
    if (t == 2 && (p.nx % PairTile::TX != 0 || p.ny % PairTile::TY != 0)) return false;
    auto pays = [&](auto tiling) {
        using TP = decltype(tiling);
        constexpr int slots = pair_slots<S, TP>();
        const Geo g = c->template column_geo<TP>(slots);
        if (t == 2 && TP::TX == 64 &&
            (p.collision != LB_BGK || g.nblocks * 10 < (g.nblocks + slots - 1) / slots * slots * 9))
            return false;
        const bool resident = g.nblocks <= slots && c->cached();
        if (resident && t < 2 && p.collision == LB_BGK) return p.ny >= 3;
        if (resident && t == 1 && p.collision == LB_TRT && n < 550000) return false;
        const double x = (double)g.gx * TP::TX / p.nx, y = (double)g.gy * TP::TY / p.ny, z = 1.0 + 2.0 * g.gz / p.nz;
        static constexpr double beyond[3][3] = {{2.7, 2.5, 2.05}, {3.05, 2.9, 2.0}, {1.4, 1.15, 0.0}};
        static constexpr double within[2][3] = {{0.0, 2.9, 1.9}, {0.0, 2.9, TP::TX == 64 ? 2.0 : 0.0}};
        const double limit = resident && t < 2 ? within[t % 2][p.collision] : beyond[t][p.collision];
        double row = 0.43 * tiles(p.nx, 64) * 64 / p.nx;
        if (!c->cached() && p.nx > 32 && p.nx % 64 != 0) row = std::max(row, 1.0 + 128.0 / (p.nx * sizeof(S)));
        return x * (1.0 + 0.75 * (y - 1.0)) * z <= limit * std::max(1.0, row);
    };
    if constexpr (sizeof(S) < 8) {
        if (c->wide_rows()) return pays(PairTileWide{});
    }
    return pays(PairTile{});
}

// A step taken alone moves the state to the other buffer, but for the first
// from a direct state; so does a pair.  A captured call has to leave the state
// in the buffer where its steps taken alone would, since a graph is replayed on
// fixed buffers: an even number of steps from a pending state ends where it
// began and advances the state at every replay.  There, pairs are taken in an
// even number (from a direct state in an odd one) and the other steps alone.
template <class S>
int run_step(lb_ctx* c, int32_t n) {
    int32_t pairs = pair_pays<S>(c) ? n / 2 : 0;
    if (pairs > 0 && (pairs & 1) == (c->pending ? 1 : 0) && capturing(c)) --pairs;
    for (; pairs > 0; --pairs, n -= 2) {
        const S* src = (const S*)c->fbuf(c->cur);
        S* dst = (S*)c->fbuf(1 - c->cur);
        const int rc = c->L.blocked ? launch_single_pair<S, true, false>(c, c->pending, src, nullptr, dst, false)
                                    : launch_single_pair<S, false, false>(c, c->pending, src, nullptr, dst, false);
        if (rc) return rc;
        c->cur = 1 - c->cur;
        c->pending = true;
    }
    for (int32_t k = 0; k < n; ++k) {
        int rc = run_collide<S>(c);
        if (rc) return rc;
        c->pending = true;
    }
    return LB_OK;
}

template <class S>
int run_init(lb_ctx* c, const double* rho, const double* u, const double* phi) {
    Timed t(c, LB_K_OTHER);
    CollParams<double> cp;
    const auto ct = coll_params<S>(c);
    cp.omega_f = ct.omega_f; cp.omega_g = ct.omega_g;
    cp.A = c->p.A; cp.B = c->p.B; cp.kappa = c->p.kappa; cp.gamma = c->p.gamma;
    cp.rho0 = c->p.storage == LB_F64 ? 0.0 : c->p.rho0;
    cp.phi0 = c->p.storage == LB_F64 ? 0.0 : c->p.phi0;
    S* f = (S*)c->fbuf(c->cur);
    S* g = (S*)c->gbuf(c->cur);
    const int rc = by_width(c, [&](auto pol) {
        using P = decltype(pol);
        if (c->p.model == LB_BINARY) k_init<P, MODEL_BINARY, S><<<c->grid(), c->block(), 0, c->stream>>>(rho, u, phi, f, g, c->geo(), cp);
        else k_init<P, MODEL_SINGLE, S><<<c->grid(), c->block(), 0, c->stream>>>(rho, u, phi, f, g, c->geo(), cp);
        return launch_status();
    });
    if (rc == LB_OK) c->pending = false;
    return rc;
}

template <class S>
int run_moments(lb_ctx* c, double* rho, double* u, double* phi) {
    Timed t(c, LB_K_OTHER);
    const double r0 = c->p.storage == LB_F64 ? 0.0 : c->p.rho0;
    const double p0 = c->p.storage == LB_F64 ? 0.0 : c->p.phi0;
    const S* f = (const S*)c->fbuf(c->cur);
    const S* g = (const S*)c->gbuf(c->cur);
    const dim3 grid = c->grid(), block = c->block();
    return by_width(c, [&](auto pol) {
        using P = decltype(pol);
        if (c->p.model == LB_BINARY) {
            if (c->pending) k_moments<P, MODEL_BINARY, S, true><<<grid, block, 0, c->stream>>>(f, g, rho, u, phi, c->geo(), r0, p0);
            else k_moments<P, MODEL_BINARY, S, false><<<grid, block, 0, c->stream>>>(f, g, rho, u, phi, c->geo(), r0, p0);
        } else {
            if (c->pending) k_moments<P, MODEL_SINGLE, S, true><<<grid, block, 0, c->stream>>>(f, g, rho, u, nullptr, c->geo(), r0, p0);
            else k_moments<P, MODEL_SINGLE, S, false><<<grid, block, 0, c->stream>>>(f, g, rho, u, nullptr, c->geo(), r0, p0);
        }
        return launch_status();
    });
}

// Blocks of a reduction over the lattice: eight 256-lane ones a CU.
constexpr int kReduceBlocks = 8 * kCUs;

// Sums of a state (f, g) in geo's layout into out, by way of `partial`; b0 and
// b4 are added to sum rho and sum phi.
template <class S, class P = Pol>
int sums_of(int model, const S* f, const S* g, const Geo& geo, double* partial, double b0, double b4, double* out,
            hipStream_t s) {
    const int nb = std::min(geo.nblocks, kReduceBlocks);
    if (model == LB_BINARY) k_sums_partial<P, MODEL_BINARY, S><<<nb, P::TPB, 0, s>>>(f, g, geo, partial);
    else k_sums_partial<P, MODEL_SINGLE, S><<<nb, P::TPB, 0, s>>>(f, nullptr, geo, partial);
    k_sums_final<Pol, 5><<<1, Pol::TPB, 0, s>>>(partial, nb, out, b0, b4, 0);
    return launch_status();
}

template <class S>
int run_sums(lb_ctx* c, double* out) {
    Timed t(c, LB_K_OTHER);
    const bool dev = c->p.storage != LB_F64;
    const double n = (double)c->L.nsite;
    const double b0 = dev ? n * c->p.rho0 : 0.0;
    const double b4 = (dev && c->p.model == LB_BINARY) ? n * c->p.phi0 : 0.0;
    return by_width(c, [&](auto pol) {
        return sums_of<S, decltype(pol)>(c->p.model, (const S*)c->fbuf(c->cur), (const S*)c->gbuf(c->cur), c->geo(),
                                         c->partial(), b0, b4, out, c->stream);
    });
}

template <class S>
int run_stats(lb_ctx* c, double* out) {
    Timed t(c, LB_K_OTHER);
    const S* f = (const S*)c->fbuf(c->cur);
    const S* g = (const S*)c->gbuf(c->cur);
    const bool dev = c->p.storage != LB_F64;
    const double r0 = dev ? c->p.rho0 : 0.0, p0 = dev ? c->p.phi0 : 0.0;
    const Geo geo = c->geo();
    const bool bin = c->p.model == LB_BINARY;
    // the 38 doubles a site of an FP64 mixture leave room for fewer blocks at once:
    // up to two rounds of one tile a block are faster (80^3, 3200 tiles, 34.8 us
    // against 36.8 in 2048 blocks)
    const int most = bin && sizeof(S) == 8 && c->L.nblocks <= 2 * kReduceBlocks ? 2 * kReduceBlocks : kReduceBlocks;
    const int nb = std::min(c->L.nblocks, most);
    by_width(c, [&](auto pol) {
        using P = decltype(pol);
        if (bin && c->pending)
            k_stats_partial<P, MODEL_BINARY, S, true><<<nb, c->block(), 0, c->stream>>>(f, g, geo, r0, p0, c->partial());
        else if (bin)
            k_stats_partial<P, MODEL_BINARY, S, false><<<nb, c->block(), 0, c->stream>>>(f, g, geo, r0, p0, c->partial());
        else if (c->pending)
            k_stats_partial<P, MODEL_SINGLE, S, true><<<nb, c->block(), 0, c->stream>>>(f, g, geo, r0, p0, c->partial());
        else
            k_stats_partial<P, MODEL_SINGLE, S, false><<<nb, c->block(), 0, c->stream>>>(f, g, geo, r0, p0, c->partial());
        return 0;
    });
    k_stats_final<Pol><<<1, c->block(), 0, c->stream>>>(c->partial(), nb, out, bin ? 1 : 0);
    return launch_status();
}

template <class S>
int run_get_state(lb_ctx* c, S* f, S* g) {
    if (c->pending) return run_stream_into<S>(c, c->cur, f, g, c->canonical_geo(), c->cached_copy());
    Timed t(c, LB_K_OTHER);
    return run_convert<S>(c, (const S*)c->fbuf(c->cur), (const S*)c->gbuf(c->cur), f, g, c->geo(),
                          c->canonical_geo(), c->cached_copy());
}

template <class S>
int run_set_state(lb_ctx* c, const S* f, const S* g) {
    Timed t(c, LB_K_OTHER);
    const int rc = run_convert<S>(c, f, g, (S*)c->fbuf(c->cur), (S*)c->gbuf(c->cur), c->canonical_geo(), c->geo(),
                                  c->cached());
    if (rc) return rc;
    c->pending = false;
    return LB_OK;
}

// nsteps binary steps whose post-collision fields go to canonical memory, f
// then g of step k to post + k*38*N; afterwards the state is pending on a copy
// of the last of them.  Captured on a pending state, the copy goes to the other
// buffer: the one the record started from stays as it is, and a graph of the call
// records the same steps at every replay.  (Always done, records of two steps
// within the cache alternate between buffers: FP16 96^3 62 us, 55.)  Step 0 collides the context's state into post[0] (128^3:
// 360 us with its phi; in the context's buffers and copied out it was 600);
// later steps march from post[k-1] to post[k] (both of direction stride N).
// A record of one step without its phi marches in the context's buffers and is
// copied out, which spares the phi pass and the copy back: FP64 128^3 464 us, as
// the others 509; 256^3 3589 and 4098; FP32 256^3 1795 and 1989.
template <class S>
int run_step_record_binary(lb_ctx* c, int32_t n, S* post, typename Compute<S>::T* phi) {
    using T = typename Compute<S>::T;
    const int64_t N = c->L.nsite;
    if (n == 1 && !phi && c->pending && march_pays<S>(c)) {
        int rc = run_binary_march<S>(c);
        if (rc) return rc;
        Timed t(c, LB_K_OTHER);
        rc = run_convert<S>(c, (const S*)c->fbuf(c->cur), (const S*)c->gbuf(c->cur), post, post + Q * N, c->geo(),
                            c->canonical_geo(), c->cached_copy());
        if (rc) return rc;
        c->pending = true;
        return LB_OK;
    }
    const auto cp = coll_params<S>(c);
    int rc = by_width(c, [&](auto pol) {              // step 0: phi of the state, then its collision
        using P = decltype(pol);
        const S* f = (const S*)c->fbuf(c->cur);
        const S* g = (const S*)c->gbuf(c->cur);
        T* ph = phi ? phi : (T*)c->phi();
        {
            Timed t(c, LB_K_PHI);
            if (c->pending) k_phi<P, S, true><<<c->grid(), c->block(), 0, c->stream>>>(g, ph, c->geo(), cp.phi0);
            else k_phi<P, S, false><<<c->grid(), c->block(), 0, c->stream>>>(g, ph, c->geo(), cp.phi0);
        }
        Timed t(c, LB_K_COLLIDE);
        by_collision(c, [&](auto coll) {
            constexpr int COLL = decltype(coll)::value;
            if (c->pending)
                k_collide<P, MODEL_BINARY, S, true, COLL, true><<<c->grid(), c->block(), 0, c->stream>>>(
                    f, g, post, post + Q * N, ph, c->geo(), cp);
            else
                k_collide<P, MODEL_BINARY, S, false, COLL, true><<<c->grid(), c->block(), 0, c->stream>>>(
                    f, g, post, post + Q * N, ph, c->geo(), cp);
        });
        return launch_status();
    });
    if (rc) return rc;
    const bool march = march_pays<S>(c);
    Geo cg = c->canonical_geo();
    for (int32_t k = 1; k < n; ++k) {
        const S* src = post + (size_t)(k - 1) * 2 * Q * N;
        S* dst = post + (size_t)k * 2 * Q * N;
        if (!march) {
            // two-pass: phi of the recorded state, then the fused collide, both on stride N
            T* ph = phi ? phi + (size_t)k * N : (T*)c->phi();
            {
                Timed t(c, LB_K_PHI);
                k_phi<Pol, S, true><<<c->grid(), c->block(), 0, c->stream>>>(src + Q * N, ph, cg, cp.phi0);
            }
            {
                Timed t(c, LB_K_COLLIDE);
                if (c->p.collision == LB_TRT)
                    k_collide<Pol, MODEL_BINARY, S, true, COLL_TRT><<<c->grid(), c->block(), 0, c->stream>>>(
                        src, src + Q * N, dst, dst + Q * N, ph, cg, cp);
                else if (c->p.collision == LB_MRT)
                    k_collide<Pol, MODEL_BINARY, S, true, COLL_MRT><<<c->grid(), c->block(), 0, c->stream>>>(
                        src, src + Q * N, dst, dst + Q * N, ph, cg, cp);
                else
                    k_collide<Pol, MODEL_BINARY, S, true><<<c->grid(), c->block(), 0, c->stream>>>(
                        src, src + Q * N, dst, dst + Q * N, ph, cg, cp);
            }
            rc = launch_status();
            if (rc) return rc;
            continue;
        }
        if (phi)
            rc = launch_march<S, false, true>(c, src, src + Q * N, dst, dst + Q * N, true, phi + (size_t)k * N);
        else
            rc = launch_march<S, false, false>(c, src, src + Q * N, dst, dst + Q * N, true, nullptr);
        if (rc) return rc;
    }
    {
        Timed t(c, LB_K_OTHER);
        const S* last = post + (size_t)(n - 1) * 2 * Q * N;
        const int dst = c->pending && capturing(c) ? 1 - c->cur : c->cur;
        rc = run_convert<S>(c, last, last + Q * N, (S*)c->fbuf(dst), (S*)c->gbuf(dst), c->canonical_geo(),
                            c->geo(), c->cached());
        if (rc) return rc;
        c->cur = dst;
    }
    c->pending = true;
    return LB_OK;
}

// The same for the single fluid, 19 N values a step: step 0 goes from the
// context's state to post[0]; the rest run in pairs where a pair beats two steps
// (the first one's values are stored too: 64^3 31.3 us a pair, 36.0 us two
// steps).
template <class S>
int run_step_record(lb_ctx* c, int32_t n, S* post, typename Compute<S>::T* phi) {
    if (c->p.model == LB_BINARY) return run_step_record_binary<S>(c, n, post, phi);
    const int64_t N = c->L.nsite;
    const auto cp = coll_params<S>(c);
    // one collision from src (layout sg; pull from a pending src when `gather`)
    // into canonical dst
    const Geo cg = c->canonical_geo();
    auto collide = [&](bool gather, const S* src, const Geo& sg, S* dst) {
        Timed t(c, LB_K_COLLIDE);
        return by_width(c, [&](auto pol) {
            using P = decltype(pol);
            const dim3 grid = c->grid(), block = c->block();
            by_collision(c, [&](auto coll) {
                constexpr int COLL = decltype(coll)::value;
                if (gather) k_collide_single_strided<P, S, true, COLL><<<grid, block, 0, c->stream>>>(src, dst, sg, cg, cp);
                else k_collide_single_strided<P, S, false, COLL><<<grid, block, 0, c->stream>>>(src, dst, sg, cg, cp);
            });
            return launch_status();
        });
    };
    int err = collide(c->pending, (const S*)c->fbuf(c->cur), c->geo(), post);
    const bool pairs = pair_pays<S>(c);
    for (int32_t k = 1; k < n && err == LB_OK;) {
        const S* src = post + (size_t)(k - 1) * Q * N;
        S* dst = post + (size_t)k * Q * N;
        if (pairs && k + 1 < n) {
            err = launch_single_pair<S, false, true>(c, true, src, dst, dst + Q * N, true);
            k += 2;
        } else {
            err = collide(true, src, cg, dst);
            k += 1;
        }
    }
    if (err) return err;
    Timed t(c, LB_K_OTHER);
    const int rc = run_convert<S>(c, post + (size_t)(n - 1) * Q * N, nullptr, (S*)c->fbuf(c->cur), nullptr, cg,
                                  c->geo(), c->cached());
    if (rc) return rc;
    c->pending = true;
    return LB_OK;
}

template <class S>
int run_sites(lb_ctx* c, const int32_t* index, int64_t m, S* f, S* g, bool set) {
    Timed t(c, LB_K_OTHER);
    const int nb = (int)((m + CB - 1) / CB);
    const Geo geo = c->geo();
    S* bufs[2] = {(S*)c->fbuf(c->cur), (S*)c->gbuf(c->cur)};
    S* packs[2] = {f, g};
    for (int d = 0; d < (c->p.model == LB_BINARY ? 2 : 1); ++d) {
        if (set) {
            if (c->pending) k_set_sites<S, true><<<nb, CB, 0, c->stream>>>(bufs[d], index, m, packs[d], geo);
            else k_set_sites<S, false><<<nb, CB, 0, c->stream>>>(bufs[d], index, m, packs[d], geo);
        } else {
            if (c->pending) k_get_sites<S, true><<<nb, CB, 0, c->stream>>>(bufs[d], index, m, packs[d], geo);
            else k_get_sites<S, false><<<nb, CB, 0, c->stream>>>(bufs[d], index, m, packs[d], geo);
        }
    }
    return launch_status();
}

// The launchers of one storage type: LB_LAUNCHERS(template, S) instantiates
// them, LB_LAUNCHERS(extern template, S) refers to another file's.
#define LB_LAUNCHERS(what, S)                                                                                     \
    what int run_collide<S>(lb_ctx*);                                                                             \
    what int run_propagate<S>(lb_ctx*);                                                                           \
    what int run_step<S>(lb_ctx*, int32_t);                                                                       \
    what int run_init<S>(lb_ctx*, const double*, const double*, const double*);                                   \
    what int run_moments<S>(lb_ctx*, double*, double*, double*);                                                  \
    what int sums_of<S>(int, const S*, const S*, const Geo&, double*, double, double, double*, hipStream_t);      \
    what int run_sums<S>(lb_ctx*, double*);                                                                       \
    what int run_stats<S>(lb_ctx*, double*);                                                                      \
    what int run_get_state<S>(lb_ctx*, S*, S*);                                                                   \
    what int run_set_state<S>(lb_ctx*, const S*, const S*);                                                       \
    what int run_step_record<S>(lb_ctx*, int32_t, S*, typename Compute<S>::T*);                                   \
    what int run_sites<S>(lb_ctx*, const int32_t*, int64_t, S*, S*, bool);

}  // namespace lbl
