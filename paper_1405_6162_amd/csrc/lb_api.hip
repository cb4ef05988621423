// C ABI of the gfx950 D3Q19 lattice-Boltzmann library: argument checks,
// workspace carving, the direct/pending state machine and kernel launches on
// the caller's stream.  See include/lb.h for the contract of every call.

#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>

#include "launch.h"

namespace lbl {
LB_LAUNCHERS(extern template, double)
LB_LAUNCHERS(extern template, float)
LB_LAUNCHERS(extern template, _Float16)
}  // namespace lbl

using namespace lbk;
using namespace lbl;

// Partial sums of lb_conserved_sums_noalloc (8 doubles per block).  In host
// code this name is only a stand-in for the symbol: kernels get the device
// address that hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) double scratch[8 * (size_t)LB_NOALLOC_MAX_BLOCKS];

namespace {

constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
double* scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per
// device (each device holds its own copy of the array).
int scratch_on_current_device(double** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LB_EDEVICE;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[dev]) {
        double* ptr = nullptr;
        if (hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return LB_EDEVICE;
        scratch_ptr[dev] = ptr;
    }
    *out = scratch_ptr[dev];
    return LB_OK;
}

}  // namespace

namespace {

// Dispatch on the storage type.
template <class F>
int by_storage(lb_ctx* c, F&& fn) {
    c->launched = true;
    switch (c->p.storage) {
        case LB_F64: return fn((double*)nullptr);
        case LB_F32: return fn((float*)nullptr);
        case LB_F16: return fn((_Float16*)nullptr);
    }
    return LB_EINVAL;
}

}  // namespace

namespace {

// True when two device ranges [a, a + na) and [b, b + nb) (in doubles) overlap.
bool overlaps(const double* a, size_t na, const double* b, size_t nb) {
    if (!a || !b) return false;
    return a < b + nb && b < a + na;
}

template <int LG>
void launch_adjoint_binary_local(lb_ctx* c, bool pending, const double* f, const double* g, const double* phi,
                                 const double* lf_next, const double* lg_next, const double* b_next, double* lf_n,
                                 double* p_out, double* afield, const Geo& geo, const CollParams<double>& cp) {
    // 32-bit byte offsets from one base per array when every array of 19
    // directions fits below 4 GiB (lattices up to about 300^3)
    const bool off32 = (uint64_t)Q * (uint64_t)geo.dstride * sizeof(double) <= ((uint64_t)1 << 32);
    auto go = [&](auto coll, auto o32) {
        constexpr int COLL = decltype(coll)::value;
        constexpr bool OFF32 = decltype(o32)::value;
        auto with = [&](auto pol) {
            using P = decltype(pol);
            if (pending)
                k_adjoint_binary<P, true, LG, COLL, OFF32><<<c->grid(), c->block(), 0, c->stream>>>(
                    f, g, phi, lf_next, lg_next, b_next, lf_n, p_out, afield, c->partial(), geo, cp);
            else
                k_adjoint_binary<P, false, LG, COLL, OFF32><<<c->grid(), c->block(), 0, c->stream>>>(
                    f, g, phi, lf_next, lg_next, b_next, lf_n, p_out, afield, c->partial(), geo, cp);
        };
        // Adjoints that stay in the memory-side cache are stored there, others
        // past it, and the states read past them: us a step (with the stencil
        // kernel), nontemporal / ordinary, 128^3 442 / 462, 100 x 90 x 77 190 /
        // 200, 64^3 56 / 53.
        if constexpr (OFF32) {
            if (c->cached()) { with(Cached<Pol>{}); return; }
        }
        with(Pol{});
    };
    auto by_coll = [&](auto o32) {
        if (c->p.collision == LB_TRT) go(std::integral_constant<int, COLL_TRT>{}, o32);
        else if (c->p.collision == LB_MRT) go(std::integral_constant<int, COLL_MRT>{}, o32);
        else go(std::integral_constant<int, COLL_BGK>{}, o32);
    };
    if (off32) by_coll(std::true_type{});
    else by_coll(std::false_type{});
}

// Gradient sums of a binary adjoint step: dL/domega_f, dL/domega_g,
// dL/dkappa; for TRT and MRT then dL/domega_minus (omega_f being the even,
// or shear, rate and omega_minus the odd, or flux, one); for MRT then the
// bulk, even-ghost and odd-ghost rates.
int binary_adjoint_grad_count(const lb_ctx* c) {
    return c->p.collision == LB_MRT ? 7 : (c->p.collision == LB_TRT ? 4 : 3);
}

// The stencil kernel of a binary adjoint step, with block 0 adding the
// local kernel's partials (one per gradient sum) into grads.
template <bool B_ONLY>
void launch_adjoint_binary_stencil(lb_ctx* c, const double* afield, const double* lg_next, double* out,
                                   const Geo& geo, double omega_g, double* grads) {
    const int ng = binary_adjoint_grad_count(c);
    if (ng == 7)
        k_adjoint_binary_stencil<Pol, B_ONLY, 7><<<c->grid(), c->block(), 0, c->stream>>>(
            afield, lg_next, out, geo, omega_g, c->partial(), c->L.nblocks, grads);
    else if (ng == 4)
        k_adjoint_binary_stencil<Pol, B_ONLY, 4><<<c->grid(), c->block(), 0, c->stream>>>(
            afield, lg_next, out, geo, omega_g, c->partial(), c->L.nblocks, grads);
    else
        k_adjoint_binary_stencil<Pol, B_ONLY, 3><<<c->grid(), c->block(), 0, c->stream>>>(
            afield, lg_next, out, geo, omega_g, c->partial(), c->L.nblocks, grads);
}

// Rate sums an adjoint step of the single fluid accumulates: 1 (BGK), 2
// (TRT) or 5 (MRT), in the order of lb_params' relaxation times.
int adjoint_rate_count(const lb_ctx* c) {
    return c->p.collision == LB_MRT ? 5 : (c->p.collision == LB_TRT ? 2 : 1);
}

// One single-fluid adjoint kernel launch writing its block partials to
// `partial`; with prev given, its block 0 also accumulates the previous
// step's partials into domega.
template <bool PEND, int COLL>
void adjoint_single_launch(lb_ctx* c, const double* f, const double* lam_next, double* lam_n, const Geo& geo,
                           const CollParams<double>& cp, double* partial, const double* prev, double* domega) {
    Timed t(c, LB_K_ADJOINT);
    k_adjoint<Pol, PEND, COLL><<<c->grid(), c->block(), 0, c->stream>>>(f, lam_next, lam_n, partial, geo, cp, prev,
                                                                        c->L.nblocks, domega);
}

template <int COLL>
void adjoint_single_sums(lb_ctx* c, const double* partial, double* domega) {
    k_sums_final<Pol, AdjointRates<COLL>::K><<<1, c->block(), 0, c->stream>>>(partial, c->L.nblocks, domega, 0.0,
                                                                               0.0, 1);
}

// One single-fluid adjoint step for the context's collision.  sums_now: the
// step's rate sums are reduced into domega by a separate launch right away;
// otherwise they stay in `partial` for the next step (prev) or the caller.
void adjoint_single_step(lb_ctx* c, const double* f, bool pending, const double* lam_next, double* lam_n,
                         const Geo& geo, const CollParams<double>& cp, double* partial, const double* prev,
                         double* domega, bool sums_now) {
    auto go = [&](auto coll) {
        constexpr int COLL = decltype(coll)::value;
        if (pending) adjoint_single_launch<true, COLL>(c, f, lam_next, lam_n, geo, cp, partial, prev, domega);
        else adjoint_single_launch<false, COLL>(c, f, lam_next, lam_n, geo, cp, partial, prev, domega);
        if (sums_now) adjoint_single_sums<COLL>(c, partial, domega);
    };
    if (c->p.collision == LB_TRT) go(std::integral_constant<int, COLL_TRT>{});
    else if (c->p.collision == LB_MRT) go(std::integral_constant<int, COLL_MRT>{});
    else go(std::integral_constant<int, COLL_BGK>{});
}

// The rate sums left in `partial` by the last step of a sweep.
void adjoint_single_flush(lb_ctx* c, const double* partial, double* domega) {
    if (c->p.collision == LB_TRT) adjoint_single_sums<COLL_TRT>(c, partial, domega);
    else if (c->p.collision == LB_MRT) adjoint_single_sums<COLL_MRT>(c, partial, domega);
    else adjoint_single_sums<COLL_BGK>(c, partial, domega);
}

}  // namespace

extern "C" {

int lb_workspace_bytes(const lb_params* p, size_t* bytes) {
    if (!bytes) return LB_EINVAL;
    int rc = check_params(p);
    if (rc) return rc;
    *bytes = layout_of(p).total;
    return LB_OK;
}

int lb_create(const lb_params* p, void* workspace, size_t workspace_bytes, void* stream, lb_ctx** out) {
    if (!out) return LB_EINVAL;
    *out = nullptr;
    int rc = check_params(p);
    if (rc) return rc;
    if (!workspace || ((uintptr_t)workspace % 256) != 0) return LB_EINVAL;
    const Layout L = layout_of(p);
    if (workspace_bytes < L.total) return LB_ENOMEM;
    lb_ctx* c = new (std::nothrow) lb_ctx();
    if (!c) return LB_ENOMEM;
    c->p = *p;
    c->L = L;
    c->stream = (hipStream_t)stream;
    c->ws = (char*)workspace;
    c->cur = 0;
    c->pending = false;
    c->profiling = false;
    c->profile_kinds = 0;
    c->launched = false;
    *out = c;
    return LB_OK;
}

int lb_set_stream(lb_ctx* c, void* stream) {
    if (!c) return LB_EINVAL;
    c->stream = (hipStream_t)stream;
    return LB_OK;
}

int lb_init_equilibrium(lb_ctx* c, const double* rho, const double* u, const double* phi) {
    if (!c || !rho || !u) return LB_EINVAL;
    if (c->p.model == LB_BINARY && !phi) return LB_EINVAL;
    return by_storage(c, [&](auto tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        return run_init<S>(c, rho, u, phi);
    });
}

int lb_collide(lb_ctx* c) {
    if (!c) return LB_EINVAL;
    return by_storage(c, [&](auto tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        return run_collide<S>(c);
    });
}

int lb_propagate(lb_ctx* c) {
    if (!c) return LB_EINVAL;
    return by_storage(c, [&](auto tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        return run_propagate<S>(c);
    });
}

int lb_step(lb_ctx* c, int32_t nsteps) {
    if (!c || nsteps < 0) return LB_EINVAL;
    if (nsteps == 0) return LB_OK;
    return by_storage(c, [&](auto tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        return run_step<S>(c, nsteps);
    });
}

int lb_moments(lb_ctx* c, double* rho, double* u, double* phi) {
    if (!c) return LB_EINVAL;
    if (phi && c->p.model != LB_BINARY) return LB_EINVAL;
    if (!rho && !u && !phi) return LB_OK;
    return by_storage(c, [&](auto tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        return run_moments<S>(c, rho, u, phi);
    });
}

int lb_conserved_sums(lb_ctx* c, double* out) {
    if (!c || !out) return LB_EINVAL;
    return by_storage(c, [&](auto tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        return run_sums<S>(c, out);
    });
}

int lb_conserved_sums_noalloc(const lb_params* p, const void* f, const void* g, double* out, void* stream) {
    if (!p || !f || !out) return LB_EINVAL;
    int rc = check_params(p);
    if (rc) return rc;
    if ((p->model == LB_BINARY) != (g != nullptr)) return LB_EINVAL;
    // the launch of lb_conserved_sums, on the canonical layout
    Geo geo;
    geo.nx = p->nx; geo.ny = p->ny; geo.nz = p->nz;
    geo.plane = (uint32_t)p->nx * (uint32_t)p->ny;
    geo.nsite = geo.plane * (uint32_t)p->nz;
    geo.dstride = geo.nsite;
    geo.zs = geo.plane; geo.ys = (uint32_t)p->nx; geo.xbs = 64;
    geo.gx = tiles(p->nx, Pol::TX);
    geo.gy = tiles(p->ny, Pol::TY);
    geo.gz = tiles(p->nz, Pol::TZ);
    const int64_t nblocks = (int64_t)geo.gx * geo.gy * geo.gz;
    if (nblocks > LB_NOALLOC_MAX_BLOCKS) return LB_ERANGE;
    geo.nblocks = (int)nblocks;
    double* partial = nullptr;
    rc = scratch_on_current_device(&partial);
    if (rc) return rc;
    const hipStream_t s = (hipStream_t)stream;
    const bool dev = p->storage != LB_F64;
    const double n = (double)geo.nsite;
    const double b0 = dev ? n * p->rho0 : 0.0;
    const double b4 = (dev && p->model == LB_BINARY) ? n * p->phi0 : 0.0;
    auto launch = [&](auto tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        return sums_of<S>(p->model, (const S*)f, (const S*)g, geo, partial, b0, b4, out, s);
    };
    if (p->storage == LB_F64) return launch((double*)nullptr);
    if (p->storage == LB_F32) return launch((float*)nullptr);
    return launch((_Float16*)nullptr);
}

int lb_field_stats(lb_ctx* c, double* out) {
    if (!c || !out) return LB_EINVAL;
    return by_storage(c, [&](auto tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        return run_stats<S>(c, out);
    });
}

int lb_get_state(lb_ctx* c, void* f, void* g) {
    if (!c || !f) return LB_EINVAL;
    if ((c->p.model == LB_BINARY) != (g != nullptr)) return LB_EINVAL;
    return by_storage(c, [&](auto tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        return run_get_state<S>(c, (S*)f, (S*)g);
    });
}

int lb_set_state(lb_ctx* c, const void* f, const void* g) {
    if (!c || !f) return LB_EINVAL;
    if ((c->p.model == LB_BINARY) != (g != nullptr)) return LB_EINVAL;
    return by_storage(c, [&](auto tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        return run_set_state<S>(c, (const S*)f, (const S*)g);
    });
}

int lb_set_tau(lb_ctx* c, double tau_f) {
    if (!c || !std::isfinite(tau_f) || !(tau_f > 0.5)) return LB_EINVAL;
    c->p.tau_f = tau_f;
    return LB_OK;
}

int lb_step_record(lb_ctx* c, int32_t nsteps, void* post, void* phi) {
    if (!c || nsteps < 0) return LB_EINVAL;
    if (phi && c->p.model != LB_BINARY) return LB_EINVAL;
    if (nsteps == 0) return LB_OK;
    if (!post) return LB_EINVAL;
    return by_storage(c, [&](auto tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        return run_step_record<S>(c, nsteps, (S*)post, (typename Compute<S>::T*)phi);
    });
}

int lb_set_params(lb_ctx* c, const lb_params* p) {
    if (!c || !p) return LB_EINVAL;
    int rc = check_params(p);
    if (rc) return rc;
    const lb_params& q = c->p;
    if (p->nx != q.nx || p->ny != q.ny || p->nz != q.nz || p->model != q.model || p->storage != q.storage ||
        p->vvl != q.vvl || p->collision != q.collision || p->binary_step != q.binary_step || p->rho0 != q.rho0 ||
        p->phi0 != q.phi0)
        return LB_EINVAL;
    c->p = *p;
    return LB_OK;
}

int lb_adjoint_step_binary(lb_ctx* c, const double* f, const double* g, const double* phi_n, int pending,
                           const double* lf_next, const double* lg_next, double* lf_n, double* lg_n,
                           double* grads) {
    if (!c || !f || !g || !lf_next || !lg_next || !lf_n || !lg_n || !grads) return LB_EINVAL;
    if (c->p.model != LB_BINARY || c->p.storage != LB_F64) return LB_ENOTSUP;
    const double* outs[2] = {lf_n, lg_n};
    const double* ins[5] = {f, g, lf_next, lg_next, phi_n};
    for (const double* o : outs)
        for (const double* i : ins)
            if (o == i) return LB_EINVAL;
    if (lf_n == lg_n) return LB_EINVAL;
    c->launched = true;
    const Geo geo = c->canonical_geo();
    const auto cp = coll_params<double>(c);
    const double* phi = phi_n;
    double* afield = (double*)c->fbuf(1 - c->cur);       // spare state buffer: >= 19 N doubles, 5 N used
    if (!phi) {
        Timed t(c, LB_K_ADJOINT);
        double* p = (double*)c->phi();
        if (pending) k_phi<Pol, double, true><<<c->grid(), c->block(), 0, c->stream>>>(g, p, geo, 0.0);
        else k_phi<Pol, double, false><<<c->grid(), c->block(), 0, c->stream>>>(g, p, geo, 0.0);
        phi = p;
    }
    {
        Timed t(c, LB_K_ADJOINT);
        launch_adjoint_binary_local<LG_GATHER>(c, pending != 0, f, g, phi, lf_next, lg_next, nullptr, lf_n, nullptr,
                                               afield, geo, cp);
    }
    {
        Timed t(c, LB_K_ADJOINT);
        launch_adjoint_binary_stencil<false>(c, afield, lg_next, lg_n, geo, cp.omega_g, grads);
    }
    return launch_status();
}

int lb_adjoint_init_binary(lb_ctx* c, const double* rho, const double* u, const double* phi, const double* lf0,
                           const double* lg0, double* dphi, double* drho, double* du, double* dkappa) {
    if (!c || !rho || !u || !phi || !lf0 || !lg0 || !dphi || !drho || !du || !dkappa) return LB_EINVAL;
    if (c->p.model != LB_BINARY || c->p.storage != LB_F64) return LB_ENOTSUP;
    c->launched = true;
    const Geo geo = c->canonical_geo();
    const auto cp = coll_params<double>(c);
    double* afield = (double*)c->fbuf(1 - c->cur);
    {
        Timed t(c, LB_K_ADJOINT);
        k_adjoint_binary_init<Pol><<<c->grid(), c->block(), 0, c->stream>>>(rho, u, phi, lf0, lg0, afield, drho, du,
                                                                           c->partial(), geo, cp);
        k_adjoint_binary_stencil<Pol, true, 1><<<c->grid(), c->block(), 0, c->stream>>>(
            afield, nullptr, dphi, geo, 1.0, c->partial(), c->L.nblocks, dkappa);
    }
    return launch_status();
}

int lb_adjoint_step(lb_ctx* c, const double* f, int f_pending, const double* lam_next, double* lam_n,
                    double* domega) {
    if (!c || !f || !lam_next || !lam_n || !domega) return LB_EINVAL;
    if (c->p.model != LB_SINGLE || c->p.storage != LB_F64) return LB_ENOTSUP;
    if (lam_n == lam_next || lam_n == f) return LB_EINVAL;
    c->launched = true;
    adjoint_single_step(c, f, f_pending != 0, lam_next, lam_n, c->canonical_geo(), coll_params<double>(c),
                        c->partial(), nullptr, domega, true);
    return launch_status();
}

int lb_adjoint_segment(lb_ctx* c, const double* f0, const double* post, int32_t length, double* lam, double* work,
                       double* domega) {
    if (!c || !f0 || !lam || !work || !domega || length < 1) return LB_EINVAL;
    if (length > 1 && !post) return LB_EINVAL;
    if (c->p.model != LB_SINGLE || c->p.storage != LB_F64) return LB_ENOTSUP;
    const size_t n19 = (size_t)Q * c->L.nsite;
    const size_t npost = length > 1 ? (size_t)(length - 1) * n19 : 0;
    const size_t nw = (size_t)adjoint_rate_count(c);
    if (overlaps(lam, n19, work, n19) || overlaps(lam, n19, f0, n19) || overlaps(work, n19, f0, n19) ||
        overlaps(lam, n19, post, npost) || overlaps(work, n19, post, npost) || overlaps(domega, nw, lam, n19) ||
        overlaps(domega, nw, work, n19) || overlaps(domega, nw, f0, n19) || overlaps(domega, nw, post, npost))
        return LB_EINVAL;
    c->launched = true;
    const Geo geo = c->canonical_geo();
    const auto cp = coll_params<double>(c);
    double* cur = lam;            // lambda^{n+1}
    double* nxt = work;
    // two partial arrays in the context's partial buffer (16 doubles per
    // block, each step using slots 8 b + k of one half): step k's block 0
    // reduces step k-1's half while the other blocks fill its own
    double* halves[2] = {c->partial(), c->partial() + 8 * (size_t)c->L.nblocks};
    const double* prev = nullptr;
    for (int32_t n = length - 1, k = 0; n >= 0; --n, ++k) {
        double* part = halves[k & 1];
        const double* fn = n > 0 ? post + (size_t)(n - 1) * n19 : f0;
        adjoint_single_step(c, fn, n > 0, cur, nxt, geo, cp, part, prev, domega, false);
        prev = part;
        std::swap(cur, nxt);
    }
    adjoint_single_flush(c, prev, domega);
    if (cur != lam) {
        Timed t(c, LB_K_OTHER);
        if (hipMemcpyAsync(lam, cur, n19 * sizeof(double), hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
            return LB_EDEVICE;
    }
    return launch_status();
}

int lb_adjoint_segment_binary(lb_ctx* c, const double* f0, const double* g0, const double* post, const double* phi,
                              int32_t length, double* lf, double* lg, double* work, double* grads) {
    if (!c || !f0 || !g0 || !lf || !lg || !work || !grads || length < 1) return LB_EINVAL;
    if (length > 1 && !post) return LB_EINVAL;
    if (c->p.model != LB_BINARY || c->p.storage != LB_F64) return LB_ENOTSUP;
    const size_t N = c->L.nsite, n19 = (size_t)Q * N;
    const size_t ng = (size_t)binary_adjoint_grad_count(c);
    const size_t npost = length > 1 ? (size_t)(length - 1) * 2 * n19 : 0;
    const size_t nphi = phi && length > 1 ? (size_t)(length - 1) * N : 0;
    struct R { const double* p; size_t n; };
    const R outs[3] = {{lf, n19}, {lg, n19}, {work, 2 * n19}};
    const R all[8] = {{lf, n19}, {lg, n19}, {work, 2 * n19}, {f0, n19}, {g0, n19}, {post, npost}, {phi, nphi},
                      {grads, ng}};
    for (int o = 0; o < 3; ++o)                      // all[o] is outs[o]
        for (int a = 0; a < 8; ++a)
            if (a != o && overlaps(outs[o].p, outs[o].n, all[a].p, all[a].n)) return LB_EINVAL;
    if (overlaps(grads, ng, f0, n19) || overlaps(grads, ng, g0, n19) || overlaps(grads, ng, post, npost))
        return LB_EINVAL;
    c->launched = true;
    const Geo geo = c->canonical_geo();
    const auto cp = coll_params<double>(c);
    double* afield = (double*)c->fbuf(1 - c->cur);   // spare state buffer: >= 19 N doubles, 6 N used
    double* bfield = afield + 5 * N;
    double* lf_cur = lf;                              // lambda_f^{n+1}
    double* lf_nxt = work;
    double* p_cur = lg;                               // lambda_g^{n+1} (first step) or P^{n+1}
    double* p_nxt = work + n19;
    for (int32_t n = length - 1; n >= 0; --n) {
        Timed t(c, LB_K_ADJOINT);
        const bool pending = n > 0;
        const double* fn = pending ? post + (size_t)(n - 1) * 2 * n19 : f0;
        const double* gn = pending ? fn + n19 : g0;
        const double* ph = (phi && n < length - 1) ? phi + (size_t)n * N : nullptr;
        if (!ph) {
            double* p = (double*)c->phi();
            if (pending) k_phi<Pol, double, true><<<c->grid(), c->block(), 0, c->stream>>>(gn, p, geo, 0.0);
            else k_phi<Pol, double, false><<<c->grid(), c->block(), 0, c->stream>>>(gn, p, geo, 0.0);
            ph = p;
        }
        if (n == length - 1)
            launch_adjoint_binary_local<LG_GATHER_KEEP>(c, pending, fn, gn, ph, lf_cur, p_cur, nullptr, lf_nxt,
                                                        p_nxt, afield, geo, cp);
        else
            launch_adjoint_binary_local<LG_PULLED_KEEP>(c, pending, fn, gn, ph, lf_cur, p_cur, bfield, lf_nxt,
                                                        p_nxt, afield, geo, cp);
        launch_adjoint_binary_stencil<true>(c, afield, nullptr, bfield, geo, 1.0, grads);
        std::swap(lf_cur, lf_nxt);
        std::swap(p_cur, p_nxt);
    }
    {
        // lambda_g^{s0} = (1 - omega_g) P^{s0} + b^{s0}, into lg (in place when P^{s0} is there)
        Timed t(c, LB_K_ADJOINT);
        k_adjoint_binary_combine<Pol><<<c->grid(), c->block(), 0, c->stream>>>(p_cur, bfield, lg, geo, cp.omega_g);
    }
    if (lf_cur != lf) {
        Timed t(c, LB_K_OTHER);
        if (hipMemcpyAsync(lf, lf_cur, n19 * sizeof(double), hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
            return LB_EDEVICE;
    }
    return launch_status();
}

int lb_mask_index(lb_ctx* c, const uint8_t* mask, int32_t* index, int64_t* count) {
    if (!c || !mask || !index || !count) return LB_EINVAL;
    c->launched = true;
    const uint32_t n = (uint32_t)c->L.nsite;
    const int nb = (int)((n + CB * CM - 1) / (CB * CM));
    int64_t* counts = reinterpret_cast<int64_t*>(c->partial());   // nb <= tiles of the launch grid
    Timed t(c, LB_K_OTHER);
    k_mask_count<<<nb, CB, 0, c->stream>>>(mask, n, counts);
    k_scan_counts<<<1, CB, 0, c->stream>>>(counts, nb, count);
    k_mask_scatter<<<nb, CB, 0, c->stream>>>(mask, n, counts, index);
    return launch_status();
}


int lb_get_sites(lb_ctx* c, const int32_t* index, int64_t m, void* f, void* g) {
    if (!c || m < 0 || m > c->L.nsite) return LB_EINVAL;
    if (m == 0) return LB_OK;
    if (!index || !f || ((c->p.model == LB_BINARY) != (g != nullptr))) return LB_EINVAL;
    return by_storage(c, [&](auto tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        return run_sites<S>(c, index, m, (S*)f, (S*)g, false);
    });
}

int lb_set_sites(lb_ctx* c, const int32_t* index, int64_t m, const void* f, const void* g) {
    if (!c || m < 0 || m > c->L.nsite) return LB_EINVAL;
    if (m == 0) return LB_OK;
    if (!index || !f || ((c->p.model == LB_BINARY) != (g != nullptr))) return LB_EINVAL;
    return by_storage(c, [&](auto tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        return run_sites<S>(c, index, m, (S*)f, (S*)g, true);
    });
}

int lb_profile_mask(lb_ctx* c, unsigned kinds) {
    if (!c || (kinds >> (LB_K_OTHER + 1)) != 0) return LB_EINVAL;
    if (kinds) {
        if (hipStreamSynchronize(c->stream) != hipSuccess) return LB_EDEVICE;
        c->release_records();
    }
    c->profiling = kinds != 0;
    c->profile_kinds = kinds;
    return LB_OK;
}

int lb_profile(lb_ctx* c, int enable) {
    return lb_profile_mask(c, enable ? (1u << (LB_K_OTHER + 1)) - 1u : 0u);
}

int lb_kernel_times(lb_ctx* c, int kind, double* total_ms, int64_t* launches) {
    if (!c || !total_ms || !launches || kind < 0 || kind > LB_K_OTHER) return LB_EINVAL;
    double ms = 0.0;
    int64_t n = 0;
    for (auto& r : c->recs) {
        if (r.kind != kind) continue;
        if (hipEventSynchronize(r.stop) != hipSuccess) return LB_EDEVICE;
        float e = 0.0f;
        if (hipEventElapsedTime(&e, r.start, r.stop) != hipSuccess) return LB_EDEVICE;
        ms += e;
        ++n;
    }
    *total_ms = ms;
    *launches = n;
    return LB_OK;
}

int lb_destroy(lb_ctx* c) {
    if (!c) return LB_OK;
    int rc = LB_OK;
    if (c->launched && hipStreamSynchronize(c->stream) != hipSuccess) rc = LB_EDEVICE;
    c->release_records();
    for (hipEvent_t e : c->pool) (void)hipEventDestroy(e);
    delete c;
    return rc;
}

int lb_stream_copy(void* dst, const void* src, size_t bytes, void* stream) {
    if (bytes == 0) return LB_OK;
    if (!dst || !src) return LB_EINVAL;
    const uintptr_t d = reinterpret_cast<uintptr_t>(dst), s = reinterpret_cast<uintptr_t>(src);
    if (d % 16 != 0 || s % 16 != 0 || bytes % 16 != 0) return LB_EINVAL;
    if (d < s + bytes && s < d + bytes) return LB_EINVAL;
    const uint64_t nwords = bytes / 16;
    const uint64_t per_block = (uint64_t)COPY_TPB * COPY_U;
    const uint64_t nblocks = (nwords + per_block - 1) / per_block;
    if (nblocks > 0x7fffffffull) return LB_EINVAL;
    k_stream_copy<<<(unsigned)nblocks, COPY_TPB, 0, (hipStream_t)stream>>>(
        static_cast<const u32x4*>(src), static_cast<u32x4*>(dst), nwords);
    return launch_status();
}

const char* lb_strerror(int status) {
    switch (status) {
        case LB_OK: return "ok";
        case LB_EINVAL: return "invalid argument";
        case LB_ENOMEM: return "workspace too small";
        case LB_EDEVICE: return "HIP runtime or kernel launch failure";
        case LB_ENOTSUP: return "not supported for this model or storage";
        case LB_ERANGE: return "lattice too large for the fixed scratch of an allocation-free call";
    }
    return "unknown status";
}

}  // extern "C"
