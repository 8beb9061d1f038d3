// Ragged batches of independent systems: the plan (work items, partial-sum layout,
// device tables and scratch, built once from the host offsets) and the batched force
// and leapfrog entry points.
//
// Work items: each system with N_k particles is cut into groups of 64 * wi i's and
// S_k j-segments of about kItemJ j's; an item is one (group, segment) pair of one system.
// Items are sorted by decreasing cost (i-lanes x j's, including padding), so large systems
// start first and small ones fill the tail.
#include <algorithm>
#include <cmath>
#include <new>
#include <vector>

#include "nbody_internal.h"
#include "tuning.h"

struct nbody_plan {
    int device = 0;
    int nsys = 0;
    int64_t total = 0;
    nbody_opts opts{};
    int jt = 256;
    int wi = 1;          // i-records per lane of the launch
    int waves = 4;       // waves per work item
    int nitems = 0;
    bool split = false;  // some system has more than one j-segment
    int64_t largest = 0; // particles of the largest system
    int64_t padded_pairs = 0;
    int64_t pairs = 0;
    // device tables
    nbody::BatchItem *items = nullptr;
    int64_t *offsets = nullptr;
    int32_t *sys_of = nullptr;
    int64_t *part_base = nullptr;
    int32_t *npad = nullptr;
    int32_t *nseg = nullptr;
    // scratch
    void *part = nullptr;
    size_t part_bytes = 0;
    float *x32 = nullptr;
    double *centre = nullptr;
};

namespace nbody {
namespace {

constexpr int64_t kItemJ = 4096;  // target j's per work item
// Largest system whose kick, drift, centre and conversion one block does in one launch: 16
// particles per thread and pass (about 5 us, against 3 launches).
constexpr int64_t kBlockSystem = 4096;

void free_plan(nbody_plan *p) {
    if (!p) return;
    void *ptrs[] = {p->items, p->offsets, p->sys_of, p->part_base, p->npad,
                    p->nseg,  p->part,    p->x32,    p->centre};
    for (void *q : ptrs)
        if (q) (void)hipFree(q);
    delete p;
}

template <typename T>
nbody_status dev_copy(T **dst, const std::vector<T> &src) {
    const size_t bytes = sizeof(T) * (src.empty() ? 1 : src.size());
    hipError_t e = hipMalloc(reinterpret_cast<void **>(dst), bytes);
    if (e != hipSuccess) {
        *dst = nullptr;
        return hip_error(e, "hipMalloc(plan)");
    }
    if (!src.empty()) {
        e = hipMemcpy(*dst, src.data(), sizeof(T) * src.size(), hipMemcpyHostToDevice);
        if (e != hipSuccess) return hip_error(e, "hipMemcpy(plan)");
    }
    return NBODY_OK;
}

nbody_status check_plan_call(const nbody_plan *p, const void *pos, const float *mass,
                             const float *eps, const double *acc) {
    if (!p) return set_error(NBODY_EINVAL, "plan must not be NULL");
    if (p->total > 0 && (!pos || !mass || !eps || !acc))
        return set_error(NBODY_EINVAL, "pos, mass, eps and acc must not be NULL");
    int dev = 0;
    NBODY_HIP_CHECK(hipGetDevice(&dev));
    if (dev != p->device) return set_error(NBODY_EINVAL, "plan was created on another device");
    return NBODY_OK;
}

// Pair kernel (+ batched finalize of the split systems) on FP32 positions.
nbody_status batched_core(const nbody_plan *p, const float *pos, const float *mass,
                          const float *eps, double *acc, double *pot, double *kick_v,
                          double kick_h, hipStream_t s) {
    const int64_t n = p->total;
    PairArgs pa{pos, pos + n, pos + 2 * n, mass, (int)n, 0, 0.0f, p->part, 0};
    FinalizeArgs out{nullptr, 1, 0, (int)n, mass, 0.0f, 0, acc, pot, kick_v, kick_h};
    BatchSched sc{p->items, p->nitems, eps, p->part};
    nbody_status st = launch_batched_pair(p->wi, p->jt, p->waves, p->opts.precision, pot != nullptr,
                                          pa, out, sc, s);
    if (st || !p->split) return st;
    BatchFinalizeArgs fa{p->part, n,   p->sys_of, p->offsets, p->part_base, p->npad, p->nseg,
                         acc,     pot, kick_v,    kick_h};
    return launch_batched_finalize(p->opts.precision, fa, s);
}

nbody_status batched_f64_core(const nbody_plan *p, const double *pos64, const float *mass,
                              const float *eps, double *acc, double *pot, double *kick_v,
                              double kick_h, hipStream_t s) {
    nbody_status st;
    const double *cen = nullptr;
    if (p->opts.centre == NBODY_CENTRE_SYSTEM && p->largest <= kBlockSystem) {
        if ((st = launch_system_step(p->nsys, p->offsets, p->total, const_cast<double *>(pos64),
                                     nullptr, nullptr, 0.0, 0.0, p->x32, s)))
            return st;
        return batched_core(p, p->x32, mass, eps, acc, pot, kick_v, kick_h, s);
    }
    if (p->opts.centre == NBODY_CENTRE_SYSTEM) {
        if ((st = launch_system_centres(p->nsys, p->offsets, p->total, pos64, p->centre, s))) return st;
        cen = p->centre;
    }
    if ((st = launch_batched_convert(p->total, pos64, p->sys_of, cen, p->x32, s))) return st;
    return batched_core(p, p->x32, mass, eps, acc, pot, kick_v, kick_h, s);
}

nbody_status enqueue_batched_steps(const nbody_plan *p, double *x, double *v, const float *m,
                                   const float *eps, double dt, int32_t nsteps, double *acc,
                                   double *pot, bool init, hipStream_t s) {
    nbody_status st;
    if (init || (nsteps == 0 && pot))
        if ((st = batched_f64_core(p, x, m, eps, acc, nsteps == 0 ? pot : nullptr, nullptr, 0.0, s)))
            return st;
    for (int32_t t = 0; t < nsteps; ++t) {
        if (p->opts.centre == NBODY_CENTRE_SYSTEM && p->largest <= kBlockSystem) {
            if ((st = launch_system_step(p->nsys, p->offsets, p->total, x, v, acc, 0.5 * dt, dt,
                                         p->x32, s)))
                return st;
            if ((st = batched_core(p, p->x32, m, eps, acc, t + 1 == nsteps ? pot : nullptr, v,
                                   0.5 * dt, s)))
                return st;
            continue;
        }
        if ((st = launch_kick_drift(p->total, x, x, v, acc, 0.5 * dt, dt, s))) return st;
        if ((st = batched_f64_core(p, x, m, eps, acc, t + 1 == nsteps ? pot : nullptr, v, 0.5 * dt, s)))
            return st;
    }
    return NBODY_OK;
}

}  // namespace
}  // namespace nbody

using namespace nbody;

extern "C" {

nbody_status nbody_plan_create_batched(int32_t nsys, const int64_t *h_offsets,
                                       const nbody_opts *opts, nbody_plan **out) {
    clear_error();
    if (!out) return set_error(NBODY_EINVAL, "out must not be NULL");
    *out = nullptr;
    if (nsys < 0) return set_error(NBODY_EINVAL, "nsys must be >= 0");
    if (nsys > 0 && !h_offsets) return set_error(NBODY_EINVAL, "offsets must not be NULL");
    nbody_opts o = resolve_opts(opts);
    if (o.precision < NBODY_PLAIN || o.precision > NBODY_COMP)
        return set_error(NBODY_EINVAL, "precision must be NBODY_PLAIN, NBODY_FP64RED or NBODY_COMP");
    if (o.centre != NBODY_CENTRE_NONE && o.centre != NBODY_CENTRE_SYSTEM)
        return set_error(NBODY_EUNSUPPORTED, "batched plans support NBODY_CENTRE_NONE and _SYSTEM");
    if (o.self_pot != 0) return set_error(NBODY_EUNSUPPORTED, "batched plans exclude the self term");
    if (o.workspace) return set_error(NBODY_EINVAL, "a plan owns its scratch; opts->workspace must be NULL");
    if (o.jlanes > 1) return set_error(NBODY_EUNSUPPORTED, "batched plans use the grid engine (jlanes 0 or 1)");
    if (o.jlanes < 0) return set_error(NBODY_EINVAL, "jlanes must be >= 0");
    if (o.symmetric < 0 || o.symmetric > 2)
        return set_error(NBODY_EINVAL, "symmetric must be 0 (tuned), 1 (off) or 2 (on)");
    if (o.symmetric == 2)
        return set_error(NBODY_EUNSUPPORTED, "batched plans use the grid engine (symmetric 0 or 1)");
    if (nsys > 0 && h_offsets[0] != 0) return set_error(NBODY_EINVAL, "offsets[0] must be 0");
    for (int32_t k = 0; k < nsys; ++k)
        if (h_offsets[k + 1] < h_offsets[k])
            return set_error(NBODY_EINVAL, "offsets must be non-decreasing");
    const int64_t total = nsys > 0 ? h_offsets[nsys] : 0;
    if (total > INT32_MAX / 2) return set_error(NBODY_EINVAL, "total particles must be < 2^30");

    TuneEntry te = tuned_shape(KERNEL_BATCHED, o.precision, total / std::max<int64_t>(1, nsys), 0);
    // i-records per lane asked for, by the caller or the table; 0: by size, as the items are.
    const int ipl = o.ipl ? o.ipl : te.set ? te.ipl : 0;
    const int jt = o.jtile ? o.jtile : te.jt;
    if (!(ipl == 0 || ipl == 1 || ipl == 2 || ipl == 4 || ipl == 8))
        return set_error(NBODY_EINVAL, "ipl must be 1, 2, 4 or 8");
    if (!(jt == 64 || jt == 128 || jt == 256 || jt == 512))
        return set_error(NBODY_EINVAL, "jtile must be 64, 128, 256 or 512");

    nbody_plan *p = new (std::nothrow) nbody_plan;
    if (!p) return set_error(NBODY_ENOMEM, "out of host memory");
    p->nsys = nsys;
    p->total = total;
    p->opts = o;
    p->jt = jt;
    hipError_t e = hipGetDevice(&p->device);
    if (e != hipSuccess) {
        free_plan(p);
        return hip_error(e, "hipGetDevice");
    }

    // i-records per lane: asked for, else by the work (pieces of 64 i's x 128 j's), as for
    // one system.
    int64_t blocks1 = 0, runs1 = 0;
    int64_t &largest = p->largest;
    for (int32_t k = 0; k < nsys; ++k) {
        const int64_t n = h_offsets[k + 1] - h_offsets[k];
        blocks1 += (n + 63) / 64 * ((n + 127) / 128);
        runs1 += (n + 63) / 64 * ((n + kItemJ - 1) / kItemJ);
        largest = std::max(largest, n);
    }
    p->wi = wave_ipl(KERNEL_BATCHED, o.precision, blocks1,
                     o.precision == NBODY_PLAIN ? runs1 : blocks1, ipl);
    // Waves per item: 4, and as many as the largest segment has FP32 blocks, up to 16, where
    // there is too little work to keep 4 waves per SIMD busy with longer runs.
    p->waves = 4;
    if (o.precision == NBODY_PLAIN) {
        p->waves = 1;
    } else if (!ipl && blocks1 < 50000) {
        const int64_t nb = (std::min(largest, kItemJ) + 127) / 128;
        p->waves = (int)std::max<int64_t>(4, std::min<int64_t>(16, nb));
    }

    // j's per item.  With the shape by size, and enough work to fill the chip with long items, the
    // largest systems of 2^14 particles stay whole as well: no partial sums, no finalize.
    const bool open_shape = !ipl && o.precision != NBODY_PLAIN;
    const int64_t item_j = open_shape && blocks1 >= 1000000 ? 4 * kItemJ : kItemJ;

    // The partial-sum layout, then the items: (system, j-segment) pairs in decreasing order
    // of their length, ties in creation order, and the groups of i's of each.
    struct Segment {
        int32_t sys, j0, nj;
        int64_t part;
    };
    const int64_t itile = (int64_t)64 * p->wi;
    const int64_t unroll = wave_unroll(p->wi);
    const int wo = 4 * (o.precision == NBODY_PLAIN ? 1 : 2);  // words per (i, segment)
    const int64_t tiles_per_seg = std::max<int64_t>(1, item_j / jt);
    std::vector<Segment> segments;
    std::vector<int64_t> base(std::max(nsys, 1)), offs(h_offsets, h_offsets + nsys + 1);
    std::vector<int32_t> npad(std::max(nsys, 1)), nseg(std::max(nsys, 1)), sys_of((size_t)total);
    int64_t words = 0, nitems = 0;
    for (int32_t k = 0; k < nsys; ++k) {
        const int64_t off = h_offsets[k], n = h_offsets[k + 1] - off;
        std::fill_n(sys_of.begin() + off, n, k);
        base[k] = words;
        npad[k] = 0;
        nseg[k] = 0;
        if (n == 0) continue;
        const int64_t t = (n + itile - 1) / itile;
        const int64_t jtiles = (n + jt - 1) / jt;
        int64_t segs = (jtiles + tiles_per_seg - 1) / tiles_per_seg;
        const int64_t per = (jtiles + segs - 1) / segs;
        segs = (jtiles + per - 1) / per;
        const int64_t seg_len = per * jt;
        npad[k] = (int32_t)(t * itile);
        nseg[k] = (int32_t)segs;
        p->split = p->split || segs > 1;
        for (int64_t si = 0; si < segs; ++si)
            segments.push_back({k, (int32_t)(off + si * seg_len),
                                (int32_t)std::min(seg_len, n - si * seg_len),
                                words + si * wo * (t * itile)});
        nitems += segs * t;
        if (segs > 1) words += segs * wo * t * itile;
        p->pairs += n * n;
    }
    std::stable_sort(segments.begin(), segments.end(),
                     [](const Segment &a, const Segment &b) { return a.nj > b.nj; });
    std::vector<BatchItem> sorted;
    sorted.reserve((size_t)nitems);
    for (const Segment &sg : segments) {
        const int32_t k = sg.sys;
        const int64_t off = h_offsets[k], n = h_offsets[k + 1] - off;
        for (int64_t c = 0; c < n; c += itile) {
            BatchItem w;
            w.sys = k;
            w.i0 = (int32_t)(off + c);
            w.ni = (int32_t)std::min(itile, n - c);
            w.j0 = sg.j0;
            w.nj = sg.nj;
            w.col0 = (int32_t)c;
            w.part = sg.part;
            w.npad = npad[k];
            w.whole = nseg[k] == 1;
            sorted.push_back(w);
            p->padded_pairs += itile * ((sg.nj + unroll - 1) / unroll * unroll);
        }
    }
    p->nitems = (int)sorted.size();

    nbody_status st = NBODY_OK;
    auto bail = [&](nbody_status code) {
        free_plan(p);
        return code;
    };
    if ((st = dev_copy(&p->items, sorted))) return bail(st);
    if ((st = dev_copy(&p->offsets, offs))) return bail(st);
    if ((st = dev_copy(&p->sys_of, sys_of))) return bail(st);
    if ((st = dev_copy(&p->part_base, base))) return bail(st);
    if ((st = dev_copy(&p->npad, npad))) return bail(st);
    if ((st = dev_copy(&p->nseg, nseg))) return bail(st);
    p->part_bytes = (size_t)std::max<int64_t>(words, 1) * 4;
    if ((e = hipMalloc(&p->part, p->part_bytes)) != hipSuccess) {
        p->part = nullptr;
        return bail(hip_error(e, "hipMalloc(plan partials)"));
    }
    if ((e = hipMalloc(reinterpret_cast<void **>(&p->x32), sizeof(float) * 3 * std::max<int64_t>(total, 1))) != hipSuccess) {
        p->x32 = nullptr;
        return bail(hip_error(e, "hipMalloc(plan positions)"));
    }
    if ((e = hipMalloc(reinterpret_cast<void **>(&p->centre), sizeof(double) * 3 * std::max(nsys, 1))) != hipSuccess) {
        p->centre = nullptr;
        return bail(hip_error(e, "hipMalloc(plan centres)"));
    }
    *out = p;
    return NBODY_OK;
}

void nbody_plan_destroy(nbody_plan *plan) {
    if (!plan) return;
    (void)hipDeviceSynchronize();
    free_plan(plan);
}

nbody_status nbody_plan_info(const nbody_plan *plan, int64_t *info) {
    clear_error();
    if (!plan || !info) return set_error(NBODY_EINVAL, "plan and info must not be NULL");
    info[0] = plan->nsys;
    info[1] = plan->total;
    info[2] = plan->nitems;
    info[3] = plan->nitems;
    info[4] = plan->pairs;
    info[5] = plan->padded_pairs;
    info[6] = plan->wi;
    info[7] = plan->jt;
    return NBODY_OK;
}

nbody_status nbody_force_batched(const nbody_plan *plan, const float *pos, const float *mass,
                                 const float *eps, double *acc, double *pot, void *stream) {
    clear_error();
    nbody_status st = check_plan_call(plan, pos, mass, eps, acc);
    if (st) return st;
    if (misaligned(pos) || misaligned(mass) || misaligned(eps) || misaligned(acc) || misaligned(pot))
        return set_error(NBODY_EINVAL, "misaligned array argument");
    if (plan->total == 0) return NBODY_OK;
    return batched_core(plan, pos, mass, eps, acc, pot, nullptr, 0.0, static_cast<hipStream_t>(stream));
}

nbody_status nbody_force_batched_f64(const nbody_plan *plan, const double *pos64, const float *mass,
                                     const float *eps, double *acc, double *pot, void *stream) {
    clear_error();
    nbody_status st = check_plan_call(plan, pos64, mass, eps, acc);
    if (st) return st;
    if (misaligned(pos64) || misaligned(mass) || misaligned(eps) || misaligned(acc) || misaligned(pot))
        return set_error(NBODY_EINVAL, "misaligned array argument");
    if (plan->total == 0) return NBODY_OK;
    return batched_f64_core(plan, pos64, mass, eps, acc, pot, nullptr, 0.0,
                            static_cast<hipStream_t>(stream));
}

nbody_status nbody_leapfrog_batched(const nbody_plan *plan, double *pos64, double *vel64,
                                    const float *mass, const float *eps, double dt, int32_t nsteps,
                                    double *acc, double *pot, int32_t flags, void *stream) {
    clear_error();
    nbody_status st = check_plan_call(plan, pos64, mass, eps, acc);
    if (st) return st;
    if (plan->total > 0 && !vel64) return set_error(NBODY_EINVAL, "vel must not be NULL");
    if (nsteps < 0) return set_error(NBODY_EINVAL, "nsteps must be >= 0");
    if (!std::isfinite(dt)) return set_error(NBODY_EINVAL, "dt must be finite");
    if (flags & ~NBODY_LF_INIT_ACC) return set_error(NBODY_EINVAL, "unknown flags");
    if (misaligned(pos64) || misaligned(vel64) || misaligned(mass) || misaligned(eps) ||
        misaligned(acc) || misaligned(pot))
        return set_error(NBODY_EINVAL, "misaligned array argument");
    if (plan->total == 0) return NBODY_OK;
    return enqueue_batched_steps(plan, pos64, vel64, mass, eps, dt, nsteps, acc, pot,
                                 (flags & NBODY_LF_INIT_ACC) != 0, static_cast<hipStream_t>(stream));
}

nbody_status nbody_graph_create_leapfrog_batched(const nbody_plan *plan, double *pos64,
                                                 double *vel64, const float *mass,
                                                 const float *eps, double dt, int32_t nsteps,
                                                 double *acc, double *pot, void *stream,
                                                 nbody_graph **out) {
    clear_error();
    if (!out) return set_error(NBODY_EINVAL, "out must not be NULL");
    *out = nullptr;
    nbody_status st = check_plan_call(plan, pos64, mass, eps, acc);
    if (st) return st;
    if (plan->total == 0 || nsteps <= 0)
        return set_error(NBODY_EINVAL, "graph needs particles and nsteps > 0");
    if (!vel64) return set_error(NBODY_EINVAL, "vel must not be NULL");
    if (!std::isfinite(dt)) return set_error(NBODY_EINVAL, "dt must be finite");
    if (stream_capturing(static_cast<hipStream_t>(stream)))
        return set_error(NBODY_ECAPTURE, "stream is already capturing");
    nbody_graph *g = new (std::nothrow) nbody_graph;
    if (!g) return set_error(NBODY_ENOMEM, "out of host memory");
    g->device = plan->device;
    st = capture_graph(g, [&](hipStream_t cs) {
        return enqueue_batched_steps(plan, pos64, vel64, mass, eps, dt, nsteps, acc, pot, false, cs);
    });
    if (st) {
        nbody_graph_destroy(g);
        return st;
    }
    *out = g;
    return NBODY_OK;
}

}  // extern "C"
