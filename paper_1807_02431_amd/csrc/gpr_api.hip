// gpr_api.hip -- host runtime behind the C ABI of include/gpr.h.
//
// Owns the device buffers of a system, drives the stepping paths and the per-check
// bookkeeping kernels, and keeps the Gen.ParRep phase machine (transient propagation,
// Fleming-Viot convergence step, parallel step; Sec. 2.4, Fig. 1) on the host: every
// decision is taken from a small status word read back once per check.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <climits>
#include <new>
#include <string>
#include <vector>

#include "gpr.h"
#include "gpr_kernels.h"
#include "gpr_room.h"

using namespace gpr;

namespace {

constexpr double COULOMB_F = 138.935458;
enum { PH_IDLE = 0, PH_DECORR = 1, PH_DEPHASE = 2, PH_CONVERGED = 3, PH_PARALLEL = 4, PH_DEPHASE_FIXED = 5 };

thread_local std::string g_thread_err;

constexpr int MAX_DEV = 64;
Room g_room[MAX_DEV];                  // by device

} // namespace

struct gpr_system {
    Dev d{};
    Dev *d_dev = nullptr;     // device copy of d, passed to every kernel
    std::vector<void *> bufs;
    hipStream_t stream = nullptr;
    int dev = 0;               // the device it was created on
    int held = 0;              // room taken on it by launches not yet waited for
    Room::Key held_by{};
    int path = GPR_PATH_PLAIN;
    int bt_persist = 0;
    int groups = 1;            // workgroups per replica on the persistent path
    Split split{};             // their atom ranges
    Split splits[NSPLIT]{};    // the atom ranges with 1, 2, 4, ... MAX_G workgroups per replica (fewer for tiny ones)
    bool split_ok[NSPLIT]{};        // whether a workgroup of that split fits on a compute unit
    // whose choice the launch shape is: 0 the library's, for the replicas of each launch
    // (run_shape), 1 the autotuner's, for launches of all replicas, 2 the caller's, for every launch
    int bt_from = 0, groups_from = 0;
    std::vector<double> work;  // per-atom work estimate that places the ranges
    // bonded units of the plain path's ranges and of every split, one after the other
    uint2 *unit_bi = nullptr;
    float4 *unit_bp = nullptr;
    int *unit_src = nullptr;   // per record: 5 * (sorted term) + kind, or -1
    int n_records = 0;
    // force-field parameters as the caller gave them (gpr_set_params rewrites the device copies)
    std::vector<double> mass_h, eps_h, sig_h, q_h, tor_k_h, tor_phi0_h;
    std::vector<int> tor_n_h, tor_order, p14_order;   // sorted term -> caller's index
    std::vector<int2> p14_h;
    double scale14 = 0.0;
    int max_coresident = 0;    // persistent-kernel workgroups that fit on the device at once
    struct Cap { int bt; size_t lds; int blocks; };
    std::vector<Cap> caps;     // persist_capacity: the launch shapes asked for and their capacities
    int n = 0, R = 0, np = 0, kind = 0, nobs = 0;
    int t_gr = 1, tcd = 1, tcp = 1;
    double tol = 0, dt = 0, kT = 0;
    long long t_min = 0;
    // phase machine
    long long s = 0, tsim = 0;
    int omega = -1, phase = PH_IDLE;
    int dc_from = -1, dc_omega = -1;
    long long dc_resid = 0, dc_steps = 0;
    long long dp_t = 0, nsamp = 0, n_branch = 0;
    long long adv_t = 0;       // steps taken by gpr_advance / gpr_batch_advance: their sampling and check phase
    long long par_M = 0, par_t = 0;   // parallel step: checks done, steps into the current check period
    // original ParRep dephasing: start configuration, samples, per-replica progress
    float *snap_x = nullptr, *snap_v = nullptr, *samp_x = nullptr, *samp_v = nullptr;
    long long *snap_F = nullptr, *samp_F = nullptr;
    std::vector<long long> resid;
    std::vector<int> done;
    // plain path as replays of a captured cycle of steps (0: off)
    int graph_cycle = 0;
    struct Graph { int nrep, code, phase; hipGraphExec_t exec; };
    std::vector<Graph> graphs;
    // persistent convergence and parallel steps as replays of captured check cycles (0: off)
    int cycles = 0;
    struct CGraph { int op; hipGraphExec_t exec; int units; };    // units: room a replay needs
    std::vector<CGraph> cgraphs;
    CycRec *cyc_dev = nullptr, *cyc_host = nullptr;
    Status *stc_dev = nullptr, *stc_host = nullptr;   // [cycles] statuses of a replay
    // scratch
    // page-locked, the three in one allocation:
    Status *st_host = nullptr;      // the status of the last check, written by k_check
    long long *adv_fec = nullptr;   // [R]: first exit checks of an advance
    char *rb = nullptr;             // [rb_bytes]: results on their way to the caller (k_read)
    size_t rb_bytes = 0;
    bool gacc_dirty = false;        // a backward pass did not get to clear gacc
    bool lists_old = false;         // some replica's pair lists may not be those of its positions (k_persist_small
                                    // keeps none, copies take none along): stepping rebuilds them, k_grad_nb reads them
    double *obs_out = nullptr;
    int *donor = nullptr, *surv = nullptr;
    long long *fec = nullptr;
    size_t lds_nb = 0, lds_stage = 0;
    int maxlds = 0;            // LDS bytes one workgroup may use on this device
    int maxlds_persist = 0;    // of which k_persist may allocate dynamically
    int persist_ok = 0;
    bool small_ok = false;     // the system may run k_persist_small (with one workgroup per replica)
    // event timing of the dominant stepping kernel
    bool prof = false;
    std::vector<hipEvent_t> ev_a, ev_b;
    size_t ev_used = 0;
    double prof_ms = 0.0;
    long long prof_n = 0;
    std::string err;
};

namespace {

gpr_status fail(gpr_system *s, gpr_status code, const std::string &msg)
{
    if (s) s->err = msg;
    g_thread_err = msg;
    return code;
}

#define HIPCHK(sys, call)                                                                        \
    do {                                                                                         \
        hipError_t e_ = (call);                                                                  \
        if (e_ != hipSuccess)                                                                    \
            return fail((sys), GPR_EDEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

#define LAUNCHCHK(sys)                                                                           \
    do {                                                                                         \
        hipError_t e_ = hipGetLastError();                                                       \
        if (e_ != hipSuccess)                                                                    \
            return fail((sys), GPR_EDEVICE, std::string("kernel launch: ") + hipGetErrorString(e_)); \
    } while (0)

template <class T>
hipError_t dalloc(gpr_system *s, T **p, size_t count, bool clear = true)
{
    void *q = nullptr;
    hipError_t e = hipMalloc(&q, std::max<size_t>(count, 1) * sizeof(T));
    if (e != hipSuccess) return e;
    s->bufs.push_back(q);
    *p = (T *)q;
    return clear ? hipMemset(q, 0, std::max<size_t>(count, 1) * sizeof(T)) : hipSuccess;
}

template <class T>
hipError_t upload(gpr_system *s, T **p, const std::vector<T> &h)
{
    hipError_t e = dalloc(s, p, h.size(), h.empty());
    if (e != hipSuccess || h.empty()) return e;
    return hipMemcpy(*p, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice);
}

bool idx_ok(const int32_t *a, long cnt, int n)
{
    if (cnt > 0 && !a) return false;
    for (long k = 0; k < cnt; ++k) if (a[k] < 0 || a[k] >= n) return false;
    return true;
}

// the order of terms of width w by their smallest atom
void sort_terms(const int32_t *atoms, int cnt, int w, std::vector<int> &order)
{
    order.resize(cnt);
    std::vector<int> mn(cnt);
    for (int t = 0; t < cnt; ++t) {
        mn[t] = *std::min_element(atoms + t * w, atoms + (t + 1) * w);
        order[t] = t;
    }
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return mn[a] < mn[b]; });
}

long long count_samples(long long t_old, long long t_new, int t_gr) { return t_new / t_gr - t_old / t_gr; }

} // namespace

static void drop_cycle_graphs(gpr_system *S);

// one more pair of timing events (created ahead by gpr_profile, so that a timed call does not
// create them; more only when a call launches the kernel more often than that)
static hipError_t prof_add_pair(gpr_system *S)
{
    hipEvent_t a, b;
    hipError_t e = hipEventCreate(&a);
    if (e != hipSuccess) return e;
    e = hipEventCreate(&b);
    if (e != hipSuccess) {
        (void)hipEventDestroy(a);
        return e;
    }
    S->ev_a.push_back(a);
    S->ev_b.push_back(b);
    return hipSuccess;
}

// event pair around the next timed launch
static hipError_t prof_begin(gpr_system *S)
{
    if (!S->prof) return hipSuccess;
    if (S->ev_used == S->ev_a.size()) {
        const hipError_t e = prof_add_pair(S);
        if (e != hipSuccess) return e;
    }
    return hipEventRecord(S->ev_a[S->ev_used], S->stream);
}

static hipError_t prof_end(gpr_system *S)
{
    if (!S->prof) return hipSuccess;
    hipError_t e = hipEventRecord(S->ev_b[S->ev_used], S->stream);
    S->ev_used++;
    return e;
}

// after the stream has drained: fold the recorded pairs into the totals
static hipError_t prof_collect(gpr_system *S)
{
    for (size_t k = 0; k < S->ev_used; ++k) {
        float ms = 0.f;
        hipError_t e = hipEventElapsedTime(&ms, S->ev_a[k], S->ev_b[k]);
        if (e != hipSuccess) return e;
        S->prof_ms += ms;
        S->prof_n += 1;
    }
    S->ev_used = 0;
    return hipSuccess;
}

static Split make_split(const std::vector<double> &work, int n, int np, int G)
{
    Split sp{};
    static_cast<AtomRanges &>(sp) = atom_ranges(work, n, np, G);
    return sp;
}

static int split_index(int G)
{
    int k = 0;
    while ((1 << k) < G) ++k;
    return k;
}

static size_t persist_lds(int n, int np, const Split &sp) { return (size_t)persist_off(n, np, sp.lmax).gn; }

// Whether workgroups of bt threads keep the next step's Gaussians in LDS too: where it fits and
// leaves as many workgroups on a compute unit (16 waves at the kernel's register count)
static bool noise_fits(int n, int np, const Split &sp, int bt, int maxlds)
{
    const PersistOff o = persist_off(n, np, sp.lmax);
    const int waves = std::max(1, 1024 / bt);
    return o.end <= maxlds && std::min(waves, maxlds / o.end) == std::min(waves, maxlds / o.gn);
}

// LDS of k_persist_small (the order of small_lds_layout) and its units of work per step
static size_t small_lds(const gpr_system *S)
{
    const Topo &T = S->d.tp;
    const size_t n = S->n, np = S->np, nterm = (size_t)T.nt + T.na + T.n14 + T.nb + T.nr;
    return 16 * np + 16 * nterm + 48 * n + 64 + (24 + sizeof(ObsDesc)) * MAX_OBS + 8 * np + 8 * 64 * ((n + 15) / 16) + 8 * nterm + 32 * n;
}
static int small_units(const gpr_system *S)
{
    const Topo &T = S->d.tp;
    auto blocks = [](int c) { return (c + 63) / 64; };
    return blocks(T.nt) + blocks(T.na) + blocks(T.n14) + blocks(T.nb) + blocks(T.nr) + blocks(S->n) +
           (S->kind == GPR_KIND_TOY2D ? 1 : (S->n + 15) / 16);
}
// Launch shape of a persistent launch of one system's first nrep replicas.  Unless the caller (or
// the autotuner) chose it:
//   workgroups per replica: those of a launch of all replicas, doubled while all workgroups of the
//   launch still get a compute unit of their own and a group keeps 32 atoms (measured, us per step:
//   one replica of 2,432 atoms 12.1 with 8 groups, 8.9 with 16, 8.3 with 32; of 4,600 atoms 19.3,
//   13.3 and 10.0; 24 replicas of 300 atoms 7.3, 6.4 and 5.8 with 2, 4 and 8; with no fewer than 64,
//   32 and 16 atoms to a group, two replicas of 161 atoms 6.7, 5.7, 5.7 and of 1,000 8.3, 7.8, 7.6);
//   threads of k_persist_small: a wave per unit of a step's work, fewer where the replicas outnumber
//   the compute units, so that they run side by side (16 waves fit on one at its register count;
//   1,024 replicas of 22 atoms: 3.6 us per step with 4 waves each, 4.3 with 2, 4.9 with 7).
struct RunShape {
    int bt;
    const Split *sp;
    bool small;                // k_persist_small, else k_persist
    bool noise_ahead;          // k_persist: the next step's Gaussians in LDS
    size_t lds;
};
static RunShape shape_on(const gpr_system *S, int bt, const Split *sp)
{
    RunShape sh{bt, sp, false, false, 0};
    // (one group draws them beside its pair tasks, which the toy system has none of)
    sh.noise_ahead = S->kind != GPR_KIND_TOY2D && noise_fits(S->n, S->np, *sp, bt, S->maxlds_persist);
    sh.lds = sh.noise_ahead ? (size_t)persist_off(S->n, S->np, sp->lmax).end : persist_lds(S->n, S->np, *sp);
    return sh;
}
static bool chosen(const gpr_system *S, int from, int nrep) { return from == 2 || (from == 1 && nrep == S->R); }
static RunShape run_shape(const gpr_system *S, int nrep)
{
    const int cus = std::max(1, S->max_coresident);
    RunShape sh{S->bt_persist, &S->split, false, false, 0};
    if (S->small_ok && S->groups == 1) {
        sh.small = true;
        if (!chosen(S, S->bt_from, nrep)) {
            const int waves = std::min(16, std::max(small_units(S), S->nobs));
            sh.bt = 64 * std::max(1, std::min(waves, 16 / ((nrep + cus - 1) / cus)));
        }
        sh.lds = small_lds(S);
        return sh;
    }
    if (!chosen(S, S->groups_from, nrep))
        for (int k = 1; k < NSPLIT; ++k) {
            const int G = 1 << k;
            if (G > sh.sp->G && S->split_ok[k] && S->n >= 32 * G && (long)nrep * G <= cus) sh.sp = &S->splits[k];
        }
    return shape_on(S, sh.bt, sh.sp);
}

// ------------------------------------------------------------------ bonded units
// The terms touching each of the atom ranges [bnd[k], bnd[k + 1]) in units of 64 terms of one kind
// (the records of gpr_device.h): first the terms inside the range, the longest kinds first, then
// those that reach outside it; a term's energy counts in the range that holds its smallest atom.
// term[kind]: the terms' atoms (-1: none) in the sorted order.  The records go to the ends of bi and
// src; returns the first unit of each range, counted from there, and the end.
static std::vector<int> write_units(const std::vector<int4> *term, int n, const int *bnd, int nr, std::vector<uint2> &bi, std::vector<int> &src)
{
    std::vector<unsigned char> range(n);
    for (int r = 0; r < nr; ++r) std::fill(range.begin() + bnd[r], range.begin() + bnd[r + 1], (unsigned char)r);
    // terms of (range, kind, inside or edge)
    std::vector<std::vector<int>> in((size_t)nr * 10);
    for (int k = 0; k < 5; ++k)
        for (int t = 0; t < (int)term[k].size(); ++t) {
            const int4 q = term[k][t];
            const int at[4] = {q.x, q.y, q.z, q.w};
            int rg[4], m = 0;
            for (int a : at) {
                if (a < 0) continue;
                const int r = range[a];
                if (std::find(rg, rg + m, r) == rg + m) rg[m++] = r;
            }
            for (int j = 0; j < m; ++j) in[(size_t)rg[j] * 10 + k + (m > 1 ? BONDED_EDGE : 0)].push_back(t);
        }
    std::vector<int> first(1, 0);
    const size_t base = src.size();
    for (int r = 0; r < nr; ++r) {
        for (int kk : {2, 7, 1, 6, 4, 9, 0, 5, 3, 8}) {
            const std::vector<int> &l = in[(size_t)r * 10 + kk];
            const int k = kk % 5;
            const size_t cnt = (l.size() + 63) / 64 * 64;
            for (size_t c = 0; c < cnt; ++c) {
                const unsigned kind0 = (unsigned)(kk & 3) << 14, kind1 = (unsigned)(kk >> 2) << 14;
                unsigned f[4] = {kind0, kind1, 0u, 0u};
                if (c < l.size()) {
                    const int4 q = term[k][l[c]];
                    const int at[4] = {q.x, q.y, q.z, q.w};
                    int mn = q.x;
                    for (int j = 0; j < 4; ++j) {
                        if (at[j] < 0) continue;
                        mn = std::min(mn, at[j]);
                        f[j] |= (unsigned)at[j] | (at[j] >= bnd[r] && at[j] < bnd[r + 1] ? (unsigned)BONDED_ATOMS : 0u);
                    }
                    f[2] |= (mn >= bnd[r] && mn < bnd[r + 1] ? 0x4000u : 0u) | 0x8000u;
                }
                bi.push_back(make_uint2(f[0] | (f[1] << 16), f[2] | (f[3] << 16)));
                src.push_back(c < l.size() ? 5 * l[c] + k : -1);
            }
        }
        first.push_back((int)((src.size() - base) / 64));
    }
    return first;
}

// The records' parameters, from the terms' current ones
static hipError_t write_unit_params(gpr_system *S)
{
    if (S->n_records == 0) return hipSuccess;
    hipLaunchKernelGGL(k_unit_params, dim3((S->n_records + 255) / 256), dim3(256), 0, S->stream, S->d.tp, S->unit_src, S->n_records, S->unit_bp);
    return hipGetLastError();
}

// The units of the plain path's blocks of 256 atoms and of every split that a launch may take (the
// caller's 1 to 8 workgroups per replica, more where run_shape takes them), in one allocation, so
// that no launch lays out any.
static gpr_status lay_units(gpr_system *S, const std::vector<int4> *term)
{
    const int n = S->n;
    std::vector<uint2> bi;
    std::vector<int> src, bnd, at(NSPLIT, -1);
    for (int a = 0; a < n; a += 256) bnd.push_back(a);
    bnd.push_back(n);
    const std::vector<int> plain = write_units(term, n, bnd.data(), (int)bnd.size() - 1, bi, src);
    for (int k = 0; k < NSPLIT; ++k) {
        Split &sp = S->splits[k];
        if (sp.G < 1 << k) {                                // (fewer groups: the units of that split)
            sp = S->splits[split_index(sp.G)];
            at[k] = at[split_index(sp.G)];
            continue;
        }
        if (!S->persist_ok || !S->split_ok[k] || (k > 3 && n < 32 << k)) continue;
        at[k] = (int)src.size();
        const std::vector<int> first = write_units(term, n, sp.bnd, sp.G, bi, src);
        std::copy(first.begin(), first.end(), sp.bu);
    }
    HIPCHK(S, upload(S, &S->unit_bi, bi));
    HIPCHK(S, upload(S, &S->unit_src, src));
    HIPCHK(S, dalloc(S, &S->unit_bp, src.size()));
    S->n_records = (int)src.size();
    HIPCHK(S, write_unit_params(S));
    for (int k = 0; k < NSPLIT; ++k)
        if (at[k] >= 0) { S->splits[k].bi = S->unit_bi + at[k]; S->splits[k].bp = S->unit_bp + at[k]; }
    S->d.pl_bi = S->unit_bi;
    S->d.pl_bp = S->unit_bp;
    HIPCHK(S, upload(S, (int **)&S->d.pl_first, plain));
    return GPR_OK;
}

// ------------------------------------------------------------------ force-field parameters
// Device copies of the per-atom parameters (sigma/2, 2 sqrt(eps), q sqrt(f), 1/m), the torsion
// parameters (k, cos phi0, sin phi0, n) and the 1-4 pair parameters (sigma_ij, 4 eps_ij s14,
// f q_i q_j s14) in the sorted term order, and 1/(2 eps_i), from the host copies.
static hipError_t write_params(gpr_system *S)
{
    const int n = S->n, np = S->np;
    Dev &d = S->d;
    const bool mol = S->kind == GPR_KIND_MOLECULAR;
    std::vector<float4> prm(np, make_float4(0, 0, 0, 0));
    std::vector<double> inv2eps(n, 0.0);
    for (int i = 0; i < n; ++i) {
        const double sig = mol ? S->sig_h[i] : 0.0, eps = mol ? S->eps_h[i] : 0.0, q = mol ? S->q_h[i] : 0.0;
        prm[i] = make_float4((float)(0.5 * sig), (float)(2.0 * std::sqrt(eps)), (float)(q * std::sqrt(COULOMB_F)),
                             (float)(1.0 / S->mass_h[i]));
        inv2eps[i] = eps > 0 ? 0.5 / eps : INFINITY;
    }
    hipError_t e = hipMemcpyAsync((void *)d.prm, prm.data(), sizeof(float4) * np, hipMemcpyHostToDevice, S->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync((void *)d.inv2eps, inv2eps.data(), sizeof(double) * n, hipMemcpyHostToDevice, S->stream);
    const Topo &T = d.tp;
    if (e == hipSuccess && mol && T.nt) {
        std::vector<float4> p(T.nt);
        for (int k = 0; k < T.nt; ++k) {
            const int t = S->tor_order[k];
            p[k] = make_float4((float)S->tor_k_h[t], (float)std::cos(S->tor_phi0_h[t]), (float)std::sin(S->tor_phi0_h[t]),
                               (float)S->tor_n_h[t]);
        }
        e = hipMemcpyAsync((void *)T.t_p, p.data(), sizeof(float4) * T.nt, hipMemcpyHostToDevice, S->stream);
    }
    if (e == hipSuccess && mol && T.n14) {
        std::vector<float4> p(T.n14);
        for (int k = 0; k < T.n14; ++k) {
            const int2 ij = S->p14_h[S->p14_order[k]];
            const double sij = 0.5 * (S->sig_h[ij.x] + S->sig_h[ij.y]);
            const double eij = std::sqrt(S->eps_h[ij.x] * S->eps_h[ij.y]);
            p[k] = make_float4((float)sij, (float)(4.0 * eij * S->scale14),
                               (float)(COULOMB_F * S->q_h[ij.x] * S->q_h[ij.y] * S->scale14), 0.f);
        }
        e = hipMemcpyAsync((void *)T.p_p, p.data(), sizeof(float4) * T.n14, hipMemcpyHostToDevice, S->stream);
    }
    if (e == hipSuccess) e = write_unit_params(S);
    if (e == hipSuccess) e = hipStreamSynchronize(S->stream);
    return e;
}

// ------------------------------------------------------------------ launches
// threads of k_obs: its time is the staging of the replica (5,200 atoms: 52 us with 256 threads, 28
// with 1,024), but many small replicas share compute units
static dim3 obs_block(const gpr_system *S) { return dim3(S->n > 1024 ? 1024 : 256); }

// forces of replicas [r_off, r_off + nrep) at their current positions.  Stepping calls
// (force_build = 0) rely on k_integrate to clear the energies and maintain the list guard;
// force-only calls (force_build = 1) rebuild the lists and clear the energies here.
static gpr_status launch_forces(gpr_system *S, int r_off, int nrep, long long s, int energy, int apply_b, int force_build,
                                bool timed = false, bool clear_e = true)
{
    const int BTN = 1024;
    if (force_build) s = S->s - 1;             // a forced build counts as built in the previous step
    if (energy && force_build && clear_e) {
        HIPCHK(S, hipMemsetAsync(S->d.E + r_off, 0, sizeof(long long) * nrep, S->stream));
    }
    dim3 gn((S->n * P + BTN - 1) / BTN, nrep);
    if (timed) HIPCHK(S, prof_begin(S));
    hipLaunchKernelGGL(k_forces, gn, dim3(BTN), S->lds_nb, S->stream, S->d_dev, s, r_off, energy, apply_b,
                       force_build);
    LAUNCHCHK(S);
    if (timed) HIPCHK(S, prof_end(S));
    if (force_build && r_off == 0 && nrep == S->R) S->lists_old = false;
    return GPR_OK;
}

// Workgroups of the persistent kernel that the device holds at once for (bt, lds): the
// occupancy query, kept per system and launch shape.
static gpr_status persist_capacity(gpr_system *S, int bt, size_t lds, int &cap)
{
    for (const auto &c : S->caps)
        if (c.bt == bt && c.lds == lds) { cap = c.blocks; return GPR_OK; }
    int dev = 0, cus = 0, per_cu = 0;
    HIPCHK(S, hipGetDevice(&dev));
    HIPCHK(S, hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    HIPCHK(S, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k_persist, bt, lds));
    S->caps.push_back({bt, lds, per_cu * cus});
    cap = per_cu * cus;
    return GPR_OK;
}

// Workgroup sets of one system in a persistent launch.  With G > 1 workgroups per replica the
// groups of a replica wait for each other, so they must be resident together: the replicas are
// shared by at most capacity / G sets (cap_blocks < 0: the whole device), so that the grid is
// no larger than what the device holds at once, and every workgroup gets a CU as soon as the
// device is free of other work.  (Other kernels hold the CUs it needs only until they end, and
// launches that wait for workgroups of their own take room first, see admit, and places as they
// start, see start_place; should a group still wait longer than the bounded spin, the call reports
// GPR_EDEVICE, never hangs.)  No cooperative launch: it adds tens of microseconds to each launch
// and is refused while another process holds the device's cooperative resources.
static gpr_status persist_item(gpr_system *S, const Split &sp, int nrep, int bt, size_t lds, int cap_blocks,
                               PersistItem &it, int &nblocks)
{
    const int G = sp.G;
    it = PersistItem{};
    it.dev = S->d_dev;
    it.sp = sp;
    if (!sp.bi) return fail(S, GPR_EDEVICE, "no bonded units for this split");
    it.nrep = nrep;
    it.boff = 0;
    if (G == 1 && cap_blocks < 0) {
        it.nsets = nrep;
        it.xcd = 0;
        nblocks = nrep;
        return GPR_OK;
    }
    if (cap_blocks < 0) {
        const gpr_status rc = persist_capacity(S, bt, lds, cap_blocks);
        if (rc) return rc;
    }
    int nsets = std::min(nrep, cap_blocks / G);
    if (nsets < 1) return fail(S, GPR_EINVAL, "a replica's workgroups do not fit on the device at once");
    // a multiple of eight sets, for their placement: more (the rest idle) where they fit, else fewer
    // where that adds no round (a second round of launches doubles the time: 12 replicas of 1,200
    // atoms used to run as 8 and then 4)
    it.xcd = 0;
    if (G > 1 && nsets >= 8) {
        const int up = (nsets + 7) / 8 * 8, down = nsets / 8 * 8;
        auto rounds = [&](int sets) { return (nrep + sets - 1) / sets; };
        if (up * G <= cap_blocks) { nsets = up; it.xcd = 1; }
        else if (rounds(down) == rounds(nsets)) { nsets = down; it.xcd = 1; }
    }
    it.nsets = nsets;
    nblocks = nsets * G;
    return GPR_OK;
}

// The room that launches held is free again: the stream has been waited for.
static void give_back(gpr_system *S)
{
    if (S->held) g_room[S->dev].give(S->held_by);
    S->held = 0;
}
static hipError_t finish(gpr_system *S)
{
    const hipError_t e = hipStreamSynchronize(S->stream);
    give_back(S);
    return e;
}
struct FinishAtEnd {                   // of a call, where it ends without having waited
    gpr_system *S;
    ~FinishAtEnd() { if (S->held) (void)finish(S); }
};
static Room::Key room_key(const gpr_system *S)
{
    return {S->stream, S->stream == hipStreamPerThread ? std::this_thread::get_id() : std::thread::id()};
}
static int room_cap(const gpr_system *S) { return std::max(8, S->max_coresident / 8 * 8); }
// Workgroups go to the eight XCDs in turn, so what counts is a launch's share of each.
static int room_units(int nblocks) { return (nblocks + 7) / 8 * 8; }
static bool hold(gpr_system *S, int units, bool wait)
{
    if (S->held >= units) return true;                     // of this call's earlier launches on the stream
    if (S->held) (void)finish(S);
    const Room::Key key = room_key(S);
    if (wait) g_room[S->dev].take(key, units, room_cap(S));
    else if (!g_room[S->dev].try_take(key, units, room_cap(S))) return false;
    S->held = units;
    S->held_by = key;
    return true;
}

// The shape and item of a launch that there is room for beside the launches of other streams that
// wait for their own workgroups too.  While others have room or wait for it, a launch takes no more
// workgroups per replica than one of all replicas does; where that has no room, fewer, down to one,
// which needs none; and it waits for room only where one does not fit or the caller chose the shape.
static gpr_status admit(gpr_system *S, int nrep, RunShape &sh, PersistItem &it, int &nblocks)
{
    const bool fixed = chosen(S, S->groups_from, nrep);
    if (sh.sp->G > S->split.G && S->held == 0 && g_room[S->dev].others(room_key(S))) sh = shape_on(S, sh.bt, &S->split);
    for (;;) {
        const gpr_status rc = persist_item(S, *sh.sp, nrep, sh.bt, sh.lds, -1, it, nblocks);
        if (rc) return rc;
        if (sh.sp->G == 1 || hold(S, room_units(nblocks), fixed)) return GPR_OK;
        int k = split_index(sh.sp->G) - 1;
        while (k >= 0 && !S->split_ok[k]) --k;
        if (k < 0) break;
        sh = shape_on(S, sh.bt, &S->splits[k]);
    }
    sh = shape_on(S, sh.bt, &S->split);
    const gpr_status rc = persist_item(S, *sh.sp, nrep, sh.bt, sh.lds, -1, it, nblocks);
    if (rc) return rc;
    (void)hold(S, room_units(nblocks), true);
    return GPR_OK;
}

// The layout of a persistent launch checked on the host before it runs, with the device's own
// placement function: items cover the grid in order without overlap, every workgroup is group
// g < G of a set < nsets, every (set, g) occurs once, the groups' atom ranges are ordered, not empty
// (the position exchange relies on it), within the system and no longer than the LDS arrays (lmax),
// and the block size is whole waves.
static gpr_status check_layout(gpr_system *S, const PersistBatch &pb, int nblocks, int bt, bool single)
{
    if (pb.nitems < 1 || pb.nitems > MAX_BATCH || bt < 64 || bt > 1024 || bt % 64) return fail(S, GPR_EDEVICE, "bad persistent launch shape");
    int next = 0;
    for (int k = 0; k < pb.nitems; ++k) {
        const PersistItem &it = pb.it[k];
        const Split &sp = it.sp;
        if (it.boff != next || it.nsets < 1 || it.nrep < 1 || sp.G < 1 || sp.G > MAX_G || !it.dev)
            return fail(S, GPR_EDEVICE, "persistent launch layout: item placement");
        if (!single && k > 0 && pb.it[k - 1].boff >= it.boff) return fail(S, GPR_EDEVICE, "persistent launch layout: item order");
        const int n = sp.bnd[sp.G];
        if (sp.bnd[0] != 0) return fail(S, GPR_EDEVICE, "persistent launch layout: atom ranges");
        for (int g = 0; g < sp.G; ++g)
            if (sp.bnd[g] >= sp.bnd[g + 1] || sp.bnd[g + 1] > n || sp.bnd[g + 1] - sp.bnd[g] > sp.lmax)
                return fail(S, GPR_EDEVICE, "persistent launch layout: atom ranges");
        std::vector<unsigned char> seen((size_t)it.nsets * sp.G, 0);
        for (int local = 0; local < it.nsets * sp.G; ++local) {
            int set = -1, g = -1;
            if (!persist_place(it, local, set, g) || set < 0 || set >= it.nsets || g < 0 || g >= sp.G ||
                seen[(size_t)set * sp.G + g]++)
                return fail(S, GPR_EDEVICE, "persistent launch layout: workgroup placement");
        }
        next = it.boff + it.nsets * sp.G;
        // the workgroups of mapped items come first, in whole rows of eight
        if (!single && it.xcd && (next > pb.mapped || next % 8)) return fail(S, GPR_EDEVICE, "persistent launch layout: mapped items");
        if (!single && !it.xcd && it.boff < pb.mapped) return fail(S, GPR_EDEVICE, "persistent launch layout: mapped items");
    }
    if (single && pb.it[0].xcd && nblocks % 8) return fail(S, GPR_EDEVICE, "persistent launch layout: mapped items");
    if (next != nblocks) return fail(S, GPR_EDEVICE, "persistent launch layout: grid size");
    return GPR_OK;
}

// One item whose sets each take one replica (roff + set) runs k_persist, or k_persist_small when
// its shape `one` says so; anything else
// (several systems, or sets that take replicas in turn) runs k_persist_batch.
static gpr_status launch_persist(gpr_system *S, PersistBatch &pb, int nblocks, int bt, size_t lds,
                                 hipStream_t stream, const RunShape *one = nullptr)
{
    const bool single = pb.nitems == 1 && (one || pb.it[0].nsets >= pb.it[0].nrep);
    {
        const gpr_status rc = check_layout(S, pb, nblocks, bt, single);
        if (rc) return rc;
    }
    const void *fn = !single ? (const void *)k_persist_batch
                             : one && one->small ? (const void *)k_persist_small : (const void *)k_persist;
    void *args_single[] = {(void *)&pb.it[0]};
    void *args_batch[] = {(void *)&pb};
    void **args = single ? args_single : args_batch;
    HIPCHK(S, hipLaunchKernel(fn, dim3(nblocks), dim3(bt), args, lds, stream));
    return GPR_OK;
}

// Step k of a captured cycle on the device clock (code DCLK_*): the kernels read the cycle's
// first step and local step from the device, so every replay continues where the last one
// stopped.  The observables of the workers: with phase >= 0 (the local step at the cycle's
// start, mod t_GR) at the steps that sample; with phase < 0 a launch every step that returns
// unless the step samples.
static gpr_status launch_step_dc(gpr_system *S, int nrep, int code, int phase, int k, hipStream_t st)
{
    const int BTI = 256, BTN = 1024;
    hipLaunchKernelGGL(k_integrate, dim3((S->n + BTI - 1) / BTI, nrep), dim3(BTI), 0, st, S->d_dev, (long long)k, 0, code);
    LAUNCHCHK(S);
    hipLaunchKernelGGL(k_forces, dim3((S->n * P + BTN - 1) / BTN, nrep), dim3(BTN), S->lds_nb, st, S->d_dev,
                       (long long)k, 0, code, 1, 0);
    LAUNCHCHK(S);
    if (code == DCLK_SAMPLE && nrep > 1) {
        if (phase < 0) {
            hipLaunchKernelGGL(k_obs, dim3(nrep - 1), obs_block(S), S->lds_stage, st, S->d_dev, 1, 3, nullptr, k);
            LAUNCHCHK(S);
        } else if ((phase + k + 1) % S->t_gr == 0) {
            hipLaunchKernelGGL(k_obs, dim3(nrep - 1), obs_block(S), S->lds_stage, st, S->d_dev, 1, 0, nullptr, 0);
            LAUNCHCHK(S);
        }
    }
    return GPR_OK;
}

// The executable graph of graph_cycle device-clocked steps and the clock advance for
// (nrep, code, phase), captured on a stream of its own the first time it is needed.
static gpr_status plain_graph(gpr_system *S, int nrep, int code, int phase, hipGraphExec_t *out)
{
    for (auto &g : S->graphs)
        if (g.nrep == nrep && g.code == code && g.phase == phase) { *out = g.exec; return GPR_OK; }
    hipStream_t cs = nullptr;
    HIPCHK(S, hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    gpr_status rc = GPR_OK;
    for (int k = 0; k < S->graph_cycle && e == hipSuccess && rc == GPR_OK; ++k)
        rc = launch_step_dc(S, nrep, code, phase, k, cs);
    if (e == hipSuccess && rc == GPR_OK) {
        hipLaunchKernelGGL(k_tick, dim3(1), dim3(1), 0, cs, S->d_dev, (long long)S->graph_cycle);
        e = hipGetLastError();
    }
    hipGraph_t g = nullptr;
    const hipError_t e2 = hipStreamEndCapture(cs, &g);
    hipGraphExec_t ex = nullptr;
    hipError_t e3 = hipSuccess;
    if (e == hipSuccess && e2 == hipSuccess && rc == GPR_OK) e3 = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
    if (g) (void)hipGraphDestroy(g);
    (void)hipStreamDestroy(cs);
    if (rc) return rc;
    if (e != hipSuccess || e2 != hipSuccess || e3 != hipSuccess)
        return fail(S, GPR_EDEVICE, std::string("graph capture: ") + hipGetErrorString(e != hipSuccess ? e : e2 != hipSuccess ? e2 : e3));
    S->graphs.push_back({nrep, code, phase, ex});
    *out = ex;
    return GPR_OK;
}

// nsteps plain steps launched from the host, local steps counted from t0
static gpr_status plain_steps(gpr_system *S, int nrep, long long nsteps, long long t0, bool sample)
{
    const int BTI = 256;
    dim3 gi((S->n + BTI - 1) / BTI, nrep);
    for (long long k = 0; k < nsteps; ++k) {
        const long long tl = t0 + k + 1;
        const bool samp = sample && nrep > 1 && (tl % S->t_gr == 0);
        const int energy = (samp && S->d.need_energy) ? 1 : 0;
        hipLaunchKernelGGL(k_integrate, gi, dim3(BTI), 0, S->stream, S->d_dev, S->s, 0, energy);
        LAUNCHCHK(S);
        gpr_status rc = launch_forces(S, 0, nrep, S->s, energy, 1, 0, true);
        if (rc) return rc;
        S->s += 1;
        if (samp) {
            hipLaunchKernelGGL(k_obs, dim3(nrep - 1), obs_block(S), S->lds_stage, S->stream, S->d_dev, 1, 0, nullptr, 0);
            LAUNCHCHK(S);
        }
    }
    return GPR_OK;
}

// advances replicas [0, nrep) by nsteps from local step counter t0; sample: accumulate the
// observables of workers every t_gr; state_end: state ids at the end
static gpr_status run_steps(gpr_system *S, int nrep, long long nsteps, long long t0, bool sample, bool state_end)
{
    if (nsteps <= 0) {
        if (state_end) {
            hipLaunchKernelGGL(k_state, dim3(nrep), dim3(256), S->lds_stage, S->stream, S->d_dev, 0);
            LAUNCHCHK(S);
        }
        return GPR_OK;
    }
    if (S->path == GPR_PATH_PERSISTENT) {
        PersistBatch pb{};
        pb.nitems = 1;
        int nblocks = 0;
        RunShape sh = run_shape(S, nrep);
        gpr_status rc = admit(S, nrep, sh, pb.it[0], nblocks);
        if (rc) return rc;
        pb.it[0].noise_ahead = sh.noise_ahead ? 1 : 0;
        // more replicas than sets that fit at once: rounds of launches, each set taking one
        // replica per launch (replicas are independent between checks)
        const int rounds = (nrep + pb.it[0].nsets - 1) / pb.it[0].nsets;
        long long done = 0;
        while (done < nsteps) {
            const int chunk = (int)std::min<long long>(nsteps - done, 1 << 20);
            const bool last = done + chunk == nsteps;
            PersistItem &it = pb.it[0];
            it.s0 = S->s + done;
            it.nsteps = chunk;
            it.t0 = (int)((t0 + done) % S->t_gr);        // the device uses it modulo t_GR only
            it.sample = sample ? 1 : 0;
            it.state_end = (state_end && last) ? 1 : 0;
            for (int k = 0; k < rounds; ++k) {
                it.roff = k * it.nsets;
                HIPCHK(S, prof_begin(S));
                rc = launch_persist(S, pb, nblocks, sh.bt, sh.lds, S->stream, &sh);
                if (rc) return rc;
                HIPCHK(S, prof_end(S));
            }
            done += chunk;
        }
        S->s += nsteps;
        if (sh.small) S->lists_old = true;
        return GPR_OK;
    }
    // whole cycles replayed from a captured graph, the steps left over launched from the host
    long long left = nsteps, tcur = t0;
    if (S->graph_cycle > 0 && left >= S->graph_cycle) {
        const int code = (sample && nrep > 1) ? DCLK_SAMPLE : DCLK_NOSAMPLE;
        const int phase = (code == DCLK_SAMPLE && S->graph_cycle % S->t_gr == 0) ? (int)(t0 % S->t_gr) : -1;
        hipGraphExec_t ex = nullptr;
        gpr_status rc = plain_graph(S, nrep, code, phase, &ex);
        if (rc) return rc;
        hipLaunchKernelGGL(k_set_clock, dim3(1), dim3(1), 0, S->stream, S->d_dev, S->s, t0);
        LAUNCHCHK(S);
        for (; left >= S->graph_cycle; left -= S->graph_cycle) {
            HIPCHK(S, hipGraphLaunch(ex, S->stream));
            S->s += S->graph_cycle;
            tcur += S->graph_cycle;
        }
    }
    gpr_status rc = plain_steps(S, nrep, left, tcur, sample);
    if (rc) return rc;
    if (state_end) {
        hipLaunchKernelGGL(k_state, dim3(nrep), dim3(256), S->lds_stage, S->stream, S->d_dev, 0);
        LAUNCHCHK(S);
    }
    return GPR_OK;
}

// the error flags of a check's status, or read back
static gpr_status flag_errors(gpr_system *S, const int *err)
{
    if (err[ERR_UNSTABLE]) return fail(S, GPR_EUNSTABLE, "non-finite or overflowing state");
    if (err[ERR_LIST]) return fail(S, GPR_EDEVICE, "pair-list capacity exceeded");
    if (err[ERR_BARRIER]) return fail(S, GPR_EDEVICE, "persistent-kernel barrier timed out");
    return GPR_OK;
}

// Up to three pieces of device memory (multiples of four bytes) into the read-back buffer, one after
// the other, at most rb_bytes; there once the stream has been waited for.
struct Piece {
    const void *src;
    size_t bytes;
};
static gpr_status read_pieces(gpr_system *S, std::initializer_list<Piece> pieces)
{
    ReadList l{};
    size_t words = 0;
    int k = 0;
    for (const Piece &p : pieces) {
        l.src[k] = (const uint32_t *)p.src;
        l.words[k++] = (unsigned)(p.bytes / 4);
        words += p.bytes / 4;
    }
    if (words * 4 > S->rb_bytes) return fail(S, GPR_EDEVICE, "read-back buffer too small");
    const unsigned blocks = (unsigned)std::min<size_t>(256, (words + 255) / 256);
    hipLaunchKernelGGL(k_read, dim3(std::max(1u, blocks)), dim3(256), 0, S->stream, l, (uint32_t *)S->rb);
    LAUNCHCHK(S);
    return GPR_OK;
}

// one launch: bookkeeping by block (0, 0), and with CHK_DEPHASE the clone-on-kill copies by
// the blocks of each killed worker's row
// (CHK_ADVANCE: fresh at the first check of a call; wait false: the caller waits and looks for errors)
static gpr_status check(gpr_system *S, int mode, int nrep, long long check_index, bool fresh = false, bool wait = true)
{
    const dim3 grid = mode == CHK_DEPHASE ? dim3((3 * S->np + 255) / 256, nrep) : dim3(1, 1);
    hipLaunchKernelGGL(k_check, grid, dim3(256), sizeof(int) * nrep, S->stream, S->d_dev, mode, S->s, S->omega, nrep,
                       S->nsamp, check_index, (long long)S->tcp, S->st_host, S->donor, S->surv, S->fec, fresh ? 1 : 0,
                       mode == CHK_ADVANCE ? S->adv_fec : (long long *)nullptr, (CycRec *)nullptr, 0);
    LAUNCHCHK(S);
    if (mode == CHK_DEPHASE) S->lists_old = true;          // (a killed worker has its donor's positions)
    if (!wait) return GPR_OK;
    HIPCHK(S, finish(S));
    HIPCHK(S, prof_collect(S));
    return flag_errors(S, S->st_host->err);
}

static gpr_status copy_replica(gpr_system *S, int dst, int src)
{
    std::vector<int> dn(S->R, -1);
    dn[dst] = src;
    HIPCHK(S, hipMemcpyAsync(S->donor, dn.data(), sizeof(int) * S->R, hipMemcpyHostToDevice, S->stream));
    hipLaunchKernelGGL(k_clone, dim3((3 * S->np + 255) / 256, S->R), dim3(256), 0, S->stream, S->d_dev, S->donor, 0);
    LAUNCHCHK(S);
    S->lists_old = true;
    return GPR_OK;
}

static gpr_status broadcast_reference(gpr_system *S)
{
    std::vector<int> dn(S->R, 0);
    dn[0] = -1;
    HIPCHK(S, hipMemcpyAsync(S->donor, dn.data(), sizeof(int) * S->R, hipMemcpyHostToDevice, S->stream));
    hipLaunchKernelGGL(k_clone, dim3((3 * S->np + 255) / 256, S->R), dim3(256), 0, S->stream, S->d_dev, S->donor, 1);
    LAUNCHCHK(S);
    S->lists_old = true;
    return GPR_OK;
}

static gpr_status state_of_ref(gpr_system *S, int *out)
{
    gpr_status rc = run_steps(S, 1, 0, 0, false, true);
    if (rc) return rc;
    rc = check(S, CHK_STATE, 1, 0);
    if (rc) return rc;
    *out = S->st_host->to_state;
    return GPR_OK;
}

// ------------------------------------------------------------------ create / destroy
extern "C" void gpr_system_destroy(gpr_system *S)
{
    if (!S) return;
    if (S->stream) (void)hipStreamSynchronize(S->stream);
    for (auto &g : S->graphs) (void)hipGraphExecDestroy(g.exec);
    for (auto &g : S->cgraphs) (void)hipGraphExecDestroy(g.exec);
    if (S->cyc_dev) (void)hipFree(S->cyc_dev);
    if (S->stc_dev) (void)hipFree(S->stc_dev);
    if (S->cyc_host) (void)hipHostFree(S->cyc_host);
    if (S->stc_host) (void)hipHostFree(S->stc_host);
    for (void *p : S->bufs) (void)hipFree(p);
    for (hipEvent_t e : S->ev_a) (void)hipEventDestroy(e);
    for (hipEvent_t e : S->ev_b) (void)hipEventDestroy(e);
    if (S->st_host) (void)hipHostFree(S->st_host);
    delete S;
}

extern "C" const char *gpr_last_error(const gpr_system *S)
{
    return S ? S->err.c_str() : g_thread_err.c_str();
}


static gpr_status create_impl(const gpr_system_desc *D, gpr_system *S)
{
    const int n = D->n_atoms, R = D->n_replicas;
    S->n = n; S->R = R; S->kind = D->kind;
    S->np = (n + 1 + 63) / 64 * 64;   // room for the dummy atom n
    const int np = S->np;
    S->t_gr = D->t_gr; S->tcd = D->t_check_dephase; S->tcp = D->t_check_parallel;
    S->tol = D->tol; S->dt = D->dt; S->t_min = D->t_min; S->kT = D->kT;
    S->nobs = D->n_obs;
    Dev &d = S->d;
    d.kind = D->kind; d.n = n; d.np = np; d.R = R;

    // per-atom parameters
    const double c1 = std::exp(-D->gamma * D->dt);
    const double c2 = std::sqrt(std::max(0.0, 1.0 - c1 * c1));
    std::vector<float4> prm(np, make_float4(0, 0, 0, 0));
    std::vector<float> sd(np, 0.f), mass(np, 0.f);
    for (int i = 0; i < n; ++i) {
        const double sig = D->kind == GPR_KIND_MOLECULAR ? D->sigma[i] : 0.0;
        const double eps = D->kind == GPR_KIND_MOLECULAR ? D->epsilon[i] : 0.0;
        const double q = D->kind == GPR_KIND_MOLECULAR ? D->charge[i] : 0.0;
        prm[i] = make_float4((float)(0.5 * sig), (float)(2.0 * std::sqrt(eps)), (float)(q * std::sqrt(COULOMB_F)),
                             (float)(1.0 / D->mass[i]));
        sd[i] = (float)(c2 * std::sqrt(D->kT / D->mass[i]));
        mass[i] = (float)D->mass[i];
    }
    HIPCHK(S, upload(S, (float4 **)&d.prm, prm));
    HIPCHK(S, upload(S, (float **)&d.sd, sd));
    HIPCHK(S, upload(S, (float **)&d.mass, mass));

    // exclusions (and 1-4 pairs) as bit masks over index offsets -32..31, and those farther
    // apart as an ascending partner list per atom
    std::vector<unsigned long long> excl(np, 0ull);
    std::vector<std::vector<int>> far(n);
    auto mark = [&](int i, int j) {
        const int off = j - i;
        if (off == 0) return;
        if (off > -32 && off < 32) {
            excl[i] |= 1ull << (off + 32);
            excl[j] |= 1ull << (-off + 32);
        } else {
            far[i].push_back(j);
            far[j].push_back(i);
        }
    };
    if (D->kind == GPR_KIND_MOLECULAR) {
        for (int e = 0; e < D->n_exclusions; ++e) mark(D->exclusion_atoms[2 * e], D->exclusion_atoms[2 * e + 1]);
        for (int p = 0; p < D->n_pairs14; ++p) mark(D->pair14_atoms[2 * p], D->pair14_atoms[2 * p + 1]);
    }
    std::vector<int> far_start(n + 1, 0), far_j;
    for (int i = 0; i < n; ++i) {
        std::sort(far[i].begin(), far[i].end());
        far[i].erase(std::unique(far[i].begin(), far[i].end()), far[i].end());
        far_start[i + 1] = far_start[i] + (int)far[i].size();
        far_j.insert(far_j.end(), far[i].begin(), far[i].end());
    }
    d.has_far = far_j.empty() ? 0 : 1;
    d.excl_span = 0;
    for (int i = 0; i < n; ++i)
        for (int b = 0; b < 64; ++b)
            if ((excl[i] >> b) & 1ull) d.excl_span = std::max(d.excl_span, std::abs(b - 32));
    HIPCHK(S, upload(S, (unsigned long long **)&d.excl, excl));
    HIPCHK(S, upload(S, (int **)&d.far_start, far_start));
    HIPCHK(S, upload(S, (int **)&d.far_j, far_j));

    // replica state: every replica starts from (pos, vel)
    const size_t rs = (size_t)R * 3 * np;
    std::vector<float> x0(3 * np, 0.f), v0(3 * np, 0.f);
    for (int c = 0; c < 3; ++c)
        for (int i = 0; i < n; ++i) {
            x0[c * np + i] = (float)D->pos[c * n + i];
            if (D->vel) v0[c * np + i] = (float)D->vel[c * n + i];
        }
    if (D->kind == GPR_KIND_TOY2D) { x0[2 * np] = 0.f; v0[2 * np] = 0.f; }
    HIPCHK(S, dalloc(S, &d.x, rs));
    HIPCHK(S, dalloc(S, &d.v, rs));
    HIPCHK(S, dalloc(S, &d.xb, rs));
    HIPCHK(S, dalloc(S, &d.F, rs));
    HIPCHK(S, dalloc(S, &d.E, R));
    HIPCHK(S, hipMemcpy(d.x, x0.data(), sizeof(float) * 3 * np, hipMemcpyHostToDevice));
    HIPCHK(S, hipMemcpy(d.v, v0.data(), sizeof(float) * 3 * np, hipMemcpyHostToDevice));

    // bonded topology, each type sorted by smallest atom
    Topo &T = d.tp;
    std::vector<int> order;
    std::vector<int4> term[5];         // by kind, as in the bonded units
    if (D->kind == GPR_KIND_MOLECULAR) {
        {
            sort_terms(D->bond_atoms, D->n_bonds, 2, order);
            std::vector<int2> ij(D->n_bonds); std::vector<float2> p(D->n_bonds);
            for (int k = 0; k < D->n_bonds; ++k) {
                const int t = order[k];
                ij[k] = make_int2(D->bond_atoms[2 * t], D->bond_atoms[2 * t + 1]);
                p[k] = make_float2((float)D->bond_r0[t], (float)D->bond_k[t]);
            }
            T.nb = D->n_bonds;
            for (int k = 0; k < T.nb; ++k) term[0].push_back(make_int4(ij[k].x, ij[k].y, -1, -1));
            HIPCHK(S, upload(S, (int2 **)&T.b_ij, ij)); HIPCHK(S, upload(S, (float2 **)&T.b_p, p));
        }
        {
            sort_terms(D->angle_atoms, D->n_angles, 3, order);
            std::vector<int4> ijk(D->n_angles); std::vector<float2> p(D->n_angles);
            for (int k = 0; k < D->n_angles; ++k) {
                const int t = order[k];
                ijk[k] = make_int4(D->angle_atoms[3 * t], D->angle_atoms[3 * t + 1], D->angle_atoms[3 * t + 2], 0);
                p[k] = make_float2((float)D->angle_theta0[t], (float)D->angle_k[t]);
            }
            T.na = D->n_angles;
            for (int k = 0; k < T.na; ++k) term[1].push_back(make_int4(ijk[k].x, ijk[k].y, ijk[k].z, -1));
            HIPCHK(S, upload(S, (int4 **)&T.a_ijk, ijk)); HIPCHK(S, upload(S, (float2 **)&T.a_p, p));
        }
        {
            sort_terms(D->torsion_atoms, D->n_torsions, 4, order);
            std::vector<int4> q(D->n_torsions); std::vector<float4> p(D->n_torsions);
            for (int k = 0; k < D->n_torsions; ++k) {
                const int t = order[k];
                q[k] = make_int4(D->torsion_atoms[4 * t], D->torsion_atoms[4 * t + 1], D->torsion_atoms[4 * t + 2],
                                 D->torsion_atoms[4 * t + 3]);
                p[k] = make_float4((float)D->torsion_k[t], (float)std::cos(D->torsion_phi0[t]),
                                   (float)std::sin(D->torsion_phi0[t]), (float)D->torsion_n[t]);
            }
            T.nt = D->n_torsions;
            term[2] = q;
            S->tor_order = order;
            HIPCHK(S, upload(S, (int4 **)&T.t_ijkl, q)); HIPCHK(S, upload(S, (float4 **)&T.t_p, p));
        }
        {
            sort_terms(D->restraint_atom, D->n_restraints, 1, order);
            std::vector<int> ia(D->n_restraints); std::vector<float4> p(D->n_restraints);
            for (int k = 0; k < D->n_restraints; ++k) {
                const int t = order[k];
                ia[k] = D->restraint_atom[t];
                p[k] = make_float4((float)D->restraint_ref[3 * t], (float)D->restraint_ref[3 * t + 1],
                                   (float)D->restraint_ref[3 * t + 2], (float)D->restraint_k[t]);
            }
            T.nr = D->n_restraints;
            for (int k = 0; k < T.nr; ++k) term[3].push_back(make_int4(ia[k], -1, -1, -1));
            HIPCHK(S, upload(S, (int **)&T.r_i, ia)); HIPCHK(S, upload(S, (float4 **)&T.r_p, p));
        }
        {
            sort_terms(D->pair14_atoms, D->n_pairs14, 2, order);
            std::vector<int2> ij(D->n_pairs14); std::vector<float4> p(D->n_pairs14);
            for (int k = 0; k < D->n_pairs14; ++k) {
                const int t = order[k];
                const int i = D->pair14_atoms[2 * t], j = D->pair14_atoms[2 * t + 1];
                ij[k] = make_int2(i, j);
                const double sij = 0.5 * (D->sigma[i] + D->sigma[j]);
                const double eij = std::sqrt(D->epsilon[i] * D->epsilon[j]);
                p[k] = make_float4((float)sij, (float)(4.0 * eij * D->scale14),
                                   (float)(COULOMB_F * D->charge[i] * D->charge[j] * D->scale14), 0.f);
            }
            T.n14 = D->n_pairs14;
            for (int k = 0; k < T.n14; ++k) term[4].push_back(make_int4(ij[k].x, ij[k].y, -1, -1));
            S->p14_order = order;
            HIPCHK(S, upload(S, (int2 **)&T.p_ij, ij)); HIPCHK(S, upload(S, (float4 **)&T.p_p, p));
        }
    }

    // nonbonded constants and pair-list capacity
    d.cutoff_on = (D->kind == GPR_KIND_MOLECULAR && D->cutoff > 0) ? 1 : 0;
    // list margins by mass
    const MarginRule margins = margin_rule(D->mass, n);
    const double heavy = margins.heavy;
    d.im_light = margins.im_light;
    {
        std::vector<unsigned char> cls((n + BLK - 1) / BLK, 0);
        for (int i = 0; i < n; ++i)
            if ((float)(1.0 / D->mass[i]) > d.im_light) cls[i / BLK] |= (unsigned char)(1u << (i % BLK));
        HIPCHK(S, upload(S, (unsigned char **)&d.cls, cls));
    }
    if (d.cutoff_on) {
        const double rc = D->cutoff;
        const double krf = (D->eps_rf - 1.0) / ((2.0 * D->eps_rf + 1.0) * rc * rc * rc);
        d.rc2 = (float)(rc * rc);
        d.krf = (float)krf;
        d.crf = (float)(1.0 / rc + krf * rc * rc);
        d.rl = (float)(rc + D->skin + 1e-4);
        const double ml = 0.5 * D->skin, mh = ml * heavy, pad = 1e-4;
        auto sq = [](double v) { return v * v; };
        d.guard2_light = (float)sq(ml);
        d.guard2_heavy = (float)sq(mh);
        d.list2_light = (float)sq(rc + ml + mh + pad);
        d.list2_heavy = (float)sq(rc + 2.0 * mh + pad);
        // the larger of the two differences (light i): a heavy i lists light partners 2 (ml - mh)^2 too far
        d.list2_j = (float)(sq(rc + 2.0 * ml + pad) - sq(rc + ml + mh + pad));
        d.period = std::max(1, D->nlist_period);
    } else {
        d.rc2 = INFINITY; d.krf = 0.f; d.crf = 0.f; d.rl = INFINITY;
        d.guard2_light = d.guard2_heavy = INFINITY; d.list2_light = d.list2_heavy = 1.0e30f; d.list2_j = 0.f;
        d.period = 1 << 30;
    }
    // capacity from the initial structure: the largest sub-list within r_list, doubled
    // per-atom work estimate for the persistent split: partners within r_list plus a constant
    // for the bonded terms, the integrator and the list build (about 72 pair evaluations' worth
    // per atom, fitted to measured per-group phase times)
    int maxsub = 0;
    S->work.assign(n, 1.0);
    if (D->kind == GPR_KIND_MOLECULAR) {
        const double rl2 = d.cutoff_on ? (double)d.rl * d.rl * 1.21 : INFINITY;
        const double rl2w = d.cutoff_on ? (double)d.rl * d.rl : INFINITY;
        std::vector<int> cnt(P);
        for (int i = 0; i < n; ++i) {
            std::fill(cnt.begin(), cnt.end(), 0);
            int nw = 0;
            for (int j = 0; j < n; ++j) {
                if (j == i) continue;
                const double dx = D->pos[i] - D->pos[j], dy = D->pos[n + i] - D->pos[n + j], dz = D->pos[2 * n + i] - D->pos[2 * n + j];
                const double r2 = dx * dx + dy * dy + dz * dz;
                if (r2 < rl2) cnt[j % P]++;
                if (r2 < rl2w) nw++;
            }
            for (int q = 0; q < P; ++q) maxsub = std::max(maxsub, cnt[q]);
            S->work[i] = nw + 72.0;
        }
    }
    const int kmax = std::max(8, d.cutoff_on ? 2 * maxsub + 8 : maxsub + 1);
    d.Kg = std::min(16383, (kmax + 3) / 4);
    HIPCHK(S, dalloc(S, &d.nbl, (size_t)R * d.Kg * np * P));
    HIPCHK(S, dalloc(S, &d.nbc, (size_t)R * np * P));
    HIPCHK(S, dalloc(S, &d.guard, 2 * R));
    HIPCHK(S, dalloc(S, &d.need_build, R));
    HIPCHK(S, dalloc(S, &d.list_pad, R));
    HIPCHK(S, dalloc(S, &d.last_build, 2 * R));
    HIPCHK(S, dalloc(S, &d.clock, 2));
    HIPCHK(S, dalloc(S, &d.err, 4));
    HIPCHK(S, dalloc(S, &d.sync, (size_t)R * 64));
    HIPCHK(S, dalloc(S, &d.ticket, (size_t)9 * 32));
    HIPCHK(S, dalloc(S, &d.xchg, (size_t)R * 4 * np));
    HIPCHK(S, dalloc(S, &d.esum, R));
    HIPCHK(S, dalloc(S, &d.acc, (size_t)R * MAX_OBS * 2));
    HIPCHK(S, dalloc(S, &d.shift, MAX_OBS));
    HIPCHK(S, dalloc(S, &d.state, R));

    // states and observables with their atom groups
    std::vector<int> groups;
    auto add_group = [&](const int32_t *g, int cnt, int &off, double &mtot) {
        off = (int)groups.size();
        mtot = 0;
        for (int k = 0; k < cnt; ++k) { groups.push_back(g[k]); mtot += D->mass[g[k]]; }
    };
    StateDesc st{};
    std::vector<ObsDesc> obs(MAX_OBS);
    st.kind = D->state.kind;
    for (int k = 0; k < 8; ++k) st.atoms[k] = D->state.atoms[k];
    st.nbox = D->state.n_boxes;
    for (int b = 0; b < GPR_MAX_BOXES; ++b)
        for (int c = 0; c < 4; ++c) st.box[b][c] = D->state.box[b][c];
    for (int c = 0; c < 3; ++c) st.center[c] = D->state.center[c];
    st.radius = D->state.radius;
    st.g_n = D->state.kind == GPR_STATE_COM_SPHERE ? D->state.n_group : 0;
    add_group(D->state.group, st.g_n, st.g_off, st.gm);
    d.nobs = D->n_obs;
    d.need_energy = 0;
    for (int j = 0; j < D->n_obs; ++j) {
        const gpr_obs_desc &o = D->obs[j];
        ObsDesc &od = obs[j];
        od.kind = o.kind;
        for (int k = 0; k < 4; ++k) od.atoms[k] = o.atoms[k];
        od.ga_n = (o.kind == GPR_OBS_COM_DISTANCE || o.kind == GPR_OBS_RMS_VELOCITY) ? o.n_a : 0;
        od.gb_n = o.kind == GPR_OBS_COM_DISTANCE ? o.n_b : 0;
        add_group(o.group_a, od.ga_n, od.ga_off, od.ma);
        add_group(o.group_b, od.gb_n, od.gb_off, od.mb);
        if (o.kind == GPR_OBS_POTENTIAL) d.need_energy = 1;
    }
    HIPCHK(S, upload(S, (int **)&d.groups, groups));
    HIPCHK(S, upload(S, (ObsDesc **)&d.obs, obs));
    HIPCHK(S, upload(S, (StateDesc **)&d.st, std::vector<StateDesc>(1, st)));

    d.h = (float)(0.5 * D->dt);
    d.c1 = (float)c1;
    d.key0 = (uint32_t)D->seed;
    d.key1 = (uint32_t)(D->seed >> 32);
    d.t_gr = D->t_gr;
    d.tol = D->tol;
    d.t_min = D->t_min;
    // force-field parameters kept on the host, device buffers of the parameter gradient
    S->mass_h.assign(D->mass, D->mass + n);
    if (D->kind == GPR_KIND_MOLECULAR) {
        S->eps_h.assign(D->epsilon, D->epsilon + n);
        S->sig_h.assign(D->sigma, D->sigma + n);
        S->q_h.assign(D->charge, D->charge + n);
        S->tor_k_h.assign(D->torsion_k, D->torsion_k + D->n_torsions);
        S->tor_phi0_h.assign(D->torsion_phi0, D->torsion_phi0 + D->n_torsions);
        S->tor_n_h.assign(D->torsion_n, D->torsion_n + D->n_torsions);
        for (int t = 0; t < D->n_pairs14; ++t)
            S->p14_h.push_back(make_int2(D->pair14_atoms[2 * t], D->pair14_atoms[2 * t + 1]));
        S->scale14 = D->scale14;
    }
    d.scale14 = (float)D->scale14;
    d.sqrt_f = std::sqrt(COULOMB_F);
    HIPCHK(S, dalloc(S, &d.gacc, (size_t)3 * np + std::max(1, d.tp.nt)));
    {
        std::vector<double> inv2eps(n, 0.0);
        HIPCHK(S, upload(S, (double **)&d.inv2eps, inv2eps));
        std::vector<int> orig(S->tor_order);
        if (orig.empty()) orig.push_back(0);
        HIPCHK(S, upload(S, (int **)&d.tor_orig, orig));
    }
    HIPCHK(S, write_params(S));
    {
        int dev = 0;
        HIPCHK(S, hipGetDevice(&dev));
        S->dev = dev < MAX_DEV ? dev : MAX_DEV - 1;
        HIPCHK(S, hipDeviceGetAttribute(&d.cus, hipDeviceAttributeMultiprocessorCount, dev));
    }

    // scratch for the per-check bookkeeping
    S->rb_bytes = std::max<size_t>((size_t)6 * np * sizeof(float), (size_t)R * MAX_OBS * 16 + MAX_OBS * 8);
    {
        const size_t at_fec = (sizeof(Status) + 255) / 256 * 256, at_rb = at_fec + (sizeof(long long) * R + 255) / 256 * 256;
        char *host = nullptr;
        HIPCHK(S, hipHostMalloc((void **)&host, at_rb + S->rb_bytes, hipHostMallocDefault));
        S->st_host = (Status *)host;
        S->adv_fec = (long long *)(host + at_fec);
        S->rb = host + at_rb;
    }
    HIPCHK(S, dalloc(S, &S->donor, R));
    HIPCHK(S, dalloc(S, &S->surv, R));
    HIPCHK(S, dalloc(S, &S->fec, R));
    HIPCHK(S, dalloc(S, &S->obs_out, (size_t)R * MAX_OBS));

    // LDS budgets
    const int nblk = (n + BLK - 1) / BLK;
    // the replica, then the boxes and scratch of a rebuild, or the force sums of 256 atoms over them
    S->lds_nb = (size_t)np * 24 + std::max((size_t)nblk * 16 + (size_t)16 * WBLK * 4, (size_t)256 * 3 * sizeof(long long));
    S->lds_stage = (size_t)np * 16;
    int dev = 0, maxlds = 0;
    HIPCHK(S, hipGetDevice(&dev));
    HIPCHK(S, hipDeviceGetAttribute(&maxlds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
    S->maxlds = maxlds;
    {
        // with the static LDS of the kernels that take them
        struct { const void *fn; size_t lds; } use[] = {{(const void *)k_forces, S->lds_nb}, {(const void *)k_grad_nb, S->lds_nb},
                                                        {(const void *)k_obs, S->lds_stage}, {(const void *)k_state, S->lds_stage}};
        for (const auto &u : use) {
            hipFuncAttributes fa{};
            HIPCHK(S, hipFuncGetAttributes(&fa, u.fn));
            if (u.lds + fa.sharedSizeBytes > (size_t)maxlds)
                return fail(S, GPR_EINVAL, "system too large for the LDS-staged pair kernel");
        }
    }
    HIPCHK(S, hipFuncSetAttribute((const void *)k_forces, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S->lds_nb));
    HIPCHK(S, hipFuncSetAttribute((const void *)k_grad_nb, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S->lds_nb));
    HIPCHK(S, hipFuncSetAttribute((const void *)k_obs, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S->lds_stage));
    HIPCHK(S, hipFuncSetAttribute((const void *)k_state, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S->lds_stage));
    {
        // dynamic LDS available to k_persist next to its static LDS
        hipFuncAttributes fa{};
        HIPCHK(S, hipFuncGetAttributes(&fa, (const void *)k_persist));
        S->maxlds_persist = maxlds - (int)fa.sharedSizeBytes;
        HIPCHK(S, hipFuncSetAttribute((const void *)k_persist, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      S->maxlds_persist));
        hipFuncAttributes fb{};
        HIPCHK(S, hipFuncGetAttributes(&fb, (const void *)k_persist_batch));
        if ((int)fb.sharedSizeBytes != (int)fa.sharedSizeBytes) return fail(S, GPR_EDEVICE, "persistent kernels differ in static LDS");
        HIPCHK(S, hipFuncSetAttribute((const void *)k_persist_batch, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      S->maxlds_persist));
    }
    S->bt_persist = std::min(1024, std::max(64, (n * P + 63) / 64 * 64));
    {
        hipFuncAttributes fa{};
        HIPCHK(S, hipFuncGetAttributes(&fa, (const void *)k_persist_small));
        const int room = maxlds - (int)fa.sharedSizeBytes;
        HIPCHK(S, hipFuncSetAttribute((const void *)k_persist_small, hipFuncAttributeMaxDynamicSharedMemorySize, room));
        // Every pair is evaluated, so the limit is where lists come out cheaper (measured, us per
        // step of 64 replicas, small / general kernel at its best shape): with a cutoff 3.4 / 6.4 at
        // 80 atoms, 5.0 / 7.1 at 128, 7.2 / 7.7 at 160, 11.2 / 9.0 at 200; without one 2.0 / 4.7 at
        // 22, 3.0 / 5.1 at 60, 5.3 / 7.3 at 128, 13.9 / 15.7 at 256 (one group per replica).
        S->small_ok = n <= (d.cutoff_on ? 160 : SMALL_MAX) && small_lds(S) <= (size_t)room;
    }
    {
        // persistent split: the fewest workgroups per replica (1, 2, 4 or 8) whose LDS fits, then
        // more while each keeps >= 256 atoms (launches of few replicas take more, see run_shape);
        // with more than one, every workgroup of the grid must be resident at once (the grid is
        // sized to what the device holds)
        int cus = 0;
        HIPCHK(S, hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        S->max_coresident = cus;
        // usable: the LDS fits and a workgroup can run; all_at_once: every replica's workgroups are
        // resident together (with fewer, sets of workgroups take the replicas in turn)
        auto usable = [&](int G, bool &ok, bool &all_at_once) -> hipError_t {
            const size_t lds = persist_lds(n, np, S->splits[split_index(G)]);
            ok = all_at_once = false;
            if ((int)lds > S->maxlds_persist) return hipSuccess;
            int per_cu = 0;
            const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k_persist,
                                                                              S->bt_persist, lds);
            ok = e == hipSuccess && per_cu >= 1;
            all_at_once = ok && (G == 1 || (long)R * G <= (long)per_cu * cus);
            return e;
        };
        for (int k = 0; k < NSPLIT; ++k) S->splits[k] = make_split(S->work, n, np, 1 << k);
        bool all[NSPLIT] = {};
        for (int k = 0; k < NSPLIT; ++k) HIPCHK(S, usable(1 << k, S->split_ok[k], all[k]));
        int G = 1;
        while (G <= 8 && !S->split_ok[split_index(G)]) G *= 2;
        S->persist_ok = G <= 8 ? 1 : 0;
        if (S->persist_ok)
            while (G < 8 && (n + 2 * G - 1) / (2 * G) >= 256 && all[split_index(2 * G)]) G *= 2;
        else
            G = 1;
        const gpr_status rc = lay_units(S, term);
        if (rc) return rc;
        S->groups = G;
        S->split = S->splits[split_index(G)];
    }
    HIPCHK(S, upload(S, &S->d_dev, std::vector<Dev>(1, d)));

    // initial velocities, copies into every replica, forces, Omega and the observable shift
    if (!D->vel) {
        hipLaunchKernelGGL(k_init_vel, dim3((n + 255) / 256), dim3(256), 0, S->stream, S->d_dev, (float)D->kT);
        LAUNCHCHK(S);
    }
    gpr_status rc = launch_forces(S, 0, 1, -1, 1, 0, 1);
    if (rc) return rc;
    rc = broadcast_reference(S);
    if (rc) return rc;
    HIPCHK(S, hipMemsetAsync(d.need_build, 0, sizeof(int) * R, S->stream));
    rc = launch_forces(S, 0, R, -1, 1, 0, 1);
    if (rc) return rc;
    hipLaunchKernelGGL(k_obs, dim3(1), obs_block(S), S->lds_stage, S->stream, S->d_dev, 0, 1, nullptr, 0);
    LAUNCHCHK(S);
    rc = state_of_ref(S, &S->omega);
    if (rc) return rc;
    S->phase = PH_IDLE;
    return GPR_OK;
}

extern "C" gpr_status gpr_system_create(const gpr_system_desc *D, gpr_system **out)
{
    if (!out) return fail(nullptr, GPR_EINVAL, "out is NULL");
    *out = nullptr;
    if (!D) return fail(nullptr, GPR_EINVAL, "descriptor is NULL");
    if (D->kind != GPR_KIND_TOY2D && D->kind != GPR_KIND_MOLECULAR) return fail(nullptr, GPR_EINVAL, "bad kind");
    if (D->n_atoms < 1 || D->n_atoms > 65535 || D->n_replicas < 2 || D->n_replicas > 4096 || !D->mass || !D->pos)
        return fail(nullptr, GPR_EINVAL, "bad sizes or missing arrays");
    if (D->kind == GPR_KIND_TOY2D && D->n_atoms != 1) return fail(nullptr, GPR_EINVAL, "the toy system has one particle");
    if (!(D->dt > 0) || !(D->kT > 0) || !(D->gamma >= 0)) return fail(nullptr, GPR_EINVAL, "bad dynamics parameters");
    if (D->t_gr < 1 || D->t_check_dephase < 1 || D->t_check_parallel < 1) return fail(nullptr, GPR_EINVAL, "bad periods");
    if (D->n_obs < 0 || D->n_obs > GPR_MAX_OBS || (D->n_obs > 0 && !D->obs)) return fail(nullptr, GPR_EINVAL, "bad observables");
    const int n = D->n_atoms;
    for (int i = 0; i < n; ++i) if (!(D->mass[i] > 0)) return fail(nullptr, GPR_EINVAL, "mass <= 0");
    if (D->kind == GPR_KIND_MOLECULAR) {
        if (!D->sigma || !D->epsilon || !D->charge) return fail(nullptr, GPR_EINVAL, "missing nonbonded parameters");
        if (!idx_ok(D->bond_atoms, 2L * D->n_bonds, n) || !idx_ok(D->angle_atoms, 3L * D->n_angles, n) ||
            !idx_ok(D->torsion_atoms, 4L * D->n_torsions, n) || !idx_ok(D->restraint_atom, D->n_restraints, n) ||
            !idx_ok(D->pair14_atoms, 2L * D->n_pairs14, n) || !idx_ok(D->exclusion_atoms, 2L * D->n_exclusions, n))
            return fail(nullptr, GPR_EINVAL, "term atom index out of range");
        if ((D->n_bonds && (!D->bond_r0 || !D->bond_k)) || (D->n_angles && (!D->angle_theta0 || !D->angle_k)) ||
            (D->n_torsions && (!D->torsion_n || !D->torsion_k || !D->torsion_phi0)) ||
            (D->n_restraints && (!D->restraint_ref || !D->restraint_k)))
            return fail(nullptr, GPR_EINVAL, "missing term parameters");
        for (int t = 0; t < D->n_torsions; ++t)
            if (D->torsion_n[t] < 0 || D->torsion_n[t] > 12) return fail(nullptr, GPR_EINVAL, "torsion multiplicity outside [0, 12]");
        if (D->cutoff > 0 && (!(D->skin > 0) || !(D->eps_rf >= 1))) return fail(nullptr, GPR_EINVAL, "bad cutoff parameters");
    }
    const gpr_state_desc &st = D->state;
    if (st.kind == GPR_STATE_SIGN_X) {
        if (!idx_ok(st.atoms, 1, n)) return fail(nullptr, GPR_EINVAL, "bad state atom");
    } else if (st.kind == GPR_STATE_DIHEDRAL_BOXES) {
        if (!idx_ok(st.atoms, 8, n) || st.n_boxes < 1 || st.n_boxes > GPR_MAX_BOXES) return fail(nullptr, GPR_EINVAL, "bad state boxes");
    } else if (st.kind == GPR_STATE_COM_SPHERE) {
        if (st.n_group < 1 || !idx_ok(st.group, st.n_group, n)) return fail(nullptr, GPR_EINVAL, "bad state group");
    } else {
        return fail(nullptr, GPR_EINVAL, "bad state kind");
    }
    for (int j = 0; j < D->n_obs; ++j) {
        const gpr_obs_desc &o = D->obs[j];
        bool ok = true;
        switch (o.kind) {
        case GPR_OBS_COORD: ok = idx_ok(o.atoms, 1, n) && o.atoms[1] >= 0 && o.atoms[1] <= 2; break;
        case GPR_OBS_POTENTIAL: case GPR_OBS_KINETIC: break;
        case GPR_OBS_DIHEDRAL: ok = idx_ok(o.atoms, 4, n); break;
        case GPR_OBS_COM_DISTANCE: ok = o.n_a >= 1 && o.n_b >= 1 && idx_ok(o.group_a, o.n_a, n) && idx_ok(o.group_b, o.n_b, n); break;
        case GPR_OBS_RMS_VELOCITY: ok = o.n_a >= 1 && idx_ok(o.group_a, o.n_a, n); break;
        default: ok = false;
        }
        if (!ok) return fail(nullptr, GPR_EINVAL, "bad observable");
    }
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) return fail(nullptr, GPR_EDEVICE, "no HIP device");
    gpr_system *S = new (std::nothrow) gpr_system();
    if (!S) return fail(nullptr, GPR_ENOMEM, "host allocation failed");
    gpr_status rc = create_impl(D, S);
    if (rc != GPR_OK) {
        g_thread_err = S->err;
        gpr_system_destroy(S);
        return rc;
    }
    *out = S;
    return GPR_OK;
}

extern "C" gpr_status gpr_set_stream(gpr_system *S, void *stream)
{
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    HIPCHK(S, hipStreamSynchronize(S->stream));
    S->stream = (hipStream_t)stream;
    return GPR_OK;
}

extern "C" gpr_status gpr_set_path(gpr_system *S, int32_t path)
{
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    if (path != GPR_PATH_PLAIN && path != GPR_PATH_PERSISTENT) return fail(S, GPR_EINVAL, "bad path");
    if (path == GPR_PATH_PERSISTENT && !S->persist_ok) return fail(S, GPR_EINVAL, "system too large for the persistent path");
    S->path = path;
    return GPR_OK;
}

extern "C" gpr_status gpr_set_launch(gpr_system *S, int32_t block_threads, int32_t groups_per_replica)
{
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    if (groups_per_replica != 0 && groups_per_replica != 1 && groups_per_replica != 2 && groups_per_replica != 4 &&
        groups_per_replica != 8)
        return fail(S, GPR_EINVAL, "groups_per_replica must be 1, 2, 4 or 8");
    if (block_threads != 0 && (block_threads < 64 || block_threads > 1024 || block_threads % 64))
        return fail(S, GPR_EINVAL, "block_threads must be a multiple of 64 in [64, 1024]");
    const int bt = block_threads != 0 ? block_threads : S->bt_persist;
    {
        const int G = groups_per_replica != 0 ? groups_per_replica : S->groups;
        const size_t lds = persist_lds(S->n, S->np, S->splits[split_index(G)]);
        if ((int)lds > S->maxlds_persist)
            return fail(S, GPR_EINVAL, "the per-workgroup LDS of this split exceeds the device limit");
        int per_cu = 0;
        HIPCHK(S, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k_persist, bt, lds));
        if (per_cu < 1) return fail(S, GPR_EINVAL, "a workgroup of this shape does not fit on a compute unit");
    }
    drop_cycle_graphs(S);                                   // captured with the old shape
    S->bt_persist = bt;
    if (block_threads != 0) S->bt_from = 2;
    if (groups_per_replica != 0) {
        S->groups_from = 2;
        S->groups = groups_per_replica;
        S->split = S->splits[split_index(groups_per_replica)];
    }
    return GPR_OK;
}

// Launch-shape autotuner of the persistent path: every (threads per workgroup, workgroups per
// replica) shape that fits is timed over nsteps steps (after a short warm-up), starting each
// time from the same saved state; the fastest is kept, or the library's own choice where that is
// faster still.  The saved state (positions,
// velocities, forces, list-reference positions and ages, step counter) is put back at the end
// with every pair list marked for a rebuild, so the run continues exactly as without the call
// (results do not depend on the shape or on when lists are rebuilt).
extern "C" gpr_status gpr_autotune(gpr_system *S, int32_t nsteps, int32_t *block_threads, int32_t *groups)
{
    if (S) drop_cycle_graphs(S);                            // captured with the old shape
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    if (nsteps < 1) return fail(S, GPR_EINVAL, "nsteps < 1");
    if (!S->persist_ok) return fail(S, GPR_EINVAL, "system too large for the persistent path");
    const int R = S->R;
    const size_t m = (size_t)R * 3 * S->np;
    Dev &d = S->d;
    // saved state, in scratch freed when the call returns
    struct Scratch {
        std::vector<void *> p;
        ~Scratch() { for (void *q : p) (void)hipFree(q); }
        hipError_t get(void **out, size_t bytes)
        {
            const hipError_t e = hipMalloc(out, bytes);
            if (e == hipSuccess) p.push_back(*out);
            return e;
        }
    } scratch;
    float *sx = nullptr, *sv = nullptr, *sxb = nullptr;
    long long *sF = nullptr, *slb = nullptr;
    HIPCHK(S, scratch.get((void **)&sx, sizeof(float) * m));
    HIPCHK(S, scratch.get((void **)&sv, sizeof(float) * m));
    HIPCHK(S, scratch.get((void **)&sxb, sizeof(float) * m));
    HIPCHK(S, scratch.get((void **)&sF, sizeof(long long) * m));
    HIPCHK(S, scratch.get((void **)&slb, sizeof(long long) * 2 * R));
    auto copy_all = [&](bool save) -> hipError_t {
        const hipMemcpyKind k = hipMemcpyDeviceToDevice;
        hipError_t e = hipMemcpyAsync(save ? sx : d.x, save ? d.x : sx, sizeof(float) * m, k, S->stream);
        if (!e) e = hipMemcpyAsync(save ? sv : d.v, save ? d.v : sv, sizeof(float) * m, k, S->stream);
        if (!e) e = hipMemcpyAsync(save ? sxb : d.xb, save ? d.xb : sxb, sizeof(float) * m, k, S->stream);
        if (!e) e = hipMemcpyAsync(save ? sF : d.F, save ? d.F : sF, sizeof(long long) * m, k, S->stream);
        if (!e) e = hipMemcpyAsync(save ? slb : d.last_build, save ? d.last_build : slb, sizeof(long long) * 2 * R, k, S->stream);
        if (!e && !save) {
            S->lists_old = true;
            std::vector<int> ones(R, 1);
            e = hipMemcpyAsync(d.need_build, ones.data(), sizeof(int) * R, hipMemcpyHostToDevice, S->stream);
            if (!e) e = hipStreamSynchronize(S->stream);
        }
        return e;
    };
    HIPCHK(S, copy_all(true));
    FinishAtEnd at_end{S};
    const long long s_saved = S->s;
    const int path_saved = S->path, bt_saved = S->bt_persist, g_saved = S->groups;
    const int btf_saved = S->bt_from, gf_saved = S->groups_from;
    const Split sp_saved = S->split;
    int dev = 0, cus = 0;
    HIPCHK(S, hipGetDevice(&dev));
    HIPCHK(S, hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    hipEvent_t e0, e1;
    HIPCHK(S, hipEventCreate(&e0));
    HIPCHK(S, hipEventCreate(&e1));
    // the time of nsteps steps on the shape that is set, from the saved state
    auto timed = [&](float &ms) -> gpr_status {
        HIPCHK(S, copy_all(false));
        S->s = s_saved;
        gpr_status rc = run_steps(S, R, std::min(20, nsteps), 0, false, false);
        if (rc) return rc;
        HIPCHK(S, hipEventRecord(e0, S->stream));
        rc = run_steps(S, R, nsteps, 0, false, false);
        if (rc) return rc;
        HIPCHK(S, hipEventRecord(e1, S->stream));
        HIPCHK(S, hipEventSynchronize(e1));
        int err[4];
        HIPCHK(S, hipMemcpy(err, d.err, sizeof err, hipMemcpyDeviceToHost));
        if (err[ERR_UNSTABLE] || err[ERR_BARRIER] || err[ERR_LIST]) return fail(S, GPR_EDEVICE, "autotune run failed");
        HIPCHK(S, hipEventElapsedTime(&ms, e0, e1));
        return GPR_OK;
    };
    float best = -1.f, own = -1.f;
    int best_bt = bt_saved, best_g = g_saved;
    gpr_status rc = GPR_OK;
    S->path = GPR_PATH_PERSISTENT;
    // the shape that launches of all replicas take by themselves (two replicas of 2,432 atoms run on 32
    // groups each, 9.2 us a step where the best of the shapes below takes 12.7)
    if (gf_saved == 0) rc = timed(own);
    S->bt_from = S->groups_from = 1;                       // the shapes tried, then the one kept
    for (int G = 1; G <= 8 && rc == GPR_OK; G *= 2) {
        const Split sp = S->splits[split_index(G)];
        const size_t lds = persist_lds(S->n, S->np, sp);
        if ((int)lds > S->maxlds_persist) continue;
        for (int bt = 256; bt <= 1024 && rc == GPR_OK; bt += 256) {
            int per_cu = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k_persist, bt, lds) != hipSuccess ||
                per_cu < 1 || (G > 1 && per_cu * cus < G))
                continue;
            S->bt_persist = bt; S->groups = G; S->split = sp;
            float ms = 0.f;
            rc = timed(ms);
            if (rc) break;
            if (best < 0.f || ms < best) { best = ms; best_bt = bt; best_g = G; }
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    // back to the saved state with the chosen shape
    S->path = path_saved;
    S->s = s_saved;
    {
        const hipError_t e = copy_all(false);
        if (e != hipSuccess && !rc) rc = fail(S, GPR_EDEVICE, std::string("autotune restore: ") + hipGetErrorString(e));
    }
    if (rc || (own >= 0.f && (best < 0.f || own <= best))) {
        S->bt_persist = bt_saved; S->groups = g_saved; S->split = sp_saved;
        S->bt_from = btf_saved; S->groups_from = gf_saved;
        if (rc) return rc;
    } else {
        S->bt_persist = best_bt;
        S->groups = best_g;
        S->split = S->splits[split_index(best_g)];
    }
    if (block_threads) *block_threads = best_bt;
    if (groups) *groups = best_g;
    return GPR_OK;
}

extern "C" gpr_status gpr_set_cycles(gpr_system *S, int32_t cycles)
{
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    if (cycles < 0 || cycles > 4096) return fail(S, GPR_EINVAL, "cycles must be in [0, 4096]");
    if (cycles > 0 && !S->persist_ok) return fail(S, GPR_EINVAL, "system too large for the persistent path");
    if (cycles == S->cycles) return GPR_OK;
    drop_cycle_graphs(S);
    if (S->stc_dev) { (void)hipFree(S->stc_dev); S->stc_dev = nullptr; }
    if (S->stc_host) { (void)hipHostFree(S->stc_host); S->stc_host = nullptr; }
    S->cycles = 0;
    if (cycles == 0) return GPR_OK;
    if (!S->cyc_dev) HIPCHK(S, hipMalloc((void **)&S->cyc_dev, sizeof(CycRec)));
    if (!S->cyc_host) HIPCHK(S, hipHostMalloc((void **)&S->cyc_host, sizeof(CycRec), hipHostMallocDefault));
    HIPCHK(S, hipMalloc((void **)&S->stc_dev, sizeof(Status) * cycles));
    HIPCHK(S, hipHostMalloc((void **)&S->stc_host, sizeof(Status) * cycles, hipHostMallocDefault));
    S->cycles = cycles;
    return GPR_OK;
}

extern "C" gpr_status gpr_set_graph(gpr_system *S, int32_t cycle_steps)
{
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    if (cycle_steps < 0 || cycle_steps > 10000) return fail(S, GPR_EINVAL, "cycle_steps must be in [0, 10000]");
    if (cycle_steps != S->graph_cycle) {
        HIPCHK(S, hipStreamSynchronize(S->stream));
        for (auto &g : S->graphs) (void)hipGraphExecDestroy(g.exec);
        S->graphs.clear();
        S->graph_cycle = cycle_steps;
    }
    return GPR_OK;
}

extern "C" gpr_status gpr_profile(gpr_system *S, int32_t enable)
{
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    HIPCHK(S, hipStreamSynchronize(S->stream));
    HIPCHK(S, prof_collect(S));
    S->prof = enable != 0;
    S->prof_ms = 0.0;
    S->prof_n = 0;
    while (S->prof && S->ev_a.size() < 8) HIPCHK(S, prof_add_pair(S));
    return GPR_OK;
}

extern "C" gpr_status gpr_profile_read(gpr_system *S, double *ms, int64_t *launches)
{
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    HIPCHK(S, hipStreamSynchronize(S->stream));
    HIPCHK(S, prof_collect(S));
    if (ms) *ms = S->prof_ms;
    if (launches) *launches = S->prof_n;
    return GPR_OK;
}

extern "C" gpr_status gpr_phase_read(gpr_system *S, double *out)
{
    if (!S || !out) return fail(S, GPR_EINVAL, "NULL argument");
    HIPCHK(S, hipStreamSynchronize(S->stream));
    std::vector<unsigned long long> acc((size_t)S->R * PHASE_MAX_G * NPHASE);
    const hipError_t e = phase_take(acc.data(), S->R, S->stream);
    if (e == hipErrorNotSupported) return fail(S, GPR_EINVAL, "library built without the phase timers");
    HIPCHK(S, e);
    int dev = 0, khz = 0;
    HIPCHK(S, hipGetDevice(&dev));
    HIPCHK(S, hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
    if (khz <= 0) return fail(S, GPR_EDEVICE, "no wall-clock rate");
    const double us_per_tick = 1000.0 / (double)khz;
    unsigned long long t0 = ~0ull;                        // the earliest start of the last launches
    for (size_t k = PH_START; k < acc.size(); k += NPHASE)
        if (acc[k]) t0 = std::min(t0, acc[k]);
    for (size_t k = 0; k < acc.size(); ++k) {
        const size_t slot = k % NPHASE;
        if (slot < PH_NSTEP) out[k] = (double)acc[k] * us_per_tick;
        else if (slot < PH_START) out[k] = (double)acc[k];
        else out[k] = acc[k] ? (double)(acc[k] - t0) * us_per_tick : 0.0;
    }
    return GPR_OK;
}

// ------------------------------------------------------------------ queries
extern "C" double gpr_simulated_time(const gpr_system *S) { return S ? (double)S->tsim * S->dt : NAN; }
extern "C" int64_t gpr_simulated_steps(const gpr_system *S) { return S ? S->tsim : -1; }
extern "C" int64_t gpr_global_step(const gpr_system *S) { return S ? S->s : -1; }
extern "C" int32_t gpr_current_state(const gpr_system *S) { return S ? S->omega : INT32_MIN; }
extern "C" int64_t gpr_advance_steps(const gpr_system *S) { return S ? S->adv_t : -1; }

extern "C" gpr_status gpr_energy_forces(gpr_system *S, int32_t r0, int32_t nr, double *energy, double *forces)
{
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    if (r0 < 0 || nr < 0 || r0 + nr > S->R) return fail(S, GPR_EINVAL, "replica range");
    if (nr == 0) return GPR_OK;
    gpr_status rc = launch_forces(S, r0, nr, -1, 1, 0, 1);
    if (rc) return rc;
    std::vector<long long> F((size_t)nr * 3 * S->np), E(nr);
    HIPCHK(S, hipMemcpyAsync(F.data(), S->d.F + (size_t)r0 * 3 * S->np, F.size() * 8, hipMemcpyDeviceToHost, S->stream));
    HIPCHK(S, hipMemcpyAsync(E.data(), S->d.E + r0, E.size() * 8, hipMemcpyDeviceToHost, S->stream));
    int err[4];
    HIPCHK(S, hipMemcpyAsync(err, S->d.err, sizeof err, hipMemcpyDeviceToHost, S->stream));
    HIPCHK(S, hipStreamSynchronize(S->stream));
    if (err[ERR_LIST]) return fail(S, GPR_EDEVICE, "pair-list capacity exceeded");
    for (int k = 0; k < nr; ++k) {
        if (energy) energy[k] = (double)E[k] * FIX_INV;
        if (forces)
            for (int c = 0; c < 3; ++c)
                for (int i = 0; i < S->n; ++i)
                    forces[((size_t)k * 3 + c) * S->n + i] = (double)F[((size_t)k * 3 + c) * S->np + i] * FIX_INV;
    }
    return GPR_OK;
}

extern "C" gpr_status gpr_set_params(gpr_system *S, const double *epsilon, const double *sigma, const double *charge,
                                     const double *torsion_k)
{
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    if (S->kind != GPR_KIND_MOLECULAR) return fail(S, GPR_EINVAL, "force-field parameters need a molecular system");
    const int n = S->n, nt = (int)S->tor_k_h.size();
    for (int i = 0; i < n; ++i) {
        if (epsilon && !(epsilon[i] >= 0 && std::isfinite(epsilon[i]))) return fail(S, GPR_EINVAL, "epsilon < 0 or not finite");
        if (sigma && !(sigma[i] >= 0 && std::isfinite(sigma[i]))) return fail(S, GPR_EINVAL, "sigma < 0 or not finite");
        if (charge && !std::isfinite(charge[i])) return fail(S, GPR_EINVAL, "charge not finite");
    }
    for (int t = 0; t < nt; ++t)
        if (torsion_k && !std::isfinite(torsion_k[t])) return fail(S, GPR_EINVAL, "torsion k not finite");
    if (epsilon) S->eps_h.assign(epsilon, epsilon + n);
    if (sigma) S->sig_h.assign(sigma, sigma + n);
    if (charge) S->q_h.assign(charge, charge + n);
    if (torsion_k) S->tor_k_h.assign(torsion_k, torsion_k + nt);
    HIPCHK(S, write_params(S));
    // the forces the integrator carries must belong to the new parameters
    gpr_status rc = launch_forces(S, 0, S->R, -1, 1, 0, 1);
    if (rc) return rc;
    HIPCHK(S, hipStreamSynchronize(S->stream));
    return GPR_OK;
}

extern "C" gpr_status gpr_energy_forces_dev(gpr_system *S, const float *x_dev, double *energy_dev, float *forces_dev)
{
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    if (!x_dev) return fail(S, GPR_EINVAL, "NULL positions");
    const int n = S->n, R = S->R;
    hipLaunchKernelGGL(k_load_x, dim3((n + 255) / 256, R), dim3(256), 0, S->stream, S->d_dev, x_dev);
    LAUNCHCHK(S);
    gpr_status rc = launch_forces(S, 0, R, -1, 1, 0, 1, false, false);
    if (rc) return rc;
    int *err = (int *)S->rb;
    hipLaunchKernelGGL(k_unfix_out, dim3((n + 255) / 256, R), dim3(256), 0, S->stream, S->d_dev, energy_dev, forces_dev, err);
    LAUNCHCHK(S);
    HIPCHK(S, hipStreamSynchronize(S->stream));
    if (err[ERR_LIST]) return fail(S, GPR_EDEVICE, "pair-list capacity exceeded");
    return GPR_OK;
}

extern "C" gpr_status gpr_energy_backward_dev(gpr_system *S, const double *w_dev, float *d_x, double *d_eps,
                                              double *d_sigma, double *d_charge, double *d_torsion_k)
{
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    if (!w_dev) return fail(S, GPR_EINVAL, "NULL weights");
    const bool params = d_eps || d_sigma || d_charge || d_torsion_k;
    if (params && S->kind != GPR_KIND_MOLECULAR) return fail(S, GPR_EINVAL, "force-field parameters need a molecular system");
    if (d_eps)
        for (double e : S->eps_h)
            if (!(e > 0)) return fail(S, GPR_EINVAL, "the epsilon gradient needs every epsilon > 0");
    const int n = S->n, np = S->np, R = S->R, nt = S->d.tp.nt, n14 = S->d.tp.n14;
    if (d_x) {
        hipLaunchKernelGGL(k_weighted_dx, dim3((n + 255) / 256, R), dim3(256), 0, S->stream, S->d_dev, w_dev, d_x);
        LAUNCHCHK(S);
    }
    const bool relist = params && S->lists_old;
    if (relist) {
        // the lists of the present positions (the forces come out as they are)
        gpr_status rc = launch_forces(S, 0, R, -1, 0, 0, 1);
        if (rc) return rc;
        rc = read_pieces(S, {{S->d.err, sizeof(int) * 4}});
        if (rc) return rc;
    }
    if (params) {
        // gacc is clear: k_grad_finish leaves it so
        if (S->gacc_dirty)
            HIPCHK(S, hipMemsetAsync(S->d.gacc, 0, sizeof(long long) * ((size_t)3 * np + std::max(1, nt)), S->stream));
        S->gacc_dirty = true;
        hipLaunchKernelGGL(k_grad_nb, dim3((n * P + 1023) / 1024, R), dim3(1024), S->lds_nb, S->stream, S->d_dev, w_dev);
        LAUNCHCHK(S);
        const int nterm = std::max(nt, n14);
        if (nterm > 0) {
            hipLaunchKernelGGL(k_grad_terms, dim3((nterm + 255) / 256, R), dim3(256), 0, S->stream, S->d_dev, w_dev);
            LAUNCHCHK(S);
        }
        hipLaunchKernelGGL(k_grad_finish, dim3((std::max(n, nt) + 255) / 256), dim3(256), 0, S->stream, S->d_dev, d_eps,
                           d_sigma, d_charge, d_torsion_k);
        LAUNCHCHK(S);
        S->gacc_dirty = false;
    }
    HIPCHK(S, hipStreamSynchronize(S->stream));
    if (relist && ((const int *)S->rb)[ERR_LIST]) return fail(S, GPR_EDEVICE, "pair-list capacity exceeded");
    return GPR_OK;
}

extern "C" gpr_status gpr_get_state(const gpr_system *Sc, int32_t r, double *q, double *v)
{
    gpr_system *S = const_cast<gpr_system *>(Sc);
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    if (r < 0 || r >= S->R) return fail(S, GPR_EINVAL, "replica index");
    const size_t m = (size_t)3 * S->np;
    const gpr_status rc = read_pieces(S, {{S->d.x + r * m, m * 4}, {S->d.v + r * m, m * 4}});
    if (rc) return rc;
    HIPCHK(S, hipStreamSynchronize(S->stream));
    const float *x = (const float *)S->rb;
    for (double *out : {q, v}) {
        if (out)
            for (int c = 0; c < 3; ++c)
                for (int i = 0; i < S->n; ++i) out[c * S->n + i] = x[c * S->np + i];
        x += m;
    }
    return GPR_OK;
}

extern "C" gpr_status gpr_set_state(gpr_system *S, int32_t r, const double *q, const double *v)
{
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    if (r < 0 || r >= S->R || !q) return fail(S, GPR_EINVAL, "replica index or NULL positions");
    std::vector<float> x(3 * S->np, 0.f), vv(3 * S->np, 0.f);
    if (!v) {
        HIPCHK(S, hipMemcpyAsync(vv.data(), S->d.v + (size_t)r * 3 * S->np, vv.size() * 4, hipMemcpyDeviceToHost, S->stream));
        HIPCHK(S, hipStreamSynchronize(S->stream));
    }
    for (int c = 0; c < 3; ++c)
        for (int i = 0; i < S->n; ++i) {
            x[c * S->np + i] = (float)q[c * S->n + i];
            if (v) vv[c * S->np + i] = (float)v[c * S->n + i];
        }
    if (S->kind == GPR_KIND_TOY2D) { x[2 * S->np] = 0.f; vv[2 * S->np] = 0.f; }
    HIPCHK(S, hipMemcpyAsync(S->d.x + (size_t)r * 3 * S->np, x.data(), x.size() * 4, hipMemcpyHostToDevice, S->stream));
    HIPCHK(S, hipMemcpyAsync(S->d.v + (size_t)r * 3 * S->np, vv.data(), vv.size() * 4, hipMemcpyHostToDevice, S->stream));
    gpr_status rc = launch_forces(S, r, 1, -1, 1, 0, 1);
    if (rc) return rc;
    HIPCHK(S, hipStreamSynchronize(S->stream));
    S->phase = PH_IDLE;
    return GPR_OK;
}

extern "C" gpr_status gpr_get_accumulators(const gpr_system *Sc, int64_t *n, double *S1, double *S2, double *shift)
{
    gpr_system *S = const_cast<gpr_system *>(Sc);
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    const gpr_status rc = read_pieces(S, {{S->d.shift, MAX_OBS * 8}, {S->d.acc, (size_t)S->R * MAX_OBS * 16}});
    if (rc) return rc;
    HIPCHK(S, hipStreamSynchronize(S->stream));
    const double *sh = (const double *)S->rb, *acc = sh + MAX_OBS;
    for (int r = 0; r < S->R; ++r)
        for (int j = 0; j < S->nobs; ++j) {
            if (S1) S1[r * S->nobs + j] = acc[((size_t)r * MAX_OBS + j) * 2];
            if (S2) S2[r * S->nobs + j] = acc[((size_t)r * MAX_OBS + j) * 2 + 1];
        }
    if (shift) for (int j = 0; j < S->nobs; ++j) shift[j] = sh[j];
    if (n) *n = S->nsamp;
    return GPR_OK;
}

extern "C" gpr_status gpr_observe(gpr_system *S, double *obs, int32_t *state)
{
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    if (S->d.need_energy) {
        gpr_status rc = launch_forces(S, 0, S->R, -1, 1, 0, 1);
        if (rc) return rc;
    }
    hipLaunchKernelGGL(k_obs, dim3(S->R), obs_block(S), S->lds_stage, S->stream, S->d_dev, 0, 2, S->obs_out, 0);
    LAUNCHCHK(S);
    hipLaunchKernelGGL(k_state, dim3(S->R), dim3(256), S->lds_stage, S->stream, S->d_dev, 0);
    LAUNCHCHK(S);
    std::vector<double> h((size_t)S->R * MAX_OBS);
    std::vector<int> st(S->R);
    HIPCHK(S, hipMemcpyAsync(h.data(), S->obs_out, h.size() * 8, hipMemcpyDeviceToHost, S->stream));
    HIPCHK(S, hipMemcpyAsync(st.data(), S->d.state, st.size() * 4, hipMemcpyDeviceToHost, S->stream));
    HIPCHK(S, hipStreamSynchronize(S->stream));
    for (int r = 0; r < S->R; ++r) {
        if (obs) for (int j = 0; j < S->nobs; ++j) obs[r * S->nobs + j] = h[(size_t)r * MAX_OBS + j];
        if (state) state[r] = st[r];
    }
    return GPR_OK;
}

// ------------------------------------------------------------------ Gen.ParRep steps
// Each call (transient propagation, convergence step, parallel step; Fig. 1) is a loop of
// chunks of steps, each ending at or before the call's next exit check, followed by that
// check.  PhaseRun holds one call in progress, so that the single-system calls and
// gpr_batch_run (several systems whose chunks share persistent launches) run one logic.
namespace {
struct PhaseRun {
    int op = 0;                          // GPR_OP_*
    long long t_corr = 0, budget = 0;    // budget: steps (transient, convergence) or checks (parallel)
    long long taken = 0;                 // steps (or checks) taken in this call
    bool done = false;
    gpr_status rc = GPR_OK;              // when done: GPR_OK (result written) or GPR_BUDGET
    gpr_event ev{};
    gpr_dephase_out dout{};
    gpr_exit_out pout{};
};
struct Chunk {
    int nrep;                            // replicas stepped
    long long k, t0;                     // steps; local step count at the start (sampling phase)
    bool sample, at_check;               // workers' observables every t_GR; the chunk ends at a check
};
} // namespace

static gpr_status phase_begin(gpr_system *S, PhaseRun &p)
{
    gpr_status rc;
    if (p.op == GPR_OP_DECORRELATE) {
        if (S->phase != PH_DECORR) {
            int st0 = -1;
            rc = state_of_ref(S, &st0);
            if (rc) return rc;
            S->phase = PH_DECORR;
            S->dc_omega = st0;
            S->dc_from = st0;
            S->dc_resid = 0;
            S->dc_steps = 0;
        }
    } else if (p.op == GPR_OP_DEPHASE) {
        if (S->phase != PH_DEPHASE) {
            if (S->omega == -1) return fail(S, GPR_EPHASE, "reference walker is in no state");
            rc = broadcast_reference(S);
            if (rc) return rc;
            HIPCHK(S, hipMemsetAsync(S->d.acc, 0, sizeof(double) * S->R * MAX_OBS * 2, S->stream));
            if (S->d.need_energy) {
                rc = launch_forces(S, 0, 1, -1, 1, 0, 1);
                if (rc) return rc;
            }
            hipLaunchKernelGGL(k_obs, dim3(1), obs_block(S), S->lds_stage, S->stream, S->d_dev, 0, 1, nullptr, 0);
            LAUNCHCHK(S);
            S->nsamp = 0;
            S->dp_t = 0;
            S->n_branch = 0;
            S->phase = PH_DEPHASE;
        }
    } else if (p.op == GPR_OP_PARALLEL_STEP) {
        if (S->phase == PH_CONVERGED) { S->phase = PH_PARALLEL; S->par_M = 0; S->par_t = 0; }
        else if (S->phase != PH_PARALLEL) return fail(S, GPR_EPHASE, "parallel step needs a converged dephasing");
    } else {
        return fail(S, GPR_EINVAL, "unknown Gen.ParRep step");
    }
    return GPR_OK;
}

// decisions taken before any further step: residence reached, or the budget spent
static void phase_ready(gpr_system *S, PhaseRun &p)
{
    if (p.done) return;
    if (p.op == GPR_OP_DECORRELATE && S->dc_omega != -1 && S->dc_resid >= p.t_corr) {
        S->omega = S->dc_omega;
        S->phase = PH_IDLE;
        p.ev.kind = GPR_EV_RESIDENT; p.ev.from_state = S->dc_from; p.ev.to_state = S->dc_omega; p.ev.pad = 0;
        p.ev.resident_steps = S->dc_resid; p.ev.steps_taken = S->dc_steps;
        p.done = true; p.rc = GPR_OK;
        return;
    }
    if (p.taken >= p.budget) { p.done = true; p.rc = GPR_BUDGET; }
}

// the next chunk, at most kmax steps
static Chunk phase_chunk(const gpr_system *S, const PhaseRun &p, long long kmax)
{
    Chunk c{};
    if (p.op == GPR_OP_DECORRELATE) {
        const long long pos = S->dc_steps % S->tcd;
        c.nrep = 1; c.k = S->tcd - pos; c.t0 = 0; c.sample = false;
        c.k = std::min(c.k, kmax);
        c.at_check = pos + c.k == S->tcd;
    } else if (p.op == GPR_OP_DEPHASE) {
        const long long pos = S->dp_t % S->tcd;
        c.nrep = S->R; c.t0 = S->dp_t; c.sample = true;
        c.k = std::min(std::min<long long>(S->tcd - pos, p.budget - p.taken), kmax);
        c.at_check = pos + c.k == S->tcd;
    } else {
        c.nrep = S->R; c.t0 = 0; c.sample = false;
        c.k = std::min<long long>(S->tcp - S->par_t, kmax);
        c.at_check = S->par_t + c.k == S->tcp;
    }
    return c;
}

// bookkeeping after a chunk of c.k steps (the steps themselves already taken), then, when
// the chunk ends at a check, the decision the check's status leads to: the status comes from
// running the check (st == nullptr) or from a replay of captured check cycles
static gpr_status phase_advance(gpr_system *S, PhaseRun &p, const Chunk &c, const Status *stc = nullptr)
{
    gpr_status rc;
    if (p.op == GPR_OP_DECORRELATE) {
        S->tsim += c.k;
        p.taken += c.k;
        S->dc_steps += c.k;
        if (!c.at_check) return GPR_OK;
        rc = check(S, CHK_STATE, 1, 0);
        if (rc) return rc;
        const int st = S->st_host->to_state;
        if (st == S->dc_omega) {
            S->dc_resid += S->tcd;
        } else if (S->dc_omega == -1) {
            S->dc_omega = st;              // entered a state: the reaching time ends here
            S->dc_resid = 0;
        } else {
            p.ev.kind = GPR_EV_EXITED; p.ev.from_state = S->dc_omega; p.ev.to_state = st; p.ev.pad = 0;
            p.ev.resident_steps = S->dc_resid + S->tcd; p.ev.steps_taken = S->dc_steps;
            S->omega = st;
            S->phase = PH_IDLE;
            p.done = true; p.rc = GPR_OK;
        }
        return GPR_OK;
    }
    if (p.op == GPR_OP_DEPHASE) {
        S->nsamp += count_samples(S->dp_t, S->dp_t + c.k, S->t_gr);
        S->dp_t += c.k;
        p.taken += c.k;
        if (!c.at_check) return GPR_OK;
        if (!stc) {
            rc = check(S, CHK_DEPHASE, S->R, 0);
            if (rc) return rc;
        }
        const Status &st = stc ? *stc : *S->st_host;
        gpr_dephase_out &o = p.dout;
        if (st.ref_exited) {
            S->tsim += S->dp_t;
            o.outcome = GPR_DEPHASE_REF_EXITED; o.to_state = st.to_state; o.t_steps = S->dp_t;
            o.n_branch = S->n_branch; o.n_samples = S->nsamp;
            for (int j = 0; j < GPR_MAX_OBS; ++j) o.rhat[j] = j < S->nobs ? st.rhat[j] : 0.0;
            S->omega = st.to_state;
            S->phase = PH_IDLE;
            p.done = true; p.rc = GPR_OK;
            return GPR_OK;
        }
        if (st.n_surv == 0 && S->R > 1) {
            S->n_branch += S->R - 1;
            S->nsamp = 0;
        } else {
            S->n_branch += st.n_exited;
        }
        bool conv = S->dp_t >= S->t_min && S->nsamp >= 2;
        for (int j = 0; j < S->nobs && conv; ++j) conv = st.rhat[j] < 1.0 + S->tol;
        if (conv) {
            S->tsim += S->dp_t;
            o.outcome = GPR_DEPHASE_CONVERGED; o.to_state = S->omega; o.t_steps = S->dp_t;
            o.n_branch = S->n_branch; o.n_samples = S->nsamp;
            for (int j = 0; j < GPR_MAX_OBS; ++j) o.rhat[j] = j < S->nobs ? st.rhat[j] : 0.0;
            S->phase = PH_CONVERGED;
            p.done = true; p.rc = GPR_OK;
        }
        return GPR_OK;
    }
    // parallel step
    S->par_t += c.k;
    if (!c.at_check) return GPR_OK;
    S->par_t = 0;
    S->par_M += 1;
    p.taken += 1;
    if (!stc) {
        rc = check(S, CHK_PARALLEL, S->R, S->par_M);
        if (rc) return rc;
    }
    const Status &st = stc ? *stc : *S->st_host;
    const int k = st.k;
    if (k == 0) return GPR_OK;
    // M, k and tau of Eq. 5, voted on the device
    const long long tau = st.tau;
    S->tsim += tau;
    if (k != 1) {
        rc = copy_replica(S, 0, k - 1);
        if (rc) return rc;
    }
    gpr_exit_out &o = p.pout;
    o.M = st.M; o.k = k; o.to_state = st.to_state; o.tau_steps = tau; o.tau = (double)tau * S->dt;
    S->omega = st.to_state;
    S->phase = PH_IDLE;
    HIPCHK(S, hipStreamSynchronize(S->stream));
    p.done = true; p.rc = GPR_OK;
    return GPR_OK;
}

static gpr_status run_cycles(gpr_system *S, PhaseRun &p, bool &ran);

static gpr_status run_phase(gpr_system *S, PhaseRun &p)
{
    FinishAtEnd at_end{S};
    gpr_status rc = phase_begin(S, p);
    if (rc) return rc;
    for (;;) {
        phase_ready(S, p);
        if (p.done) return p.rc;
        bool ran = false;
        rc = run_cycles(S, p, ran);
        if (rc) return rc;
        if (ran) continue;
        const Chunk c = phase_chunk(S, p, 1LL << 62);
        rc = run_steps(S, c.nrep, c.k, c.t0, c.sample, c.at_check);
        if (rc) return rc;
        rc = phase_advance(S, p, c);
        if (rc) return rc;
        if (p.done) return p.rc;
    }
}

static void drop_cycle_graphs(gpr_system *S)
{
    if (S->stream) (void)hipStreamSynchronize(S->stream);
    for (auto &g : S->cgraphs) (void)hipGraphExecDestroy(g.exec);
    S->cgraphs.clear();
}

// The captured run of S->cycles check cycles of the convergence step (op GPR_OP_DEPHASE) or
// the parallel step on the persistent path, captured on a stream of its own the first time
// it is needed.  Per cycle: the persistent launch(es) of one check period with the state test at
// the end, then the check with its clone-on-kill copies.  Steps, check indices and Omega come from
// the cycle record, which the host writes before each replay.
static gpr_status cycle_graph(gpr_system *S, int op, gpr_system::CGraph *out)
{
    for (auto &g : S->cgraphs)
        if (g.op == op) { *out = g; return GPR_OK; }
    const int nrep = S->R;
    const bool dep = op == GPR_OP_DEPHASE;
    const int nsteps = dep ? S->tcd : S->tcp;
    PersistBatch pb{};
    pb.nitems = 1;
    int nblocks = 0;
    const RunShape sh = run_shape(S, nrep);
    gpr_status rc = persist_item(S, *sh.sp, nrep, sh.bt, sh.lds, -1, pb.it[0], nblocks);
    if (rc) return rc;
    pb.it[0].noise_ahead = sh.noise_ahead ? 1 : 0;
    const int rounds = (nrep + pb.it[0].nsets - 1) / pb.it[0].nsets;
    rc = check_layout(S, pb, nblocks, sh.bt, true);
    if (rc) return rc;
    const dim3 cgrid = dep ? dim3((3 * S->np + 255) / 256, nrep) : dim3(1, 1);
    hipStream_t cs = nullptr;
    HIPCHK(S, hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    for (int j = 0; j < S->cycles && e == hipSuccess; ++j) {
        PersistItem it = pb.it[0];
        it.s0 = 0; it.t0 = 0; it.nsteps = nsteps; it.sample = dep ? 1 : 0; it.state_end = 1;
        it.cyc = S->cyc_dev;
        it.cycle = j;
        for (int k = 0; k < rounds && e == hipSuccess; ++k) {
            it.roff = k * it.nsets;
            void *args[] = {(void *)&it};
            e = hipLaunchKernel(sh.small ? (const void *)k_persist_small : (const void *)k_persist, dim3(nblocks), dim3(sh.bt),
                                args, sh.lds, cs);
        }
        if (e != hipSuccess) break;
        hipLaunchKernelGGL(k_check, cgrid, dim3(256), sizeof(int) * nrep, cs, S->d_dev, dep ? CHK_DEPHASE : CHK_PARALLEL,
                           0LL, 0, nrep, 0LL, 0LL, (long long)S->tcp, S->stc_dev, S->donor, S->surv, S->fec, 0, (long long *)nullptr,
                           S->cyc_dev, j);
        e = hipGetLastError();
    }
    hipGraph_t g = nullptr;
    const hipError_t e2 = hipStreamEndCapture(cs, &g);
    hipGraphExec_t ex = nullptr;
    hipError_t e3 = hipSuccess;
    if (e == hipSuccess && e2 == hipSuccess) e3 = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
    if (g) (void)hipGraphDestroy(g);
    (void)hipStreamDestroy(cs);
    if (e != hipSuccess || e2 != hipSuccess || e3 != hipSuccess)
        return fail(S, GPR_EDEVICE, std::string("check-cycle capture: ") +
                                        hipGetErrorString(e != hipSuccess ? e : e2 != hipSuccess ? e2 : e3));
    S->cgraphs.push_back({op, ex, sh.sp->G > 1 && !sh.small ? room_units(nblocks) : 0});
    *out = S->cgraphs.back();
    return GPR_OK;
}

// S->cycles check cycles replayed from the captured graph, when the call stands at a check
// boundary with room in its budget for all of them; then the host takes, cycle by cycle, the
// decision each status leads to, exactly as after a check it runs itself, and verifies that
// the call ends at the cycle the device stopped at.
static gpr_status run_cycles(gpr_system *S, PhaseRun &p, bool &ran)
{
    ran = false;
    const int C = S->cycles;
    if (C <= 0 || S->path != GPR_PATH_PERSISTENT || (p.op != GPR_OP_DEPHASE && p.op != GPR_OP_PARALLEL_STEP))
        return GPR_OK;
    const bool dep = p.op == GPR_OP_DEPHASE;
    const long long per = dep ? S->tcd : S->tcp;
    if (dep ? (S->dp_t % S->tcd != 0 || p.budget - p.taken < C * per) : (S->par_t != 0 || p.budget - p.taken < C))
        return GPR_OK;
    gpr_system::CGraph g{};
    gpr_status rc = cycle_graph(S, p.op, &g);
    if (rc) return rc;
    if (g.units) (void)hold(S, g.units, true);
    CycRec &h = *S->cyc_host;
    h.s_start = S->s; h.t_start = dep ? S->dp_t : 0; h.M_start = S->par_M; h.nsamp = S->nsamp;
    h.nsteps = (int)per; h.halt_cycle = NO_HALT; h.omega = S->omega; h.pad = 0;
    HIPCHK(S, hipMemcpyAsync(S->cyc_dev, S->cyc_host, sizeof(CycRec), hipMemcpyHostToDevice, S->stream));
    S->lists_old = true;
    HIPCHK(S, hipGraphLaunch(g.exec, S->stream));
    HIPCHK(S, hipMemcpyAsync(S->stc_host, S->stc_dev, sizeof(Status) * C, hipMemcpyDeviceToHost, S->stream));
    HIPCHK(S, hipMemcpyAsync(S->cyc_host, S->cyc_dev, sizeof(CycRec), hipMemcpyDeviceToHost, S->stream));
    HIPCHK(S, finish(S));
    ran = true;
    const int halt = S->cyc_host->halt_cycle;
    const int ncyc = halt == NO_HALT ? C : halt + 1;
    for (int j = 0; j < ncyc; ++j) {
        const Status &st = S->stc_host[j];
        rc = flag_errors(S, st.err);
        if (rc) return rc;
        Chunk c{};
        c.nrep = S->R; c.k = per; c.t0 = dep ? S->dp_t : 0; c.sample = dep; c.at_check = true;
        S->s += per;
        rc = phase_advance(S, p, c, &st);
        if (rc) return rc;
        if (p.done != (j == halt)) return fail(S, GPR_EDEVICE, "check cycles: device and host disagree on the end of the call");
        if (p.done) break;
    }
    return GPR_OK;
}

extern "C" gpr_status gpr_decorrelate(gpr_system *S, int64_t t_corr, int64_t max_steps, gpr_event *ev)
{
    if (!S || !ev) return fail(S, GPR_EINVAL, "NULL argument");
    PhaseRun p;
    p.op = GPR_OP_DECORRELATE; p.t_corr = t_corr; p.budget = max_steps;
    const gpr_status rc = run_phase(S, p);
    if (rc == GPR_OK) *ev = p.ev;
    return rc;
}

extern "C" gpr_status gpr_dephase(gpr_system *S, int64_t max_steps, gpr_dephase_out *o)
{
    if (!S || !o) return fail(S, GPR_EINVAL, "NULL argument");
    PhaseRun p;
    p.op = GPR_OP_DEPHASE; p.budget = max_steps;
    const gpr_status rc = run_phase(S, p);
    if (rc == GPR_OK) *o = p.dout;
    return rc;
}

// copies the (x, v, F) of one replica between the system and a replica-sized buffer set
static gpr_status move_replica(gpr_system *S, float *dx, float *dv, long long *dF, const float *sx, const float *sv,
                               const long long *sF)
{
    const size_t m = (size_t)3 * S->np;
    HIPCHK(S, hipMemcpyAsync(dx, sx, sizeof(float) * m, hipMemcpyDeviceToDevice, S->stream));
    HIPCHK(S, hipMemcpyAsync(dv, sv, sizeof(float) * m, hipMemcpyDeviceToDevice, S->stream));
    HIPCHK(S, hipMemcpyAsync(dF, sF, sizeof(long long) * m, hipMemcpyDeviceToDevice, S->stream));
    return GPR_OK;
}

extern "C" gpr_status gpr_dephase_fixed(gpr_system *S, int64_t t_phase, int64_t max_steps, gpr_dephase_out *o)
{
    if (!S || !o) return fail(S, GPR_EINVAL, "NULL argument");
    FinishAtEnd at_end{S};
    const int R = S->R;
    const size_t m = (size_t)3 * S->np;
    Dev &d = S->d;
    gpr_status rc;
    if (S->phase != PH_DEPHASE_FIXED) {
        if (S->omega == -1) return fail(S, GPR_EPHASE, "reference walker is in no state");
        if (t_phase < 0) return fail(S, GPR_EINVAL, "t_phase < 0");
        if (!S->snap_x) {
            HIPCHK(S, dalloc(S, &S->snap_x, m)); HIPCHK(S, dalloc(S, &S->snap_v, m)); HIPCHK(S, dalloc(S, &S->snap_F, m));
            HIPCHK(S, dalloc(S, &S->samp_x, m * R)); HIPCHK(S, dalloc(S, &S->samp_v, m * R));
            HIPCHK(S, dalloc(S, &S->samp_F, m * R));
        }
        rc = move_replica(S, S->snap_x, S->snap_v, S->snap_F, d.x, d.v, d.F);
        if (rc) return rc;
        rc = broadcast_reference(S);
        if (rc) return rc;
        S->resid.assign(R, 0);
        S->done.assign(R, 0);
        S->dp_t = 0;
        S->n_branch = 0;
        S->phase = PH_DEPHASE_FIXED;
    }
    const int one = 1;
    std::vector<int> st(R);
    long long taken = 0;
    while (taken < max_steps) {
        const long long k = std::min<long long>(S->tcd - S->dp_t % S->tcd, max_steps - taken);
        const bool at_check = (S->dp_t + k) % S->tcd == 0;
        rc = run_steps(S, R, k, S->dp_t, false, at_check);
        if (rc) return rc;
        S->dp_t += k;
        taken += k;
        if (!at_check) break;
        HIPCHK(S, hipMemcpyAsync(st.data(), d.state, sizeof(int) * R, hipMemcpyDeviceToHost, S->stream));
        int err[4];
        HIPCHK(S, hipMemcpyAsync(err, d.err, sizeof err, hipMemcpyDeviceToHost, S->stream));
        HIPCHK(S, finish(S));
        if (err[ERR_UNSTABLE]) return fail(S, GPR_EUNSTABLE, "non-finite or overflowing state");
        if (err[ERR_BARRIER]) return fail(S, GPR_EDEVICE, "persistent kernel barrier timed out");
        if (err[ERR_LIST]) return fail(S, GPR_EDEVICE, "pair-list capacity exceeded");
        bool all = true;
        for (int r = 0; r < R; ++r) {
            if (S->done[r]) continue;
            const size_t b = (size_t)r * m;
            if (st[r] != S->omega) {
                rc = move_replica(S, d.x + b, d.v + b, d.F + b, S->snap_x, S->snap_v, S->snap_F);
                if (rc) return rc;
                S->lists_old = true;
                HIPCHK(S, hipMemcpyAsync(d.need_build + r, &one, sizeof(int), hipMemcpyHostToDevice, S->stream));
                S->resid[r] = 0;
                S->n_branch += 1;
                all = false;
            } else if ((S->resid[r] += S->tcd) >= t_phase) {
                rc = move_replica(S, S->samp_x + b, S->samp_v + b, S->samp_F + b, d.x + b, d.v + b, d.F + b);
                if (rc) return rc;
                S->done[r] = 1;
            } else {
                all = false;
            }
        }
        if (all) {
            S->lists_old = true;
            for (int r = 0; r < R; ++r) {
                const size_t b = (size_t)r * m;
                rc = move_replica(S, d.x + b, d.v + b, d.F + b, S->samp_x + b, S->samp_v + b, S->samp_F + b);
                if (rc) return rc;
            }
            std::vector<int> ones(R, 1);
            HIPCHK(S, hipMemcpyAsync(d.need_build, ones.data(), sizeof(int) * R, hipMemcpyHostToDevice, S->stream));
            HIPCHK(S, hipStreamSynchronize(S->stream));
            o->outcome = GPR_DEPHASE_CONVERGED; o->to_state = S->omega; o->t_steps = S->dp_t;
            o->n_branch = S->n_branch; o->n_samples = 0;
            for (int j = 0; j < GPR_MAX_OBS; ++j) o->rhat[j] = 0.0;
            S->phase = PH_CONVERGED;
            return GPR_OK;
        }
        HIPCHK(S, hipStreamSynchronize(S->stream));
    }
    return GPR_BUDGET;
}

extern "C" gpr_status gpr_parallel_step(gpr_system *S, int64_t max_checks, gpr_exit_out *o)
{
    if (!S || !o) return fail(S, GPR_EINVAL, "NULL argument");
    PhaseRun p;
    p.op = GPR_OP_PARALLEL_STEP; p.budget = max_checks;
    const gpr_status rc = run_phase(S, p);
    if (rc == GPR_OK) *o = p.pout;
    return rc;
}

extern "C" gpr_status gpr_advance(gpr_system *S, int64_t nsteps, int64_t *first_exit_check)
{
    if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
    if (nsteps < 0) return fail(S, GPR_EINVAL, "nsteps < 0");
    // the sampling (every t_GR) and check (every t_check_dephase) schedule runs on the steps
    // counted over all calls, so that short calls sample and check as one long call would
    FinishAtEnd at_end{S};
    long long t = S->adv_t;
    const long long end = S->adv_t + nsteps;
    bool checked = false, at_check = false;
    while (t < end) {
        const long long k = std::min<long long>(S->tcd - t % S->tcd, end - t);
        at_check = (t + k) % S->tcd == 0;
        gpr_status rc = run_steps(S, S->R, k, t, true, at_check);
        if (rc) return rc;
        S->nsamp += count_samples(t, t + k, S->t_gr);
        t += k;
        S->adv_t = t;
        if (at_check) {
            rc = check(S, CHK_ADVANCE, S->R, t / S->tcd, !checked, t < end);
            if (rc) return rc;
            checked = true;
        }
    }
    // one wait for the steps and the results: the error flags come with the check that ends the call,
    // the first exit checks with its last check
    if (!at_check) {
        const gpr_status rc = read_pieces(S, {{S->d.err, sizeof(int) * 4}});
        if (rc) return rc;
    }
    HIPCHK(S, finish(S));
    HIPCHK(S, prof_collect(S));
    const gpr_status rc = flag_errors(S, at_check ? S->st_host->err : (const int *)S->rb);
    if (rc) return rc;
    if (first_exit_check) for (int r = 0; r < S->R; ++r) first_exit_check[r] = checked ? S->adv_fec[r] : 0;
    return GPR_OK;
}

// ------------------------------------------------------------------ several systems in one launch
// validation shared by the batch calls
static gpr_status batch_check(gpr_system *const *systems, int32_t nsys)
{
    if (!systems || nsys < 1 || nsys > MAX_BATCH) return fail(nullptr, GPR_EINVAL, "1 to 8 systems");
    for (int k = 0; k < nsys; ++k) {
        gpr_system *S = systems[k];
        if (!S) return fail(nullptr, GPR_EINVAL, "NULL system");
        for (int j = 0; j < k; ++j)
            if (systems[j] == S) return fail(S, GPR_EINVAL, "a system appears twice");
        if (!S->persist_ok) return fail(S, GPR_EINVAL, "system too large for the persistent path");
        if (S->stream != systems[0]->stream) return fail(S, GPR_EINVAL, "all systems must use one stream");
    }
    return GPR_OK;
}

// block size of a shared launch (the largest of the systems'), LDS (with their own splits, then
// of the layout), the workgroups the device holds at once and the most LDS that keeps that number;
// w[k]: work estimate of one step of one of system k's replicas
struct BatchShape {
    int bt = 64;
    size_t lds0 = 0, lds = 0, lds_most = 0;
    int capacity = 0;
    int units = 0;             // room that the workgroups that wait for one another need (0: none do)
    std::vector<double> w;
};

static gpr_status batch_shape(gpr_system *const *systems, int32_t nsys, BatchShape &sh)
{
    sh.w.assign(nsys, 0.0);
    for (int k = 0; k < nsys; ++k) {
        gpr_system *S = systems[k];
        sh.bt = std::max(sh.bt, S->bt_persist);
        sh.lds0 = std::max(sh.lds0, persist_lds(S->n, S->np, S->split));
        double per = 0.0;
        for (double x : S->work) per += x;
        sh.w[k] = per;
    }
    int dev = 0, cus = 0, per_cu = 0;
    HIPCHK(systems[0], hipGetDevice(&dev));
    HIPCHK(systems[0], hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    HIPCHK(systems[0], hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k_persist_batch, sh.bt, sh.lds0));
    sh.capacity = per_cu * cus;
    sh.lds_most = per_cu == 1 ? (size_t)systems[0]->maxlds_persist : sh.lds0;
    return GPR_OK;
}

// Items of a shared launch for the systems with nrep[k] > 0 replicas stepped: workgroups per replica
// and sets for each, so that the longest takes the least time by the estimate (rounds of replicas
// per set) x (us of one replica's step on G workgroups).  That is 4 + 1.7 (G > 1) + (1.55e-4 + 1e-5 G)
// w / G, within 8 % of steps measured from 160 to 4,600 atoms on 1 to 8 workgroups.  The splits are
// the system's own where the caller or the autotuner chose it.  (One set at a time for the longest,
// with each system's own split: 45.8 us a step for the mix of 22, 300, 1,200 and 2,432 atoms with 48
// replicas each; this way 38.)  slot[k]: the item of system k (-1: none).
static gpr_status batch_layout(gpr_system *const *systems, int32_t nsys, const std::vector<int> &nrep,
                               BatchShape &sh, PersistBatch &pb, std::vector<int> &slot, int &nblocks)
{
    gpr_system *S0 = systems[0];
    struct Choice {
        const Split *sp = nullptr;
        int sets = 0;
    };
    std::vector<Choice> pick(nsys);
    // the fewest workgroups with which every system takes at most T
    auto need = [&](double T) {
        long used = 0;
        for (int k = 0; k < nsys; ++k) {
            if (nrep[k] <= 0) continue;
            const gpr_system *S = systems[k];
            pick[k] = Choice{};
            for (int j = 0; j < 4; ++j) {
                const Split *sp = (1 << j) == S->groups ? &S->split : &S->splits[j];
                const int G = sp->G;
                if ((1 << j) != S->groups && (S->groups_from != 0 || !S->split_ok[j] || S->n < 64 << j)) continue;
                if (persist_lds(S->n, S->np, *sp) > sh.lds_most) continue;
                const double t = 4.0 + (G > 1 ? 1.7 : 0.0) + (1.55e-4 + 1e-5 * G) * sh.w[k] / G;
                const long rounds = (long)(T / t);
                if (rounds < 1) continue;
                const int sets = (int)((nrep[k] + rounds - 1) / rounds);
                if (!pick[k].sp || (long)sets * G < (long)pick[k].sets * pick[k].sp->G) pick[k] = {sp, sets};
            }
            if (!pick[k].sp) return LONG_MAX;
            used += (long)pick[k].sets * pick[k].sp->G;
        }
        return used;
    };
    double lo = 0.0, hi = 1.0;
    while (hi < 1e12 && need(hi) > sh.capacity) hi *= 2.0;
    if (need(hi) > sh.capacity) return fail(S0, GPR_EINVAL, "the systems' workgroups do not fit on the device at once");
    for (int it = 0; it < 40 && hi - lo > 1e-3 * hi; ++it) {
        const double mid = 0.5 * (lo + hi);
        (need(mid) > sh.capacity ? lo : hi) = mid;
    }
    (void)need(hi);
    std::vector<PersistItem> items(nsys);
    std::vector<int> nb(nsys, 0);
    sh.lds = 0;
    for (int k = 0; k < nsys; ++k) {
        if (nrep[k] <= 0) continue;
        gpr_system *S = systems[k];
        const Split &sp = *pick[k].sp;
        gpr_status rc = persist_item(S, sp, nrep[k], sh.bt, sh.lds_most, pick[k].sets * sp.G, items[k], nb[k]);
        if (rc) return rc;
        const size_t with = (size_t)persist_off(S->n, S->np, sp.lmax).end;
        items[k].noise_ahead = with <= sh.lds_most && S->kind != GPR_KIND_TOY2D;   // (drawn beside the pair tasks)
        sh.lds = std::max(sh.lds, items[k].noise_ahead ? with : persist_lds(S->n, S->np, sp));
    }
    slot.assign(nsys, -1);
    pb = PersistBatch{};
    int boff = 0, j = 0;
    for (int pass = 1; pass >= 0; --pass)
        for (int k = 0; k < nsys; ++k) {
            if (nrep[k] <= 0 || items[k].xcd != pass) continue;
            items[k].boff = boff;
            boff += nb[k];
            slot[k] = j;
            pb.it[j++] = items[k];
            if (pass == 1) pb.mapped = boff;
        }
    pb.nitems = j;
    if (boff > sh.capacity) return fail(S0, GPR_EINVAL, "the systems' workgroups do not fit on the device at once");
    nblocks = boff;
    int waiting = 0;
    for (int k = 0; k < nsys; ++k)
        if (nrep[k] > 0 && items[k].sp.G > 1) waiting += room_units(nb[k]);
    sh.units = waiting;
    return GPR_OK;
}

// gpr_advance of every system, with the persistent steps of all systems in shared launches:
// each launch runs up to the next exit check of any of them, then the systems at a check run
// it.  Workgroups are shared out so as to even out the systems' estimated times per step.
extern "C" gpr_status gpr_batch_advance(gpr_system *const *systems, int32_t nsys, int64_t nsteps,
                                        int64_t *const *first_exit_check)
{
    gpr_status rc = batch_check(systems, nsys);
    if (rc) return rc;
    if (nsteps < 0) return fail(systems[0], GPR_EINVAL, "nsteps < 0");
    gpr_system *S0 = systems[0];
    hipStream_t stream = S0->stream;
    BatchShape sh;
    rc = batch_shape(systems, nsys, sh);
    if (rc) return rc;
    std::vector<int> nrep(nsys), slot;
    for (int k = 0; k < nsys; ++k) nrep[k] = systems[k]->R;
    PersistBatch pb{};
    int nblocks = 0;
    rc = batch_layout(systems, nsys, nrep, sh, pb, slot, nblocks);
    if (rc) return rc;
    FinishAtEnd at_end{S0};
    std::vector<long long> t(nsys, 0);
    for (int k = 0; k < nsys; ++k) t[k] = systems[k]->adv_t;
    std::vector<char> checked(nsys, 0);
    long long done = 0;
    while (done < nsteps) {
        long long kstep = nsteps - done;
        for (int k = 0; k < nsys; ++k) kstep = std::min<long long>(kstep, systems[k]->tcd - t[k] % systems[k]->tcd);
        kstep = std::min<long long>(kstep, 1 << 20);
        for (int k = 0; k < nsys; ++k) {
            gpr_system *S = systems[k];
            PersistItem &it = pb.it[slot[k]];
            it.s0 = S->s;
            it.nsteps = (int)kstep;
            it.t0 = (int)(t[k] % S->t_gr);
            it.sample = 1;
            it.state_end = (t[k] + kstep) % S->tcd == 0 ? 1 : 0;
        }
        if (sh.units) (void)hold(S0, sh.units, true);
        rc = launch_persist(S0, pb, nblocks, sh.bt, sh.lds, stream);
        if (rc) return rc;
        for (int k = 0; k < nsys; ++k) {
            gpr_system *S = systems[k];
            S->s += kstep;
            S->nsamp += count_samples(t[k], t[k] + kstep, S->t_gr);
            t[k] += kstep;
            S->adv_t = t[k];
            if (t[k] % S->tcd == 0) {
                rc = check(S, CHK_ADVANCE, S->R, t[k] / S->tcd, !checked[k]);
                if (rc) return rc;
                checked[k] = 1;
                give_back(S0);                             // (the check has waited for the launch)
            }
        }
        done += kstep;
    }
    for (int k = 0; k < nsys; ++k) {
        rc = read_pieces(systems[k], {{systems[k]->d.err, sizeof(int) * 4}});
        if (rc) return rc;
    }
    HIPCHK(S0, finish(S0));
    for (int k = 0; k < nsys; ++k) {
        gpr_system *S = systems[k];
        rc = flag_errors(S, (const int *)S->rb);
        if (rc) return rc;
        if (first_exit_check && first_exit_check[k])
            for (int r = 0; r < S->R; ++r) first_exit_check[k][r] = checked[k] ? S->adv_fec[r] : 0;
    }
    return GPR_OK;
}

// The Gen.ParRep calls of several systems (Fig. 1 steps), their chunks of steps in shared
// launches: each launch takes every running system up to the nearest exit check among them.
extern "C" gpr_status gpr_batch_run(gpr_system *const *systems, int32_t nsys, gpr_batch_op *ops)
{
    gpr_status rc = batch_check(systems, nsys);
    if (rc) return rc;
    if (!ops) return fail(systems[0], GPR_EINVAL, "NULL ops");
    gpr_system *S0 = systems[0];
    hipStream_t stream = S0->stream;
    BatchShape sh;
    rc = batch_shape(systems, nsys, sh);
    if (rc) return rc;
    FinishAtEnd at_end{S0};
    std::vector<PhaseRun> p(nsys);
    for (int k = 0; k < nsys; ++k) {
        p[k].op = ops[k].op;
        p[k].t_corr = ops[k].t_corr;
        p[k].budget = ops[k].max_steps;
        ops[k].status = GPR_BUDGET;
    }
    auto hand_over = [&](int k) {
        ops[k].status = p[k].rc;
        if (p[k].rc == GPR_OK) {
            if (p[k].op == GPR_OP_DECORRELATE) ops[k].event = p[k].ev;
            else if (p[k].op == GPR_OP_DEPHASE) ops[k].dephase = p[k].dout;
            else ops[k].exit = p[k].pout;
        }
    };
    for (int k = 0; k < nsys; ++k) {
        rc = phase_begin(systems[k], p[k]);
        if (rc) { ops[k].status = rc; return rc; }
    }
    std::vector<int> nrep(nsys), slot, last_nrep;
    std::vector<Chunk> c(nsys);
    PersistBatch pb{};
    int nblocks = 0;
    for (;;) {
        long long kstep = 1LL << 20;
        int active = 0;
        for (int k = 0; k < nsys; ++k) {
            phase_ready(systems[k], p[k]);
            nrep[k] = 0;
            if (p[k].done) continue;
            c[k] = phase_chunk(systems[k], p[k], 1LL << 62);
            kstep = std::min(kstep, c[k].k);
            nrep[k] = c[k].nrep;
            ++active;
        }
        if (active == 0) break;
        if (nrep != last_nrep) {                          // the running systems or their replica counts changed
            rc = batch_layout(systems, nsys, nrep, sh, pb, slot, nblocks);
            if (rc) return rc;
            last_nrep = nrep;
        }
        for (int k = 0; k < nsys; ++k) {
            if (nrep[k] == 0) continue;
            gpr_system *S = systems[k];
            c[k] = phase_chunk(S, p[k], kstep);
            PersistItem &it = pb.it[slot[k]];
            it.s0 = S->s;
            it.nsteps = (int)kstep;
            it.t0 = (int)(c[k].t0 % S->t_gr);
            it.sample = c[k].sample ? 1 : 0;
            it.state_end = c[k].at_check ? 1 : 0;
        }
        if (sh.units) (void)hold(S0, sh.units, true);
        rc = launch_persist(S0, pb, nblocks, sh.bt, sh.lds, stream);
        if (rc) return rc;
        for (int k = 0; k < nsys; ++k) {
            if (nrep[k] == 0) continue;
            systems[k]->s += kstep;
            rc = phase_advance(systems[k], p[k], c[k]);
            if (rc) { ops[k].status = rc; return rc; }
            if (c[k].at_check) give_back(S0);              // (the check has waited for the launch)
        }
    }
    for (int k = 0; k < nsys; ++k) hand_over(k);
    return GPR_OK;
}

// ------------------------------------------------------------------ building blocks
template <class T>
static hipError_t tmp_alloc(std::vector<void *> &v, T **p, size_t count)
{
    void *q = nullptr;
    hipError_t e = hipMalloc(&q, std::max<size_t>(count, 1) * sizeof(T));
    if (e == hipSuccess) { v.push_back(q); *p = (T *)q; }
    return e;
}

struct TmpBufs {
    std::vector<void *> v;
    ~TmpBufs() { for (void *p : v) (void)hipFree(p); }
};

#define TMPCHK(call)                                                                                \
    do {                                                                                            \
        hipError_t e_ = (call);                                                                     \
        if (e_ != hipSuccess) return fail(nullptr, GPR_EDEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

extern "C" gpr_status gpr_philox_noise(uint64_t seed, int32_t replica, int64_t step, int32_t stream, int32_t n_atoms,
                                       uint32_t *out_words, float *out_gauss)
{
    if (n_atoms < 0 || stream < 0 || stream > 255) return fail(nullptr, GPR_EINVAL, "bad arguments");
    if (n_atoms == 0) return GPR_OK;
    TmpBufs t;
    uint32_t *w = nullptr;
    float *g = nullptr;
    TMPCHK(tmp_alloc(t.v, &w, 4 * (size_t)n_atoms));
    TMPCHK(tmp_alloc(t.v, &g, 3 * (size_t)n_atoms));
    hipLaunchKernelGGL(k_noise_test, dim3((n_atoms + 255) / 256), dim3(256), 0, 0, (uint32_t)seed,
                       (uint32_t)(seed >> 32), replica, (long long)step, stream, n_atoms, w, g);
    TMPCHK(hipGetLastError());
    if (out_words) TMPCHK(hipMemcpy(out_words, w, 16 * (size_t)n_atoms, hipMemcpyDeviceToHost));
    if (out_gauss) TMPCHK(hipMemcpy(out_gauss, g, 12 * (size_t)n_atoms, hipMemcpyDeviceToHost));
    TMPCHK(hipDeviceSynchronize());
    return GPR_OK;
}

extern "C" gpr_status gpr_fv_plan(uint64_t seed, int64_t step, int32_t R, const uint8_t *exited, int32_t *donor)
{
    if (R < 1 || !exited || !donor) return fail(nullptr, GPR_EINVAL, "bad arguments");
    TmpBufs t;
    uint8_t *ex = nullptr;
    int *dn = nullptr, *sv = nullptr;
    TMPCHK(tmp_alloc(t.v, &ex, R));
    TMPCHK(tmp_alloc(t.v, &dn, R));
    TMPCHK(tmp_alloc(t.v, &sv, R));
    TMPCHK(hipMemcpy(ex, exited, R, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(k_fvplan_test, dim3(1), dim3(256), 0, 0, (uint32_t)seed, (uint32_t)(seed >> 32), (long long)step, R, ex, dn, sv);
    TMPCHK(hipGetLastError());
    TMPCHK(hipMemcpy(donor, dn, sizeof(int) * R, hipMemcpyDeviceToHost));
    return GPR_OK;
}

// ------------------------------------------------------------------ branching plan without allocation
// Device array that gpr_fv_plan_noalloc stages through, for up to GPR_NOALLOC_MAX_R replicas:
// donors (int) at byte 0, the survivor list (int) at 4 * max, the exited flags at 8 * max.
// Every device the library runs on holds its own copy until the process ends.  In host code
// its name is not a device address: the address is taken per device with
// hipGetSymbolAddress and only that address is used.
constexpr size_t NOALLOC_BYTES = (size_t)9 * GPR_NOALLOC_MAX_R;
static __device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];

namespace {
constexpr int NOALLOC_MAX_DEV = 64;
std::mutex g_scratch_mu;
unsigned char *g_scratch_ptr[NOALLOC_MAX_DEV] = {};

// the device address of `scratch` on the current device, taken on the first call there
hipError_t scratch_of_current_device(unsigned char **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= NOALLOC_MAX_DEV) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = (unsigned char *)ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}
} // namespace

extern "C" gpr_status gpr_fv_plan_noalloc(uint64_t seed, int64_t step, int32_t R, const uint8_t *exited, int32_t *donor)
{
    if (R < 1 || !exited || !donor) return fail(nullptr, GPR_EINVAL, "bad arguments");
    if (R > GPR_NOALLOC_MAX_R)
        return fail(nullptr, GPR_EINVAL, "R exceeds GPR_NOALLOC_MAX_R (" + std::to_string(GPR_NOALLOC_MAX_R) + ")");
    unsigned char *base = nullptr;
    TMPCHK(scratch_of_current_device(&base));
    int *dn = (int *)base;
    int *sv = (int *)(base + (size_t)4 * GPR_NOALLOC_MAX_R);
    uint8_t *ex = base + (size_t)8 * GPR_NOALLOC_MAX_R;
    // every word the kernel reads is written first (flags copied in, survivors and donors
    // written before they are read), so nothing needs clearing between calls
    TMPCHK(hipMemcpy(ex, exited, R, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(k_fvplan_test, dim3(1), dim3(256), 0, 0, (uint32_t)seed, (uint32_t)(seed >> 32), (long long)step, R, ex, dn, sv);
    TMPCHK(hipGetLastError());
    TMPCHK(hipMemcpy(donor, dn, sizeof(int) * R, hipMemcpyDeviceToHost));
    return GPR_OK;
}

extern "C" gpr_status gpr_rhat(int32_t nw, int32_t n_obs, int64_t n, const double *S1, const double *S2, double *rhat)
{
    if (nw < 1 || n_obs < 0 || n_obs > 64 || n < 1 || (n_obs && (!S1 || !S2 || !rhat)))
        return fail(nullptr, GPR_EINVAL, "bad arguments");
    if (n_obs == 0) return GPR_OK;
    TmpBufs t;
    double *a = nullptr, *b = nullptr, *o = nullptr;
    const size_t cnt = (size_t)nw * n_obs;
    TMPCHK(tmp_alloc(t.v, &a, cnt));
    TMPCHK(tmp_alloc(t.v, &b, cnt));
    TMPCHK(tmp_alloc(t.v, &o, n_obs));
    TMPCHK(hipMemcpy(a, S1, cnt * 8, hipMemcpyHostToDevice));
    TMPCHK(hipMemcpy(b, S2, cnt * 8, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(k_rhat_test, dim3(n_obs), dim3(64), 0, 0, nw, n_obs, (long long)n, a, b, o);
    TMPCHK(hipGetLastError());
    TMPCHK(hipMemcpy(rhat, o, 8 * (size_t)n_obs, hipMemcpyDeviceToHost));
    return GPR_OK;
}

extern "C" gpr_status gpr_exit_vote(int32_t R, const int64_t *fec, int64_t t_check, int64_t *M, int32_t *k, int64_t *tau)
{
    if (R < 1 || !fec || !M || !k || !tau) return fail(nullptr, GPR_EINVAL, "bad arguments");
    TmpBufs t;
    long long *f = nullptr, *o = nullptr;
    TMPCHK(tmp_alloc(t.v, &f, R));
    TMPCHK(tmp_alloc(t.v, &o, 3));
    TMPCHK(hipMemcpy(f, fec, 8 * (size_t)R, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(k_vote_test, dim3(1), dim3(256), 0, 0, R, f, (long long)t_check, o);
    TMPCHK(hipGetLastError());
    long long h[3];
    TMPCHK(hipMemcpy(h, o, sizeof h, hipMemcpyDeviceToHost));
    if (h[0] == 0) return GPR_BUDGET;
    *M = h[0];
    *k = (int32_t)h[1];
    *tau = h[2];
    return GPR_OK;
}
