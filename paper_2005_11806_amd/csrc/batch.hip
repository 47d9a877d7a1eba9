// Batched uneven solves: one plan per problem, every pass of every problem
// expressed as tiles of the same block-level tile functions as the single
// solve (pass_x.hpp, pass_yz.hpp). Two executors share the task code:
//  * per-pass batched kernels: one launch per pass covers the tiles of all
//    problems (a block finds its problem by a prefix table); the sequence of
//    launches, refinement rounds included, is captured once in a HIP graph and
//    replayed;
//  * a persistent kernel: blocks take tickets from a global task queue (passes
//    in dependency order, problems largest first), wait on per-(problem, pass)
//    completion counters with a bounded spin, run the tile and release the
//    counter.
// Mixed precision runs the refinement rounds with device-side convergence
// flags: once a problem converges its remaining tiles return immediately.
#include <algorithm>
#include <cstring>
#include <numeric>
#include <vector>

#include "batch_tasks.hpp"

struct psv_batch;

namespace psv {

__global__ void k_persist_reset(ProblemDesc* desc, int n, int* counters, int ncount, int* ticket,
                                int* error) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        desc[i].flags[F_DONE] = 0;
        desc[i].flags[F_STEPS] = 0;
    }
    if (i < ncount) counters[i] = 0;
    if (i == 0) {
        *ticket = 0;
        *error = 0;
    }
}

}  // namespace psv

struct psv_batch {
    std::vector<psv::Plan*> plans;
    psv_opts opts{};
    int n = 0;
    bool fp32 = false;
    psv::ProblemDesc* d_desc = nullptr;
    psv::ProblemIO* d_io = nullptr;
    psv::ProblemIO* h_io = nullptr;  // pinned
    // the copy of h_io to d_io reads h_io when the stream reaches it: the next
    // call waits for this event before it rewrites the table
    hipEvent_t io_copied = nullptr;
    bool io_pending = false;
    std::vector<psv::PassLaunch> seq[2];  // per graph: without / with the final check
    std::vector<int*> starts[2];
    hipGraph_t graph[2] = {nullptr, nullptr};
    hipGraphExec_t exec[2] = {nullptr, nullptr};
    int device = 0;
    // persistent executor (per graph)
    int persistent = 0;
    int4* d_tasks[2] = {nullptr, nullptr};
    int* d_kinds[2] = {nullptr, nullptr};
    int ntasks[2] = {0, 0};
    int nlevels[2] = {0, 0};
    size_t plds[2] = {0, 0};
    int* d_counters = nullptr;  // sized for the longer sequence
    int ncounters = 0;
    int* d_ticket = nullptr;    // [0] ticket, [1] error
    int* h_err = nullptr;       // pinned
};

namespace psv {

void plan_init(Plan& p, const psv_grid& g, const psv_opts& o, bool alloc_ws);
void plan_free(Plan& p);

static size_t kind_lds(const Plan& p, int kind, bool fp32) {
    const size_t cs = fp32 ? sizeof(float2) : sizeof(double2);
    switch (kind) {
        case K_FWD: case K_RES:
            return fwd_x_lds(make_xgeom(p), cs, kind == K_RES ? FWD_RESID : p.opts.method == PSV_SPLIT_RHO0 ? FWD_METHOD1 : FWD_CONST,
                             bx_compiled(p.nx / 2));
        case K_INV: case K_INVADD: return inv_x_lds(make_xgeom(p, true), cs, bx_compiled(p.nx / 2));
        case K_Y: case K_YI: return yz_lds(p.ny, p.lp.kc, cs, yz_batch_compiled(p.ny));
        case K_Z: case K_Z2: return ifc_lds(p);
        default: return 0;
    }
}

__global__ void k_batch_reset(ProblemDesc* desc, int n) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) {
        desc[p].flags[F_DONE] = 0;
        desc[p].flags[F_STEPS] = 0;
    }
}

std::vector<int> batch_sequence(bool fp32, int method, int rounds, bool check) {
    std::vector<int> k;
    if (method == PSV_SPLIT_RHO0) {
        k.push_back(K_MINP);
        k.push_back(K_MINF);
    }
    k.push_back(K_FWD);
    if (fp32) k.push_back(K_MEAN);
    k.insert(k.end(), {K_Y, K_Z, K_YI, K_INV});
    if (fp32) {
        for (int r = 0; r < rounds; ++r) k.insert(k.end(), {K_RES, K_NRM, K_Y, K_Z2, K_YI, K_INVADD});
    }
    if (check || fp32) k.insert(k.end(), {K_CHK, K_CHKF});
    return k;
}

void batch_build(psv_batch& B, bool check) {
    const int gi = check ? 1 : 0;
    const int rounds = B.fp32 ? std::max(1, std::min(B.opts.max_refine, 3)) : 0;
    const std::vector<int> kinds = batch_sequence(B.fp32, B.opts.method, rounds, check);
    B.seq[gi].clear();
    for (int kind : kinds) {
        // the forward x kinds of a Method-I batch run as one launch per stencil
        // variant and the y kinds as one per chunk size, each over the problems
        // whose plan takes it; the interface kinds as one launch
        auto variant = [&](int p) {
            const Plan& P = *B.plans[p];
            if ((kind == K_FWD && B.opts.method == PSV_SPLIT_RHO0) || kind == K_RES) return P.lp.xstage;
            if (kind == K_Y || kind == K_YI) return P.lp.kc;
            return 1;
        };
        int qm = 4;
        for (const Plan* P : B.plans) qm = std::max(qm, ifc_qmax(2 * ((P->nz + P->lp.kc - 1) / P->lp.kc)));
        for (int sel : {1, 0, 4, 8, 16}) {
            PassLaunch L{};
            L.kind = kind;
            L.sel = kind == K_Z || kind == K_Z2 ? qm : sel;
            std::vector<int> st(B.n + 1, 0);
            size_t lds = 0;
            for (int p = 0; p < B.n; ++p) {
                const bool mine = variant(p) == sel;
                st[p + 1] = st[p] + (mine ? kind_tiles(*B.plans[p], kind) : 0);
                if (mine) lds = std::max(lds, kind_lds(*B.plans[p], kind, B.fp32));
            }
            if (st[B.n] == 0) continue;
            L.nblk = st[B.n];
            L.lds = lds;
            int* d = nullptr;
            PSV_HIP(hipMalloc(&d, st.size() * sizeof(int)));
            PSV_HIP(hipMemcpy(d, st.data(), st.size() * sizeof(int), hipMemcpyHostToDevice));
            B.starts[gi].push_back(d);
            L.d_start = d;
            B.seq[gi].push_back(L);
        }
    }
    // persistent queue: level by level, problems largest first (LPT)
    std::vector<int> order(B.n);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        return B.plans[a]->ncell() > B.plans[b]->ncell();
    });
    std::vector<int4> tasks;
    const int nlev = (int)kinds.size();
    size_t plds = 0;
    for (int lev = 0; lev < nlev; ++lev) {
        for (int p : order) {
            const int nt = kind_tiles(*B.plans[p], kinds[lev]);
            const int dep = lev > 0 ? kind_tiles(*B.plans[p], kinds[lev - 1]) : 0;
            for (int t = 0; t < nt; ++t) tasks.push_back(int4{p, lev, t, dep});
            plds = std::max(plds, kind_lds(*B.plans[p], kinds[lev], B.fp32));
        }
    }
    B.ntasks[gi] = (int)tasks.size();
    B.nlevels[gi] = nlev;
    B.plds[gi] = plds;
    PSV_HIP(hipMalloc(&B.d_tasks[gi], tasks.size() * sizeof(int4)));
    PSV_HIP(hipMemcpy(B.d_tasks[gi], tasks.data(), tasks.size() * sizeof(int4), hipMemcpyHostToDevice));
    PSV_HIP(hipMalloc(&B.d_kinds[gi], kinds.size() * sizeof(int)));
    PSV_HIP(hipMemcpy(B.d_kinds[gi], kinds.data(), kinds.size() * sizeof(int), hipMemcpyHostToDevice));
    if (B.n * nlev > B.ncounters) {
        if (B.d_counters) PSV_HIP(hipFree(B.d_counters));
        B.ncounters = B.n * nlev;
        PSV_HIP(hipMalloc(&B.d_counters, B.ncounters * sizeof(int)));
    }
}

static void launch_persistent(const psv_batch& B, int gi, hipStream_t s) {
    const int ncount = B.n * B.nlevels[gi];
    const int rn = std::max(B.n, ncount);
    hipLaunchKernelGGL(k_persist_reset, dim3((rn + 255) / 256), dim3(256), 0, s, B.d_desc, B.n,
                       B.d_counters, ncount, B.d_ticket, B.d_ticket + 1);
    const PersistArgs A{B.d_desc, B.d_io, B.d_tasks[gi], B.d_kinds[gi], B.d_counters,
                        B.d_ticket, B.d_ticket + 1, B.ntasks[gi], B.nlevels[gi], 0};
    if (B.fp32)
        launch_queue32(A, B.plds[gi], B.device, s);
    else
        launch_queue64(A, B.plds[gi], B.device, s);
}

void batch_enqueue(const psv_batch& B, int gi, hipStream_t s) {
    if (B.persistent) {
        launch_persistent(B, gi, s);
        return;
    }
    hipLaunchKernelGGL(k_batch_reset, dim3((B.n + 255) / 256), dim3(256), 0, s, B.d_desc, B.n);
    for (const PassLaunch& L : B.seq[gi]) {
        if (B.fp32)
            launch_pass32(L, B.d_desc, B.d_io, B.n, s);
        else
            launch_pass64(L, B.d_desc, B.d_io, B.n, s);
    }
}

void batch_create(psv_batch& B, int n, const psv_grid* grids, const psv_opts& o) {
    B.n = n;
    B.opts = o;
    B.fp32 = o.precision == PSV_MIXED;
    PSV_HIP(hipGetDevice(&B.device));
    std::vector<ProblemDesc> desc(n);
    for (int p = 0; p < n; ++p) {
        Plan* pl = new Plan();
        B.plans.push_back(pl);
        plan_init(*pl, grids[p], o, true);
        const int need = 2 * kind_tiles(*pl, K_CHK) + 64;
        if (need > pl->n_partials) {
            PSV_HIP(hipFree(pl->partials));
            pl->n_partials = need;
            PSV_HIP(hipMalloc(&pl->partials, need * sizeof(double)));
        }
        ProblemDesc& D = desc[p];
        std::memset(&D, 0, sizeof(D));
        D.xg = make_xgeom(*pl);
        D.xgi = make_xgeom(*pl, true);
        D.st = Stencil{pl->t.inv_h, pl->t.inv_g, pl->t.vol};
        D.z = make_zargs(*pl, pl->scal + S_RHS_MEAN);
        D.method = o.method;
        D.fp32 = B.fp32 ? 1 : 0;
        D.rad_y = pl->rad_y;
        D.twx = B.fp32 ? (const void*)pl->t.twx32 : (const void*)pl->t.twx64;
        D.twy = B.fp32 ? (const void*)pl->t.twy32 : (const void*)pl->t.twy64;
        D.spec = pl->spec;
        D.r_ws = pl->r_ws;
        D.partials = pl->partials;
        D.scal = pl->scal;
        D.flags = pl->flags;
        D.tol = pl->opts.tol;
        double hsum = 0.0;
        for (double h : pl->h) hsum += h;
        D.vtotal = pl->dx * pl->dy * hsum * pl->nx * pl->ny;
        D.ncell = pl->ncell();
        for (int k = 0; k < K_NKIND; ++k) D.ntiles[k] = kind_tiles(*pl, k);
    }
    PSV_HIP(hipMalloc(&B.d_desc, n * sizeof(ProblemDesc)));
    PSV_HIP(hipMemcpy(B.d_desc, desc.data(), n * sizeof(ProblemDesc), hipMemcpyHostToDevice));
    PSV_HIP(hipMalloc(&B.d_io, n * sizeof(ProblemIO)));
    PSV_HIP(hipHostMalloc(&B.h_io, n * sizeof(ProblemIO)));
    std::memset(B.h_io, 0, n * sizeof(ProblemIO));
    PSV_HIP(hipEventCreateWithFlags(&B.io_copied, hipEventDisableTiming));
    PSV_HIP(hipMalloc(&B.d_ticket, 2 * sizeof(int)));
    PSV_HIP(hipHostMalloc(&B.h_err, sizeof(int)));
    *B.h_err = 0;
    B.persistent = (o.batch_executor == 2) ? 1 : 0;
}

void batch_free(psv_batch& B) {
    for (int i = 0; i < 2; ++i) {
        if (B.exec[i]) (void)hipGraphExecDestroy(B.exec[i]);
        if (B.graph[i]) (void)hipGraphDestroy(B.graph[i]);
    }
    for (int i = 0; i < 2; ++i) {
        for (int* d : B.starts[i]) (void)hipFree(d);
        if (B.d_tasks[i]) (void)hipFree(B.d_tasks[i]);
        if (B.d_kinds[i]) (void)hipFree(B.d_kinds[i]);
    }
    if (B.d_counters) (void)hipFree(B.d_counters);
    if (B.d_ticket) (void)hipFree(B.d_ticket);
    if (B.h_err) (void)hipHostFree(B.h_err);
    for (Plan* p : B.plans) {
        plan_free(*p);
        delete p;
    }
    if (B.d_desc) (void)hipFree(B.d_desc);
    if (B.d_io) (void)hipFree(B.d_io);
    if (B.h_io) (void)hipHostFree(B.h_io);
    if (B.io_copied) (void)hipEventDestroy(B.io_copied);
}

// One batched solve: upload the per-call pointer table, then replay the
// captured graph (captured on first use for this `check` setting).
void batch_solve(psv_batch& B, hipStream_t s, bool check) {
    PSV_HIP(hipMemcpyAsync(B.d_io, B.h_io, B.n * sizeof(ProblemIO), hipMemcpyHostToDevice, s));
    PSV_HIP(hipEventRecord(B.io_copied, s));
    B.io_pending = true;
    const int gi = check ? 1 : 0;
    if (!B.exec[gi]) {
        batch_build(B, check);
        hipStream_t cs;
        PSV_HIP(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
        PSV_HIP(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
        batch_enqueue(B, gi, cs);
        PSV_HIP(hipStreamEndCapture(cs, &B.graph[gi]));
        PSV_HIP(hipGraphInstantiate(&B.exec[gi], B.graph[gi], nullptr, nullptr, 0));
        PSV_HIP(hipStreamDestroy(cs));
    }
    PSV_HIP(hipGraphLaunch(B.exec[gi], s));
}

psv_batch* batch_new() { return new psv_batch(); }

void batch_delete(psv_batch* b) {
    batch_free(*b);
    delete b;
}

int batch_size(const psv_batch& B) { return B.n; }
int batch_method(const psv_batch& B) { return B.opts.method; }
bool batch_fp32(const psv_batch& B) { return B.fp32; }

void batch_set_io(psv_batch& B, int p, const double* f, const double* rho, const double* pprev,
                  double* pout, double rho0, bool want_r) {
    // the previous call's copy of the table may still be queued behind work
    // on its stream
    if (B.io_pending) {
        PSV_HIP(hipEventSynchronize(B.io_copied));
        B.io_pending = false;
    }
    ProblemIO& io = B.h_io[p];
    io.f = f;
    io.rho = rho;
    io.pprev = pprev;
    io.pout = pout;
    io.rho0 = rho0;
    io.want_r = want_r ? 1 : 0;
}

// Synchronises and fills one psv_info per problem; false if a mixed-precision
// problem missed its tolerance.
bool batch_infos(psv_batch& B, hipStream_t s, psv_info* infos) {
    PSV_HIP(hipStreamSynchronize(s));
    if (B.persistent) {
        PSV_HIP(hipMemcpy(B.h_err, B.d_ticket + 1, sizeof(int), hipMemcpyDeviceToHost));
        if (*B.h_err) fail(PSV_ERR_HIP, "persistent batch: a dependency wait exceeded its spin budget");
    }
    bool ok = true;
    for (int p = 0; p < B.n; ++p) {
        Plan& P = *B.plans[p];
        PSV_HIP(hipMemcpy(P.host_scal, P.scal, SCAL_BYTES, hipMemcpyDeviceToHost));
        infos[p].refine_steps = P.host_flags[F_STEPS];
        infos[p].relres = P.host_scal[S_RELRES];
        infos[p].rhs_mean_removed = P.host_scal[S_RHS_MEAN];
        infos[p].rho0_used = P.host_scal[S_RHO0];
        for (int i = 0; i < PSV_RELRES_HISTORY; ++i) infos[p].relres_sweep[i] = NAN;
        if (B.fp32 && !(infos[p].relres <= P.opts.tol)) ok = false;
    }
    return ok;
}

}  // namespace psv
