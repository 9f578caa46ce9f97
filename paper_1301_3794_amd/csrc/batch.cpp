// Batched cavities: one fused FP32 V-cycle for every operator of a batch.
//
// The V-cycles of the members are merged level by level into batched
// launches (kernels.hip, launch_batched): at depth d every member that still
// has a coarser level smooths, forms its residual and restricts; a member
// whose coarsest level is d solves it there; on the way up the members
// prolong and post-smooth.  Each member takes the steps of its own V-cycle
// in their order; only the launches are shared.  Its values do not depend on
// the other members (LDS sweeps and launches round alike), and differ from
// those of its own FP32 V-cycle by rounding: the cut rows are summed in FP64
// here, from centre weights in FP64.  The fused sequence is recorded in one HIP graph,
// for the block size (64, 128 or 256 threads) that the autotuner timed fastest.
//
// dm_batch_eigs runs every member's eigensolve on its own host thread and
// stream; at each FP32 preconditioner call the threads meet, and the last to
// arrive launches the graph once for all of them (ordered after every
// member's input by events, and every member waits for its completion).
#include <algorithm>
#include <chrono>
#include <cstring>

#include "op.h"

namespace dm {

namespace {

struct HostStep {
    int kind, comp;
    std::vector<BJob> jobs;
};

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

struct LevelBufs {
    const float *c;
    float *f, *x, *r;
};

LevelBufs bufs(dm_op *op, int l) {
    Level &L = op->lv[l];
    if (l == 0) return {L.coef32, op->fg_f32, op->fg_x32, L.r32};
    return {L.coef32, L.f32, L.x32, L.r32};
}

int64_t cells(const Grid &g) { return (int64_t)g.nx * g.ny * g.nz; }

// whether member op smooths its level l in LDS when the whole depth does
bool lds_at(dm_op *op, int l) { return lds_level(op->lv[l].g.P, op->lv[l].n_act_faces, sizeof(float), false); }

// the fused V-cycle as a list of batched steps
std::vector<HostStep> schedule(dm_batch *b) {
    std::vector<HostStep> st;
    int dmax = 0;
    for (dm_op *op : b->ops) dmax = std::max(dmax, op->nlev());
    const int nu_pre = b->ops[0]->opt.nu_pre, nu_post = b->ops[0]->opt.nu_post;
    auto add = [&](int kind, int comp, std::vector<BJob> jobs) {
        if (!jobs.empty()) st.push_back({kind, comp, std::move(jobs)});
    };
    auto job = [&](dm_op *op, int l) {
        BJob J{};
        J.g = op->lv[l].g;
        if (l + 1 < op->nlev()) {
            J.gc = op->lv[l + 1].g;
            J.cc = op->lv[l + 1].coef32;
        }
        J.c = op->lv[l].coef32;
        J.sigma = (float)op->sigma;
        return J;
    };
    // the rows of a class update or of the residual
    auto rows = [&](BJob &J, const ClassList &cl) {
        J.cut = cl.idx;
        J.w = cl.w32;
        J.w0 = cl.w64;
        J.s = static_cast<float *>(cl.s);
        J.runs = cl.runs;
        J.cells = cl.cells;
        J.n = cl.n;
        J.nruns = (uint32_t)cl.nruns;
        J.colour = cl.colour;
        J.pair = cl.pair;
        J.items = cl.nruns << kRunLog;
    };
    // the smoothing sweeps of every member with a coarser level than d: one
    // launch of one workgroup per member where all of them fit LDS, else a
    // launch per class (a member that fits joins it at no cost)
    auto smooth = [&](int d, int sweeps, bool reverse) {
        std::vector<dm_op *> at;
        bool lds = true;
        for (dm_op *op : b->ops)
            if (d < op->nlev() - 1) {
                at.push_back(op);
                lds = lds && lds_at(op, d);
            }
        auto jobs_of = [&](auto &&fill) {
            std::vector<BJob> v;
            for (dm_op *op : at) {
                const LevelBufs B = bufs(op, d);
                BJob J = job(op, d);
                J.in = B.f;
                J.out = B.x;
                fill(J, op);
                v.push_back(J);
            }
            return v;
        };
        if (lds) {
            add(BS_SWEEPS, 0, jobs_of([&](BJob &J, dm_op *op) {
                    J.lds = op->lv[d].lds;
                    J.sweeps = sweeps;
                    J.reverse = reverse;
                }));
            return;
        }
        for (int it = 0; it < sweeps; ++it)
            for (int q = 0; q < 6; ++q) {
                const int cls = reverse ? 5 - q : q, comp = cls / 2, col = cls % 2;
                add(BS_SMOOTH, comp, jobs_of([&](BJob &J, dm_op *op) {
                        rows(J, op->lv[d].cut_list(comp, col, q % 2 == 0 ? kPairFirst : kPairSecond, op->cut_s));
                    }));
            }
    };
    for (int d = 0; d < dmax; ++d) {
        std::vector<BJob> zero, coarse, resid, restr;
        for (dm_op *op : b->ops) {
            const int nl = op->nlev();
            if (d >= nl) continue;
            const LevelBufs B = bufs(op, d);
            if (d == 0) {   // coarser iterates are set to zero by the restriction
                BJob z = job(op, d);
                z.out = B.x;
                z.items = 3 * z.g.P;
                zero.push_back(z);
            }
            if (d == nl - 1) {
                BJob c = job(op, d);
                c.in = B.f;
                c.out = B.x;
                c.inv = op->cinv;
                c.idx = op->cidx;
                c.ncoarse = op->nc;
                c.items = op->nc;
                coarse.push_back(c);
                continue;
            }
            // residual, restriction and prolongation visit the grid rows
            // holding an active face: what they write is zero elsewhere
            const Level &C = op->lv[d + 1];
            BJob R = job(op, d);
            R.in = B.f;
            R.aux = B.x;
            R.out = B.r;
            rows(R, op->lv[d].cut_cells_rows());
            resid.push_back(R);
            BJob T = job(op, d);
            T.in = B.r;
            T.out = bufs(op, d + 1).f;
            T.xz = bufs(op, d + 1).x;
            T.rows = C.frows;
            T.nrows = C.nfrows;
            T.items = C.frows ? C.nfrows * T.gc.nx : cells(T.gc);
            restr.push_back(T);
        }
        add(BS_ZERO, 0, zero);
        add(BS_COARSE, 0, coarse);
        smooth(d, nu_pre, false);
        add(BS_RESID, 0, resid);
        add(BS_RESTRICT, 0, restr);
    }
    for (int d = dmax - 2; d >= 0; --d) {
        std::vector<BJob> pro;
        for (dm_op *op : b->ops)
            if (d < op->nlev() - 1) {
                const Level &L = op->lv[d];
                BJob P = job(op, d);
                P.in = bufs(op, d + 1).x;
                P.out = bufs(op, d).x;
                P.rows = L.frows;
                P.nrows = L.nfrows;
                P.items = L.frows ? L.nfrows * P.g.nx : cells(P.g);
                pro.push_back(P);
            }
        add(BS_PROLONG, 0, pro);
        smooth(d, nu_post, true);
    }
    return st;
}

void free_tables(dm_batch *b) {
    for (void *p : b->tables) (void)hipFree(p);
    b->tables.clear();
}

// job tables for block size tpb, then the fused V-cycle recorded into a graph
hipGraphExec_t capture(dm_batch *b, const std::vector<HostStep> &steps, int tpb) {
    struct Launch {
        const BJob *jobs;
        const int32_t *job_of;
        int64_t blocks;
        size_t lds;
    };
    std::vector<Launch> launches;
    auto table = [&](const void *host, size_t bytes) {
        void *dev = nullptr;
        DM_HIP(hipMalloc(&dev, bytes));
        b->tables.push_back(dev);
        DM_HIP(hipMemcpy(dev, host, bytes, hipMemcpyHostToDevice));
        return dev;
    };
    for (const HostStep &h : steps) {
        std::vector<BJob> jobs = h.jobs;
        std::vector<int32_t> job_of;
        size_t lds = 0;
        for (size_t q = 0; q < jobs.size(); ++q) {
            BJob &J = jobs[q];
            J.block0 = (int64_t)job_of.size();
            int64_t blocks = 1;
            if (h.kind == BS_COARSE) {
                blocks = J.items;
            } else if (h.kind == BS_SWEEPS) {
                lds = std::max(lds, (size_t)(3 * J.g.P) * sizeof(float));
            } else {
                // the residual's cut part: a wave per component of 64 cells (apply_cut_part)
                J.ncut = h.kind == BS_RESID ? cdiv(3 * 64 * cdiv(J.n, 64), tpb) : cdiv(J.n, tpb);
                blocks = J.ncut + cdiv(J.items, tpb);
            }
            job_of.resize(job_of.size() + (size_t)blocks, (int32_t)q);
        }
        if (h.kind != BS_SWEEPS)
            while (job_of.size() % 8) job_of.push_back(-1);
        if (job_of.empty()) job_of.assign(8, -1);
        launches.push_back({(const BJob *)table(jobs.data(), jobs.size() * sizeof(BJob)),
                            (const int32_t *)table(job_of.data(), job_of.size() * sizeof(int32_t)),
                            (int64_t)job_of.size(), lds});
    }
    hipGraph_t gph = nullptr;
    hipGraphExec_t exec = nullptr;
    DM_HIP(hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal));
    for (size_t q = 0; q < steps.size(); ++q)
        launch_batched(steps[q].kind, steps[q].comp, launches[q].jobs, launches[q].job_of, launches[q].blocks, tpb,
                       launches[q].lds, b->stream);
    const hipError_t e1 = hipStreamEndCapture(b->stream, &gph);
    if (e1 != hipSuccess) {
        if (gph) (void)hipGraphDestroy(gph);
        DM_HIP(e1);
    }
    const hipError_t e2 = hipGraphInstantiate(&exec, gph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(gph);
    DM_HIP(e2);
    return exec;
}

double time_graph(dm_batch *b, hipGraphExec_t g, int reps) {
    hipEvent_t e0, e1;
    DM_HIP(hipEventCreate(&e0));
    DM_HIP(hipEventCreate(&e1));
    DM_HIP(hipGraphLaunch(g, b->stream));
    DM_HIP(hipEventRecord(e0, b->stream));
    for (int r = 0; r < reps; ++r) DM_HIP(hipGraphLaunch(g, b->stream));
    DM_HIP(hipEventRecord(e1, b->stream));
    DM_HIP(hipEventSynchronize(e1));
    float ms = 0.f;
    DM_HIP(hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return ms / reps;
}

// launch the fused V-cycle for the members that submitted (caller holds mu)
void run_round(dm_batch *b) {
    for (size_t i = 0; i < b->ops.size(); ++i)
        if (b->pending[i]) DM_HIP(hipStreamWaitEvent(b->stream, b->ev_in[i], 0));
    DM_HIP(hipGraphLaunch(b->graph, b->stream));
    DM_HIP(hipEventRecord(b->ev_done, b->stream));
    std::fill(b->pending.begin(), b->pending.end(), 0);
    b->submitted = 0;
    ++b->round;
    b->cv.notify_all();
}

}  // namespace

void batch_setup(dm_batch *b) {
    for (dm_op *op : b->ops) {
        if (op->lv[0].g.pmc) throw DmError{DM_EINVAL, "batched cavities without PMC planes only"};
        if (op->opt.nu_pre != b->ops[0]->opt.nu_pre || op->opt.nu_post != b->ops[0]->opt.nu_post)
            throw DmError{DM_EINVAL, "batch members need the same smoothing counts"};
        ensure_krylov_small(op);   // fg_f32 / fg_x32: the fused V-cycle's level-0 buffers
    }
    DM_HIP(hipDeviceSynchronize());
    if (b->graph) (void)hipGraphExecDestroy(b->graph);
    b->graph = nullptr;
    free_tables(b);
    const std::vector<HostStep> steps = schedule(b);
    b->nsteps = (int)steps.size();
    // autotuner: time the fused V-cycle at 64, 128 and 256 threads per block
    const int cand[3] = {64, 128, 256};
    double best = 1e300;
    int best_tpb = 256;
    for (int q = 0; q < 3; ++q) {
        hipGraphExec_t g = capture(b, steps, cand[q]);
        b->tuned_ms[q] = time_graph(b, g, 5);
        (void)hipGraphExecDestroy(g);
        if (b->tuned_ms[q] < best) {
            best = b->tuned_ms[q];
            best_tpb = cand[q];
        }
        DM_HIP(hipStreamSynchronize(b->stream));
        free_tables(b);
    }
    b->tpb = best_tpb;
    b->graph = capture(b, steps, best_tpb);
    DM_HIP(hipStreamSynchronize(b->stream));
}

void batch_release(dm_batch *b) {
    if (b->stream) (void)hipStreamSynchronize(b->stream);
    if (b->graph) (void)hipGraphExecDestroy(b->graph);
    b->graph = nullptr;
    free_tables(b);
}

void batch_vcycle_lockstep(dm_op *op, hipStream_t s) {
    dm_batch *b = op->batch;
    const int me = op->batch_index;
    DM_HIP(hipEventRecord(b->ev_in[me], s));
    {
        std::unique_lock<std::mutex> lk(b->mu);
        const uint64_t my_round = b->round;
        b->pending[me] = 1;
        ++b->submitted;
        if (b->submitted == b->active) run_round(b);
        else b->cv.wait(lk, [&] { return b->round != my_round; });
    }
    DM_HIP(hipStreamWaitEvent(s, b->ev_done, 0));
}

void batch_leave(dm_batch *b) {
    std::unique_lock<std::mutex> lk(b->mu);
    --b->active;
    if (b->submitted > 0 && b->submitted == b->active) run_round(b);
}

}  // namespace dm
