// batch.cpp -- many runs of uneven size in one launch.
//
// psa_jobs_step_batch advances a set of existing jobs by up to k steps each
// with one launch of the batch kernel: a work list holds one item per
// (job, trial); each workgroup reads its job's arguments from a device table
// and runs the kernel variant that job needs.  Work items are placed so that
// a job's workgroups land on one XCD (workgroups are dispatched to the eight
// XCDs round-robin by index), heaviest jobs first.  psa_anneal_batch wraps it:
// create the jobs, run them to the end, write energies, cuts and spins.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <memory>
#include <numeric>
#include <string>
#include <vector>

#include "engine.hpp"
#include "psa.h"

using psa::set_error;

namespace {

constexpr int kXcds = 8;
constexpr int kChunk = 16;  // work items placed on one XCD together


// Grow-only device buffer kept by the context between batched launches.
psa_status ensure(void **buf, size_t *cap, size_t bytes) {
    if (*cap >= bytes) return PSA_OK;
    if (*buf) (void)hipFree(*buf);
    *buf = nullptr;
    *cap = 0;
    if (hipMalloc(buf, bytes) != hipSuccess) {
        *buf = nullptr;
        set_error("batch: device allocation failed");
        return PSA_ENOMEM;
    }
    *cap = bytes;
    return PSA_OK;
}

}  // namespace

namespace psa {

// Build the XCD-aware work list of a batch: items[j] work items of job j, each
// of modelled time cost[j]; `slots` workgroups run at once on an XCD.  Chunks of
// a job's items go whole to one XCD, costliest first, to the one that then ends
// first: an XCD ends with its longest item as long as its items all run at
// once, past that with its work spread over its slots, if that is later, and
// one item more.  A list that fits the slots leaves no XCD more items than slots,
// a chunk that no XCD can take whole going item by item where there is room
// (12 graphs and a denser one, 256 items for 256 compute units: dealt by work
// alone 5.9 ms, with the second rule alone 4.1, this way 3.4).
void build_work_list(const std::vector<int32_t> &items, const std::vector<double> &cost, int32_t slots,
                     std::vector<int2> *work) {
    struct Chunk {
        int32_t job, q0, q1;
    };
    std::vector<Chunk> chunks;
    for (size_t j = 0; j < items.size(); ++j)
        for (int32_t q = 0; q < items[j]; q += kChunk)
            chunks.push_back(Chunk{static_cast<int32_t>(j), q, std::min(items[j], q + kChunk)});
    std::stable_sort(chunks.begin(), chunks.end(),
                     [&](const Chunk &a, const Chunk &b) { return cost[static_cast<size_t>(a.job)] > cost[static_cast<size_t>(b.job)]; });
    const bool all_run = std::accumulate(items.begin(), items.end(), int64_t{0}) <= int64_t{kXcds} * slots;
    std::vector<std::vector<int2>> queue(kXcds);
    std::vector<double> sum(kXcds, 0.0), longest(kXcds, 0.0);
    for (const Chunk &c : chunks) {
        const double each = cost[static_cast<size_t>(c.job)];
        const int32_t n = c.q1 - c.q0;
        int best = 0;
        double best_end = 0.0;
        for (int x = 0; x < kXcds; ++x) {
            const double most = std::max(longest[x], each);
            const int64_t count = static_cast<int64_t>(queue[x].size()) + n;
            const double end = count <= slots ? most
                                              : std::max(most, (sum[x] + n * each) / slots) + (all_run ? 1e30 : each);
            if (x == 0 || end < best_end || (end == best_end && sum[x] < sum[best])) {
                best = x;
                best_end = end;
            }
        }
        const bool split = all_run && static_cast<int64_t>(queue[best].size()) + n > slots;
        for (int32_t q = c.q0; q < c.q1; ++q) {
            if (split)
                for (int x = 0; x < kXcds; ++x)
                    if (queue[x].size() < queue[best].size()) best = x;
            queue[best].push_back(make_int2(c.job, q));
            sum[best] += each;
            longest[best] = std::max(longest[best], each);
        }
    }
    size_t len = 0;
    for (const auto &qu : queue) len = std::max(len, qu.size());
    work->assign(len * kXcds, make_int2(-1, 0));
    for (int x = 0; x < kXcds; ++x)
        for (size_t s = 0; s < queue[x].size(); ++s) (*work)[s * kXcds + x] = queue[x][s];
}

// Automatic path choice: modelled time of a step (period timing: of a
// sub-step) on either path.  Fitted to 2,610 runs of 300 to 4,500 p-bits of
// degree 6 to 180, +-1 and integer weights, 8 to 2,048 trials, with and without
// gate, SpSA, TApSA (window 4) and periods of 10 (each on both paths): the choice
// takes 0.8 % longer than the better path over all of them, and none longer than
// 1.8 times it.
constexpr double kCsrStepFloorSeconds = 1.5e-6;
constexpr double kDenseStepFloorSeconds = 5.5e-6;    // fp4 couplings: the launch
constexpr double kDenseI8StepFloorSeconds = 7.0e-6;  // int8

double csr_step_seconds(const DevGraph &g, const DevRun &run, const AnnealPlan &plan) {
    const double n = g.n, nnz = static_cast<double>(g.nnz), deg = nnz / std::max(n, 1.0);
    const double wgs = plan.tpw == 4 ? run.t4 / 4 : run.trials;
    const double rounds = wgs * plan.block / (256.0 * 1024.0), whole = std::max(1.0, std::ceil(rounds));
    if (run.t_res > 0 && plan.tpw == 1)  // the class sweep visits the p-bits that fire
        return std::max(kCsrStepFloorSeconds, whole * (0.5e-6 + n / run.t_res * (2.5e-9 + 0.35e-9 * deg)));
    if (plan.ell) {
        // streaming sweeps: lane-operations per update, on the compute units the
        // workgroups reach in whole rounds of them (sums in halves issue half as
        // much again; a sub-step of periods passes by the wavefronts that hold);
        // TApSA windows and SpSA inputs in device memory at about 4 TB/s, 16
        // bytes for the 4 a one-trial workgroup uses, and the latency of window
        // reads where a lane takes several tasks
        double ops = plan.tpw == 4 ? 35.0 + (g.e4_mode == 0 ? 4.0 : 6.0) * deg : 50.0 + 7.0 * deg;
        if (run.t_res > 0) ops *= 0.45;
        const double words = run.ring ? run.alpha : (run.xs ? 2.0 : 0.0);
        const double state = words * (plan.tpw == 4 ? 4.0 : 16.0) / 4.0e12;
        const double share = rounds > 1.0 ? rounds / whole : std::min(1.0, wgs / 256.0);
        const double wait = run.ring && plan.tpw == 1 && g.n4 / 4 > 1024 ? 3.5e-6 * run.alpha * whole : 0.0;
        return std::max(kCsrStepFloorSeconds, n * run.trials * (ops / (kValuOpsPerSecond * share) + state)) + wait;
    }
    // (rows of unit weights: 950 p-bits of degree 45, 284 trials, two rounds 4.4 us, the
    // dense step 5.3; 950 of 29, 520 trials, three rounds 5.0 and 6.8)
    if (plan.csr_lds)
        return std::max(kCsrStepFloorSeconds, whole * (1.0e-6 + nnz * (plan.csr == kCsrUnit ? 0.05e-9 : 0.08e-9)));
    // rows read from device memory by the few lanes of a workgroup: a latency
    // per 1,024 entries
    return whole * nnz / 1024.0 * (plan.csr == kCsrUnit ? 0.4e-6 : 0.23e-6) * (1.0 + std::min(run.trials, 256) / 200.0);
}

double dense_step_seconds(int32_t n, const DevRun &run, bool two_bit, bool one_bit, bool identity) {
    const bool fp4 = two_bit || one_bit;
    const int32_t np = fp4 ? (n + 255) / 256 * 256 : (n + 127) / 128 * 128, t4 = run.t4;
    const int32_t nb = t4 >= 64 ? 4 : (t4 >= 32 ? 2 : 1);
    const double tiles = std::ceil(t4 / (16.0 * nb)), tp = tiles * 16.0 * nb, np2 = static_cast<double>(np) * np;
    const double mfma = 2.0 * np2 * tp / (0.4 * (fp4 ? kMfmaF4OpsPerSecond : kMfmaI8OpsPerSecond));
    const double bytes = np2 * (one_bit ? 0.125 : (two_bit ? 0.25 : 1.0)) * tiles / kHbmBytesPerSecond;
    double t = (fp4 ? kDenseStepFloorSeconds : kDenseI8StepFloorSeconds) + 1.2 * std::max(mfma, bytes) +
               static_cast<double>(n) * t4 * 40.0 / kValuOpsPerSecond;
    // the general epilogue, and its window or input reads: for each (row block,
    // trial block) pair of a wavefront one after the other
    const int32_t most = fp4 ? std::min(nb, 2) : nb;
    const double items = (np + 255) / 256 * std::ceil(t4 / (16.0 * most));
    if (dense_splits(static_cast<int64_t>(items), static_cast<int64_t>(items), fp4)) {
        int32_t k = 1;
        while (k < most && np / 64 * std::ceil(t4 / (16.0 * k)) > 2.0 * kDenseSplitItems) k *= 2;
        t += k * (run.ring ? 0.75e-6 * run.alpha : (run.xs ? 1.3e-6 : 0.0));
    } else if (!identity) {
        const double turns = std::max(1.0, items / (fp4 ? 512.0 : 256.0));
        t += turns * (run.ring ? (fp4 ? 9.0e-6 : 12.5e-6) * run.alpha : (run.xs ? (fp4 ? 11.0e-6 : 18.0e-6) : 4.0e-6));
    }
    return t;
}

bool dense_two_bit(const psa_graph *g) {
    int32_t mag = 0;
    for (int32_t v : g->val_host) {
        const int32_t a = v < 0 ? -v : v;
        if (a == 0) return false;
        if (mag == 0) mag = a;
        if (a != mag) return false;
    }
    return true;
}

bool dense_one_bit(const psa_graph *g) {
    if (g->val_host.empty() || g->val_host[0] == 0) return false;
    return std::all_of(g->val_host.begin(), g->val_host.end(), [&](int32_t v) { return v == g->val_host[0]; });
}

// A graph without its dense matrix pays for it at the first dense run: about 0.11
// ns per entry of it, encoded and uploaded (5,000 p-bits 2.7 ms, where 10 steps of
// 8 trials take 0.2 ms there and 0.7 on the rows).  A run that is over after its
// schedule takes the rows until what such runs on the graph have forgone, each
// its own modelled gain, comes to that cost; a job that its caller keeps may be reset
// and stepped again and has the matrix at once (3 graphs of 800 to 5,000 p-bits, 27
// trials, 53 steps a pass: 0.85 ms with it, 3.0 on the rows).
constexpr double kDenseEncodeSecondsPerEntry = 0.11e-9;

bool prefer_dense(psa_graph *g, const DevRun &run, const AnnealPlan &plan, bool identity, bool once) {
    if (g->info.n < 256) return false;
    const bool two_bit = dense_two_bit(g);
    if (!two_bit && std::any_of(g->val_host.begin(), g->val_host.end(),
                                [](int32_t v) { return v < -127 || v > 127; }))
        return false;
    const double steps = static_cast<double>(run.steps) * std::max(run.t_res, 1);
    const double gain = 0.7 * csr_step_seconds(g->dev, run, plan) -
                        dense_step_seconds(g->info.n, run, two_bit, dense_one_bit(g), identity);
    if (gain <= 0.0) return false;
    if (!once || g->d_dense) return true;
    g->dense_gain += gain * steps;
    return g->dense_gain > kDenseEncodeSecondsPerEntry * g->info.n * static_cast<double>(g->info.n);
}

// Work list of the dense runs `idx` of `table` (one encoding): items (job,
// group of `rows` rows, trial tile) in chunks of up to 16 items -- consecutive row
// groups, each with its trial tiles next to each other -- each chunk given
// whole to the least loaded of the 8 XCDs, heaviest runs first.  Workgroup b
// of a launch runs on XCD b % 8, so slot b takes item b / 8 of that XCD's
// queue (or an empty slot): a chunk's items share their spin tiles in one L2,
// and the trial tiles of a row group read its couplings at about the same
// time there.
static void dense_work_list(const std::vector<DenseJob> &table, const std::vector<int32_t> &idx,
                            int32_t nb, int32_t rows, std::vector<int4> *out) {
    constexpr int32_t kXcd = 8, kChunk = 16;
    std::vector<int32_t> order(idx);
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
        const DenseJob &x = table[a], &y = table[b];
        return static_cast<double>(x.np) * x.np * x.tp > static_cast<double>(y.np) * y.np * y.tp;
    });
    std::vector<std::vector<int4>> bins(kXcd);
    std::vector<double> load(kXcd, 0.0);
    for (int32_t j : order) {
        const DenseJob &d = table[j];
        const int32_t groups = (d.np + rows - 1) / rows, tiles = d.tp / (16 * nb);
        const int32_t span = std::max(1, kChunk / tiles);  // row groups per chunk
        for (int32_t g0 = 0; g0 < groups; g0 += span) {
            const int32_t g1 = std::min(groups, g0 + span);
            const int32_t x = static_cast<int32_t>(std::min_element(load.begin(), load.end()) - load.begin());
            for (int32_t g = g0; g < g1; ++g)
                for (int32_t tt = 0; tt < tiles; ++tt) bins[x].push_back(make_int4(j, g, tt, 0));
            load[x] += static_cast<double>(g1 - g0) * tiles * d.np;
        }
    }
    size_t len = 0;
    for (const auto &b : bins) len = std::max(len, b.size());
    out->assign(len * kXcd, make_int4(-1, 0, 0, 0));
    for (int32_t x = 0; x < kXcd; ++x)
        for (size_t q = 0; q < bins[x].size(); ++q) (*out)[q * kXcd + x] = bins[x][q];
}

// One dense step sequence on stream s, launched step by step: replayed from a
// captured graph of the same shape, captured now (evicting the least recently
// used graph past kDenseGraphCache, after the stream has drained), or --
// use_graph false, or a single step -- launched one by one.  *graph: it ran
// as a graph.
static psa_status dense_sequence(psa_ctx *ctx, hipStream_t s, const DenseJob *table, const int4 *work,
                                 int32_t nwork, int32_t nb, bool split, const DenseJob *one, int32_t enc, int32_t mode,
                                 int32_t steps, bool use_graph, bool *graph) {
    *graph = false;
    if (!use_graph || steps < kDenseGraphMinSteps) {
        PSA_HIP(launch_dense_steps(s, table, work, nwork, nb, split, one, enc, mode, steps), "dense step launch");
        return PSA_OK;
    }
    auto &cache = ctx->dense_graph_cache;
    auto it = std::find_if(cache.begin(), cache.end(), [&](const DenseGraph &d) {
        return d.table == table && d.work == work && d.nwork == nwork && d.nb == nb && d.enc == enc &&
               d.mode == mode && d.steps == steps && d.split == split;
    });
    if (it == cache.end()) {
        PSA_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeRelaxed), "hipStreamBeginCapture");
        const hipError_t le = launch_dense_steps(s, table, work, nwork, nb, split, nullptr, enc, mode, steps);
        hipGraph_t g = nullptr;
        const hipError_t ce = hipStreamEndCapture(s, &g);
        if (le != hipSuccess || ce != hipSuccess) {
            if (g) (void)hipGraphDestroy(g);
            PSA_HIP(le != hipSuccess ? le : ce, "dense step capture");
        }
        hipGraphExec_t exec = nullptr;
        const hipError_t ie = hipGraphInstantiate(&exec, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        PSA_HIP(ie, "hipGraphInstantiate");
        if (cache.size() >= kDenseGraphCache) {
            PSA_HIP(hipStreamSynchronize(s), "hipStreamSynchronize");
            (void)hipGraphExecDestroy(cache.front().exec);
            cache.erase(cache.begin());
        }
        cache.push_back(DenseGraph{table, work, nwork, nb, enc, mode, steps, split, exec});
        it = cache.end() - 1;
    } else {
        std::rotate(it, it + 1, cache.end());  // most recently used last
        it = cache.end() - 1;
    }
    PSA_HIP(hipGraphLaunch(it->exec, s), "hipGraphLaunch");
    *graph = true;
    return PSA_OK;
}

// Task list of the persistent launch: whole runs dealt to kDenseQueues queues
// (heaviest first, each to the least loaded queue), each queue's items run by
// run (256-row group, then trial tile), no empty slots; q->off the queues'
// bounds in the list.
static void dense_task_list(const std::vector<DenseJob> &table, const std::vector<int32_t> &idx, int32_t nb,
                            std::vector<int4> *out, DenseQueues *q) {
    std::vector<int32_t> order(idx);
    auto cost = [&](int32_t j) { return static_cast<double>(table[j].np) * table[j].np * table[j].tp; };
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return cost(a) > cost(b); });
    std::vector<std::vector<int32_t>> queue(kDenseQueues);
    std::vector<double> load(kDenseQueues, 0.0);
    for (int32_t j : order) {
        const int32_t x = static_cast<int32_t>(std::min_element(load.begin(), load.end()) - load.begin());
        queue[x].push_back(j);
        load[x] += cost(j);
    }
    out->clear();
    for (int32_t x = 0; x < kDenseQueues; ++x) {
        q->off[x] = static_cast<int32_t>(out->size());
        for (int32_t j : queue[x]) {
            const DenseJob &d = table[j];
            const int32_t groups = (d.np + 255) / 256, tiles = d.tp / (16 * nb);
            for (int32_t g = 0; g < groups; ++g)
                for (int32_t tt = 0; tt < tiles; ++tt) out->push_back(make_int4(j, g, tt, 0));
        }
    }
    q->off[kDenseQueues] = static_cast<int32_t>(out->size());
}

psa_status dense_step_jobs(psa_ctx *ctx, psa_job *const *jobs, int32_t count, int32_t k, double share) {
    std::vector<psa::DenseJob> table;
    std::vector<psa_job *> live;
    constexpr int kE = kDenseEncodings;
    std::vector<int32_t> by_enc[kE];
    int32_t max_steps = 0, nb[kE] = {4, 4, 4};
    bool plain[kE] = {true, true, true};     // every run of the encoding is plain pSA
    bool identity[kE] = {true, true, true};  // ... with identity factors and no gate
    for (int32_t j = 0; j < count; ++j) {
        psa_job *job = jobs[j];
        const psa_graph *g = job->g;
        const int32_t te = static_cast<int32_t>(std::min<int64_t>(int64_t{job->t} + k, job->run.steps));
        if (te <= job->t) continue;
        psa::DenseJob d;
        d.n = g->info.n;
        d.n4 = g->dev.n4;
        d.np = g->np;
        d.t4 = job->run.t4;
        d.tp = job->tp;
        d.t = job->t;
        d.t_end = te;
        d.scale = g->dense_scale;
        d.items = 0;
        d.J = g->d_dense;
        d.m0 = job->d_m;
        d.m1 = job->d_m + static_cast<size_t>(job->tp) * g->np;
        d.h = g->dev.h;
        d.i0 = job->run.i0;
        d.lam = job->run.lambda;
        d.dlt = job->run.delta;
        d.thr = job->run.thr24;
        d.k0 = job->run.key0;
        d.k1 = job->run.key1;
        d.xs = job->run.xs;
        d.stall24 = job->run.stall24;
        d.ring = job->run.ring;
        d.alpha = job->run.alpha;
        d.t_res = job->run.t_res;
        const int32_t e = g->dense_enc;
        plain[e] = plain[e] && d.xs == nullptr && d.ring == nullptr && d.t_res == 0;
        identity[e] = identity[e] && job->identity_factors;
        by_enc[e].push_back(static_cast<int32_t>(table.size()));
        nb[e] = std::min(nb[e], job->plan.nb);
        table.push_back(d);
        live.push_back(job);
        max_steps = std::max(max_steps, (te - job->t) * std::max(job->run.t_res, 1));
    }
    if (live.empty()) return PSA_OK;
    // fp4 couplings: trial tiles of at most 32 trials.  The two tiles of a
    // 64-trial row group read the same couplings (the second mostly from L2,
    // the work list keeping them together), and twice the items per launch
    // both outnumber the resident workgroup slots, so that items start in
    // waves and their coupling and epilogue phases overlap, and even out the
    // items per compute unit in the vector-bound epilogue (48 runs of n
    // 2,000-4,000 at 64 trials, 1-bit couplings: 25.1-25.5 against 26.8-26.9
    // us per step, the second tile's coupling reads adding 4.5 MB of HBM
    // traffic to 70 MB; 16-trial tiles 30.7 us; 2-bit couplings 32.5 us
    // either way).
    for (int e = 0; e < kE; ++e)
        if (dense_fp4(e)) nb[e] = std::min(nb[e], 2);
    const int32_t how = max_steps >= kDenseGraphMinSteps ? ctx->dense_launch : kDenseLaunchSteps;
    std::vector<int4> work, part;
    size_t off[kE] = {0, 0, 0}, len[kE] = {0, 0, 0};
    bool split[kE] = {false, false, false};
    DenseQueues queues[kE] = {};
    for (int e = 0; e < kE; ++e) {
        if (by_enc[e].empty()) continue;
        if (how == kDenseLaunchPersistent && plain[e])
            dense_task_list(table, by_enc[e], nb[e], &part, &queues[e]);
        else {
            // fewer 256-row items than compute units: 64-row items whose waves
            // split the columns, in the narrowest trial tiles that keep them
            // to two per compute unit (graphs of density 0.06, us per step: 3,000
            // p-bits x 64 trials, 24 items, 10.6 -> 5.0, with 32-trial tiles 6.2;
            // 4,000 x 256, 128 items, 13.2 -> 9.9; 2,000 x 1,024, 256 items, 10.6
            // either way; 4,000 x 1,024, 512 items, 17.1 against 23.5 split: each
            // 64 rows read the trial tile's spins again)
            int64_t items = 0;
            for (int32_t j : by_enc[e]) items += static_cast<int64_t>((table[j].np + 255) / 256) * (table[j].tp / (16 * nb[e]));
            dense_work_list(table, by_enc[e], nb[e], 256, &part);
            split[e] = dense_splits(items, static_cast<int64_t>(part.size()), dense_fp4(e));
            if (split[e]) {
                const int32_t most = nb[e];
                auto fine = [&](int32_t b) {
                    int64_t n64 = 0;
                    for (int32_t j : by_enc[e]) n64 += static_cast<int64_t>(table[j].np / 64) * (table[j].tp / (16 * b));
                    return n64;
                };
                nb[e] = 1;
                while (nb[e] < most && fine(nb[e]) > 2 * kDenseSplitItems) nb[e] *= 2;
                dense_work_list(table, by_enc[e], nb[e], 64, &part);
            }
        }
        off[e] = work.size();
        len[e] = part.size();
        work.insert(work.end(), part.begin(), part.end());
    }
    for (const int4 &w : work)
        if (w.x >= 0) ++table[static_cast<size_t>(w.x)].items;
    PSA_HIP(hipStreamSynchronize(ctx->stream2), "hipStreamSynchronize");
    if (ctx->h_dense_err && (ctx->h_dense_err[0] | ctx->h_dense_err[1] | ctx->h_dense_err[2])) {
        ctx->h_dense_err[0] = ctx->h_dense_err[1] = ctx->h_dense_err[2] = 0u;
        set_error("dense step sequence: a workgroup waited past its limit for another work item of its run; "
                  "the spins of that quantum are not valid");
        return PSA_EHIP;
    }
    psa_status st;
    if ((st = ensure(&ctx->d_dense_table, &ctx->dense_table_cap, table.size() * sizeof(psa::DenseJob))) != PSA_OK)
        return st;
    if ((st = ensure(&ctx->d_dense_work, &ctx->dense_work_cap, work.size() * sizeof(int4))) != PSA_OK)
        return st;
    const int32_t sync_words = dense_sync_words(static_cast<int32_t>(table.size()));
    if (how == kDenseLaunchPersistent) {
        void *p = ctx->d_dense_sync;
        if ((st = ensure(&p, &ctx->dense_sync_cap, kE * static_cast<size_t>(sync_words) * sizeof(uint32_t))) !=
            PSA_OK)
            return st;
        ctx->d_dense_sync = static_cast<uint32_t *>(p);
        if (!ctx->h_dense_err) {
            void *h = nullptr;
            PSA_HIP(hipHostMalloc(&h, kE * sizeof(uint32_t), hipHostMallocDefault), "hipHostMalloc");
            ctx->h_dense_err = static_cast<uint32_t *>(h);
            ctx->h_dense_err[0] = ctx->h_dense_err[1] = ctx->h_dense_err[2] = 0u;
        }
    }
    ctx->h_dense_table = table;
    ctx->h_dense_work = work;
    for (psa_job *job : live)
        for (int half = 0; half < 2; ++half)  // both buffers: a fully defined state
            PSA_HIP(psa::launch_to_dense(ctx->stream2, job->g->dense_enc, job->g->info.n, job->run.t4, job->g->np,
                                         job->tp, job->d_spins,
                                         job->d_m + static_cast<size_t>(half) * job->tp * job->g->np),
                    "dense layout");
    PSA_HIP(hipMemcpyAsync(ctx->d_dense_table, ctx->h_dense_table.data(),
                           table.size() * sizeof(psa::DenseJob), hipMemcpyHostToDevice, ctx->stream2),
            "dense table upload");
    PSA_HIP(hipMemcpyAsync(ctx->d_dense_work, ctx->h_dense_work.data(), work.size() * sizeof(int4),
                           hipMemcpyHostToDevice, ctx->stream2),
            "dense work upload");
    const int4 *dwork = static_cast<const int4 *>(ctx->d_dense_work);
    const psa::DenseJob *dtable = static_cast<const psa::DenseJob *>(ctx->d_dense_table);
    hipEvent_t ev = nullptr;
    if ((st = time_begin(ctx, ctx->stream2, &ev)) != PSA_OK) return st;
    int64_t launches = 0, replayed = 0;
    // launched step by step, the sequences of a second (and third) encoding
    // run on the third stream beside the first encoding's: a few runs of one
    // encoding take latency-bound steps that would otherwise follow the
    // other encoding's whole sequence (in a mix of 256 graphs, 24 runs of
    // 2-bit couplings took 15 ms per 1,000 steps alone, 127 runs of 1-bit
    // ones 62-64 ms, and the two 72.7 ms side by side)
    int32_t present = 0;
    for (int e = 0; e < kE; ++e) present += len[e] > 0 ? 1 : 0;
    const bool side = how == kDenseLaunchSteps && present > 1;
    if (side) {
        PSA_HIP(hipEventRecord(ctx->ev_fork3, ctx->stream2), "hipEventRecord");
        PSA_HIP(hipStreamWaitEvent(ctx->stream3, ctx->ev_fork3, 0), "hipStreamWaitEvent");
    }
    bool first = true;
    for (int e = 0; e < kE; ++e) {
        if (len[e] == 0) continue;
        const int32_t enc = e;
        const int32_t mode = plain[e] ? (identity[e] ? 2 : 1) : 0;
        if (how == kDenseLaunchPersistent && mode != 0) {
            uint32_t *sync = ctx->d_dense_sync + static_cast<size_t>(e) * sync_words;
            const int32_t cus = std::clamp(static_cast<int32_t>(std::lround(share * ctx->num_cu)), kDenseQueues,
                                           ctx->num_cu);
            PSA_HIP(psa::launch_dense_persistent(ctx->stream2, dtable, dwork + off[e], queues[e], nb[e], enc, mode,
                                                 max_steps, sync, sync_words, ctx->dense_max_polls, cus),
                    "dense step sequence launch");
            PSA_HIP(hipMemcpyAsync(ctx->h_dense_err + e, sync + 32 * kDenseQueues, sizeof(uint32_t),
                                   hipMemcpyDeviceToHost, ctx->stream2),
                    "dense step error flag");
            launches += 1;
            continue;
        }
        bool graph = false;
        hipStream_t s = side && !first ? ctx->stream3 : ctx->stream2;
        first = false;
        if ((st = dense_sequence(ctx, s, dtable, dwork + off[e], static_cast<int32_t>(len[e]), nb[e], split[e],
                                 split[e] && by_enc[e].size() == 1 ? &table[static_cast<size_t>(by_enc[e][0])] : nullptr, enc, mode,
                                 max_steps, how == kDenseLaunchGraph, &graph)) != PSA_OK)
            return st;
        launches += max_steps;
        replayed += graph ? max_steps : 0;
    }
    if (side) {
        PSA_HIP(hipEventRecord(ctx->ev_join3, ctx->stream3), "hipEventRecord");
        PSA_HIP(hipStreamWaitEvent(ctx->stream2, ctx->ev_join3, 0), "hipStreamWaitEvent");
    }
    if (ev) ctx->timed_graph_launches += replayed;
    if ((st = time_end(ctx, ctx->stream2, kTimeDense, ev, launches)) != PSA_OK) return st;
    for (size_t j = 0; j < live.size(); ++j) {
        psa_job *job = live[j];
        const psa::DenseJob &d = table[j];
        const int8_t *fin = (((d.t_end - d.t) * std::max(d.t_res, 1)) & 1) ? d.m1 : d.m0;
        PSA_HIP(psa::launch_from_dense(ctx->stream2, job->g->dense_enc, job->g->info.n, job->run.t4, job->g->np, fin,
                                       job->d_spins),
                "dense layout");
        job->t = d.t_end;
    }
    return PSA_OK;
}

}  // namespace psa

namespace psa {

// Modelled step (all its sub-steps) of one workgroup of a batch, fitted to runs
// alone: its time with the compute unit to itself (a chain of latencies for small
// runs), and the compute unit's time it takes in issue and in about 4 TB/s of
// TApSA windows and SpSA inputs.  us, modelled and measured alone: 2,000 p-bits of
// degree 6, four trials 4.1 and 4.2, of 60 11.8 and 11.7; 4,500 of 6, one trial 3.9
// and 4.0; TApSA 800 of 24, four trials 8.8 and 8.8.
BatchItemTime batch_item_time(const DevGraph &g, const DevRun &run, const AnnealPlan &plan) {
    const double n = g.n, nnz = static_cast<double>(g.nnz), deg = nnz / std::max(n, 1.0);
    constexpr double kUnitOps = kValuOpsPerSecond / 256.0, kUnitBytes = 4.0e12 / 256.0;
    // (one trial's inputs of up to 2,048 p-bits stay in L2)
    const double words = run.ring ? run.alpha : (run.xs ? (plan.tpw == 4 ? 0.5 : (n <= 2048.0 ? 0.25 : 1.3)) : 0.0);
    double alone, unit;
    if (plan.tpw == 4) {
        unit = 3.6 * n * (38.0 + 3.2 * deg) / kUnitOps;
        alone = std::max(2.4e-6 + 0.1e-6 * deg + n * (0.4e-9 + 0.022e-9 * deg), unit) + (run.xs ? 1.2e-6 : 0.0);
    } else if (plan.ell) {
        unit = n * (50.0 + 7.0 * deg) / kUnitOps;
        alone = 1.2e-6 + unit;
    } else {
        unit = n * (130.0 + 5.0 * deg) / kUnitOps;
        alone = (plan.csr_lds ? 1.0e-6 + nnz * 0.08e-9 : nnz / 1024.0 * (plan.csr == kCsrUnit ? 0.8e-6 : 0.46e-6)) *
                (run.ring ? 1.15 : (run.xs ? 1.1 : 1.0));
    }
    if (plan.tpw == 4 || plan.ell) {  // (resident lanes keep their state)
        unit += 16.0 * words * n / kUnitBytes;
        alone += 16.0 * words * n / kUnitBytes;
    }
    // wavefronts none of whose p-bits fire pass a sub-step by
    const double subs = run.t_res > 0 ? run.t_res * (plan.tpw == 4 ? 0.5 : 0.65) : 1.0;
    return BatchItemTime{alone * subs, unit * subs};
}

// Which runs of a batch take four trials per workgroup (those whose trials per
// workgroup are the library's choice and whose rows the four-trial streaming
// sweep reads).  A four-trial workgroup walks its rows once for the four and
// issues fewer instructions per update, but takes two to five times as long per
// step.  The batch ends with its longest workgroup, its workgroups' times over
// the slots they have, or the compute units' time over the units, whichever is
// latest (where workgroups share a unit, plus the longest one's, which may meet
// another); a slot is a launch's share of a unit, by the largest workgroup and LDS
// of all its runs, so a single one-trial run of wide lanes may halve the slots of
// every other.  Starting with four for every run, the run with the longest
// workgroup goes back to one again and again; the earliest end of these, and of one
// for every run, wins.
// Measured, all one and all four, us per step: 12 graphs of degree 4-8 and 2,069 to
// 4,044 p-bits, 64 trials 9.1 and 6.3, 32 6.3 and 6.3, 16 3.5 and 6.3; 16 requests
// of 4,951 to 19,606 p-bits, degree 4 to 50, 131 and 75; 20 graphs of 60 to 500 p-bits,
// degree 4-8, 100 to 500 trials 15.1 and 8.7 (19 of them four: 13.0); 40 such, TApSA, 8
// to 64 trials 4.5 and 8.8; six of 3,000 of degree 6, 8 trials 3.0 and 5.6.
std::vector<char> choose_four_trials(const psa_ctx *ctx, psa_job *const *jobs, const std::vector<int32_t> &idx,
                                     const std::vector<int32_t> &t_end) {
    struct Form {
        BatchItemTime t{0.0, 0.0};
        int64_t items = 0;
        int32_t lanes = 0;
        size_t lds = 0;
    };
    const size_t count = idx.size();
    std::vector<char> four(count, 0), fixed(count, 1);
    std::vector<std::array<Form, 2>> forms(count);  // one and four trials
    for (size_t x = 0; x < count; ++x) {
        const psa_job *job = jobs[idx[x]];
        const DevGraph &g = job->g->dev;
        const double steps = t_end[static_cast<size_t>(idx[x])] - job->t;
        bool have[2], ell4 = false;
        for (int f = 0; f < 2; ++f) {
            AnnealPlan p;
            int32_t variant = 0;
            have[f] = plan_batch_item(g, job->run, f ? 4 : 1, !f && job->plan.tpw == 1 ? job->plan.lpt : 0, ctx->max_lds, &p, &variant, nullptr);
            if (!have[f]) continue;
            const BatchItemTime t = batch_item_time(g, job->run, p);
            forms[x][f] = Form{{t.alone * steps, t.unit * steps}, f ? job->run.t4 / 4 : job->run.trials, g.n4 / 4 * p.lpt, p.lds_bytes};
            if (f) ell4 = p.ell != 0;
        }
        fixed[x] = !(job->auto_tpw && job->plan.tpw == 1 && job->run.pps && have[0] && have[1] && ell4);
        four[x] = fixed[x] ? job->plan.tpw == 4 : 1;
    }
    // modelled end, and the run with the longest workgroup
    auto end_of = [&](const std::vector<char> &form, size_t *at) {
        size_t lds = 1;
        double longest = 0.0, shortest = 1e30, alone = 0.0, unit = 0.0, most_unit = 0.0;
        int64_t items = 0;
        int32_t lanes = 0;
        *at = count;
        for (size_t x = 0; x < count; ++x) {
            const Form &f = forms[x][form[x] ? 1 : 0];
            if (f.t.alone > longest) {
                longest = f.t.alone;
                *at = x;
            }
            shortest = std::min(shortest, f.t.alone);
            most_unit = std::max(most_unit, f.t.unit);
            alone += f.t.alone * f.items;
            unit += f.t.unit * f.items;
            items += f.items;
            lanes = std::max(lanes, f.lanes);
            lds = std::max(lds, f.lds);
        }
        const int64_t per_unit = std::min<int64_t>(1024 / batch_block(lanes), std::max<int64_t>(1, ctx->max_lds / lds));
        const double slots = static_cast<double>(ctx->num_cu * per_unit);
        return std::max({longest, alone / slots, unit / ctx->num_cu}) + (items > slots ? 0.5 * shortest : 0.0) +
               (per_unit > 1 && items > ctx->num_cu ? most_unit : 0.0);
    };
    constexpr double kMixed = 1.15;  // a mixture has to be clearly earlier: its lanes and LDS are the larger of both forms'
    size_t at = count;
    std::vector<char> best = four, ones = four;
    double best_end = end_of(four, &at);
    for (size_t x = 0; x < count; ++x) ones[x] = fixed[x] ? four[x] : 0;
    size_t unused = 0;
    const double ones_end = end_of(ones, &unused);
    if (ones_end < best_end) {
        best = ones;
        best_end = ones_end;
    }
    while (at < count && four[at] && !fixed[at]) {
        four[at] = 0;
        const double end = kMixed * end_of(four, &at);
        if (end < best_end) {
            best = four;
            best_end = end;
        }
    }
    return best;
}

}  // namespace psa

extern "C" {

psa_status psa_jobs_step_batch(psa_ctx *ctx, int32_t count, psa_job *const *jobs, int32_t k) {
    return psa::guarded("psa_jobs_step_batch", [&]() -> psa_status {
        if (!ctx || count < 0 || (count > 0 && !jobs) || k < 0) {
            set_error("psa_jobs_step_batch: invalid arguments");
            return PSA_EINVAL;
        }
        std::vector<psa::BatchJob> table;
        std::vector<int32_t> trials;
        std::vector<double> cost;
        std::vector<int32_t> t_end;
        std::vector<psa_job *> dense_jobs;
        size_t lds = 0;
        int32_t max_lanes = 0;
        std::vector<int32_t> sweep_jobs;  // indices of the runs on the CSR path
        double dense_s = 0.0, csr_s = 0.0;  // model estimates of the two families' device time
        for (int32_t j = 0; j < count; ++j) {
            psa_job *job = jobs[j];
            if (!job || job->ctx != ctx) {
                set_error("psa_jobs_step_batch: job " + std::to_string(j) + " is NULL or belongs to "
                          "another context");
                return PSA_EINVAL;
            }
            for (int32_t i = 0; i < j; ++i)
                if (jobs[i] == job) {
                    set_error("psa_jobs_step_batch: job listed twice");
                    return PSA_EINVAL;
                }
            const int32_t te = static_cast<int32_t>(
                std::min<int64_t>(int64_t{job->t} + k, job->run.steps));
            t_end.push_back(te);
            if (te <= job->t) continue;
            if (job->plan.dense) {
                dense_jobs.push_back(job);
                dense_s += psa::dense_step_seconds(job->g->info.n, job->run, job->g->dense_enc == psa::kDenseT2,
                                                   job->g->dense_enc == psa::kDenseB1, job->identity_factors) *
                           (te - job->t);
                continue;
            }
            sweep_jobs.push_back(j);
        }
        std::vector<char> four = psa::choose_four_trials(ctx, jobs, sweep_jobs, t_end);
        for (size_t x = 0; x < sweep_jobs.size(); ++x) {
            const int32_t j = sweep_jobs[x];
            psa_job *job = jobs[j];
            const int32_t te = t_end[static_cast<size_t>(j)];
            psa::AnnealPlan plan;
            int32_t variant = 0;
            std::string why;
            const int32_t tpw = four[x] ? 4 : job->plan.tpw;
            if (!psa::plan_batch_item(job->g->dev, job->run, tpw, tpw == 1 ? job->plan.lpt : 0, ctx->max_lds, &plan,
                                      &variant, &why)) {
                set_error("psa_jobs_step_batch: " + why);
                return PSA_EUNSUPPORTED;
            }
            csr_s += psa::csr_step_seconds(job->g->dev, job->run, plan) * (te - job->t);
            psa::BatchJob bj;
            psa::fill_anneal_args(&bj.a, job->g->dev, job->run, job->d_order, job->t, te);
            bj.variant = variant;
            table.push_back(bj);
            trials.push_back(plan.tpw == 4 ? job->run.t4 / 4 : job->run.trials);  // work items
            cost.push_back(psa::batch_item_time(job->g->dev, job->run, plan).alone * (te - job->t));
            lds = std::max(lds, plan.lds_bytes);
            max_lanes = std::max(max_lanes, job->g->dev.n4 / 4 * plan.lpt);
        }
        PSA_HIP(hipSetDevice(ctx->device), "hipSetDevice");
        if (!dense_jobs.empty()) {
            // dense runs on the second stream, concurrently with the CSR launch
            PSA_HIP(hipEventRecord(ctx->ev_fork, ctx->stream), "hipEventRecord");
            PSA_HIP(hipStreamWaitEvent(ctx->stream2, ctx->ev_fork, 0), "hipStreamWaitEvent");
            // a persistent dense launch keeps its workgroups resident: it gets
            // the dense family's modelled share of the device
            const double share = csr_s > 0.0 ? dense_s / (dense_s + csr_s) : 1.0;
            psa_status st = psa::dense_step_jobs(ctx, dense_jobs.data(),
                                                 static_cast<int32_t>(dense_jobs.size()), k, share);
            if (st != PSA_OK) return st;
            PSA_HIP(hipEventRecord(ctx->ev_join, ctx->stream2), "hipEventRecord");
        }
        if (table.empty()) {
            if (!dense_jobs.empty())
                PSA_HIP(hipStreamWaitEvent(ctx->stream, ctx->ev_join, 0), "hipStreamWaitEvent");
            return PSA_OK;
        }
        const int32_t block = psa::batch_block(max_lanes);
        std::vector<int2> work;
        psa::build_work_list(trials, cost, psa::batch_slots(std::accumulate(trials.begin(), trials.end(), int64_t{0}), ctx->num_cu, block), &work);
        // the staging buffers are reused: the previous batched launch must be done
        PSA_HIP(hipStreamSynchronize(ctx->stream), "hipStreamSynchronize");
        psa_status st;
        if ((st = ensure(&ctx->d_batch_table, &ctx->batch_table_cap,
                         table.size() * sizeof(psa::BatchJob))) != PSA_OK)
            return st;
        if ((st = ensure(&ctx->d_batch_work, &ctx->batch_work_cap, work.size() * sizeof(int2))) != PSA_OK)
            return st;
        ctx->h_batch_table = table;
        ctx->h_batch_work = work;
        PSA_HIP(hipMemcpyAsync(ctx->d_batch_table, ctx->h_batch_table.data(),
                               table.size() * sizeof(psa::BatchJob), hipMemcpyHostToDevice, ctx->stream),
                "batch table upload");
        PSA_HIP(hipMemcpyAsync(ctx->d_batch_work, ctx->h_batch_work.data(), work.size() * sizeof(int2),
                               hipMemcpyHostToDevice, ctx->stream),
                "batch work upload");
        hipEvent_t ev = nullptr;
        if ((st = psa::time_begin(ctx, ctx->stream, &ev)) != PSA_OK) return st;
        PSA_HIP(psa::launch_anneal_batch(ctx->stream, static_cast<const psa::BatchJob *>(ctx->d_batch_table),
                                         static_cast<const int2 *>(ctx->d_batch_work),
                                         static_cast<int32_t>(work.size()), block, lds),
                "batch anneal launch");
        if ((st = psa::time_end(ctx, ctx->stream, psa::kTimeBatch, ev, 1)) != PSA_OK) return st;
        for (int32_t j = 0; j < count; ++j) jobs[j]->t = std::max(jobs[j]->t, t_end[j]);
        if (!dense_jobs.empty())
            PSA_HIP(hipStreamWaitEvent(ctx->stream, ctx->ev_join, 0), "hipStreamWaitEvent");
        return PSA_OK;
    });
}

psa_status psa_anneal_batch(psa_ctx *ctx, int32_t count, const psa_batch_item *items,
                            uint32_t flags) {
    return psa::guarded("psa_anneal_batch", [&]() -> psa_status {
        if (!ctx || count < 0 || (count > 0 && !items) ||
            (flags & ~(PSA_OUT_DEVICE | PSA_BATCH_SEQUENTIAL)) != 0) {
            set_error("psa_anneal_batch: invalid arguments");
            return PSA_EINVAL;
        }
        for (int32_t j = 0; j < count; ++j)
            if (!items[j].graph || !items[j].energy_out || !items[j].cut_out) {
                set_error("psa_anneal_batch: item " + std::to_string(j) +
                          " needs a graph, energy_out and cut_out");
                return PSA_EINVAL;
            }
        std::vector<std::unique_ptr<psa_job, void (*)(psa_job *)>> owned;
        std::vector<psa_job *> jobs;
        int32_t max_steps = 0;
        for (int32_t j = 0; j < count; ++j) {
            psa_run_desc d = items[j].desc;
            if (!(flags & PSA_BATCH_SEQUENTIAL)) {
                if (d.flags & PSA_TUNE) {
                    psa_status st = psa::tuned_desc(ctx, items[j].graph, &d, PSA_TUNE_BATCH);
                    if (st != PSA_OK) {
                        set_error("psa_anneal_batch: item " + std::to_string(j) + ": " + psa_last_error());
                        return st;
                    }
                }
            }
            psa_job *job = nullptr;
            psa_status st = (flags & PSA_BATCH_SEQUENTIAL) ? psa_job_create(ctx, items[j].graph, &d, &job)
                                                           : psa::create_batch_job(ctx, items[j].graph, &d, &job);
            if (st != PSA_OK) {
                set_error("psa_anneal_batch: item " + std::to_string(j) + ": " + psa_last_error());
                return st;
            }
            owned.emplace_back(job, psa_job_destroy);
            jobs.push_back(job);
            max_steps = std::max(max_steps, d.steps);
        }
        psa_status st;
        if (flags & PSA_BATCH_SEQUENTIAL) {
            for (psa_job *job : jobs)
                if ((st = psa_job_step(job, job->run.steps)) != PSA_OK) return st;
        } else {
            if ((st = psa_jobs_step_batch(ctx, count, jobs.data(), max_steps)) != PSA_OK) return st;
        }
        const uint32_t out = flags & PSA_OUT_DEVICE;
        if (!(flags & PSA_BATCH_SEQUENTIAL)) {
            // the batch's read-outs in two launches
            std::vector<int64_t *> energy(static_cast<size_t>(count)), cut(static_cast<size_t>(count));
            for (int32_t j = 0; j < count; ++j) {
                energy[static_cast<size_t>(j)] = items[j].energy_out;
                cut[static_cast<size_t>(j)] = items[j].cut_out;
            }
            if ((st = psa_jobs_energy_cut(ctx, count, jobs.data(), energy.data(), cut.data(), out)) != PSA_OK)
                return st;
        }
        for (int32_t j = 0; j < count; ++j) {
            if ((flags & PSA_BATCH_SEQUENTIAL) &&
                (st = psa_job_energy_cut(jobs[j], items[j].energy_out, items[j].cut_out, out)) != PSA_OK)
                return st;
            if (items[j].spins_out &&
                (st = psa_job_read_spins(jobs[j], items[j].spins_out, out)) != PSA_OK)
                return st;
        }
        PSA_HIP(hipStreamSynchronize(ctx->stream), "hipStreamSynchronize");
        return PSA_OK;
    });
}

}  // extern "C"
