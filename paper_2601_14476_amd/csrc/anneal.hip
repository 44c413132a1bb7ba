// anneal.hip -- launches of the persistent sweep of one run, and its planning
// (the kernel body is in sweep.hpp, the streaming sweeps' in ell_sweep.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <numeric>

#include "engine.hpp"
#include "sweep.hpp"

namespace psa {
namespace {

// At most 128 registers (four wavefronts per SIMD) for the smaller blocks too:
// with a few more, a compute unit holds three workgroups of 256 or one of 512
// fewer, and runs of more trials than units take another round (289 p-bits of
// degree 27, 837 trials 4.1 us per step with 131 registers).
template <int TPW, int LPT, int CSR, bool CSR_LDS, int BLOCK, bool ALONE>
__global__ __launch_bounds__(BLOCK, 4) void anneal_kernel(AnnealArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    anneal_body<TPW, LPT, CSR, CSR_LDS, BLOCK, ALONE>(a, static_cast<int32_t>(blockIdx.x), smem);
}

template <int TPW, int LPT, int CSR, bool LDS, int BLOCK>
hipError_t launch_variant(hipStream_t stream, const AnnealArgs &args, const AnnealPlan &plan) {
    auto kern = anneal_kernel<TPW, LPT, CSR, LDS, BLOCK, false>;
    if constexpr (LPT == 4) {
        if (plan.alone) kern = anneal_kernel<TPW, LPT, CSR, LDS, BLOCK, true>;
    }
    hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                         hipFuncAttributeMaxDynamicSharedMemorySize,
                                         static_cast<int>(plan.lds_bytes));
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(plan.grid), dim3(BLOCK), plan.lds_bytes, stream, args);
    return hipGetLastError();
}

template <int TPW, int LPT, int CSR, bool LDS>
hipError_t launch_block(hipStream_t stream, const AnnealArgs &args, const AnnealPlan &plan) {
    switch (plan.block) {
        case 256: return launch_variant<TPW, LPT, CSR, LDS, 256>(stream, args, plan);
        case 512: return launch_variant<TPW, LPT, CSR, LDS, 512>(stream, args, plan);
        case 1024: return launch_variant<TPW, LPT, CSR, LDS, 1024>(stream, args, plan);
        default: return hipErrorInvalidValue;
    }
}

template <int TPW, int LPT, int CSR>
hipError_t launch_lds(hipStream_t stream, const AnnealArgs &args, const AnnealPlan &plan) {
    return plan.csr_lds ? launch_block<TPW, LPT, CSR, true>(stream, args, plan)
                        : launch_block<TPW, LPT, CSR, false>(stream, args, plan);
}

template <int LPT>
hipError_t launch_one_trial(hipStream_t stream, const AnnealArgs &args, const AnnealPlan &plan) {
    switch (plan.csr) {
        case kCsrPair: return launch_lds<1, LPT, kCsrPair>(stream, args, plan);
        case kCsrPack32: return launch_lds<1, LPT, kCsrPack32>(stream, args, plan);
        case kCsrUnit: return launch_lds<1, LPT, kCsrUnit>(stream, args, plan);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_four_trials(hipStream_t stream, const AnnealArgs &args, const AnnealPlan &plan) {
    switch (plan.csr) {
        case kCsrPair: return launch_lds<4, 1, kCsrPair>(stream, args, plan);
        case kCsrPack32: return launch_lds<4, 1, kCsrPack32>(stream, args, plan);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

// Rounds of one-trial workgroups up to which a run on a graph with ELL rows
// keeps them: about the ratio of a four-trial step to one round (us per step, one
// and four trials per workgroup).
//   streaming sweep: 2 (4,000 p-bits of degree 6, 512 trials 5.8 and 6.0, 600 8.1
//     and 5.9), and so resident lanes whose rows are weighted or outgrow their
//     cached slots (64 for one row, most of them; 32 for two) (1,000 of degree 6,
//     weights, 1,000 trials 5.9 and 3.7; 2,000 of 24, 520 trials 14.3 and 6.3; 950 of 63,
//     520 trials 9.6 and 8.2, but 800 of 47, up to 70, 5.9 and 7.0);
//   resident lanes with cached rows: 3 (600 of degree 6, 760 trials 3.1 and 3.4,
//     780 4.1 and 3.4; SpSA 1,500 of degree 6, 760 trials 4.1 and 4.7), but 2 where
//     two rows fill more than 800 lanes (2,000 of degree 6, 760 trials 4.1 and 3.7;
//     1,200 of degree 6 3.3 and 3.5); TApSA 4, the
//     window in LDS against 16 bytes per p-bit from memory (1,500 of degree 6, 1,000
//     trials 5.6 and 8.1; 600 of degree 6, 1,000 4.7 and 6.0);
//   period classes, which visit only the p-bits that fire: by the entries, and longer
//     with weights, whose four-trial sums take more instructions.  One row per lane: 4
//     to 10,000 entries (800 of degree 12, sub-steps of 10, 760 trials 15.7 and 21.3,
//     1,000 20.6 and 21.3), with weights to 30,000 (500 of degree 48, 1,000 trials 45
//     and 52), 3 to 30,000 (300 of degree 72, 760 trials 39 and 43, 780 51 and 43), else
//     2 (1,000 of degree 40, 520 trials 51 and 39).  Two rows: 3 to 25,000 (1,200 of
//     degree 12, 760 trials 23.4 and 24.5; 1,100 of 24 32.3 and 30.4), with weights to
//     40,000 (1,500 of 24, 760 trials 37.1 and 38.8), else 2.
static int64_t one_trial_rounds(const DevGraph &g, const DevRun &run, const AnnealPlan &one) {
    const int64_t n = g.n;
    if (run.t_res > 0) {
        const bool unit = one.csr == kCsrUnit;
        if (one.lpt == 4) return g.nnz <= (unit ? 10000 : 30000) ? 4 : (g.nnz <= 30000 ? 3 : 2);
        return one.lpt == 2 && g.nnz <= (unit ? 25000 : 40000) ? 3 : 2;
    }
    if (one.ell || one.csr != kCsrUnit || !one.csr_lds || one.lpt == 1) return 2;
    if (one.lpt == 4 ? g.nnz > 56 * n : (g.nnz > 8 * n || g.max_degree > 32)) return 2;
    return run.ring ? 4 : (run.xs || one.lpt == 4 || n <= 1600 ? 3 : 2);
}

// Lanes per task of a one-trial run that leaves them open: as many as the
// workgroup has.  But two rows a lane of a weighted graph lie in LDS one behind the
// other, and rows of one length put a wavefront's lanes on few banks (47 x 38
// torus, weights, 140 trials: 2.5 us per step, streamed rows 1.4; random rows 2,000
// of degree 6 2.4 and 1.9, SpSA 2.6 and 2.3, 1,100 of degree 6 2.0 and 1.9, SpSA 2.2
// and 2.3, of 24 4.3 and 3.6; 1,500 of 60, past LDS, 30 and 6.0): these stream, pSA
// always, SpSA but for few short rows of up to a trial per unit.  TApSA keeps its
// sums in the lanes (1,100 of degree 6 2.2 and 3.2).
static int32_t lanes_per_task(const DevGraph &g, const DevRun &run, size_t max_lds, int32_t num_cu) {
    const int32_t tasks = g.n4 / 4;
    const int32_t spread = tasks * 4 <= 1024 ? 4 : (tasks * 2 <= 1024 ? 2 : 1);
    const bool streams = spread == 2 && !g.ux16 && g.e1 && !run.ring && run.t_res == 0 && 2 * ell1_stride(g.n4) <= max_lds &&
                         (!run.xs || g.n >= 1300 || g.max_degree <= 8 || g.nnz >= 10 * static_cast<int64_t>(g.n) || run.trials > num_cu);
    return streams ? 1 : spread;
}

bool plan_anneal(const DevGraph &g, const DevRun &run, int32_t tpw_req, int32_t lpt_req,
                 int32_t block_req, size_t max_lds, int32_t num_cu, AnnealPlan *plan,
                 std::string *why) {
    AnnealPlan p;
    const int32_t n4 = g.n4;
    const int32_t tasks = n4 / 4;
    const bool ell_ok = g.e1 != nullptr;
    if (tpw_req == 1 || tpw_req == 4) {
        p.tpw = tpw_req;
    } else {
        // One trial per workgroup exposes four times the workgroups; four
        // share each walk of the rows and issue fewer instructions.  Four pay
        // once the one-trial workgroups take too many rounds of the compute
        // units (one_trial_rounds; a unit runs 1,024 of their threads at once,
        // and one workgroup of the period-class sweep).
        AnnealPlan one;
        const int32_t spread = lanes_per_task(g, run, max_lds, num_cu);
        if (ell_ok && g.e4_mode >= 0 && plan_anneal(g, run, 1, lpt_req ? lpt_req : spread, block_req, max_lds, num_cu, &one, nullptr)) {
            // (streams of up to 2,048 p-bits: two workgroups of 512 threads on a unit
            // get in each other's way: 2,000 of degree 6, 400 trials 3.0 and 4.0 us per
            // step, 760 4.5 and 4.1)
            const int64_t threads = run.t_res > 0 || (lpt_req == 0 && one.ell && g.n <= 2048) ? 1024 : one.block;
            p.tpw = run.trials * threads > one_trial_rounds(g, run, one) * static_cast<int64_t>(num_cu) * 1024 ? 4 : 1;
        } else {
            p.tpw = (run.t4 / 4 >= num_cu) ? 4 : 1;
        }
    }
    p.grid = p.tpw == 4 ? run.t4 / 4 : run.trials;
    p.alone = p.grid <= num_cu ? 1 : 0;
    if (p.tpw == 4) {
        p.csr = g.pk32 ? kCsrPack32 : kCsrPair;
        p.lpt = 1;
        p.ell = ell_ok && g.e4_mode >= 0 && ell4_lds(n4) <= max_lds ? 1 : 0;
    } else {
        p.csr = g.ux16 ? kCsrUnit : (g.pk32 ? kCsrPack32 : kCsrPair);
        if (lpt_req == 1 || lpt_req == 2 || lpt_req == 4)
            p.lpt = lpt_req;
        else
            p.lpt = lanes_per_task(g, run, max_lds, num_cu);
        // but with workgroups to share the compute units, two lanes per task
        // issue less for short rows, whose random blocks outweigh their sums,
        // as long as two rows fit a lane's 32 cached slots (us per step with
        // four and two: 364 p-bits of degree 4, 843 trials, SpSA 2.93 and 1.39;
        // 1,000 of degree 6, 300 trials 2.17 and 1.37; 250 of degree 6, 300
        // trials 0.89 and 0.88; 404 of mean degree 11, 466 trials 1.14 and 1.50;
        // 263 of 18, 438 trials 1.16 and 2.23): from the first trial that has to share
        // on where four lanes fill a unit (1,023 of degree 4, 284 trials 2.18 and 1.00),
        // from a quarter more on below
        if (lpt_req == 0 && p.lpt == 4 && p.csr == kCsrUnit && g.nnz <= 8 * static_cast<int64_t>(g.n) && g.max_degree <= 16 &&
            (tasks * 4 > 512 ? 5 : 4) * static_cast<int64_t>(run.trials) > 5 * static_cast<int64_t>(num_cu))
            p.lpt = 2;
        // (a lane that keeps its task's input-stage state and edges in
        // registers steps SpSA and TApSA faster: 3,000 p-bits of degree 6, 30
        // trials, TApSA 3.5 against 4.5 us per step)
        const bool keeps_state = (run.xs || run.ring) && p.csr == kCsrUnit && tasks <= 1024;
        p.ell = ell_ok && p.lpt == 1 && !keeps_state && 2 * ell1_stride(n4) <= max_lds ? 1 : 0;
    }
    auto set_block = [&]() {
        const int32_t lanes = tasks * p.lpt;
        if (block_req == 256 || block_req == 512 || block_req == 1024)
            p.block = block_req;
        else
            p.block = lanes > 512 ? 1024 : (lanes > 256 ? 512 : 256);
    };
    if (p.ell) {
        p.csr_lds = 0;
        p.lds_bytes = p.tpw == 4 ? ell4_lds(n4) : 2 * ell1_stride(n4);
        set_block();
        *plan = p;
        return true;
    }
    const size_t sp = 2 * spin_stride(n4, p.tpw, p.lpt, p.csr) +
                      ring_lds_bytes(n4, p.tpw, p.lpt, p.csr, run.ring != nullptr, run.alpha);
    if (sp > max_lds) {
        // four trials' spin state too large: one trial per workgroup if the
        // choice was the planner's
        if (p.tpw == 4 && tpw_req != 4)
            return plan_anneal(g, run, 1, lpt_req, block_req, max_lds, num_cu, plan, why);
        if (why)
            *why = "n = " + std::to_string(g.n) + " does not fit the LDS-resident spin state (" +
                   std::to_string(sp) + " > " + std::to_string(max_lds) + " bytes)";
        return false;
    }
    const size_t full = sp + params_bytes(n4) + align16(static_cast<size_t>(g.nnz) * edge_bytes(p.csr));
    p.csr_lds = full <= max_lds ? 1 : 0;
    p.lds_bytes = p.csr_lds ? full : sp;
    set_block();
    *plan = p;
    return true;
}

void task_order(const DevGraph &g, const std::vector<int32_t> &row_ptr_host, const AnnealPlan &plan,
                std::vector<int32_t> *order) {
    const int32_t tasks = g.n4 / 4;
    std::vector<int64_t> key(static_cast<size_t>(tasks));
    for (int32_t m = 0; m < tasks; ++m) {
        int64_t d[4];
        for (int p = 0; p < 4; ++p) d[p] = row_ptr_host[4 * m + p + 1] - row_ptr_host[4 * m + p];
        if (plan.tpw == 1 && plan.lpt == 2)
            key[m] = std::max(d[0] + d[1], d[2] + d[3]);
        else if (plan.tpw == 1 && plan.lpt == 4)
            key[m] = std::max(std::max(d[0], d[1]), std::max(d[2], d[3]));
        else
            key[m] = d[0] + d[1] + d[2] + d[3];
    }
    order->resize(static_cast<size_t>(tasks));
    for (int32_t m = 0; m < tasks; ++m) (*order)[m] = m;
    // heaviest tasks first: lanes of a wavefront walk rows of similar length
    std::stable_sort(order->begin(), order->end(),
                     [&](int32_t x, int32_t y) { return key[x] > key[y]; });
}

// LDS the kernel carves for a run under a plan (the layout above).
size_t lds_need(const DevGraph &g, const DevRun &run, const AnnealPlan &p) {
    if (p.ell) return p.tpw == 4 ? ell4_lds(g.n4) : 2 * ell1_stride(g.n4);
    size_t b = 2 * spin_stride(g.n4, p.tpw, p.lpt, p.csr) +
               ring_lds_bytes(g.n4, p.tpw, p.lpt, p.csr, run.ring != nullptr, run.alpha);
    if (p.csr_lds) b += params_bytes(g.n4) + align16(static_cast<size_t>(g.nnz) * edge_bytes(p.csr));
    return b;
}

hipError_t launch_anneal(hipStream_t stream, const DevGraph &g, const DevRun &run,
                         const AnnealPlan &plan, const int32_t *order, int32_t t_begin,
                         int32_t t_end) {
    if (t_end <= t_begin) return hipSuccess;
    // a plan made for another input stage would leave the kernel's LDS
    // layout outside the allocation
    if (lds_need(g, run, plan) > plan.lds_bytes) return hipErrorInvalidValue;
    // the streaming sweeps read the graph's ELL rows and the run's constants
    if (plan.ell && (!g.e1 || !run.pps || (plan.tpw == 4 && !g.e4))) return hipErrorInvalidValue;
    AnnealArgs a;
    fill_anneal_args(&a, g, run, order, t_begin, t_end);
    if (plan.ell) return launch_ell(stream, a, plan, g.e4_mode);
    if (plan.tpw == 4) return launch_four_trials(stream, a, plan);
    switch (plan.lpt) {
        case 1: return launch_one_trial<1>(stream, a, plan);
        case 2: return launch_one_trial<2>(stream, a, plan);
        case 4: return launch_one_trial<4>(stream, a, plan);
        default: return hipErrorInvalidValue;
    }
}

void fill_anneal_args(AnnealArgs *a, const DevGraph &g, const DevRun &run, const int32_t *order,
                      int32_t t_begin, int32_t t_end) {
    a->n = g.n;
    a->n4 = g.n4;
    a->t4 = run.t4;
    a->t_begin = t_begin;
    a->t_end = t_end;
    a->nnz = static_cast<int32_t>(g.nnz);
    a->tasks = g.n4 / 4;
    a->row_ptr = g.row_ptr;
    a->col = g.col;
    a->val = g.val;
    a->pk32 = g.pk32;
    a->ux16 = g.ux16;
    a->gorder = g.gorder;
    a->wofs = g.wofs;
    a->e4 = g.e4;
    a->e1 = g.e1;
    a->e1j = g.e1j;
    a->pps = run.pps;
    a->groups = g.ell_groups;
    a->i0_lim = run.i0_lim;
    a->gated = run.gated;
    a->h = g.h;
    a->i0 = run.i0;
    a->lam = run.lambda;
    a->dlt = run.delta;
    a->thr = run.thr24;
    a->order = order;
    a->k0 = run.key0;
    a->k1 = run.key1;
    a->spins = run.spins;
    a->xs = run.xs;
    a->stall24 = run.stall24;
    a->ring = run.ring;
    a->alpha = run.alpha;
    a->t_res = run.t_res;
}

bool plan_batch_item(const DevGraph &g, const DevRun &run, int32_t tpw_req, int32_t lpt_req,
                     size_t max_lds, AnnealPlan *plan, int32_t *variant, std::string *why) {
    AnnealPlan p;
    if (tpw_req == 4) {
        if (!plan_anneal(g, run, 4, 1, 0, max_lds, 1 << 30, &p, why)) return false;
        if (p.ell) {
            *variant = kBatchEll4 + g.e4_mode;
        } else if (p.csr == kCsrPack32) {
            *variant = p.csr_lds ? kBatchP32Lds4T : kBatchP32Glb4T;
        } else {
            *variant = kBatchPairGlb4T;
            p.csr_lds = 0;
            p.lds_bytes = 2 * spin_buf_bytes(g.n4, 4, kCsrPair);
        }
        *plan = p;
        return true;
    }
    if (lpt_req == 1 && plan_anneal(g, run, 1, 1, 0, max_lds, 1 << 30, &p, why) && p.ell) {
        *variant = g.e1j ? kBatchEll1 : kBatchEll1Unit;
        *plan = p;
        return true;
    }
    if (!plan_anneal(g, run, 1, lpt_req == 4 ? 4 : 2, 0, max_lds, 1 << 30, &p, why)) return false;
    if (p.csr == kCsrUnit) {
        *variant = p.lpt == 4 ? (p.csr_lds ? kBatchUnitLds4 : kBatchUnitGlb4)
                              : (p.csr_lds ? kBatchUnitLds2 : kBatchUnitGlb2);
    } else {
        p.lpt = 2;
        if (p.csr == kCsrPack32) {
            *variant = p.csr_lds ? kBatchP32Lds2 : kBatchP32Glb2;
        } else {
            *variant = kBatchPairGlb2;
            p.csr_lds = 0;
            p.lds_bytes = 2 * spin_buf_bytes(g.n4, 1, kCsrPair);
        }
    }
    *plan = p;
    return true;
}

}  // namespace psa
