// kernels.hip -- gfx950 kernels of the pSA hot path.
//
//   init_spins_kernel   initial state: m = +1 iff bit 31 of the INIT word
//   local_field_kernel  L = h + J m (Eq. 3 without I0)
//   energy_partial_kernel, energy_finish_kernel   Eq. 2 energy and MAX-CUT value per trial
//   spins_{to,from}_tn  layout conversion [n][t4] <-> [trials][n]
//
// (The persistent sweep kernel is in anneal.hip.)  Random words: Philox4x32-10
// block of counter (t, i/4, k, purpose) serves the four p-bits 4m..4m+3
// (m = i/4) of trial k; word i mod 4.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_math.hpp"
#include "engine.hpp"

namespace psa {
namespace {

__device__ __forceinline__ uint32_t load_word(const int8_t *spins, int32_t t4, int32_t i,
                                              int32_t q) {
    return *reinterpret_cast<const uint32_t *>(spins + static_cast<size_t>(i) * t4 + 4 * q);
}

__device__ __forceinline__ void store_word(int8_t *spins, int32_t t4, int32_t i, int32_t q,
                                           uint32_t w) {
    *reinterpret_cast<uint32_t *>(spins + static_cast<size_t>(i) * t4 + 4 * q) = w;
}

__device__ __forceinline__ Words4 block_of(uint32_t t, uint32_t m, uint32_t k, uint32_t tag,
                                           uint32_t k0, uint32_t k1) {
    return philox4x32_10(t, m, k, tag, k0, k1);
}

// ---------------------------------------------------------------------------
// Initial spins: thread per (task m, trial k) over all t4 trials; p-bit
// 4m+p of trial k is +1 iff bit 31 of word p of block (0, m, k, INIT).
// ---------------------------------------------------------------------------
__global__ void init_spins_kernel(int32_t n, int32_t tasks, int32_t t4, uint32_t k0,
                                  uint32_t k1, int8_t *__restrict__ spins) {
    const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= static_cast<int64_t>(tasks) * t4) return;
    const int32_t m = static_cast<int32_t>(idx / t4);
    const int32_t k = static_cast<int32_t>(idx % t4);
    const Words4 w = block_of(0u, static_cast<uint32_t>(m), static_cast<uint32_t>(k), kTagInit,
                              k0, k1);
    const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int32_t i = 4 * m + p;
        if (i < n) spins[static_cast<size_t>(i) * t4 + k] = (ws[p] >> 31) ? int8_t(1) : int8_t(-1);
    }
}

// ---------------------------------------------------------------------------
// Energy and cut.  With
// S_k = sum_i m_i sum_j J_ij m_j (= 2 sum_{i<j} J_ij m_i m_j) and
// W2 = sum_i sum_j J_ij:
//   E_k   = -sum_i h_i m_i - S_k / 2
//   cut_k = sum_{i<j} w_ij [m_i != m_j] = (S_k - W2) / 4     (w = -J)
// ---------------------------------------------------------------------------
constexpr int kEnergyRows = 256;   // rows of a partial sum
constexpr int kEnergyBlock = 1024;  // most threads of a partial pass
constexpr int kFieldBlock = 256;

// Number of a workgroup of a wide_grid; those past the last one that a launch
// asked for have one, too (at most 2^31 - 1).
__device__ __forceinline__ int32_t wide_index() {
    const uint32_t b = blockIdx.y * gridDim.x + blockIdx.x;
    return static_cast<int32_t>(min(b, 0x7FFFFFFFu));
}

// Final pass: a wavefront sums the row blocks' terms of one trial group, eight
// lanes (the group's S and h terms) to a block, then reduces over the blocks:
//   E_k   = -sum_i h_i m_i - S_k / 2
//   cut_k = sum_{i<j} w_ij [m_i != m_j] = (S_k - W2) / 4     (w = -J)
// A thread per trial walking the blocks one by one took 20 us at 20,000 p-bits
// (79 dependent loads); this 4.7 us.
__device__ __forceinline__ void energy_finish(const EnergyJob &e, int32_t q) {
    const int lane = threadIdx.x & 63, c = lane & 7;
    const int32_t groups = e.t4 / 4;
    if (q >= groups) return;  // past the last wavefront of the grid (wide_grid)
    int64_t v = 0;
    for (int32_t b = lane >> 3; b < e.blocks; b += 8) v += e.part[(static_cast<size_t>(b) * groups + q) * 8 + c];
#pragma unroll
    for (int off = 8; off < 64; off <<= 1) v += __shfl_xor(v, off);
    const int64_t H = __shfl_down(v, 4);
    const int32_t k = 4 * q + c;
    if (lane < 4 && k < e.trials) {
        e.energy[k] = -H - v / 2;
        e.cut[k] = (v - e.w2) / 4;
    }
}

// One run (its table entry as the argument).
__global__ __launch_bounds__(64) void energy_finish_kernel(EnergyJob e) {
    energy_finish(e, wide_index());
}

// The run of a batched read-out that index x (a workgroup of the partial
// pass, or a trial group of the final pass) belongs to: the last run whose
// first index is at most x (first indices ascending, the first one 0).
template <bool WG>
__device__ __forceinline__ int32_t energy_run_of(const EnergyJob *__restrict__ jobs, int32_t count, int32_t x) {
    int32_t lo = 0, hi = count - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if ((WG ? jobs[mid].wg0 : jobs[mid].q0) <= x)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// Read-out work split.  A lane holds sixteen trials (a chunk of Q = 4 trial
// groups) of a row: the `cpl` lanes of consecutive chunks read a neighbour's
// spins as one contiguous piece of up to 256 bytes, and `lpr` such groups share
// a long row's edges; at most 16 lanes to a row in the partial pass, at most a
// wavefront for the local fields.  Runs too small to fill the chip that way
// take Q = 1, four trials to a lane (energy_split, field_split).
struct ReadLane {
    int32_t c, sub, row;      // chunk, share of the row, row of the block
    int32_t q0, nq;           // first trial group of the chunk, groups in it (none: <= 0)
    int32_t rows;             // rows in flight together
};
template <int Q>
__device__ __forceinline__ ReadLane read_lane(const EnergyJob &e, int32_t y) {
    ReadLane l;
    const int32_t tid = static_cast<int32_t>(threadIdx.x);
    l.c = tid & (e.cpl - 1);
    l.sub = (tid / e.cpl) & (e.lpr - 1);
    l.row = tid / (e.cpl * e.lpr);
    l.rows = static_cast<int32_t>(blockDim.x) / (e.cpl * e.lpr);
    l.q0 = (y * e.cpl + l.c) * Q;
    l.nq = min(e.t4 / 4 - l.q0, Q);
    return l;
}

// A lane's share of sum_j J_ij m_j of row i: edges sub, sub + lpr, ...  A
// whole chunk's spins are one 16-byte load, aligned to 4 bytes.
typedef u32x4 __attribute__((aligned(4))) u32x4_word;
template <int Q>
__device__ __forceinline__ void row_sums(const EnergyJob &e, int32_t i, const ReadLane &l, int32_t (&L)[Q][4]) {
    const int32_t e1 = e.row_ptr[i + 1];
#pragma unroll 4
    for (int32_t x = e.row_ptr[i] + l.sub; x < e1; x += e.lpr) {
        const int32_t j = e.col[x];
        const int32_t J = e.val[x];
        uint32_t w[Q] = {};
        if (Q == 4 && l.nq == Q) {
            const u32x4 v = *reinterpret_cast<const u32x4_word *>(e.spins + static_cast<size_t>(j) * e.t4 + 4 * l.q0);
#pragma unroll
            for (int qq = 0; qq < Q; ++qq) w[qq] = v[qq];
        } else {
#pragma unroll
            for (int qq = 0; qq < Q; ++qq)
                if (qq < l.nq) w[qq] = load_word(e.spins, e.t4, j, l.q0 + qq);
        }
#pragma unroll
        for (int qq = 0; qq < Q; ++qq)
#pragma unroll
            for (int k = 0; k < 4; ++k) L[qq][k] += J * spin_of(w[qq], k);
    }
}

// Partial pass: workgroup (256-row block, group y of cpl chunks) sums m_i
// sum_j J_ij m_j and h_i m_i over its rows into part[(block * groups + q) * 8
// + c]: c < 4 the S terms of trial 4q + c, c >= 4 the h terms.  S is linear
// in each row's inner sum, so a lane multiplies its share of it by m_i and
// keeps the product; the h terms (none when every h is 0) are taken by the
// row's first share.  SUM: the type a block's sums fit -- int32 when 256 rows
// of the field bound do (then a reduction step is one exchange), else int64.
// A lane's own sum is over at most 16 rows (256 threads, at most 16 to a row)
// of terms below 2^24: int32.
template <typename SUM, int Q>
__device__ __forceinline__ void energy_partial_run(const EnergyJob &e, int32_t local) {
    const int32_t groups = e.t4 / 4;
    const int32_t ys = (groups + Q * e.cpl - 1) / (Q * e.cpl);
    const int32_t blk = local / ys;
    if (blk >= e.blocks) return;  // past the last workgroup of the grid (wide_grid)
    const ReadLane l = read_lane<Q>(e, local % ys);
    const bool has_h = e.h != nullptr;
    int32_t s32[Q][4] = {}, hm32[Q][4] = {};
    if (l.nq > 0)
        for (int32_t r = l.row; r < kEnergyRows; r += l.rows) {
            const int32_t i = blk * kEnergyRows + r;
            if (i >= e.n) break;
            int32_t L[Q][4] = {};
            row_sums<Q>(e, i, l, L);
            const int32_t hi = has_h && l.sub == 0 ? e.h[i] : 0;
#pragma unroll
            for (int qq = 0; qq < Q; ++qq) {
                if (qq < l.nq) {
                    const uint32_t wi = load_word(e.spins, e.t4, i, l.q0 + qq);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int32_t mi = spin_of(wi, k);
                        s32[qq][k] += mi * L[qq][k];
                        hm32[qq][k] += mi * hi;
                    }
                }
            }
        }
    // over the lanes of a chunk, then over the wavefronts
    extern __shared__ __align__(16) unsigned char energy_lds[];  // energy_lds_bytes
    SUM *red = reinterpret_cast<SUM *>(energy_lds);              // [wavefronts][cpl][Q][8]
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    SUM v[Q * 8];  // the S terms, then the h terms
#pragma unroll
    for (int x = 0; x < 4 * Q; ++x) {
        v[x] = s32[x >> 2][x & 3];
        v[4 * Q + x] = hm32[x >> 2][x & 3];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)  // every value's exchange of a step in flight together
        if (off >= e.cpl) {
#pragma unroll
            for (int x = 0; x < 4 * Q; ++x) v[x] += __shfl_xor(v[x], off);
            if (has_h) {
#pragma unroll
                for (int x = 4 * Q; x < 8 * Q; ++x) v[x] += __shfl_xor(v[x], off);
            }
        }
    if (lane < e.cpl) {
#pragma unroll
        for (int x = 0; x < 4 * Q; ++x) {
            SUM *to = red + ((wave * e.cpl + lane) * Q + (x >> 2)) * 8 + (x & 3);
            to[0] = v[x];
            to[4] = v[4 * Q + x];
        }
    }
    __syncthreads();
    for (int32_t x = threadIdx.x; x < 8 * Q * e.cpl; x += static_cast<int32_t>(blockDim.x)) {
        const int32_t ch = x / (8 * Q), qq = (x >> 3) % Q, c = x & 7;
        const int32_t q = ((local % ys) * e.cpl + ch) * Q + qq;
        if (q < groups) {
            int64_t sum = 0;
            for (int wv = 0; wv < static_cast<int>(blockDim.x) / 64; ++wv) sum += red[((wv * e.cpl + ch) * Q + qq) * 8 + c];
            e.part[(static_cast<size_t>(blk) * groups + q) * 8 + c] = sum;
        }
    }
}

// One run: 20,000 p-bits of degree 20, 256 trials: 48 us (a thread per row
// and four trials, which the one-run read-out used before: 224 us).
template <typename SUM, int Q>
__global__ __launch_bounds__(kEnergyBlock) void energy_partial_kernel(EnergyJob e) {
    energy_partial_run<SUM, Q>(e, wide_index());
}

// Many runs: workgroup b is workgroup b - wg0 of its run.
template <typename SUM, int Q>
__global__ __launch_bounds__(kEnergyBlock) void energy_partial_batch_kernel(const EnergyJob *__restrict__ jobs,
                                                                            int32_t count) {
    const int32_t b = wide_index();
    const EnergyJob &e = jobs[energy_run_of<true>(jobs, count, b)];
    energy_partial_run<SUM, Q>(e, b - e.wg0);
}

// Many runs' final pass: wavefront x is trial group x - q0 of its run.
__global__ __launch_bounds__(64) void energy_finish_batch_kernel(const EnergyJob *__restrict__ jobs, int32_t count) {
    const int32_t x = wide_index();
    const EnergyJob &e = jobs[energy_run_of<false>(jobs, count, x)];
    energy_finish(e, x - e.q0);
}

// Local fields L = h + J m, int32 [trials][n]: the same split of lanes; the
// shares of a row are reduced and divide its stores.  Bound by the spin
// gathers from L2 (20,000 p-bits of degree 20, 256 trials: 103 MB): 35 us,
// against 375 us with a thread per p-bit and four trials (4-byte gathers) and
// 60 us with a chunk's rows on neighbouring lanes (16-byte gathers).
template <int Q>
__global__ __launch_bounds__(kFieldBlock) void local_field_kernel(EnergyJob e, int32_t *__restrict__ out) {
    const ReadLane l = read_lane<Q>(e, static_cast<int32_t>(blockIdx.z * gridDim.y + blockIdx.y));
    const int32_t i = static_cast<int32_t>(blockIdx.x) * l.rows + l.row;
    int32_t L[Q][4] = {};
    if (i < e.n && l.nq > 0) row_sums<Q>(e, i, l, L);
    const int32_t h = i < e.n && e.h ? e.h[i] : 0;
#pragma unroll
    for (int x = 0; x < 4 * Q; ++x) {
        int32_t v = L[x >> 2][x & 3];
        for (int off = e.cpl; off < e.cpl * e.lpr; off <<= 1) v += __shfl_xor(v, off);
        const int32_t trial = 4 * l.q0 + x;
        if ((x & (e.lpr - 1)) == l.sub && i < e.n && trial < e.trials) out[static_cast<size_t>(trial) * e.n + i] = h + v;
    }
}

// Layout changes between [n][t4] (trials innermost) and [trials][n], 64 p-bits
// x 64 trials per workgroup through LDS so that both sides are read and
// written in runs of 64 bytes (a thread per byte of the output, reading one
// byte of a row each, took 24.6 us at 20,000 p-bits x 256 trials; this 5.6 us).
constexpr int kTile = 64;

// Workgroup b's tile: the p-bits' tiles next to each other.
struct TileAt {
    int32_t i0, k0;
};
__device__ __forceinline__ TileAt tile_at(int32_t n) {
    const uint32_t across = static_cast<uint32_t>((n + kTile - 1) / kTile);
    return TileAt{static_cast<int32_t>(blockIdx.x % across) * kTile, static_cast<int32_t>(blockIdx.x / across) * kTile};
}
inline unsigned tile_grid(int32_t n, int32_t trials) {
    return static_cast<unsigned>((static_cast<int64_t>(n) + kTile - 1) / kTile * ((static_cast<int64_t>(trials) + kTile - 1) / kTile));
}

// spins -> out
__global__ __launch_bounds__(256) void spins_to_tn_kernel(int32_t n, int32_t t4, int32_t trials,
                                                          const int8_t *__restrict__ spins, int8_t *__restrict__ out) {
    __shared__ int8_t tile[kTile][kTile + 4];
    const TileAt at = tile_at(n);
    const int32_t i0 = at.i0, k0 = at.k0;
    // 16 words of four trials per row
    for (int32_t x = threadIdx.x; x < kTile * 16; x += 256) {
        const int32_t r = x / 16, w = x % 16;
        if (i0 + r < n && k0 + 4 * w < t4)
            *reinterpret_cast<uint32_t *>(&tile[r][4 * w]) = load_word(spins, t4, i0 + r, k0 / 4 + w);
    }
    __syncthreads();
    const int32_t c = threadIdx.x & 63;
    if (i0 + c >= n) return;
    for (int32_t r = threadIdx.x >> 6; r < kTile && k0 + r < trials; r += 4)
        out[static_cast<size_t>(k0 + r) * n + i0 + c] = tile[c][r];
}

// in -> spins; padding trials (k >= trials) are left unchanged.
__global__ __launch_bounds__(256) void spins_from_tn_kernel(int32_t n, int32_t t4, int32_t trials,
                                                            const int8_t *__restrict__ in, int8_t *__restrict__ spins) {
    __shared__ int8_t tile[kTile][kTile + 4];
    const TileAt at = tile_at(n);
    const int32_t i0 = at.i0, k0 = at.k0;
    const int32_t c = threadIdx.x & 63;
    if (i0 + c < n)
        for (int32_t r = threadIdx.x >> 6; r < kTile && k0 + r < trials; r += 4)
            tile[c][r] = in[static_cast<size_t>(k0 + r) * n + i0 + c];
    __syncthreads();
    if (k0 + c >= trials) return;
    for (int32_t r = threadIdx.x >> 6; r < kTile && i0 + r < n; r += 4)
        spins[static_cast<size_t>(i0 + r) * t4 + k0 + c] = tile[r][c];
}

inline unsigned grid_for(int64_t items, int block) {
    return static_cast<unsigned>((items + block - 1) / block);
}

// ---------------------------------------------------------------------------
// Value-level checks of the per-update arithmetic (test entry points): the
// device tanh_f32 of every x, and the decision pbit_up of every (x, word)
// with the branch it took (bit 0: +1, bit 1: the estimate was within 2^-16
// of r, so tanh_f32 decided).  Grid-stride over count elements.
// ---------------------------------------------------------------------------
__global__ void debug_tanh_kernel(int64_t count, const float *__restrict__ x,
                                  float *__restrict__ y) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < count;
         i += stride)
        y[i] = tanh_f32(x[i]);
}

__global__ void debug_decide_kernel(int64_t count, const float *__restrict__ x,
                                    const uint32_t *__restrict__ word, uint8_t *__restrict__ out) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < count;
         i += stride) {
        const float diff = tanh_estimate_minus(x[i], r_of(word[i]));
        out[i] = static_cast<uint8_t>((pbit_up(x[i], word[i]) ? 1u : 0u) |
                                      (estimate_decides(diff) ? 0u : 2u));
    }
}

}  // namespace

hipError_t launch_init_spins(hipStream_t stream, int32_t n, const DevRun &run) {
    const int32_t tasks = (n + 3) / 4;
    const int block = 256;
    hipLaunchKernelGGL(init_spins_kernel, dim3(grid_for(static_cast<int64_t>(tasks) * run.t4, block)),
                       dim3(block), 0, stream, n, tasks, run.t4, run.key0, run.key1, run.spins);
    return hipGetLastError();
}

EnergyJob energy_job(const DevGraph &g, const DevRun &run) {
    EnergyJob e;
    e.n = g.n;
    e.t4 = run.t4;
    e.trials = run.trials;
    e.blocks = (g.n + kEnergyRows - 1) / kEnergyRows;
    e.degree = g.n > 0 ? static_cast<int32_t>(g.nnz / g.n) : 0;
    read_out_split(run.t4, e.degree, &e.cpl, &e.lpr);
    e.w2 = g.w2;
    e.row_ptr = g.row_ptr;
    e.col = g.col;
    e.val = g.val;
    e.h = g.any_h ? g.h : nullptr;
    e.narrow = g.max_field < (1 << 23) ? 1 : 0;
    e.spins = run.spins;
    return e;
}

hipError_t launch_local_field(hipStream_t stream, const DevGraph &g, const DevRun &run,
                              int32_t *out_tn) {
    EnergyJob e = energy_job(g, run);
    field_split(&e);
    const int32_t chunks = (run.t4 + 4 * e.quads - 1) / (4 * e.quads), ys = (chunks + e.cpl - 1) / e.cpl;
    const int32_t y = std::min(ys, kMostGridY);
    hipLaunchKernelGGL(e.quads == 1 ? local_field_kernel<1> : local_field_kernel<4>,
                       dim3(grid_for(static_cast<int64_t>(g.n) * e.cpl * e.lpr, kFieldBlock), y, (ys + y - 1) / y),
                       dim3(kFieldBlock), 0, stream, e, out_tn);
    return hipGetLastError();
}

size_t energy_partial_bytes(int32_t n, int32_t t4) {
    return static_cast<size_t>((n + kEnergyRows - 1) / kEnergyRows) * (t4 / 4) * 8 * sizeof(int64_t);
}

// LDS of a partial pass: a partial sum per wavefront, chunk and term.  At most
// 64 KB (1,024 threads, 16 chunks of 16 trials, int64).
static size_t energy_lds_bytes(const EnergyJob &e, int32_t block, bool narrow) {
    return static_cast<size_t>(block / 64) * e.cpl * e.quads * 8 * (narrow ? 4 : 8);
}

hipError_t launch_energy_cut(hipStream_t stream, const DevGraph &g, const DevRun &run,
                             int64_t *part, int64_t *energy, int64_t *cut) {
    EnergyJob e = energy_job(g, run);
    energy_split(&e, energy_waves(e), energy_batch_wgs(e), true);
    e.part = part;
    e.energy = energy;
    e.cut = cut;
    auto kern = e.quads == 1 ? (e.narrow ? energy_partial_kernel<int32_t, 1> : energy_partial_kernel<int64_t, 1>)
                             : (e.narrow ? energy_partial_kernel<int32_t, 4> : energy_partial_kernel<int64_t, 4>);
    const int32_t block = energy_block(e);
    hipLaunchKernelGGL(kern, wide_grid(energy_batch_wgs(e)), dim3(block),
                       energy_lds_bytes(e, block, e.narrow), stream, e);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(energy_finish_kernel, wide_grid(run.t4 / 4), dim3(64), 0, stream, e);
    return hipGetLastError();
}

hipError_t launch_energy_cut_batch(hipStream_t stream, const EnergyJob *jobs, const EnergyJob *host, int32_t count,
                                   int32_t wgs, int32_t groups) {
    if (count <= 0 || wgs <= 0 || groups <= 0) return hipSuccess;
    int32_t block = 64;
    bool narrow = true;
    for (int32_t j = 0; j < count; ++j) {
        if (host[j].quads != host[0].quads) return hipErrorInvalidValue;
        block = std::max(block, energy_block(host[j]));
        narrow = narrow && host[j].narrow;
    }
    size_t lds = 0;
    for (int32_t j = 0; j < count; ++j) lds = std::max(lds, energy_lds_bytes(host[j], block, narrow));
    auto kern = host[0].quads == 1
                    ? (narrow ? energy_partial_batch_kernel<int32_t, 1> : energy_partial_batch_kernel<int64_t, 1>)
                    : (narrow ? energy_partial_batch_kernel<int32_t, 4> : energy_partial_batch_kernel<int64_t, 4>);
    hipLaunchKernelGGL(kern, wide_grid(wgs), dim3(block), lds, stream, jobs, count);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(energy_finish_batch_kernel, wide_grid(groups), dim3(64), 0, stream, jobs, count);
    return hipGetLastError();
}

hipError_t launch_spins_to_tn(hipStream_t stream, int32_t n, const DevRun &run, int8_t *out_tn) {
    hipLaunchKernelGGL(spins_to_tn_kernel, dim3(tile_grid(n, run.trials)), dim3(256), 0, stream, n,
                       run.t4, run.trials, run.spins, out_tn);
    return hipGetLastError();
}

hipError_t launch_spins_from_tn(hipStream_t stream, int32_t n, const DevRun &run,
                                const int8_t *in_tn) {
    hipLaunchKernelGGL(spins_from_tn_kernel, dim3(tile_grid(n, run.trials)), dim3(256), 0, stream, n,
                       run.t4, run.trials, in_tn, run.spins);
    return hipGetLastError();
}

hipError_t launch_debug_tanh(hipStream_t stream, int64_t count, const float *x, float *y) {
    const int block = 256;
    const int64_t grid = std::min<int64_t>((count + block - 1) / block, 8192);
    hipLaunchKernelGGL(debug_tanh_kernel, dim3(static_cast<uint32_t>(grid)), dim3(block), 0, stream,
                       count, x, y);
    return hipGetLastError();
}

hipError_t launch_debug_decide(hipStream_t stream, int64_t count, const float *x,
                               const uint32_t *word, uint8_t *out) {
    const int block = 256;
    const int64_t grid = std::min<int64_t>((count + block - 1) / block, 8192);
    hipLaunchKernelGGL(debug_decide_kernel, dim3(static_cast<uint32_t>(grid)), dim3(block), 0,
                       stream, count, x, word, out);
    return hipGetLastError();
}

}  // namespace psa
