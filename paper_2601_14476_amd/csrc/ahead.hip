// ahead.hip -- sweep of small runs with the decisions' thresholds drawn ahead
// of the spins (gfx950).
//
// An update's random words and factors do not depend on the spins: p-bit i of
// trial k at step t turns up iff tanh(I0 lambda (L + delta)) > r, and for a
// positive I0 lambda that is iff its count of neighbours c (L = h - sum |J| +
// 2 c) reaches a whole number.  A run of few trials leaves most of the chip
// idle and spends its steps on random blocks and exponentials in a serial
// chain, so here each launch does two things at once: workgroup k < trials
// runs the steps of one chunk for trial k from the thresholds that the launch
// before has left, and the other workgroups write the thresholds of the next
// chunk (a byte per update: 128 - the least count that turns the p-bit up, 0
// where the timing gate holds it).
//
// What bounds it: the running side by a step's latency and the issue of about
// three vector instructions per neighbour, the drawing side by vector issue.
// A gather of spin bytes or words costs about 10 cycles per wavefront in bank
// conflicts (measured with a word of four trials per p-bit: 1.30 us per step
// for 2,000 p-bits of degree 6); so the spins lie as bits, 32 p-bits to a
// word, and every word 64 times, once per bank: each lane reads its own bank,
// and a wavefront's 64 new spins are one mask, written to all banks by four
// stores.  Threshold loads run eight steps ahead in registers; the reads of a
// row are all issued before the first is used (1.08 -> 0.96 us).
//
// Measured against the sweeps that draw as they go, timing gate, us per step:
// 2,000 p-bits of degree 6, 100 trials 1.23 -> 1.00; 4,001 of degree 12,
// weights +-1..+-7, 37 trials 4.0 -> 3.05; 2,000 of degree 24, 100 trials 4.6
// -> 2.4; as masks, 800 of degree 48, 10 trials, no gate 1.78 -> 0.65; 250 of
// degree 6 0.81 -> 0.37.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ell_sweep.hpp"
#include "engine.hpp"

namespace psa {
namespace {

// Rows of 64 equal words, one per bank: row 0 is zero, rows 1 .. 2 bw hold the
// bits u = (m + 1) / 2 (bw wavefronts of 64 positions), the next 2 bw 1 - u.
constexpr int32_t kRowBytes = 256;
// Distance between the two buffers with K positions per lane of 1,024.
constexpr int32_t ahead_stride(int K) { return (1 + 4 * (K == 4 ? kAheadMaxN / 64 : 16 * K)) * kRowBytes; }

struct AheadArgs {
    int32_t n, n4, t4, tasks, waves, trials;
    int32_t consumers;         // workgroups that run steps: trials or 0
    int32_t c_begin, c_end;    // their steps
    int32_t p_begin, p_end;    // the steps whose thresholds are drawn
    const uint8_t *in;         // [step][trial][256 waves]
    uint8_t *out;
    const int32_t *gorder;
    const uint32_t *pps;
    const int32_t *border, *bofs;  // positions (longest rows first) and their entries
    const uint32_t *be, *bm;
    int32_t bw;
    const float *i0, *lam, *dlt;
    uint32_t k0, k1;
    int32_t gated;
    int8_t *spins;
};

// Least count in 0 .. 127 that turns the p-bit up, by the decision itself.
// The decision is monotone in the count: counts are two apart in L, so with
// I0 lambda of 2^-12 and more their pre-activations differ by far more than
// the roundings of tanh_f32's exponential, and every later operation of it
// rounds a monotone function.
__device__ __noinline__ int32_t exact_threshold(float a, float d, float base, uint32_t rword, int32_t k) {
    auto up = [&](int32_t c) { return pbit_up(a * ((base + 2.0f * static_cast<float>(c)) + d), rword); };
    while (k > 0 && up(k - 1)) --k;
    while (k < 127 && !up(k)) ++k;
    return k;
}

// The thresholds of steps p_begin .. p_end-1; this workgroup is number `id`
// of `count`.  A wavefront keeps one set of 64 tasks and takes every stride-th
// (step, trial).
//
// tanh(x) > r iff v = 2 log2(e) x > z = log2((1 + r) / (1 - r)); v is linear
// in the count, so the threshold is the next whole number past c* = z / (I0
// P1) - delta / 2 - (h - sum |J|) / 2 (P1 = 4 lambda log2 e).  Where c* lies
// within its error of a whole number the decision itself is evaluated.  That
// error, in v: 2^-15 for the two logarithms (2^-19 each), the rounding of 1 +-
// r to 24 bits and relative roundings (|z| <= 25, 2^-20 of it); tanh_f32 is
// within 2^-22 of tanh, which moves z by at most 32 / (2^24 (1 - |r|)) (2.89 *
// 2^-22 / (1 - r^2) where that is small, and near |r| = 1 at most the 4 that
// lie between z >= 22 and the 26 of |x| = 9); and 2^-20 of delta / 2 and of the
// count range directly in counts.
__device__ __forceinline__ void draw_thresholds(const AheadArgs &a, int32_t id, int32_t count) {
    const uint32_t lane = threadIdx.x & 63u;
    const int32_t per = static_cast<int32_t>(blockDim.x >> 6);
    const int32_t gw = __builtin_amdgcn_readfirstlane(id * per + static_cast<int32_t>(threadIdx.x >> 6));
    const int32_t stride = count * per / a.waves;  // sets of wavefronts
    const int32_t w = gw % a.waves;
    if (gw >= stride * a.waves) return;
    const uint32_t m = static_cast<uint32_t>((a.gorder + 64 * w)[lane]);
    const bool valid = 64 * w + static_cast<int32_t>(lane) < a.tasks;
    float hd[4], p1[4], off[4], eps[4];
    uint32_t th[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const u32x4 c = load_lane_x4(a.pps + static_cast<size_t>(w) * 1024 + p * 256, lane * 16u);
        hd[p] = __uint_as_float(c.x);
        p1[p] = valid ? __uint_as_float(c.y) : 1.0f;
        const float half_d = __uint_as_float(c.z) / p1[p];
        off[p] = -(half_d + hd[p]);
        eps[p] = fmaf(fabsf(half_d) + fabsf(hd[p]) + 1.0f, 0x1p-20f, 0.0f);
        th[p] = c.w;
    }
    const RoundKeys keys = round_keys(a.k0, a.k1);
    const int32_t items = (a.p_end - a.p_begin) * a.trials;
    for (int32_t it = gw / a.waves; it < items; it += stride) {
        const int32_t dt = it / a.trials;
        const uint32_t t = static_cast<uint32_t>(a.p_begin + dt), k = static_cast<uint32_t>(it - dt * a.trials);
        const float i0t = load_uniform(a.i0 + t);
        const Words4 rb = block_of_task(m, block_prefix(t, k, kTagR, a.k0, a.k1), keys);
        const uint32_t rw[4] = {rb.x, rb.y, rb.z, rb.w};
        float b[4];  // the bytes
        bool close[4], any = false;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const float inv = __builtin_amdgcn_rcpf(i0t * p1[p]);
            const uint32_t ai = (rw[p] >> 7) | 1u;  // 2^24 (1 + r)
            const float fa = static_cast<float>(ai), fb = static_cast<float>(0x2000000u - ai);
            const float z = __builtin_amdgcn_logf(fa) - __builtin_amdgcn_logf(fb);
            const float tol_v = fmaf(32.0f, __builtin_amdgcn_rcpf(fminf(fa, fb)), 0x1.8p-15f);
            const float cs = __builtin_amdgcn_fmed3f(fmaf(z, inv, off[p]), -0.5f, 126.5f);
            const float fr = __builtin_amdgcn_fractf(cs);
            close[p] = fabsf(fr - 0.5f) > 0.5f - fmaf(tol_v, inv, eps[p]);
            any = any || close[p];
            b[p] = 127.0f + fr - cs;
        }
        if (__ballot(any && valid) != 0u) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                if (close[p] && valid) {
                    const int32_t i = static_cast<int32_t>(4 * m) + p;
                    b[p] = static_cast<float>(128 - exact_threshold(i0t * a.lam[i], a.dlt[i], 2.0f * hd[p], rw[p],
                                                                    128 - static_cast<int32_t>(b[p])));
                }
            }
        }
        if (a.gated) {
            const Words4 gb = block_of_task(m, block_prefix(t, k, kTagGate, a.k0, a.k1), keys);
            const uint32_t gv[4] = {gb.x, gb.y, gb.z, gb.w};
#pragma unroll
            for (int p = 0; p < 4; ++p) b[p] = fires(gv[p], th[p]) ? b[p] : 0.0f;
        }
        uint32_t word = 0u;
#pragma unroll
        for (int p = 0; p < 4; ++p) word = __builtin_amdgcn_cvt_pk_u8_f32(b[p], p, word);
        // in the order of the p-bits (idle lanes have no p-bits)
        if (valid) reinterpret_cast<uint32_t *>(a.out)[static_cast<size_t>(it) * a.waves * 64 + m] = word;
    }
}

// f(std::integral_constant<int, 0>{}), ... N of them.
template <int N, typename F>
__device__ __forceinline__ void unroll(F &&f) {
    if constexpr (N > 0) {
        unroll<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// Steps c_begin .. c_end-1 of trial k.  Position s blockDim + tid is a lane's
// slot s (K slots); the first kCached entries of each slot's row are kept in
// registers, the rest of longer rows read from the graph's at every step.
template <int K, bool WEIGHTS>
__device__ __forceinline__ void run_steps(const AheadArgs &a, int32_t k, unsigned char *smem) {
    constexpr int kCached = K == 1 ? 48 : (K == 2 ? 24 : 12);
    constexpr int kFirst = K == 4 ? 4 : 8, kChunk = 4;
    constexpr int32_t kStride = ahead_stride(K);
    const uint32_t lane = threadIdx.x & 63u;
    const int32_t w = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(threadIdx.x >> 6));
    const int32_t per = static_cast<int32_t>(blockDim.x >> 6);
    const uint32_t mine = lane << 18;  // the lane's bank in an entry's address
    int32_t idx[K], len[K];
    bool valid[K];
    const uint32_t *rows[K];
    uint32_t ent[K][kCached];
    uint64_t up[K];  // the slots' spins
#pragma unroll
    for (int s = 0; s < K; ++s) {
        const int32_t wv = s * per + w;
        const bool have = wv < a.bw;
        valid[s] = have && 64 * wv + static_cast<int32_t>(lane) < a.n;
        idx[s] = valid[s] ? (a.border + 64 * wv)[lane] : 0;
        const int32_t b = have ? load_uniform(a.bofs + wv) : 0;
        len[s] = have ? load_uniform(a.bofs + wv + 1) - b : 0;
        rows[s] = a.be + static_cast<size_t>(b) * 64;
        // every load at once (at a clamped index), then the rest made the zero row
#pragma unroll
        for (int e = 0; e < kCached; ++e)
            ent[s][e] = a.be[static_cast<size_t>(bit_row_entry(b, len[s], e)) * 64 + lane];
#pragma unroll
        for (int e = 0; e < kCached; ++e) {
            asm volatile("" : "+v"(ent[s][e]));
            ent[s][e] = (e < len[s] ? ent[s][e] : 0u) + mine;
        }
        const bool u = valid[s] && a.spins[static_cast<size_t>(idx[s]) * a.t4 + k] > 0;
        up[s] = __ballot(u);
    }
    int32_t longest = 0;
#pragma unroll
    for (int s = 0; s < K; ++s) longest = max(longest, len[s]);
    auto store = [&](auto par_tag) __attribute__((always_inline)) {
        unsigned char *at = smem + decltype(par_tag)::value * kStride + lane * 4u;
#pragma unroll
        for (int s = 0; s < K; ++s) {
            const int32_t wv = s * per + w;
            if (wv >= a.bw) continue;
            const uint32_t lo = static_cast<uint32_t>(up[s]), hi = static_cast<uint32_t>(up[s] >> 32);
            uint32_t *r0 = reinterpret_cast<uint32_t *>(at + (1 + 2 * wv) * kRowBytes);
            uint32_t *r1 = reinterpret_cast<uint32_t *>(at + (1 + 2 * wv + 2 * a.bw) * kRowBytes);
            r0[0] = lo;
            r0[64] = hi;
            r1[0] = ~lo;
            r1[64] = ~hi;
        }
    };
    store(std::integral_constant<int, 0>{});
    if (w == 0) {
        *reinterpret_cast<uint32_t *>(smem + lane * 4u) = 0u;
        *reinterpret_cast<uint32_t *>(smem + kStride + lane * 4u) = 0u;
    }
    const int32_t steps = a.c_end - a.c_begin;
    const size_t step_bytes = static_cast<size_t>(a.trials) * a.waves * 256;
    const uint8_t *kin = a.in + static_cast<size_t>(k) * a.waves * 256;
    // thresholds of kBlock steps, and of the next kBlock, on their way meanwhile
    constexpr int kBlock = K == 4 ? 4 : 8;
    uint32_t kb[kBlock][K], next[kBlock][K];
    auto load_block = [&](int32_t t) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < kBlock; ++v) {
            const uint8_t __attribute__((address_space(1))) *at =
                (const uint8_t __attribute__((address_space(1))) *)(kin +
                                                                    static_cast<size_t>(min(t + v, steps - 1)) * step_bytes);
#pragma unroll
            for (int s = 0; s < K; ++s) next[v][s] = at[static_cast<uint32_t>(idx[s])];
        }
    };
    load_block(0);
    __syncthreads();
    auto step = [&](auto par_tag, const uint32_t(&kw)[K]) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par_tag)::value;
        const unsigned char *cur = smem + PAR * kStride;
        auto word_at = [&](uint32_t e) { return *reinterpret_cast<const uint32_t *>(cur + (e >> 16)); };
        auto add = [](uint32_t sum, uint32_t e, uint32_t word) {
            const uint32_t bit = __builtin_amdgcn_ubfe(word, e, 1u);
            if constexpr (WEIGHTS) return __umul24(__builtin_amdgcn_ubfe(e, 5u, 7u), bit) + sum;
            return sum + bit;
        };
        uint32_t sum[K];
#pragma unroll
        for (int s = 0; s < K; ++s) sum[s] = kw[s];
        // N entries of slot S from C on; the reads all before the first sum
        // (left to itself the compiler waits for each)
        auto read = [&](auto s_tag, auto c_tag, auto &x) __attribute__((always_inline)) {
            constexpr int S = decltype(s_tag)::value, C = decltype(c_tag)::value;
            constexpr int N = sizeof(x) / sizeof(x[0]);
            // opaque, or the addresses are taken apart once for all steps and
            // need twice the registers
#pragma unroll
            for (int e = 0; e < N; ++e) asm volatile("" : "+v"(ent[S][C + e]));
#pragma unroll
            for (int e = 0; e < N; ++e) x[e] = word_at(ent[S][C + e]);
        };
        auto sum_up = [&](auto s_tag, auto c_tag, auto &x) __attribute__((always_inline)) {
            constexpr int S = decltype(s_tag)::value, C = decltype(c_tag)::value;
            constexpr int N = sizeof(x) / sizeof(x[0]);
#pragma unroll
            for (int e = 0; e < N; ++e) sum[S] = add(sum[S], ent[S][C + e], x[e]);
        };
        constexpr std::integral_constant<int, 0> at0{};
        // the first kFirst entries of every slot with no branch between them,
        // then each slot's rest four at a time
        uint32_t first[K][kFirst];
        unroll<K>([&](auto s_tag) __attribute__((always_inline)) { read(s_tag, at0, first[decltype(s_tag)::value]); });
        __builtin_amdgcn_sched_barrier(0);
        unroll<K>([&](auto s_tag) __attribute__((always_inline)) { sum_up(s_tag, at0, first[decltype(s_tag)::value]); });
        unroll<(kCached - kFirst) / kChunk>([&](auto n_tag) __attribute__((always_inline)) {
            constexpr int C = kFirst + kChunk * decltype(n_tag)::value;
            if (longest <= C) return;
            unroll<K>([&](auto s_tag) __attribute__((always_inline)) {
                if (len[decltype(s_tag)::value] > C) {
                    uint32_t x[kChunk];
                    read(s_tag, std::integral_constant<int, C>{}, x);
                    __builtin_amdgcn_sched_barrier(0);
                    sum_up(s_tag, std::integral_constant<int, C>{}, x);
                }
            });
        });
#pragma unroll
        for (int s = 0; s < K; ++s) {
#pragma unroll 1
            for (int32_t c = kCached; c < len[s]; c += 2) {
                const uint32_t e0 = rows[s][c * 64 + lane] + mine, e1 = rows[s][(c + 1) * 64 + lane] + mine;
                const uint32_t x0 = word_at(e0), x1 = word_at(e1);
                sum[s] = add(add(sum[s], e0, x0), e1, x1);
            }
        }
#pragma unroll
        for (int s = 0; s < K; ++s) {
            // 128 - threshold + count reaches 128 iff the p-bit turns up; a
            // byte 0 holds it
            const uint64_t on = __ballot(sum[s] >= 128u), live = __ballot(kw[s] != 0u);
            up[s] = (on & live) | (up[s] & ~live);
        }
        store(std::integral_constant<int, 1 - PAR>{});
        __syncthreads();
    };
    for (int32_t t = 0; t < steps; t += kBlock) {
#pragma unroll
        for (int v = 0; v < kBlock; ++v)
#pragma unroll
            for (int s = 0; s < K; ++s) {
                // waited for here, before the next loads are issued
                asm volatile("" : "+v"(next[v][s]));
                kb[v][s] = valid[s] ? next[v][s] : 0u;
            }
        load_block(t + kBlock);
#pragma unroll
        for (int v = 0; v < kBlock; v += 2) {
            if (t + v < steps) step(std::integral_constant<int, 0>{}, kb[v]);
            if (t + v + 1 < steps) step(std::integral_constant<int, 1>{}, kb[v + 1]);
        }
    }
#pragma unroll
    for (int s = 0; s < K; ++s)
        if (valid[s])
            a.spins[static_cast<size_t>(idx[s]) * a.t4 + k] = (up[s] >> lane & 1u) != 0u ? int8_t(1) : int8_t(-1);
}

// acc + the ones of x, in the instruction that does both (the compiler counts
// from zero and adds up afterwards).
__device__ __forceinline__ uint32_t count_bits(uint32_t x, uint32_t acc) {
    uint32_t r;
    asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(acc));
    return r;
}

// The same for at most 1,024 p-bits and weights +-1, one position per lane:
// its row as W words of bits (neighbours, and those with J < 0) in registers,
// the step's spins as W words read by every lane.  Two instructions per 32
// p-bits whatever the row's length.
template <int W>
__device__ __forceinline__ void run_steps_masked(const AheadArgs &a, int32_t k, uint32_t *spin) {
    const uint32_t lane = threadIdx.x & 63u;
    const int32_t w = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(threadIdx.x >> 6));
    const bool have = w < a.bw;
    const bool valid = have && 64 * w + static_cast<int32_t>(lane) < a.n;
    const int32_t idx = valid ? (a.border + 64 * w)[lane] : 0;
    const int32_t np = 64 * a.bw;
    const uint32_t *mask = a.bm + (have ? 64 * w : 0) + lane;
    uint32_t nz[W], neg[W];
#pragma unroll
    for (int j = 0; j < W; ++j) {
        const int32_t at = min(j, 2 * a.bw - 1);
        nz[j] = mask[(2 * at) * np];
        neg[j] = mask[(2 * at + 1) * np];
    }
#pragma unroll
    for (int j = 0; j < W; ++j) {
        asm volatile("" : "+v"(nz[j]), "+v"(neg[j]));
        nz[j] = j < 2 * a.bw ? nz[j] : 0u;
    }
    uint64_t up = __ballot(valid && a.spins[static_cast<size_t>(idx) * a.t4 + k] > 0);
    auto store = [&](int par) __attribute__((always_inline)) {
        if (lane == 0 && have) reinterpret_cast<uint64_t *>(spin + par * 32)[w] = up;
    };
    if (threadIdx.x < 64) spin[threadIdx.x] = 0u;
    __syncthreads();
    store(0);
    const int32_t steps = a.c_end - a.c_begin;
    const size_t step_bytes = static_cast<size_t>(a.trials) * a.waves * 256;
    const uint8_t *kin = a.in + static_cast<size_t>(k) * a.waves * 256;
    constexpr int kBlock = 8;
    uint32_t kb[kBlock], next[kBlock];
    auto load_block = [&](int32_t t) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < kBlock; ++v)
            next[v] = ((const uint8_t __attribute__((address_space(1))) *)(
                kin + static_cast<size_t>(min(t + v, steps - 1)) * step_bytes))[static_cast<uint32_t>(idx)];
    };
    load_block(0);
    __syncthreads();
    for (int32_t t = 0; t < steps; t += kBlock) {
#pragma unroll
        for (int v = 0; v < kBlock; ++v) {
            asm volatile("" : "+v"(next[v]));
            kb[v] = valid ? next[v] : 0u;
        }
        load_block(t + kBlock);
#pragma unroll
        for (int v = 0; v < kBlock; ++v) {
            if (t + v < steps) {
                const u32x4 *cur = reinterpret_cast<const u32x4 *>(spin + (v & 1) * 32);
                u32x4 u[W / 4];
#pragma unroll
                for (int j = 0; j < W / 4; ++j) u[j] = cur[j];
                uint32_t sum[2] = {kb[v], 0u};
#pragma unroll
                for (int j = 0; j < W; ++j)  // (u ^ neg) & nz
                    sum[j & 1] = count_bits(__builtin_amdgcn_bitop3_b32(u[j / 4][j % 4], neg[j], nz[j], 0x28), sum[j & 1]);
                const uint64_t on = __ballot(sum[0] + sum[1] >= 128u), live = __ballot(kb[v] != 0u);
                up = (on & live) | (up & ~live);
                store(1 - (v & 1));
                __syncthreads();
            }
        }
    }
    if (valid) a.spins[static_cast<size_t>(idx) * a.t4 + k] = (up >> lane & 1u) != 0u ? int8_t(1) : int8_t(-1);
}

template <int W>
__global__ __launch_bounds__(1024) void ahead_masked_kernel(AheadArgs a) {
    __shared__ __align__(16) uint32_t spin[64];
    const int32_t b = static_cast<int32_t>(blockIdx.x);
    if (b < a.consumers)
        run_steps_masked<W>(a, b, spin);
    else
        draw_thresholds(a, b - a.consumers, static_cast<int32_t>(gridDim.x) - a.consumers);
}

template <int K, bool WEIGHTS>
__global__ __launch_bounds__(1024) void ahead_kernel(AheadArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int32_t b = static_cast<int32_t>(blockIdx.x);
    if (b < a.consumers)
        run_steps<K, WEIGHTS>(a, b, smem);
    else
        draw_thresholds(a, b - a.consumers, static_cast<int32_t>(gridDim.x) - a.consumers);
}

// Workgroup (wv, c) writes kBuildEntries entries of positions 64 wv .. 64 wv +
// 63 (longest rows first, so the first wavefront's are the most): the
// neighbour's row of words (1 - u for J < 0) as a byte address << 16, |J| << 5
// and its bit; 0 (the zero row) past a row's end.
constexpr int32_t kBuildEntries = 4;
__global__ __launch_bounds__(64) void build_bit_rows_kernel(int32_t n, int32_t bw, const int32_t *__restrict__ row_ptr,
                                                            const int32_t *__restrict__ col,
                                                            const int32_t *__restrict__ val,
                                                            const int32_t *__restrict__ border,
                                                            const int32_t *__restrict__ place,
                                                            const int32_t *__restrict__ bofs, uint32_t *__restrict__ be) {
    const int32_t wv = static_cast<int32_t>(blockIdx.x), lane = static_cast<int32_t>(threadIdx.x);
    const int32_t pos = 64 * wv + lane;
    const int32_t i = pos < n ? border[pos] : 0;
    const int32_t b = pos < n ? row_ptr[i] : 0, e = pos < n ? row_ptr[i + 1] : 0;
    const int32_t g0 = bofs[wv] + static_cast<int32_t>(blockIdx.y) * kBuildEntries;
    const int32_t g1 = min(g0 + kBuildEntries, bofs[wv + 1]);
    for (int32_t g = g0; g < g1; ++g) {
        const int32_t x = b + (g - bofs[wv]);
        uint32_t word = 0u;
        if (x < e) {
            const int32_t p = place[col[x]], J = val[x];
            const int32_t row = 1 + (p >> 5) + (J < 0 ? 2 * bw : 0);
            word = static_cast<uint32_t>(row * kRowBytes) << 16 | static_cast<uint32_t>(J < 0 ? -J : J) << 5 |
                   static_cast<uint32_t>(p & 31);
        }
        be[static_cast<size_t>(g) * 64 + lane] = word;
    }
}

// Workgroup wv writes the masks of positions 64 wv .. 64 wv + 63 from their
// entries, collected in LDS: words 2 j and 2 j + 1 of a position, 64 bw apart,
// hold its neighbours among positions 32 j .. 32 j + 31 and those with J < 0.
__global__ __launch_bounds__(64) void build_masks_kernel(int32_t bw, const int32_t *__restrict__ bofs,
                                                         const uint32_t *__restrict__ be, uint32_t *__restrict__ bm) {
    __shared__ uint32_t word[64][64];
    const int32_t wv = static_cast<int32_t>(blockIdx.x), lane = static_cast<int32_t>(threadIdx.x);
    for (int32_t j = 0; j < 4 * bw; ++j) word[j][lane] = 0u;  // each lane its own column
    for (int32_t g = bofs[wv]; g < bofs[wv + 1]; ++g) {
        const uint32_t e = be[static_cast<size_t>(g) * 64 + lane];
        if (e == 0u) continue;  // past the row's end
        const int32_t row = static_cast<int32_t>(e >> 16) / kRowBytes - 1;
        const int32_t neg = row >= 2 * bw ? 1 : 0, j = row - 2 * bw * neg;
        word[2 * j][lane] |= 1u << (e & 31u);
        if (neg) word[2 * j + 1][lane] |= 1u << (e & 31u);
    }
    for (int32_t j = 0; j < 4 * bw; ++j) bm[j * 64 * bw + 64 * wv + lane] = word[j][lane];
}

}  // namespace

hipError_t launch_build_bit_rows(hipStream_t stream, int32_t n, int32_t bw, int32_t most, const int32_t *row_ptr, const int32_t *col,
                                 const int32_t *val, const int32_t *border, const int32_t *place, const int32_t *bofs,
                                 uint32_t *be, uint32_t *bm) {
    if (bw <= 0 || most <= 0) return hipSuccess;
    const int32_t parts = (most + kBuildEntries - 1) / kBuildEntries;
    hipLaunchKernelGGL(build_bit_rows_kernel, dim3(bw, parts), dim3(64), 0, stream, n, bw, row_ptr, col, val, border,
                       place, bofs, be);
    if (bm) hipLaunchKernelGGL(build_masks_kernel, dim3(bw), dim3(64), 0, stream, bw, bofs, be, bm);
    return hipGetLastError();
}

hipError_t launch_ahead(hipStream_t stream, const DevGraph &g, const DevRun &run, uint8_t *buf, size_t buf_bytes,
                        int32_t num_cu, int32_t t_begin, int32_t t_end, int64_t *launches) {
    *launches = 0;
    AheadArgs a{};
    a.n = g.n;
    a.n4 = g.n4;
    a.t4 = run.t4;
    a.tasks = g.n4 / 4;
    a.waves = (a.tasks + 63) / 64;
    a.trials = run.trials;
    a.gorder = g.gorder;
    a.pps = run.pps;
    a.border = g.border;
    a.bofs = g.bofs;
    a.be = g.be;
    a.bm = g.bm;
    a.bw = (g.n + 63) / 64;
    a.i0 = run.i0;
    a.lam = run.lambda;
    a.dlt = run.delta;
    a.k0 = run.key0;
    a.k1 = run.key1;
    a.gated = run.gated;
    a.spins = run.spins;
    const size_t step_bytes = static_cast<size_t>(a.trials) * a.waves * 256;
    const int64_t most = std::min<int64_t>(kAheadChunk, static_cast<int64_t>(buf_bytes / 2 / step_bytes));
    if (g.n > kAheadMaxN || !g.be || !g.gorder || !run.pps || a.trials >= num_cu || most < 1) return hipErrorInvalidValue;
    uint8_t *half[2] = {buf, buf + buf_bytes / 2};
    const int32_t K = g.n <= 1024 ? 1 : (g.n <= 2048 ? 2 : 4);
    // at least a wavefront for every set of tasks
    const int32_t block = K == 1 ? std::max(256, 64 * a.bw) : 1024;
    // a compute unit holds 1,024 threads of this kernel's registers
    const int32_t per_cu = 1024 / block;
    // masks: two instructions per 32 p-bits (2 bw words), against three per
    // entry of the longest rows (800 p-bits of degree 48 in 640 ns per step
    // against 2.2 us by entries; 250 of degree 6 in 0.22 against 0.46)
    const bool masked = g.bm != nullptr && 4 * a.bw + 8 <= 3 * std::max(g.max_degree, 16);
    const size_t lds = masked ? 0 : 2 * static_cast<size_t>(ahead_stride(K));
    void (*kern)(AheadArgs);
    if (masked)
        kern = a.bw <= 4 ? ahead_masked_kernel<8> : (a.bw <= 8 ? ahead_masked_kernel<16>
                                                                : (a.bw <= 14 ? ahead_masked_kernel<28> : ahead_masked_kernel<32>));
    else if (K == 1)
        kern = g.e1j ? ahead_kernel<1, true> : ahead_kernel<1, false>;
    else if (K == 2)
        kern = g.e1j ? ahead_kernel<2, true> : ahead_kernel<2, false>;
    else
        kern = g.e1j ? ahead_kernel<4, true> : ahead_kernel<4, false>;
    const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (err != hipSuccess) return err;
    // the first chunks are short (nothing runs while the first is drawn) and
    // double up to the most
    int32_t next = t_begin, len = 16;
    a.c_begin = a.c_end = t_begin;
    for (int32_t k = 0; next < t_end || a.c_begin < a.c_end; ++k) {
        a.p_begin = next;
        a.p_end = static_cast<int32_t>(std::min<int64_t>(t_end, int64_t{next} + std::min<int64_t>(len, most)));
        a.consumers = a.c_begin < a.c_end ? a.trials : 0;
        a.in = half[(k + 1) & 1];
        a.out = half[k & 1];
        const int64_t items = int64_t{a.p_end - a.p_begin} * a.trials * a.waves;
        const int64_t wanted = items > 0 ? (std::max<int64_t>(items, a.waves) * 64 + block - 1) / block : 0;
        const int32_t draw = static_cast<int32_t>(std::min<int64_t>(int64_t{num_cu - a.consumers} * per_cu, wanted));
        hipLaunchKernelGGL(kern, dim3(a.consumers + draw), dim3(block), lds, stream, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        ++*launches;
        a.c_begin = a.p_begin;
        a.c_end = a.p_end;
        next = a.p_end;
        len = std::min(2 * len, kAheadChunk);
    }
    return hipSuccess;
}

}  // namespace psa
