// ell_sweep.hpp -- sweep of graphs whose rows stream from device memory (gfx950).
//
// One workgroup owns one trial or four trials of a run, keeps their spins in
// LDS and runs every step of the launch; a lane updates a whole task (four
// consecutive p-bits, one random block per purpose and trial).  The rows are
// read at every step as ELL groups laid out for the wavefront that reads
// them: the tasks in one order per graph (longest rows first), 64 tasks to a
// wavefront, every row of a wavefront padded to the wavefront's longest, so
// that a load is 1 KB contiguous, the loop bounds are scalar and no entry is
// masked.  The per-p-bit constants lie in the same order (16 bytes per p-bit).
//
// What bounds it: vector issue (four trials) and, with one trial, LDS gathers
// and issue about equally.  An all-register add, xor, shift right, bitop3 or
// float multiply-add of a wavefront takes about 2.8 cycles, one with a scalar
// operand, a compare, a convert or a 32-bit product 4.6 to 5, an exponential
// or reciprocal 8.6 (measured on this chip).  Hence: round keys in vector
// registers; the parts of the first three random rounds that depend only on
// step, trial and purpose on the scalar unit, once per step (34 vector
// instructions per block instead of 40); the signed logistic form of the
// decision (no absolute value, sign or clamp); decisions and gates combined
// as sign masks rather than compares and selects.
//
// Measured against the sweep over per-task rows it took the place of (20,000
// p-bits of degree 4, timing gate): 1,024 trials, four per workgroup, 30.1 ->
// 21.2 us per step (9.7e11 updates/s); 100 trials, one per workgroup (100 of
// the 256 compute units), 14.7 -> 7.3 us; 4,001 p-bits of degree 12, weights
// +-1..+-7, 37 trials, 13.6 -> 4.0 us.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_math.hpp"
#include "engine.hpp"

namespace psa {
namespace {

// Keep a value in a vector register (round keys and mask constants: as a
// scalar operand or literal they would cost the slower form at each use).
__device__ __forceinline__ uint32_t in_vgpr(uint32_t x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Keys of rounds 3..9 of the random block (the earlier ones enter the scalar
// prefix), in vector registers.
struct RoundKeys {
    uint32_t k0[7], k1[7];
};
template <bool VGPR = true>
__device__ __forceinline__ RoundKeys round_keys(uint32_t k0, uint32_t k1) {
    RoundKeys K;
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        K.k0[i] = k0 + static_cast<uint32_t>(i + 3) * 0x9E3779B9u;
        K.k1[i] = k1 + static_cast<uint32_t>(i + 3) * 0xBB67AE85u;
        if constexpr (VGPR) {
            K.k0[i] = in_vgpr(K.k0[i]);
            K.k1[i] = in_vgpr(K.k1[i]);
        }
    }
    return K;
}

// The part of blocks (t, m, k, tag) that is the same for every task m.  With
// c0 = t, c2 = k and c3 = tag uniform and c1 = m, round 0 leaves c0 = x ^ m
// and the rest uniform; round 1 needs one lane product, round 2 the other.
struct BlockPrefix {
    uint32_t x;  // round 0: hi(M1 k) ^ k0[0]
    uint32_t a;  // round 1: lo(M0 t) ^ k1[1]
    uint32_t b;  // round 2: lo(M1 c2) ^ k0[2], c2 of round 0
    uint32_t c;  // round 2: hi(M0 c0) ^ k1[2], c0 of round 1
    uint32_t e;  // round 3: lo(M0 c0) ^ k1[3]
};
__device__ __forceinline__ BlockPrefix block_prefix(uint32_t t, uint32_t k, uint32_t tag, uint32_t k0,
                                                    uint32_t k1) {
    const uint64_t p0 = static_cast<uint64_t>(0xD2511F53u) * t;
    const uint64_t p1 = static_cast<uint64_t>(0xCD9E8D57u) * k;
    const uint32_t c2 = static_cast<uint32_t>(p0 >> 32) ^ tag ^ k1;
    const uint64_t q1 = static_cast<uint64_t>(0xCD9E8D57u) * c2;
    const uint32_t c0 = static_cast<uint32_t>(q1 >> 32) ^ static_cast<uint32_t>(p1) ^ (k0 + 0x9E3779B9u);
    const uint64_t s0 = static_cast<uint64_t>(0xD2511F53u) * c0;
    BlockPrefix P;
    P.x = static_cast<uint32_t>(p1 >> 32) ^ k0;
    P.a = static_cast<uint32_t>(p0) ^ (k1 + 0xBB67AE85u);
    P.b = static_cast<uint32_t>(q1) ^ (k0 + 2u * 0x9E3779B9u);
    P.c = static_cast<uint32_t>(s0 >> 32) ^ (k1 + 2u * 0xBB67AE85u);
    P.e = static_cast<uint32_t>(s0) ^ (k1 + 3u * 0xBB67AE85u);
    return P;
}
// The block of task m under its prefix: the same ten rounds as philox4x32_10.
__device__ __forceinline__ Words4 block_of_task(uint32_t m, const BlockPrefix &P, const RoundKeys &K) {
    const uint64_t r1 = static_cast<uint64_t>(0xD2511F53u) * (P.x ^ m);
    const uint32_t n2 = static_cast<uint32_t>(r1 >> 32) ^ P.a;
    const uint64_t r2 = static_cast<uint64_t>(0xCD9E8D57u) * n2;
    uint32_t c0 = static_cast<uint32_t>(r2 >> 32) ^ P.b;
    uint32_t c2 = static_cast<uint32_t>(r1) ^ P.c;
    uint32_t c1 = static_cast<uint32_t>(r2), c3 = 0u;
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        const uint64_t p0 = static_cast<uint64_t>(0xD2511F53u) * c0;
        const uint64_t p1 = static_cast<uint64_t>(0xCD9E8D57u) * c2;
        c0 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(p1 >> 32), c1, K.k0[i], 0x96);
        c2 = i == 0 ? (static_cast<uint32_t>(p0 >> 32) ^ P.e)  // c3 of round 3 is uniform
                    : __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(p0 >> 32), c3, K.k1[i], 0x96);
        c1 = static_cast<uint32_t>(p1);
        c3 = static_cast<uint32_t>(p0);
    }
    return Words4{c0, c1, c2, c3};
}

// Decision as a signed distance.  With f in [1, 2) holding the top 23 bits of
// the r word, (1 + r) / 2 = f - 1 to within 2^-23, and tanh(x) = 1 - 2 q with
// q = 1 / (2^v + 1), v = 2 log2(e) x, so tanh(x) > r iff D = q + (f - 2) < 0,
// and |tanh(x) - r| = 2 |D|.  The estimate of D is off by less than 2^-20:
// f by 2^-23; q by 2^-22 relative (hardware exponential and reciprocal), and
// through v = I0 (L/2 P1 + P2), P1 = 4 lambda log2 e and P2 = 2 lambda delta
// log2 e rounded once, sum and product once: relative errors of v move q by
// less than 2^-22 (v q^2 2^v <= 0.33), and the rounding of P2 by 0.18 * 2^-24
// |2 I0 lambda delta log2 e|, which the bound on |I0 lambda delta|
// (kEstimateLimit) keeps below 2^-19; where the sum in v may overflow no I0
// passes.  Past |D| = kCloseD the sign is therefore tanh_f32's decision; the
// rest evaluates tanh_f32.
constexpr float kCloseD = 0x1p-17f;
constexpr float kTwoLog2e = 0x1.715476p+1f;
__device__ __forceinline__ float decision_distance(float v, uint32_t rword) {
    const float f = __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, rword, 9u));  // 1.0 | top 23 bits
    return __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(v) + 1.0f) + (f - 2.0f);
}
// Least magnitude of four distances.  minnum passes over a not-a-number: with
// four of them the result is one and no `> close_d` holds; with fewer, close_d
// is infinite (a schedule within i0_lim overflows nothing) and none holds either.
__device__ __forceinline__ float least_of(const float (&d)[4]) {
    return fminf(fminf(fminf(fabsf(d[0]), fabsf(d[1])), fabsf(d[2])), fabsf(d[3]));
}
// Bytes 0 and 1 (HALF 0) or 2 and 3 (HALF 1) all ones where lo or hi is
// negative; the other bytes 0.
template <int HALF>
__device__ __forceinline__ uint32_t sign_bytes(uint32_t lo, uint32_t hi) {
    return __builtin_amdgcn_perm(hi, lo, HALF == 0 ? 0x0C0C0B09u : 0x0B090C0Cu);
}
// Uniform loads of run arrays the kernel never writes, through the scalar unit.
template <typename T>
__device__ __forceinline__ T load_uniform(const T *p) {
    return *(const T __attribute__((address_space(4))) *)(p);
}
// 16-byte load at a uniform address plus a lane's byte offset.
__device__ __forceinline__ u32x4 load_lane_x4(const uint32_t *base, uint32_t off) {
    const char __attribute__((address_space(1))) *b = (const char __attribute__((address_space(1))) *)(base);
    return *(const u32x4 __attribute__((address_space(1))) *)(b + off);
}
// All ones when negative, else 0.
__device__ __forceinline__ uint32_t sign_mask(uint32_t x) {
    return static_cast<uint32_t>(static_cast<int32_t>(x) >> 31);
}

enum : int { kEllUnit = 0, kEllByte = 1, kEllHalf = 2 };

// LDS of the four-trial body: [n4 + 1] pairs of words (the two step parities
// of a p-bit's four 0/1 bytes side by side, the last pair zero).
// LDS of the one-trial body: per parity n4 bytes u = (m + 1) / 2, n4 bytes
// 1 - u, and a zero byte (and up to 15 of padding).

// One group word of four trials: neighbour's word address (bits 0..17, 8 per
// p-bit), |J| (bits 18..30; 0 in padding, unused with unit weights), sign.
constexpr uint32_t kEll4Addr = 0x3FFFFu;

template <int MODE>
struct Ell4Sum {
    uint32_t lo[4];  // per row of the task: byte counts, or (kEllHalf) trials 0 and 2
    uint32_t hi[MODE == kEllHalf ? 4 : 1];  // kEllHalf: trials 1 and 3
};

template <int MODE>
__device__ __forceinline__ void ell4_add(Ell4Sum<MODE> &s, int p, uint32_t ev, uint32_t w, uint32_t ones) {
    // the sign complements the four 0/1 bytes
    const uint32_t x = __builtin_amdgcn_bitop3_b32(w, sign_mask(ev), ones, 0x78);  // w ^ (sign & ones)
    if constexpr (MODE == kEllUnit) {
        s.lo[p] += x;
    } else {
        const uint32_t j = (ev >> 18) & 0x1FFFu;
        if constexpr (MODE == kEllByte) {
            s.lo[p] += j * x;
        } else {
            s.lo[p] += j * (x & 0x00FF00FFu);
            s.hi[p] += j * ((x >> 8) & 0x00FF00FFu);
        }
    }
}

// Count of trial kk as a float.
template <int MODE>
__device__ __forceinline__ float ell4_count(const Ell4Sum<MODE> &s, int p, int kk) {
    if constexpr (MODE == kEllHalf) {
        const uint32_t w = (kk & 1) ? s.hi[p] : s.lo[p];
        return static_cast<float>((kk & 2) ? w >> 16 : w & 0xFFFFu);
    } else {
        return static_cast<float>((s.lo[p] >> (8 * kk)) & 0xFFu);
    }
}

// Four trials per workgroup: trial group q of the run, steps a.t_begin ..
// a.t_end-1; any workgroup size (a multiple of 64).
template <int MODE, int ALG>
__device__ __forceinline__ void ell4_steps(const AnnealArgs &a, int32_t q, unsigned char *smem) {
    const int32_t n4 = a.n4, tasks = a.tasks;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t ones = in_vgpr(0x01010101u);
    const bool need_gate = ALG != kAlgPeriod && a.gated != 0;
    const RoundKeys keys = round_keys(a.k0, a.k1);
    const bool resident = tasks <= static_cast<int32_t>(blockDim.x);
    const int32_t nsub = ALG == kAlgPeriod ? a.t_res : 1;
    u32x4 c[4] = {};
    uint32_t m = 0;
    // wavefronts of tasks; the last one's idle lanes run along and store nothing
    const int32_t waves = (tasks + 63) >> 6;
    const int32_t wave = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(threadIdx.x >> 6));
    const int32_t nwaves = static_cast<int32_t>(blockDim.x >> 6);
    bool load = true;
    uint32_t par = 0;  // byte offset of the current parity's word: 0 or 4
    for (int32_t t = a.t_begin; t < a.t_end; ++t) {
        const float i0s = load_uniform(a.i0 + t);
        const float i0t = __uint_as_float(in_vgpr(__float_as_uint(i0s)));
        const float close_d = fabsf(i0s) <= a.i0_lim ? kCloseD : __builtin_inff();
        for (int32_t s = 0; s < nsub; ++s) {
            const uint32_t tau = static_cast<uint32_t>(t) * static_cast<uint32_t>(nsub) + static_cast<uint32_t>(s);
            BlockPrefix pr[4], pg[4];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                pr[kk] = block_prefix(tau, static_cast<uint32_t>(4 * q + kk), kTagR, a.k0, a.k1);
                if (ALG != kAlgPeriod) pg[kk] = block_prefix(tau, static_cast<uint32_t>(4 * q + kk), kTagGate, a.k0, a.k1);
            }
            for (int32_t w = wave; w < waves; w += nwaves) {
                const bool valid = 64 * w + static_cast<int32_t>(lane) < tasks;
                if (load) {
                    m = static_cast<uint32_t>((a.gorder + 64 * w)[lane]);
                    const uint32_t *pp = a.pps + static_cast<size_t>(w) * 1024;
#pragma unroll
                    for (int p = 0; p < 4; ++p) c[p] = load_lane_x4(pp + p * 256, lane * 16u);
                }
                const unsigned char *cur = smem + par;
                uint32_t word[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) word[p] = *reinterpret_cast<const uint32_t *>(cur + (m << 5) + 8 * p);
                unsigned char *to = smem + (par ^ 4u) + (m << 5);
                if constexpr (ALG == kAlgPeriod) {
                    // p-bits whose period does not divide the sub-step hold
                    const bool any = period_fires(tau, c[0].w) | period_fires(tau, c[1].w) |
                                     period_fires(tau, c[2].w) | period_fires(tau, c[3].w);
                    if (__ballot(any) == 0u) {
                        if (valid) {
#pragma unroll
                            for (int p = 0; p < 4; ++p) *reinterpret_cast<uint32_t *>(to + 8 * p) = word[p];
                        }
                        continue;
                    }
                }
                // neighbour sums: groups four (then two) at a time
                Ell4Sum<MODE> sum = {};
                const int32_t g0 = load_uniform(a.wofs + w), g1 = load_uniform(a.wofs + w + 1);  // pairs of groups
                const uint32_t *ep = a.e4 + static_cast<size_t>(g0) * 512;
                auto groups = [&](auto u_tag) __attribute__((always_inline)) {
                    constexpr int U = decltype(u_tag)::value;
                    u32x4 ev[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) ev[u] = load_lane_x4(ep + u * 256, lane * 16u);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const uint32_t e[4] = {ev[u].x, ev[u].y, ev[u].z, ev[u].w};
                        uint32_t x[4];
#pragma unroll
                        for (int p = 0; p < 4; ++p)
                            x[p] = *reinterpret_cast<const uint32_t *>(cur + (e[p] & kEll4Addr));
#pragma unroll
                        for (int p = 0; p < 4; ++p) ell4_add<MODE>(sum, p, e[p], x[p], ones);
                    }
                    ep += U * 256;
                };
                int32_t g = g0;
                for (; g + 2 <= g1; g += 2) groups(std::integral_constant<int, 4>{});
                if (g < g1) groups(std::integral_constant<int, 2>{});
                float ac[4], bc[4], hd[4];
                uint32_t th[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    hd[p] = __uint_as_float(c[p].x);
                    ac[p] = i0t * __uint_as_float(c[p].y);
                    // SpSA and TApSA: I0 lambda and delta themselves
                    bc[p] = ALG == kAlgPsa || ALG == kAlgPeriod ? i0t * __uint_as_float(c[p].z) : __uint_as_float(c[p].z);
                    th[p] = c[p].w;
                }
                const int32_t i0 = static_cast<int32_t>(4 * m);
                // TApSA window sums (without this step's field) and SpSA held
                // inputs of the task's four trials, 16 bytes per access
                const uint32_t al = static_cast<uint32_t>(a.alpha);
                const uint32_t count = tau + 1 < al ? tau + 1 : al;
                const size_t row = static_cast<size_t>(q) * n4 + i0;
                u32x4 state[4] = {};
                if constexpr (ALG == kAlgTapsa) {
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        for (uint32_t s2 = 1; s2 < count; ++s2)
                            state[p] += load_global_x4(a.ring + ((row + p) * al + (tau - s2) % al) * 4);
                } else if constexpr (ALG == kAlgSpsa) {
                    if (t > 0) {
#pragma unroll
                        for (int p = 0; p < 4; ++p) state[p] = load_global_x4(a.xs + (row + p) * 4);
                    }
                }
                uint32_t up[4] = {0u, 0u, 0u, 0u}, fire[4] = {0u, 0u, 0u, 0u};
                // trials two at a time: a byte pair of the new words each
#pragma unroll
                for (int H = 0; H < 2; ++H) {
                    uint32_t gs[2][4] = {};
                    float d[2][4];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int kk = 2 * H + h;
                        const uint32_t k = static_cast<uint32_t>(4 * q + kk);
                        if (need_gate) {
                            const Words4 gb = block_of_task(m, pg[kk], keys);
                            const uint32_t gw[4] = {gb.x, gb.y, gb.z, gb.w};
#pragma unroll
                            for (int p = 0; p < 4; ++p)  // negative iff (gw >> 8) < th, both below 2^25
                                gs[h][p] = (gw[p] >> 8) - th[p];
                        }
                        const Words4 rb = block_of_task(m, pr[kk], keys);
                        const uint32_t rw[4] = {rb.x, rb.y, rb.z, rb.w};
                        float x[4];
                        bool close;
                        if constexpr (ALG == kAlgPsa || ALG == kAlgPeriod) {
#pragma unroll
                            for (int p = 0; p < 4; ++p)
                                d[h][p] = decision_distance(fmaf(ell4_count(sum, p, kk) + hd[p], ac[p], bc[p]), rw[p]);
                            close = !(least_of(d[h]) > close_d);
                        } else {
                            uint32_t sw[4] = {0u, 0u, 0u, 0u};
                            if (ALG == kAlgSpsa && t > 0) {
                                const Words4 b = philox4x32_10(tau, m, k, kTagStall, a.k0, a.k1);
                                sw[0] = b.x;
                                sw[1] = b.y;
                                sw[2] = b.z;
                                sw[3] = b.w;
                            }
                            close = false;
#pragma unroll
                            for (int p = 0; p < 4; ++p) {
                                const float Lf = 2.0f * (ell4_count(sum, p, kk) + hd[p]);
                                if constexpr (ALG == kAlgTapsa) {
                                    const int32_t L = static_cast<int32_t>(Lf);
                                    const int32_t total = static_cast<int32_t>(state[p][kk]) + L;
                                    state[p][kk] = static_cast<uint32_t>(L);
                                    x[p] = ac[p] * (static_cast<float>(total) / static_cast<float>(count) + bc[p]);
                                } else {
                                    x[p] = t > 0 && (sw[p] >> 8) < a.stall24 ? __uint_as_float(state[p][kk])
                                                                             : ac[p] * (Lf + bc[p]);
                                    state[p][kk] = __float_as_uint(x[p]);
                                }
                                d[h][p] = decision_distance(x[p] * kTwoLog2e, rw[p]);
                                close = close || !(fabsf(d[h][p]) > kCloseD);  // not a number: tanh_f32 decides
                            }
                        }
                        if (__ballot(close) != 0u) {
#pragma unroll
                            for (int p = 0; p < 4; ++p) {
                                if constexpr (ALG == kAlgPsa || ALG == kAlgPeriod)
                                    x[p] = (i0t * a.lam[i0 + p]) * (2.0f * (ell4_count(sum, p, kk) + hd[p]) + a.dlt[i0 + p]);
                                d[h][p] = tanh_f32(x[p]) > r_of(rw[p]) ? -1.0f : 1.0f;
                            }
                        }
                    }
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const uint32_t d0 = __float_as_uint(d[0][p]), d1 = __float_as_uint(d[1][p]);
                        up[p] |= H == 0 ? sign_bytes<0>(d0, d1) : sign_bytes<1>(d0, d1);
                        if (need_gate) fire[p] |= H == 0 ? sign_bytes<0>(gs[0][p], gs[1][p]) : sign_bytes<1>(gs[0][p], gs[1][p]);
                    }
                }
                if constexpr (ALG == kAlgTapsa || ALG == kAlgSpsa) {
                    // this step's fields into their window slot; the inputs held
                    if (valid) {
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            void *to4 = ALG == kAlgTapsa ? static_cast<void *>(a.ring + ((row + p) * al + tau % al) * 4)
                                                         : static_cast<void *>(a.xs + (row + p) * 4);
                            *reinterpret_cast<u32x4 *>(to4) = state[p];
                        }
                    }
                }
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    up[p] &= ones;
                    if constexpr (ALG == kAlgPeriod) {
                        if (!period_fires(tau, th[p])) up[p] = word[p];
                    } else if (need_gate) {
                        up[p] = __builtin_amdgcn_bitop3_b32(fire[p], up[p], word[p], 0xCA);  // fire ? up : word
                    }
                    if (valid) *reinterpret_cast<uint32_t *>(to + 8 * p) = up[p];
                }
            }
            load = !resident;
            __syncthreads();
            par ^= 4u;
        }
    }
    const uint32_t *S = reinterpret_cast<const uint32_t *>(smem + par);
    for (int32_t i = static_cast<int32_t>(threadIdx.x); i < a.n; i += static_cast<int32_t>(blockDim.x)) {
        const uint32_t w = ((S[2 * i] ^ 0x01010101u) * 0xFEu) ^ 0x01010101u;  // 0/1 -> -1/+1
        *reinterpret_cast<uint32_t *>(a.spins + static_cast<size_t>(i) * a.t4 + 4 * q) = w;
    }
}

template <int MODE>
__device__ __forceinline__ void ell4_body(const AnnealArgs &a, int32_t q, unsigned char *smem) {
    uint32_t *S = reinterpret_cast<uint32_t *>(smem);
    for (int32_t i = static_cast<int32_t>(threadIdx.x); i <= a.n4; i += static_cast<int32_t>(blockDim.x)) {
        uint32_t w = 0u;  // the zero pair and padding p-bits
        if (i < a.n)
            w = (~*reinterpret_cast<const uint32_t *>(a.spins + static_cast<size_t>(i) * a.t4 + 4 * q) >> 7) & 0x01010101u;
        S[2 * i] = w;
        if (i == a.n4) S[2 * i + 1] = 0u;
    }
    __syncthreads();
    if (a.t_res > 0)
        ell4_steps<MODE, kAlgPeriod>(a, q, smem);
    else if (a.ring != nullptr)
        ell4_steps<MODE, kAlgTapsa>(a, q, smem);
    else if (a.xs != nullptr)
        ell4_steps<MODE, kAlgSpsa>(a, q, smem);
    else
        ell4_steps<MODE, kAlgPsa>(a, q, smem);
}

// One trial per workgroup.  A pair word holds two neighbours of a row as
// 16-bit byte indices into [u | 1 - u] (n4 + j for J < 0, the zero byte 2 n4
// past the row); with weights a second word holds their |J|.
template <bool WEIGHTS>
__device__ __forceinline__ void ell1_add(uint32_t &acc, uint32_t x0, uint32_t x1, uint32_t j) {
    if constexpr (WEIGHTS) {
        acc += x0 * (j & 0xFFFFu);
        acc += x1 * (j >> 16);
    } else {
        acc += x0 + x1;
        (void)j;
    }
}

template <bool WEIGHTS, int ALG>
__device__ __forceinline__ void ell1_steps(const AnnealArgs &a, int32_t q, unsigned char *smem, uint32_t stride) {
    const int32_t n4 = a.n4, tasks = a.tasks;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t ones = in_vgpr(0x01010101u);
    const bool need_gate = ALG != kAlgPeriod && a.gated != 0;
    const RoundKeys keys = round_keys(a.k0, a.k1);
    const InputState st{a.xs, a.stall24, a.ring, a.alpha, n4};
    const bool resident = tasks <= static_cast<int32_t>(blockDim.x);
    const int32_t nsub = ALG == kAlgPeriod ? a.t_res : 1;
    const uint32_t k = static_cast<uint32_t>(q);
    // The constants and the first two groups of the task a lane updates next
    // are loaded one task ahead (a lane's first task follows its last one),
    // so that their latency does not follow the step's barrier.
    // wavefronts of tasks; the last one's idle lanes run along and store nothing
    const int32_t waves = (tasks + 63) >> 6;
    const int32_t wave = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(threadIdx.x >> 6));
    const int32_t nwaves = static_cast<int32_t>(blockDim.x >> 6);
    u32x4 c[4] = {}, e0[2] = {}, j0[2] = {};
    uint32_t mn = 0;
    int32_t gn0 = 0, gn1 = 0;
    auto fetch = [&](int32_t w) __attribute__((always_inline)) {
        mn = static_cast<uint32_t>((a.gorder + 64 * w)[lane]);
        const uint32_t *pp = a.pps + static_cast<size_t>(w) * 1024;
#pragma unroll
        for (int p = 0; p < 4; ++p) c[p] = load_lane_x4(pp + p * 256, lane * 16u);
        gn0 = load_uniform(a.wofs + w);
        gn1 = load_uniform(a.wofs + w + 1);
        // a wavefront of empty rows reads group 0 or the last one and adds nothing
        const int32_t last = a.groups - 1;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const size_t at = static_cast<size_t>(min(gn0 + u, last)) * 256;
            e0[u] = load_lane_x4(a.e1 + at, lane * 16u);
            if constexpr (WEIGHTS) j0[u] = load_lane_x4(a.e1j + at, lane * 16u);
        }
    };
    if (wave < waves) fetch(wave);
    uint32_t m = mn;
    bool first = true;  // first step: load the input-stage state
    // input stage of a lane that keeps its task (resident): TApSA window sums
    // of the steps before t, SpSA held inputs
    int32_t wsum[4] = {0, 0, 0, 0};
    float held[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    const uint32_t al = static_cast<uint32_t>(a.alpha);
    auto window = [&](int p) __attribute__((always_inline)) {
        return a.ring + (static_cast<size_t>(k >> 2) * n4 + 4 * m + p) * al * 4 + (k & 3u);
    };
    auto input = [&](int p) __attribute__((always_inline)) {
        return a.xs + (static_cast<size_t>(k >> 2) * n4 + 4 * m + p) * 4 + (k & 3u);
    };
    uint32_t base = 0;  // the current parity's buffer: 0 or stride
    for (int32_t t = a.t_begin; t < a.t_end; ++t) {
        const float i0s = load_uniform(a.i0 + t);
        const float i0t = __uint_as_float(in_vgpr(__float_as_uint(i0s)));
        const float close_d = fabsf(i0s) <= a.i0_lim ? kCloseD : __builtin_inff();
        for (int32_t s = 0; s < nsub; ++s) {
            const uint32_t tau = static_cast<uint32_t>(t) * static_cast<uint32_t>(nsub) + static_cast<uint32_t>(s);
            const BlockPrefix pr = block_prefix(tau, k, kTagR, a.k0, a.k1);
            const BlockPrefix pg = block_prefix(tau, k, kTagGate, a.k0, a.k1);
            const unsigned char *cur = smem + base;
            unsigned char *nxt = smem + (stride - base);
            for (int32_t w = wave; w < waves; w += nwaves) {
                m = mn;
                const bool valid = 64 * w + static_cast<int32_t>(lane) < tasks;
                const int32_t g0 = gn0, g1 = gn1;
                const int32_t i0 = static_cast<int32_t>(4 * m);
                float hd[4], p1[4], p2[4];
                uint32_t th[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    hd[p] = __uint_as_float(c[p].x);
                    p1[p] = __uint_as_float(c[p].y);
                    p2[p] = __uint_as_float(c[p].z);
                    th[p] = c[p].w;
                }
                if (first) {
                    if (ALG == kAlgTapsa && resident && valid) {
                        const uint32_t cnt = static_cast<uint32_t>(t) < al ? static_cast<uint32_t>(t) : al;
#pragma unroll
                        for (int p = 0; p < 4; ++p)
                            for (uint32_t i = 1; i <= cnt; ++i) wsum[p] += window(p)[((static_cast<uint32_t>(t) - i) % al) * 4];
                    }
                    if (ALG == kAlgSpsa && resident && valid) {
#pragma unroll
                        for (int p = 0; p < 4; ++p) held[p] = *input(p);
                    }
                }
                // TApSA, resident: the field that leaves the window sits in the
                // slot this step's field takes; its load is issued first
                int32_t leaving[4] = {0, 0, 0, 0};
                const uint32_t at = (static_cast<uint32_t>(t) % al) * 4;
                if (ALG == kAlgTapsa && resident && valid && static_cast<uint32_t>(t) >= al) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) leaving[p] = window(p)[at];
                }
                const uint32_t old = *reinterpret_cast<const uint32_t *>(cur + 4 * m);
                unsigned char *to = nxt + 4 * m;
                if constexpr (ALG == kAlgPeriod) {
                    const bool any = period_fires(tau, th[0]) | period_fires(tau, th[1]) | period_fires(tau, th[2]) |
                                     period_fires(tau, th[3]);
                    if (__ballot(any) == 0u) {
                        if (valid) {
                            *reinterpret_cast<uint32_t *>(to) = old;
                            *reinterpret_cast<uint32_t *>(to + n4) = old ^ 0x01010101u;
                        }
                        if (!resident) fetch(w + nwaves < waves ? w + nwaves : wave);
                        continue;
                    }
                }
                uint32_t acc[4] = {0u, 0u, 0u, 0u};
                auto add = [&](const u32x4 ev, const u32x4 jv) __attribute__((always_inline)) {
                    const uint32_t e[4] = {ev.x, ev.y, ev.z, ev.w}, j[4] = {jv.x, jv.y, jv.z, jv.w};
                    uint32_t x0[4], x1[4];
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        x0[p] = cur[e[p] & 0xFFFFu];
                        x1[p] = cur[e[p] >> 16];
                    }
#pragma unroll
                    for (int p = 0; p < 4; ++p) ell1_add<WEIGHTS>(acc[p], x0[p], x1[p], j[p]);
                };
                const uint32_t *ep = a.e1 + static_cast<size_t>(g0 + 2) * 256;
                const uint32_t *jp = WEIGHTS ? a.e1j + static_cast<size_t>(g0 + 2) * 256 : nullptr;
                auto groups = [&](auto u_tag) __attribute__((always_inline)) {
                    constexpr int U = decltype(u_tag)::value;
                    u32x4 ev[U], jv[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        ev[u] = load_lane_x4(ep + u * 256, lane * 16u);
                        jv[u] = u32x4{0u, 0u, 0u, 0u};
                        if constexpr (WEIGHTS) jv[u] = load_lane_x4(jp + u * 256, lane * 16u);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) add(ev[u], jv[u]);
                    ep += U * 256;
                    jp += U * 256;
                };
                if (g0 < g1) add(e0[0], j0[0]);
                if (g0 + 1 < g1) add(e0[1], j0[1]);
                int32_t g = g0 + 2;
                for (; g + 4 <= g1; g += 4) groups(std::integral_constant<int, 4>{});
                if (g + 2 <= g1) {
                    groups(std::integral_constant<int, 2>{});
                    g += 2;
                }
                if (g < g1) groups(std::integral_constant<int, 1>{});
                if (!resident) fetch(w + nwaves < waves ? w + nwaves : wave);
                uint32_t up, fire = 0u;
                if (need_gate) {
                    const Words4 gb = block_of_task(m, pg, keys);
                    const uint32_t gw[4] = {gb.x, gb.y, gb.z, gb.w};
                    uint32_t gs[4];  // negative iff (gw >> 8) < th, both below 2^25
#pragma unroll
                    for (int p = 0; p < 4; ++p) gs[p] = (gw[p] >> 8) - th[p];
                    fire = sign_bytes<0>(gs[0], gs[1]) | sign_bytes<1>(gs[2], gs[3]);
                }
                const Words4 rb = block_of_task(m, pr, keys);
                const uint32_t rw[4] = {rb.x, rb.y, rb.z, rb.w};
                float d[4], x[4], lh[4];
#pragma unroll
                for (int p = 0; p < 4; ++p)  // half the field, exact
                    lh[p] = static_cast<float>(acc[p]) + hd[p];
                bool close;
                if constexpr (ALG == kAlgPsa || ALG == kAlgPeriod) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) d[p] = decision_distance(i0t * fmaf(lh[p], p1[p], p2[p]), rw[p]);
                    close = !(least_of(d) > close_d);
                } else {
                    uint32_t sw[4] = {0u, 0u, 0u, 0u};
                    if (ALG == kAlgSpsa && t > 0) {
                        const Words4 b = philox4x32_10(tau, m, k, kTagStall, a.k0, a.k1);
                        sw[0] = b.x;
                        sw[1] = b.y;
                        sw[2] = b.z;
                        sw[3] = b.w;
                    }
                    close = false;
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const int32_t L = static_cast<int32_t>(2.0f * lh[p]);
                        const float av = i0t * p1[p], dl = p2[p];  // SpSA and TApSA: lambda and delta themselves
                        if (ALG == kAlgTapsa && resident) {
                            wsum[p] += L - leaving[p];
                            if (valid) window(p)[at] = L;
                            const uint32_t cnt = tau + 1 < al ? tau + 1 : al;
                            x[p] = av * (static_cast<float>(wsum[p]) / static_cast<float>(cnt) + dl);
                        } else if (ALG == kAlgSpsa && resident) {
                            x[p] = t > 0 && (sw[p] >> 8) < st.s24 ? held[p] : av * (static_cast<float>(L) + dl);
                            held[p] = x[p];
                        } else {
                            x[p] = 0.0f;
                            if (valid) x[p] = input_of<ALG>(av, dl, L, st, i0 + p, k, tau, sw[p]);
                        }
                        d[p] = decision_distance(x[p] * kTwoLog2e, rw[p]);
                        close = close || !(fabsf(d[p]) > kCloseD);
                    }
                }
                if (__ballot(close) != 0u) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        if constexpr (ALG == kAlgPsa || ALG == kAlgPeriod)
                            x[p] = (i0t * a.lam[i0 + p]) * (2.0f * lh[p] + a.dlt[i0 + p]);
                        d[p] = tanh_f32(x[p]) > r_of(rw[p]) ? -1.0f : 1.0f;
                    }
                }
                up = __builtin_amdgcn_bitop3_b32(sign_bytes<0>(__float_as_uint(d[0]), __float_as_uint(d[1])),
                                                 sign_bytes<1>(__float_as_uint(d[2]), __float_as_uint(d[3])), ones,
                                                 0xA8);  // (a | b) & c
                if constexpr (ALG == kAlgPeriod) {
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        if (period_fires(tau, th[p])) fire |= 1u << (8 * p);
                    up = __builtin_amdgcn_bitop3_b32(fire, up, old, 0xCA);
                } else if (need_gate) {
                    up = __builtin_amdgcn_bitop3_b32(fire, up, old, 0xCA);
                }
                if (valid) {
                    *reinterpret_cast<uint32_t *>(to) = up;
                    *reinterpret_cast<uint32_t *>(to + n4) = up ^ 0x01010101u;
                }
            }
            first = false;
            __syncthreads();
            base = stride - base;
        }
    }
    if (ALG == kAlgSpsa && resident && static_cast<int32_t>(threadIdx.x) < tasks) {
#pragma unroll
        for (int p = 0; p < 4; ++p) *input(p) = held[p];
    }
    for (int32_t i = static_cast<int32_t>(threadIdx.x); i < a.n; i += static_cast<int32_t>(blockDim.x))
        a.spins[static_cast<size_t>(i) * a.t4 + q] = smem[base + i] ? int8_t(1) : int8_t(-1);
}

template <bool WEIGHTS>
__device__ __forceinline__ void ell1_body(const AnnealArgs &a, int32_t q, unsigned char *smem) {
    const int32_t n4 = a.n4;
    const uint32_t stride = static_cast<uint32_t>(ell1_stride(n4));
    for (int32_t i = static_cast<int32_t>(threadIdx.x); i < n4; i += static_cast<int32_t>(blockDim.x)) {
        const unsigned char u = i < a.n && a.spins[static_cast<size_t>(i) * a.t4 + q] > 0 ? 1 : 0;
        smem[i] = u;
        smem[n4 + i] = u ^ 1u;
    }
    if (threadIdx.x == 0) smem[2 * n4] = smem[stride + 2 * n4] = 0;
    __syncthreads();
    if (a.t_res > 0)
        ell1_steps<WEIGHTS, kAlgPeriod>(a, q, smem, stride);
    else if (a.ring != nullptr)
        ell1_steps<WEIGHTS, kAlgTapsa>(a, q, smem, stride);
    else if (a.xs != nullptr)
        ell1_steps<WEIGHTS, kAlgSpsa>(a, q, smem, stride);
    else
        ell1_steps<WEIGHTS, kAlgPsa>(a, q, smem, stride);
}

}  // namespace
}  // namespace psa
