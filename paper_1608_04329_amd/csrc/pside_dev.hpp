// The p-side role of the sweep kernel: the conditionals of Eq. (12) other
// than z, in float64, computed by a group of gp blocks that run next to the
// z-pass blocks of the same launch.
//
//   lambda_j^-2 ~ Exp(nu_j^-1 + tau^-2 beta_j^2 / 2)
//   tau^-2      ~ Gamma((p+1)/2, rate xi^-1 + sum_j lambda_j^-2 beta_j^2 / 2)
//   nu_j^-1     ~ Exp(1 + lambda_j^-2),   xi^-1 ~ Exp(1 + tau^-2)
//   beta        ~ N(Q^-1 X^T z, Q^-1),  Q = X^T X + tau^-2 Lambda^-2
// (rate parameterisation, Eq. 11; tau^-2 is the Gamma draw of Section 5's
// sampling step, so tau^2 is inverse-gamma).  lambda, tau, nu, xi and the
// Cholesky factorisation of Q depend only on the previous sweep, so the group
// runs them while the z pass streams X; beta waits for the z pass.
//
// beta for p <= 16 (one block): Q in the registers of one wave, factored while the
// z pass runs, then two triangular solves on 16 lanes.
//
// beta for p > 16 (gp blocks, 64 x 64 tiles): a right-looking blocked Cholesky,
// and after the z pass either of two ways to
//   y = U^-T b + s,   beta = U^-1 y = U^-1 U^-T b + U^-1 s,
// mean Q^-1 b plus noise with covariance U^-1 U^-T = Q^-1.  From 7 to 24 tiles
// (p = 385 .. 1536) the factorisation applies its row operations to an identity
// block as well, so it produces U and L^-1 = U^-T together ([Q | I]), and y and
// beta are two parallel triangular products.  With fewer or more tiles, and for
// the chains of a multi-chain pass, it forms the diagonal tiles of L^-1 only, and
// y and beta come from blocked substitution (subst_solve).
//
// Group barriers use a monotonic device counter; every wait is bounded in
// time and sets kErrTimeout instead of hanging.
#pragma once
#include <float.h>

#include "hsp_internal.hpp"
#include "philox.hpp"
#include "sync_dev.hpp"

namespace hsp {

// ---- bounded waits and group barriers ---------------------------------------------
struct Group {
    uint64_t* trace;           // this block's timestamp slots, or null
    Ctrl* ctrl;
    unsigned long long base;   // bar_count when this launch started
    unsigned long long zbase;  // z_count when this launch started
    uint32_t size;
    uint32_t n;                // barriers passed
    uint32_t slot;             // next trace slot
    uint32_t npotrf;           // diagonal tiles factored by this block
    uint64_t timeout;
};

// Sleep about 64 * n cycles between polls.  Polls are coherent loads that
// bypass the L2 and all land on one memory channel: a tight loop from many
// blocks slows the z pass's stream, so every wait backs off exponentially.
__device__ __forceinline__ void backoff(uint32_t& n, uint32_t cap) {
    for (uint32_t i = 0; i < n; ++i) __builtin_amdgcn_s_sleep(1);
    n = n < cap ? 2 * n : cap;
}

// Thread 0 only: wait until *ctr >= target, or give up after the timeout.
// Relaxed polls; what the caller reads afterwards it loads coherently.
__device__ __forceinline__ void wait_count(unsigned long long* ctr, unsigned long long target,
                                        Ctrl* ctrl, uint64_t timeout, uint32_t cap = 16) {
    const uint64_t t0 = wall_clock64();
    uint32_t nap = 1;
    while (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
        if (__hip_atomic_load(&ctrl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrTimeout)
            break;
        if (wall_clock64() - t0 > timeout) {
            atomicOr(&ctrl->err, kErrTimeout);
            break;
        }
        backoff(nap, cap);
    }
}

// Thread 0: next trace timestamp, or a given value (diagnostics only).
__device__ __forceinline__ void stamp(Group& g) {
    if (g.trace && threadIdx.x == 0 && g.slot + 1 < (uint32_t)kTraceSeq) g.trace[++g.slot] = wall_clock64();
}
__device__ __forceinline__ void stamp_value(Group& g, uint64_t v) {
    if (g.trace && threadIdx.x == 0 && g.slot + 1 < (uint32_t)kTraceSeq) g.trace[++g.slot] = v;
}

// Thread 0: timestamp into slot s of a diagonal-factorisation record (or none).
__device__ __forceinline__ void stamp_at(uint64_t* rec, int s) {
    if (rec && threadIdx.x == 0) rec[s] = wall_clock64();
}

// Thread 0 only: wait until *v[i] >= need[i] for i < n (the n loads of a poll
// are in flight together); false if the group is failing or the wait timed
// out.  The tiles read after a success are loaded coherently (ldc).
__device__ __forceinline__ bool wait_vers(uint32_t* const (&v)[3], const uint32_t (&need)[3], int n,
                                          Ctrl* ctrl, uint64_t timeout) {
    uint64_t t0 = 0;
    uint32_t nap = 1;
    for (int it = 0;; ++it) {
        uint32_t got[3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
            got[i] = i < n ? __hip_atomic_load(v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        bool ok = true;
#pragma unroll
        for (int i = 0; i < 3; ++i) ok = ok && (i >= n || got[i] >= need[i]);
        if (ok) return true;
        if (it == 0) t0 = wall_clock64();
        if (__hip_atomic_load(&ctrl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
            (kErrTimeout | kErrNotPD))
            return false;
        if (wall_clock64() - t0 > timeout) {
            atomicOr(&ctrl->err, kErrTimeout);
            return false;
        }
        backoff(nap, 8);
    }
}

// Publish *ver = val (and *ver2 = val2) once this block's coherent tile
// stores are complete: every wave waits for its own stores first.
__device__ __forceinline__ void publish(uint32_t* ver, uint32_t val, uint32_t* ver2 = nullptr,
                                        uint32_t val2 = 0) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        __hip_atomic_store(ver, val, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (ver2) __hip_atomic_store(ver2, val2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__device__ __forceinline__ void group_sync(Group& g) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicAdd(&g.ctrl->bar_count, 1ull);
        if (g.size > 1)
            wait_count(&g.ctrl->bar_count, g.base + (unsigned long long)(g.n + 1) * g.size, g.ctrl,
                       g.timeout);
    }
    g.n++;
    stamp(g);
    __syncthreads();
}

// This block has drawn lambda and tau, and what it stored of them is complete; it
// does not wait for the others.  (A count of its own: on bar_count, a block that
// has run ahead to the next barrier would be taken for one still to come.)
__device__ __forceinline__ void hyper_arrive(Group& g) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(&g.ctrl->hyper_count, 1ull);
    stamp(g);
}

// Every block of the group has arrived there.
__device__ __forceinline__ void hyper_wait(Group& g) {
    if (threadIdx.x == 0 && g.size > 1) wait_count(&g.ctrl->hyper_count, g.size, g.ctrl, g.timeout);
    __syncthreads();
}

// Arrive, then wait for the group and, with a target, for the z pass (z_count
// >= ztarget), both polled in the same loads; the last to arrive knows it from
// its own arrival.  The failure flags are read by the caller, later: a block sets
// them before it arrives.
__device__ __forceinline__ void group_sync_z(Group& g, unsigned long long ztarget) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    g.n++;
    if (threadIdx.x == 0) {
        const unsigned long long target = g.base + (unsigned long long)g.n * g.size;
        bool here = atomicAdd(&g.ctrl->bar_count, 1ull) + 1 >= target;
        stamp(g);
        const uint64_t t0 = wall_clock64();
        uint32_t nap = 1;
        while (!here || ztarget) {
            const unsigned long long bars = __hip_atomic_load(&g.ctrl->bar_count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long zs = __hip_atomic_load(&g.ctrl->z_count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t err = __hip_atomic_load(&g.ctrl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            here = here || bars >= target;
            if ((here && zs >= ztarget) || (err & kErrTimeout)) break;
            if (wall_clock64() - t0 > g.timeout) {
                atomicOr(&g.ctrl->err, kErrTimeout);
                break;
            }
            backoff(nap, here ? 16 : 8);
        }
        if (g.trace && ztarget) g.trace[kTraceSlots - 1] = wall_clock64();
    }
    __syncthreads();
}

// Block-wide float64 sum in a fixed order (identical result in every block).
__device__ __forceinline__ double block_sum(double v, double* red) {
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < kThreads / kWave; ++w) s += red[w];
    __syncthreads();
    return s;
}

__device__ __forceinline__ uint32_t record_slot(Args& a, uint32_t k, bool* keep) {
    const uint32_t since = k - a.ctrl->draw_base;
    *keep = (a.mode & kModeRecord) && since % a.thin == 0;
    return *keep ? (since / a.thin - 1u) % a.capacity : 0u;
}

// LDS offsets (doubles) of what hyper_lambda_tau leaves in red: on the one-block
// path lambda^-2 (16).
constexpr int kRedGamma = 9, kRedLambda = 16;

// ---- lambda^-2 and tau^-2 (every block of the group computes them) ---------------
// Returns tau^-2 (new if kModeTau).  Block `writer` stores lambda^-2 and tau^-2.
// The gamma variate behind tau^-2 does not depend on the data: the last wave draws
// it before its share of the lambda^-2, beside the other waves.  The caller's next
// use of red comes after a block barrier.
__device__ double hyper_lambda_tau(Args& a, uint32_t k, bool writer, double* red) {
    const uint32_t p = a.x.p;
    const double tau_old = *a.tau_m2, xi = *a.xi_m1;
    if ((a.mode & kModeTau) && threadIdx.x >= kThreads - kWave) {
        // Cheng's GB: proposal m = 64 * round + lane, uniforms of Philox round m/2
        // (words 0-1 for even m, 2-3 for odd m); the lowest accepted m wins, which
        // is the first acceptance of the sequential algorithm.  (Section 5 uses 32
        // threads and a serial scan for the same purpose.)
        const int lane = threadIdx.x & (kWave - 1);
        const double sh = ((double)p + 1.0) / 2.0;
        const double A = 1.0 / sqrt(2.0 * sh - 1.0);
        const double B = sh - log(4.0);
        const double C = sh + 1.0 / A;
        const double D = 1.0 + log(4.5);
        double g = __builtin_nan("");
        for (uint32_t round = 0; round < (1u << 16); ++round) {
            const uint32_t m = round * kWave + lane;
            const Words4 w = draw_words(a.seed, 0, k, kTagTau, m >> 1, a.chain);
            const double u1 = u01d((m & 1u) ? w.w2 : w.w0);
            const double u2 = u01d((m & 1u) ? w.w3 : w.w1);
            const double V = A * log(u1 / (1.0 - u1));
            const double X = sh * exp(V);
            const double Z = u1 * u1 * u2;
            const double R = B + C * V - X;
            const bool ok = (R + D - 4.5 * Z >= 0.0) || (R >= log(Z));
            const unsigned long long mask = __ballot(ok);
            if (mask) {
                g = __shfl(X, (int)(__ffsll((long long)mask) - 1));
                break;
            }
        }
        if (lane == 0) red[kRedGamma] = g;
    }
    double acc = 0.0;
    uint32_t clamps = 0;
    bool bad = false;
    for (uint32_t j = threadIdx.x; j < p; j += kThreads) {
        const double bj = a.beta[j];
        double lam;
        if (a.mode & kModeLambda) {
            double rate = a.nu_m1[j] + tau_old * bj * bj / 2.0;
            if (!(rate >= DBL_MIN)) {
                rate = DBL_MIN;
                ++clamps;
            }
            const Words4 w = draw_words(a.seed, j, k, kTagLambda, 0, a.chain);
            lam = -log(u01d(w.w0)) / rate;
            if (!isfinite(lam)) bad = true;
            if (writer) stc(&a.lam_m2[j], lam);
        } else {
            lam = a.lam_m2[j];
        }
        if (p <= (uint32_t)kSmallP) red[kRedLambda + j] = lam;
        acc += lam * bj * bj;
    }
    if (writer) {
        if (clamps) atomicAdd(&a.ctrl->clamps, (unsigned long long)clamps);
        if (bad) atomicOr(&a.ctrl->err, kErrNonFinite);
    }
    if (!(a.mode & kModeTau)) return tau_old;
    const double sum = block_sum(acc, red);
    const double tau = red[kRedGamma] / (xi + sum / 2.0);
    // the other blocks may still be reading the old value: the new one goes to
    // a scratch slot and is published when the launch closes
    if (writer && threadIdx.x == 0) {
        stc(&a.vec[2 * p], tau);
        if (!isfinite(tau) || !(tau > 0.0)) atomicOr(&a.ctrl->err, kErrNonFinite);
    }
    return tau;
}

// tau^-2 of this sweep: the scratch slot if it was drawn in this launch.
__device__ __forceinline__ double current_tau(Args& a) {
    // written by block 0 of the group in this launch: read past the scalar cache
    return (a.mode & kModeTau)
               ? __hip_atomic_load(a.vec + 2 * a.x.p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
               : *a.tau_m2;
}

// nu^-1 and xi^-1 from the (new) lambda^-2 and tau^-2 in memory.
__device__ void hyper_nu_xi(Args& a, uint32_t k) {
    const uint32_t p = a.x.p;
    for (uint32_t j = threadIdx.x; j < p; j += kThreads) {
        const Words4 w = draw_words(a.seed, j, k, kTagNu, 0, a.chain);
        a.nu_m1[j] = -log(u01d(w.w0)) / (1.0 + ldc(&a.lam_m2[j]));
    }
    if (threadIdx.x == 0) {
        const Words4 w = draw_words(a.seed, 0, k, kTagXi, 0, a.chain);
        *a.xi_m1 = -log(u01d(w.w0)) / (1.0 + current_tau(a));
    }
}

// ---- tile path, p > 16 ----------------------------------------------------------
// The tile path works on P x P matrices, P = p rounded up to a multiple of 64,
// leading dimension P: Gp holds G with an identity block on the padding, so
// the factor, L^-1 and Q^-1 carry an identity block there too and no tile
// ever needs a bounds check.
typedef double Tile[kTile][kTileLd];

__device__ __forceinline__ uint32_t padded(uint32_t p) { return (p + kTile - 1) / kTile * kTile; }

// T[r][c] = M[(r0 + r) P + c0 + c] (+ tau * lam on the diagonal of Q when
// add_diag).  Thread t reads column t % 64 of rows t / 64 + 4q: every load
// instruction of a wave is one contiguous 512-byte row segment, and all 16
// loads of a thread are in flight together.
__device__ __forceinline__ void load_tile(Tile& T, const double* M, uint32_t P, uint32_t r0,
                                          uint32_t c0, bool add_diag, double tau,
                                          const double* lam, uint32_t p) {
    const int c = threadIdx.x & (kTile - 1), rb = threadIdx.x >> 6;
    const double* src = M + (size_t)(r0 + rb) * P + c0 + c;
    double v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = ldc(src + (size_t)(4 * q) * P);
    if (add_diag) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const uint32_t gi = r0 + rb + 4 * q;
            if (gi == c0 + c && gi < p) v[q] += tau * ldc(lam + gi);
        }
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) T[rb + 4 * q][c] = v[q];
}

// Two tiles on their way from memory to LDS (load_tile's layout).
struct TilePair {
    double v[16], w[16];
};
__device__ __forceinline__ void fetch_tiles(TilePair& o, const double* MS, uint32_t rs, uint32_t cs, const double* MT,
                                            uint32_t rt, uint32_t ct, uint32_t P) {
    const int c = threadIdx.x & (kTile - 1), rb = threadIdx.x >> 6;
    const double* s0 = MS + (size_t)(rs + rb) * P + cs + c;
    const double* t0 = MT + (size_t)(rt + rb) * P + ct + c;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        o.v[q] = ldc(s0 + (size_t)(4 * q) * P);
        o.w[q] = ldc(t0 + (size_t)(4 * q) * P);
    }
}
__device__ __forceinline__ void put_tiles(const TilePair& o, Tile& S, Tile& T) {
    const int c = threadIdx.x & (kTile - 1), rb = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        S[rb + 4 * q][c] = o.v[q];
        T[rb + 4 * q][c] = o.w[q];
    }
}

// load_tile for two tiles with every global load issued before any LDS store.
__device__ __forceinline__ void load_tiles(Tile& S, const double* MS, uint32_t rs, uint32_t cs,
                                           Tile& T, const double* MT, uint32_t rt, uint32_t ct,
                                           uint32_t P) {
    TilePair x;
    fetch_tiles(x, MS, rs, cs, MT, rt, ct, P);
    put_tiles(x, S, T);
}

// ---- 64 x 64 x 64 tile products on the FP64 matrix cores ----------------------
// v_mfma_f64_16x16x4f64 computes D(16x16) += A(16x4) B(4x16); lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16] and holds D[l / 16 + 4 r][l % 16]
// in its r-th result.  Wave w owns the 32 x 32 quadrant at rows 32 (w / 2),
// columns 32 (w % 2) as 2 x 2 blocks of 16 x 16; per k-step of 4 it reads
// four 64-lane fragments from LDS for four matrix operations.
typedef double Acc4 __attribute__((ext_vector_type(4)));
struct MAcc {
    Acc4 v[2][2];
};

__device__ __forceinline__ void zero_acc(MAcc& acc) {
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) acc.v[bi][bj] = Acc4{0.0, 0.0, 0.0, 0.0};
}

// acc += S^T T
__device__ __forceinline__ void gemm_tn(const Tile& S, const Tile& T, MAcc& acc) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i0 = 32 * (wave >> 1), j0 = 32 * (wave & 1);
    const int kr = lane >> 4, cc = lane & 15;
#pragma unroll 4
    for (int q0 = 0; q0 < kTile; q0 += 4) {
        const double a0 = S[q0 + kr][i0 + cc], a1 = S[q0 + kr][i0 + 16 + cc];
        const double b0 = T[q0 + kr][j0 + cc], b1 = T[q0 + kr][j0 + 16 + cc];
        acc.v[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc.v[0][0], 0, 0, 0);
        acc.v[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc.v[0][1], 0, 0, 0);
        acc.v[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc.v[1][0], 0, 0, 0);
        acc.v[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc.v[1][1], 0, 0, 0);
    }
}

// The matrix-core layout of a 64 x 64 tile at (r0, c0) of M: lane l of wave w
// holds rows r0 + 32 (w / 2) + 16 bi + l / 16 + 4 r, column c0 + 32 (w % 2) +
// 16 bj + l % 16; each group of 16 lanes covers a 128-byte row segment.
struct MTile {
    double v[2][2][4];
};

// Load a tile in that layout (zeros for a null M), with tau * lam added on
// Q's diagonal when add_diag.  Issued before a product, the loads overlap it.
__device__ __forceinline__ void load_tile_m(MTile& o, const double* M, uint32_t P, uint32_t r0,
                                            uint32_t c0, bool add_diag, double tau, const double* lam,
                                            uint32_t p) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t ri = r0 + 32 * (wave >> 1) + (lane >> 4);
    const uint32_t cj = c0 + 32 * (wave & 1) + (lane & 15);
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                o.v[bi][bj][r] = M ? ldc(M + (size_t)(ri + 16 * bi + 4 * r) * P + cj + 16 * bj) : 0.0;
    if (add_diag) {
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int bj = 0; bj < 2; ++bj)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint32_t gi = ri + 16 * bi + 4 * r, gj = cj + 16 * bj;
                    if (gi == gj && gi < p) o.v[bi][bj][r] += tau * ldc(lam + gi);
                }
    }
}

// M(r0.., c0..) = old + sign * acc, sixteen stores back to back.
__device__ __forceinline__ void put_tile_m(double* M, uint32_t P, uint32_t r0, uint32_t c0,
                                           const MAcc& acc, double sign, const MTile& old) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t ri = r0 + 32 * (wave >> 1) + (lane >> 4);
    const uint32_t cj = c0 + 32 * (wave & 1) + (lane & 15);
    double out[2][2][4];
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int r = 0; r < 4; ++r) out[bi][bj][r] = fma(sign, acc.v[bi][bj][r], old.v[bi][bj][r]);
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int r = 0; r < 4; ++r) stc(M + (size_t)(ri + 16 * bi + 4 * r) * P + cj + 16 * bj, out[bi][bj][r]);
}

// v, or zero, with no branch (a branch around a load or store would make the
// next one wait for it).
__device__ __forceinline__ double keep_if(bool keep, double v) {
    const long long m = keep ? -1ll : 0ll;
    return __longlong_as_double(__double_as_longlong(v) & m);
}

// 1 / sqrt(d) for d > 0: the hardware estimate and one Newton step.
__device__ __forceinline__ double rsqrt_nr(double d) {
    const double y = __builtin_amdgcn_rsq(d);
    const double e = fma(-d * y, y, 1.0);  // 1 - d y^2
    return fma(0.5 * y, e, y);
}

// Lane C of each row of 16 lanes, in every lane of that row.
template <int C>
__device__ __forceinline__ double row_bcast(double v) {
    return __builtin_amdgcn_update_dpp(0.0, v, 0x150 + C, 0xf, 0xf, true);
}
// A vector register that is written needs two wait states before a cross-lane
// operand reads it, and the compiler, which keeps to that for its own instructions,
// sees neither the write nor the read of one inside asm.  settle() stands between a
// write inside asm and a cross-lane operand of the compiler's.
__device__ __forceinline__ void settle(double& x) { asm("s_nop 1" : "+v"(x)); }

// acc -= (lane C of x's row of 16 lanes) * y is one instruction (HSP_FMSUB).  Blocks
// of them wait for x themselves, in the same asm: whatever the compiler puts before
// it, a copy or a reload of x from a spill among others, has then settled.  (Their
// results are early clobbers: no operand read later may share a register with one.)
#define HSP_FMSUB(acc, x, y, lane) \
    "v_fmac_f64_dpp %" #acc ", -%" #x ", %" #y " row_newbcast:%" #lane " row_mask:0xf bank_mask:0xf\n\t"

// Pivots of a 16-row panel: d holds the panel's diagonal block (column l % 16 in
// lane l, a copy in each row of 16 lanes), a the 64 other columns of the panel, one
// per lane.  Row C is scaled by 1 / sqrt(pivot), then every later row i loses (row
// C's entry at column i) times row C: the multiplier is lane i's entry of row C's
// diagonal part, which a row of 16 lanes broadcasts to itself, so each row costs
// two instructions and no scalar registers.
//
// The n rows I .. 15 lose their part of row I - 1 in one asm block, which also
// returns 1 / sqrt(pivot I) (rsqrt_nr's operations) for the next step: the first
// row is done first, and the root's chain runs between the other rows' instructions,
// with two of them or waits before the pivot's broadcast and one after the
// hardware's estimate.  N = 1e5, p = 100, us per 8 sweeps: one asm statement per
// instruction, arranged by the compiler (which could put a copy before any) 348,
// blocks of up to four with a wait each 366, this 337.
#define HSP_D(r) "v_fmac_f64_dpp %[d" #r "], -%[x], %[x] row_newbcast:%[l" #r "] row_mask:0xf bank_mask:0xf\n\t"
#define HSP_A(r) "v_fmac_f64_dpp %[a" #r "], -%[x], %[y] row_newbcast:%[l" #r "] row_mask:0xf bank_mask:0xf\n\t"
#define HSP_DA(r) HSP_D(r) HSP_A(r)
#define HSP_ROOT1 "v_mov_b64_dpp %[t], %[d0] row_newbcast:%[l0] row_mask:0xf bank_mask:0xf\n\t"
#define HSP_ROOT2 "v_rsq_f64 %[rs], %[t]\n\t"
#define HSP_ROOT3 "v_mul_f64 %[e], %[rs], -%[t]\n\t"
#define HSP_ROOT4 "v_fma_f64 %[e], %[e], %[rs], 1.0\n\tv_mul_f64 %[t], %[rs], 0.5\n\t"
#define HSP_ROOT5 "v_fmac_f64 %[rs], %[t], %[e]\n\t"
#define HSP_T1 "s_nop 1\n\t" HSP_DA(0) "s_nop 0\n\t" HSP_ROOT1 HSP_ROOT2 "s_nop 0\n\t" HSP_ROOT3 HSP_ROOT4 HSP_ROOT5
#define HSP_T2 "s_nop 1\n\t" HSP_DA(0) HSP_D(1) HSP_ROOT1 HSP_ROOT2 HSP_A(1) HSP_ROOT3 HSP_ROOT4 HSP_ROOT5
#define HSP_HEAD "s_nop 1\n\t" HSP_DA(0) HSP_D(1) HSP_ROOT1 HSP_A(1) HSP_ROOT2 HSP_DA(2)
#define HSP_T3 HSP_HEAD HSP_ROOT3 HSP_ROOT4 HSP_ROOT5
#define HSP_T4 HSP_HEAD HSP_ROOT3 HSP_DA(3) HSP_ROOT4 HSP_ROOT5
#define HSP_T5 HSP_HEAD HSP_ROOT3 HSP_DA(3) HSP_ROOT4 HSP_DA(4) HSP_ROOT5
#define HSP_T6 HSP_HEAD HSP_DA(3) HSP_ROOT3 HSP_DA(4) HSP_ROOT4 HSP_DA(5) HSP_ROOT5
#define HSP_T7 HSP_T6 HSP_DA(6)
#define HSP_T8 HSP_T7 HSP_DA(7)
#define HSP_T9 HSP_T8 HSP_DA(8)
#define HSP_T10 HSP_T9 HSP_DA(9)
#define HSP_T11 HSP_T10 HSP_DA(10)
#define HSP_T12 HSP_T11 HSP_DA(11)
#define HSP_T13 HSP_T12 HSP_DA(12)
#define HSP_T14 HSP_T13 HSP_DA(13)
#define HSP_T15 HSP_T14 HSP_DA(14)
#define HSP_OUT(r) [d##r] "+&v"(d[I + r]), [a##r] "+&v"(a[I + r])
#define HSP_O1 HSP_OUT(0)
#define HSP_O2 HSP_O1, HSP_OUT(1)
#define HSP_O3 HSP_O2, HSP_OUT(2)
#define HSP_O4 HSP_O3, HSP_OUT(3)
#define HSP_O5 HSP_O4, HSP_OUT(4)
#define HSP_O6 HSP_O5, HSP_OUT(5)
#define HSP_O7 HSP_O6, HSP_OUT(6)
#define HSP_O8 HSP_O7, HSP_OUT(7)
#define HSP_O9 HSP_O8, HSP_OUT(8)
#define HSP_O10 HSP_O9, HSP_OUT(9)
#define HSP_O11 HSP_O10, HSP_OUT(10)
#define HSP_O12 HSP_O11, HSP_OUT(11)
#define HSP_O13 HSP_O12, HSP_OUT(12)
#define HSP_O14 HSP_O13, HSP_OUT(13)
#define HSP_O15 HSP_O14, HSP_OUT(14)
#define HSP_LANE(r) [l##r] "n"(I + r)
#define HSP_L1 HSP_LANE(0)
#define HSP_L2 HSP_L1, HSP_LANE(1)
#define HSP_L3 HSP_L2, HSP_LANE(2)
#define HSP_L4 HSP_L3, HSP_LANE(3)
#define HSP_L5 HSP_L4, HSP_LANE(4)
#define HSP_L6 HSP_L5, HSP_LANE(5)
#define HSP_L7 HSP_L6, HSP_LANE(6)
#define HSP_L8 HSP_L7, HSP_LANE(7)
#define HSP_L9 HSP_L8, HSP_LANE(8)
#define HSP_L10 HSP_L9, HSP_LANE(9)
#define HSP_L11 HSP_L10, HSP_LANE(10)
#define HSP_L12 HSP_L11, HSP_LANE(11)
#define HSP_L13 HSP_L12, HSP_LANE(12)
#define HSP_L14 HSP_L13, HSP_LANE(13)
#define HSP_L15 HSP_L14, HSP_LANE(14)
#define HSP_PIVOT(n)                                                                                                  \
    if constexpr (16 - I == n)                                                                                        \
        asm(HSP_T##n : HSP_O##n, [rs] "=&v"(rs), [t] "=&v"(t), [e] "=&v"(e) : [x] "v"(d[I - 1]), [y] "v"(a[I - 1]), HSP_L##n);
template <int I>
__device__ __forceinline__ double panel_rows(double (&d)[16], double (&a)[16]) {
    double rs, t, e;
    HSP_PIVOT(1)
    HSP_PIVOT(2)
    HSP_PIVOT(3)
    HSP_PIVOT(4)
    HSP_PIVOT(5)
    HSP_PIVOT(6)
    HSP_PIVOT(7)
    HSP_PIVOT(8)
    HSP_PIVOT(9)
    HSP_PIVOT(10)
    HSP_PIVOT(11)
    HSP_PIVOT(12)
    HSP_PIVOT(13)
    HSP_PIVOT(14)
    HSP_PIVOT(15)
    return rs;
}
template <int C = 0>
__device__ __forceinline__ void panel_pivots(double (&d)[16], double (&a)[16], double rs) {
    d[C] *= rs;
    a[C] *= rs;
    if constexpr (C < 15) panel_pivots<C + 1>(d, a, panel_rows<C + 1>(d, a));
}

// acc += sum_j x_j y[j], x_j being lane j of x's row of 16 lanes.
__device__ __forceinline__ void dot_bcast(double& acc, double minus_x, const double (&y)[16]) {
    asm("s_nop 1\n\t" HSP_FMSUB(0, 1, 2, 18) HSP_FMSUB(0, 1, 3, 19) HSP_FMSUB(0, 1, 4, 20) HSP_FMSUB(0, 1, 5, 21)
            HSP_FMSUB(0, 1, 6, 22) HSP_FMSUB(0, 1, 7, 23) HSP_FMSUB(0, 1, 8, 24) HSP_FMSUB(0, 1, 9, 25)
                HSP_FMSUB(0, 1, 10, 26) HSP_FMSUB(0, 1, 11, 27) HSP_FMSUB(0, 1, 12, 28) HSP_FMSUB(0, 1, 13, 29)
                    HSP_FMSUB(0, 1, 14, 30) HSP_FMSUB(0, 1, 15, 31) HSP_FMSUB(0, 1, 16, 32) HSP_FMSUB(0, 1, 17, 33)
        : "+&v"(acc)
        : "v"(minus_x), "v"(y[0]), "v"(y[1]), "v"(y[2]), "v"(y[3]), "v"(y[4]), "v"(y[5]), "v"(y[6]), "v"(y[7]), "v"(y[8]),
          "v"(y[9]), "v"(y[10]), "v"(y[11]), "v"(y[12]), "v"(y[13]), "v"(y[14]), "v"(y[15]), "n"(0), "n"(1), "n"(2), "n"(3),
          "n"(4), "n"(5), "n"(6), "n"(7), "n"(8), "n"(9), "n"(10), "n"(11), "n"(12), "n"(13), "n"(14), "n"(15));
}

// One wave eliminates row panel P (16 rows from r0 = 16 P) of [S | T]: the
// panel's columns are its 16 x 16 diagonal block of S, S's 48 - r0 columns to
// the right of it and T's first r0 + 16 columns, the last 16 of which start as
// the identity: 64 columns beside the diagonal block whatever P.  Returns
// whether every pivot was positive (a failed one leaves NaN in the last).
__device__ __forceinline__ bool factor_panel(Tile& S, Tile& T, int P) {
    const int lane = threadIdx.x & 63, r0 = 16 * P, right = 48 - r0;
    const int tcol = lane - right;  // this lane's column of T, if not negative
    double* col = tcol < 0 ? &S[r0][r0 + 16 + lane] : &T[r0][tcol];
    const double* dcol = &S[r0][r0 + (lane & 15)];
    double d[16], a[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        d[i] = dcol[i * kTileLd];
        a[i] = col[i * kTileLd];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) a[i] = tcol < r0 ? a[i] : (tcol - r0 == i ? 1.0 : 0.0);
    panel_pivots(d, a, rsqrt_nr(row_bcast<0>(d[0])));
    if (lane < 16) {
        double* dw = &S[r0][r0 + lane];
#pragma unroll
        for (int i = 0; i < 16; ++i) dw[i * kTileLd] = d[i];  // valid on and above the diagonal
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) col[i * kTileLd] = a[i];
    return row_bcast<15>(d[15]) > 0.0;
}

// B(I, J) -= S(P, I)^T B(P, J) on 16 x 16 blocks; fresh: B(I, J) starts at zero.
__device__ __forceinline__ void panel_update(const Tile& S, Tile& B, int P, int I, int J, bool fresh) {
    const int lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
    double x[4], y[4];
    Acc4 acc;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        x[kk] = -S[16 * P + 4 * kk + kr][16 * I + cc];
        y[kk] = B[16 * P + 4 * kk + kr][16 * J + cc];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = fresh ? 0.0 : B[16 * I + kr + 4 * r][16 * J + cc];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[kk], y[kk], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) B[16 * I + kr + 4 * r][16 * J + cc] = acc[r];
}

// Factor a 64 x 64 diagonal block by row operations on [S | I]: on return the
// upper part of S is U and the lower part of T is U^-T (the rest of both tiles
// is not written or read).  Only the upper part of S is read; rows 16.. of it
// may still be completed by waves 1..3 in `rest`, which runs beside the first
// panel (wave 0).
//
// Four row panels of 16, each on wave 0 (factor_panel); then the blocks of the
// next panel's rows take the panel's rank-16 update on the matrix cores -- there
// are four of them whatever the panel, one per wave: S(P+1, J > P) and
// T(P+1, J <= P) -- and the blocks of later rows take it on waves 1..3 while
// wave 0 eliminates the next panel.
//
// Bound by wave 0's chain of 64 pivots.  Whole tile, phase trace at N = 1e6,
// p = 1000: 11.3 -> 7.5 us (a panel 2.1 -> 1.4) against multipliers broadcast
// through scalar registers, the identity in a second set of columns and every
// update before the next panel; a panel step of the chain block 17.3 -> 10.8 us.
template <class F>
__device__ __forceinline__ bool factor_diag(Tile& S, Tile& T, double* flag, uint64_t* rec, F rest) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll 1
    for (int P = 0; P < 4; ++P) {
        if (wave == 0) {
            const bool ok = factor_panel(S, T, P);
            if (threadIdx.x == 0) *flag = ok ? 0.0 : 1.0;
        } else if (P == 0) {
            rest();
        } else {
            // the rank-16 update of panel P - 1 on the rows after panel P
            int n = 0;
            for (int I = P + 1; I < 4; ++I) {
                for (int J = I; J < 4; ++J)
                    if (n++ % 3 == wave - 1) panel_update(S, S, P - 1, I, J, false);
                for (int J = 0; J < P; ++J)
                    if (n++ % 3 == wave - 1) panel_update(S, T, P - 1, I, J, J == P - 1);
            }
        }
        __syncthreads();
        stamp_at(rec, 1 + 2 * P);
        if (*flag != 0.0) return false;
        if (P < 3) {
            const int J = P + 1 + wave;
            if (J < 4) panel_update(S, S, P, P + 1, J, false);
            else panel_update(S, T, P, P + 1, J - 4, J - 4 == P);
            __syncthreads();
        }
        stamp_at(rec, 2 + 2 * P);
    }
    stamp_at(rec, 9);
    return true;
}

// Factor diagonal block kb held in S (its upper part; the rest is not read)
// and store L^-1_kk = U_kk^-T into Linv, zeros above its diagonal: the
// triangular solves read it from there (U_kk itself is needed by nothing after
// this block).  Reports a failed pivot.  On return the lower part of T is U_kk^-T.
template <class F>
__device__ __forceinline__ void diag_factor(Args& a, uint32_t kb, Tile& S, Tile& T, double* flag, uint64_t* rec, F rest) {
    const uint32_t P = padded(a.x.p), k0 = kb * kTile;
    stamp_at(rec, 0);
    if (factor_diag(S, T, flag, rec, rest)) {
        const int c = threadIdx.x & (kTile - 1), rb = threadIdx.x >> 6;
        double v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = T[rb + 4 * q][c];
#pragma unroll
        for (int q = 0; q < 16; ++q)
            stc(a.Linv + (size_t)(k0 + rb + 4 * q) * P + k0 + c, keep_if(c <= rb + 4 * q, v[q]));
    } else if (threadIdx.x == 0) {
        atomicOr(&a.ctrl->err, kErrNotPD);
        atomicCAS(&a.ctrl->chol_info, 0, (int)(k0 + 1));
    }
    __syncthreads();
    stamp_at(rec, 10);
}

// Four 16 x 16 blocks of a tile in the matrix-core layout, one block column:
// block I's r-th value of lane l is row 16 I + l / 16 + 4 r, column l % 16.
struct MCol {
    Acc4 v[4];
};

// Wave w's block column of W X for a lower triangular W (its upper part is
// not read): rows of block I need only the column blocks K <= I of W, 40
// matrix operations instead of 64.
__device__ __forceinline__ void trsm_tri(const Tile& W, const Tile& X, MCol& out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, kr = lane >> 4, cc = lane & 15;
#pragma unroll
    for (int I = 0; I < 4; ++I) out.v[I] = Acc4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int K = 0; K < 4; ++K) {
        double y[4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) y[kk] = X[16 * K + 4 * kk + kr][16 * wave + cc];
#pragma unroll
        for (int I = K; I < 4; ++I)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const int k = 16 * K + 4 * kk + kr, i = 16 * I + cc;
                const double w = I > K ? W[i][k] : keep_if(k <= i, W[i][k]);
                out.v[I] = __builtin_amdgcn_mfma_f64_16x16x4f64(w, y[kk], out.v[I], 0, 0, 0);
            }
    }
}

// Store a wave's block column of the tile at (r0, c0) of M.
__device__ __forceinline__ void put_col(double* M, uint32_t P, uint32_t r0, uint32_t c0, const MCol& v) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, kr = lane >> 4, cc = lane & 15;
#pragma unroll
    for (int I = 0; I < 4; ++I)
#pragma unroll
        for (int r = 0; r < 4; ++r) stc(M + (size_t)(r0 + 16 * I + kr + 4 * r) * P + c0 + 16 * wave + cc, v.v[I][r]);
}

// The blocks (I, J), I <= J, of a diagonal tile that each wave updates in a
// panel step: first (0, wave), which the first row panel needs, then for waves
// 1..3 two of the other six.
__device__ __forceinline__ void rest_block(int wave, int n, int& I, int& J) {
    I = wave == 3 && n == 0 ? 2 : wave == 3 ? 3 : wave == 2 && n == 1 ? 2 : 1;
    J = wave == 1 ? 1 + n : wave == 2 ? 3 - n : 3;
}

// D(I, J) = old - (U^T U)(I, J) over 64 rows, U in LDS: the sums and the
// subtraction a GEMM task does (a group of one block factors with those).
__device__ __forceinline__ void syrk_block(const Tile& U, Tile& D, int I, int J, const Acc4& old) {
    const int lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
    Acc4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q0 = 0; q0 < kTile; q0 += 4)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(U[q0 + kr][16 * I + cc], U[q0 + kr][16 * J + cc], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) D[16 * I + kr + 4 * r][16 * J + cc] = fma(-1.0, acc[r], old[r]);
}

// Wave 0: wait for the inputs of a run of n updates of tile (i, j) from step k on:
// U_k'i and U_k'j final for each step k', and the tile updated up to k; false if
// the group is failing or the wait timed out.
__device__ __forceinline__ bool wait_run(const uint32_t* vU, uint32_t nt, uint32_t k, uint32_t n, uint32_t i, uint32_t j,
                                         Ctrl* ctrl, uint64_t timeout) {
    const uint32_t l = threadIdx.x & 63u, s = l < n ? l : l - n;
    const bool tile = l >= 2 * n;  // (lanes past 2 n all look at the tile itself)
    const uint32_t* v = tile ? vU + i * nt + j : vU + (k + s) * nt + (l < n ? i : j);
    const uint32_t need = tile ? k : k + s + 1;
    uint64_t t0 = 0;
    uint32_t nap = 1;
    for (int it = 0;; ++it) {
        const uint32_t got = __hip_atomic_load(const_cast<uint32_t*>(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__ballot(got < need) == 0ull) return true;
        if (it == 0) t0 = wall_clock64();
        if (__hip_atomic_load(&ctrl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & (kErrTimeout | kErrNotPD))
            return false;
        if (wall_clock64() - t0 > timeout) {
            if (l == 0) atomicOr(&ctrl->err, kErrTimeout);
            return false;
        }
        backoff(nap, 8);
    }
}

// Run block `rank`'s list of factorisation tasks.  Tile versions: U tile
// (i, j), i <= j, has had v of its i updates (plus 1 once final); L^-1 tile
// (i, j), j <= i, v of its i - j updates (plus 1 once final).  Each task waits
// for the versions it reads, then publishes the version it wrote.  Returns
// false if the group is failing.
__device__ __forceinline__ bool run_tasks(Args& a, Group& g, uint32_t rank, double tau, Tile& S, Tile& T,
                          double* flag) {
    const uint32_t p = a.x.p, P = padded(p), nt = P / kTile;
    // flags of the factorisation and of the queue, in T's padding columns
    double* fact_flag = &T[kTile - 1][kTile];
    double* next_lds = &T[kTile - 2][kTile];
    bool swapped = false;  // the chain block's two tiles trade places with every panel step
    uint32_t* vU = a.ver;
    uint32_t* vL = a.ver + nt * nt;
    // Block 0 (or a group of one) runs its own list; the others claim tasks
    // from the shared queue in order, each reserving its next task when it
    // starts one.  The claimed index travels to the block through LDS.
    const bool queue = g.size > 1 && rank > 0;
    const uint32_t n0 = queue ? a.task_off[1] : 0u, n1 = queue ? a.task_off[2] : a.task_off[1];
    // With runs (no L^-1) the queue's items, and a lone block's, are numbered by
    // a.runs; an item is claimed when the block is free, a reservation would hold
    // up the tasks next to the chain for as long as a run takes.
    const bool by_runs = a.runs && (queue || g.size == 1);
    uint32_t x = 0;
    uint32_t n = n0;
    if (queue) {
        if (threadIdx.x == 0) *next_lds = (double)atomicAdd(&a.ctrl->task_next, 1u);
        __syncthreads();
        x = (uint32_t)*next_lds;
        n = n0 + x;
        __syncthreads();
    }
    while (by_runs ? x < a.nruns : n < n1) {
        uint32_t len = 1;
        if (by_runs) {
            n = a.runs[x];
            len = a.runs[x + 1] - n;
        }
        const uint32_t code = a.tasks[n];
        const uint32_t type = code & 3u, part = (code >> 2) & 1u, kb = (code >> 3) & kTaskField,
                       ib = (code >> 11) & kTaskField, jb = (code >> 19) & kTaskField;
        uint32_t reserved = 0;
        if (len > 1) {
            if (threadIdx.x < (uint32_t)kWave) {
                const bool w = wait_run(vU, nt, kb, len, ib, jb, a.ctrl, g.timeout);
                if (threadIdx.x == 0) *flag = w ? 0.0 : 1.0;
            }
        } else if (threadIdx.x == 0) {
            if (queue && !by_runs) reserved = atomicAdd(&a.ctrl->task_next, 1u);
            uint32_t* v[3] = {nullptr, nullptr, nullptr};
            uint32_t need[3] = {0u, 0u, 0u};
            int nv;
            if (type == kTaskPotrf) {
                v[0] = &vU[kb * nt + kb], need[0] = kb;
                nv = 1;
            } else if (type == kTaskPanel) {
                v[0] = &vU[(kb - 1) * nt + kb], need[0] = kb - 1;
                v[1] = &vU[kb * nt + kb], need[1] = kb - 1;
                nv = 2;
            } else if (type == kTaskTrsm) {
                v[0] = &vU[kb * nt + kb], need[0] = kb + 1;
                if (part == 0) v[1] = &vU[kb * nt + jb], need[1] = kb;
                else v[1] = &vL[kb * nt + jb], need[1] = kb - jb;
                nv = 2;
            } else {
                v[0] = &vU[kb * nt + ib], need[0] = kb + 1;
                if (part == 0) {
                    v[1] = &vU[kb * nt + jb], need[1] = kb + 1;
                    v[2] = &vU[ib * nt + jb], need[2] = kb;
                } else {
                    v[1] = &vL[kb * nt + jb], need[1] = kb - jb + 1;
                    v[2] = &vL[ib * nt + jb], need[2] = kb - jb;
                }
                nv = 3;
            }
            const bool w = wait_vers(v, need, nv, a.ctrl, g.timeout);
            *flag = w ? 0.0 : 1.0;
        }
        __syncthreads();
        stamp_value(g, n + 1u);
        stamp(g);
        if (*flag != 0.0) return false;
        const uint32_t k0 = kb * kTile;
        uint32_t* out = nullptr;   // version published when the task is done
        uint32_t* out2 = nullptr;  // a diagonal L^-1 tile, final at version 1
        uint32_t val = 0;
        if (type == kTaskPotrf || type == kTaskPanel) {
            uint64_t* rec = nullptr;
            if (g.trace && g.npotrf < (uint32_t)kTraceRecs) rec = g.trace + kTraceSeq + kTraceRec * g.npotrf;
            g.npotrf++;
            Acc4 dg[3];
            int I1 = 0, J1 = 0, I2 = 0, J2 = 0;
            Tile& Sc = swapped ? T : S;  // (a step's tiles trade places with the previous one's)
            Tile& Tc = swapped ? S : T;
            if (type == kTaskPotrf) {
                load_tile(Sc, kb == 0 ? a.Gp : a.A, P, k0, k0, kb == 0, tau, a.lam_m2, p);
                __syncthreads();
                stamp(g);
            } else {
                // U_{k-1,k} = L^-1_{k-1,k-1} A_{k-1,k} with L^-1_{k-1,k-1} still in
                // T, then A_kk -= U_{k-1,k}^T U_{k-1,k} and its factorisation, all
                // in this block.  U overwrites A_{k-1,k} in S (a wave reads and
                // writes its own 16 columns only), the updated A_kk takes T's
                // place, and the new inverse takes S's: the six blocks of A_kk
                // outside its first 16 rows read U's columns 16.. while the first
                // panel is factored, which writes columns 0..15 only.
                const uint32_t km = kb - 1, r1 = km * kTile;
                const double* src = km == 0 ? a.Gp : a.A;
                const int lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
                const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
                // this wave's blocks of A_kk: (0, wave), then rest_block's
                auto diag_block = [&](int I, int J) {
                    const uint32_t i0 = k0 + 16 * I + kr, j = k0 + 16 * J + cc;
                    Acc4 v;
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = ldc(src + (size_t)(i0 + 4 * r) * P + j);
                    if (km == 0 && I == J) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (i0 + 4 * r == j && j < p) v[r] += tau * ldc(a.lam_m2 + j);
                    }
                    return v;
                };
                rest_block(wave, 0, I1, J1);
                rest_block(wave, 1, I2, J2);
                dg[0] = diag_block(0, wave);
                if (wave != 0) {
                    dg[1] = diag_block(I1, J1);
                    dg[2] = diag_block(I2, J2);
                }
                load_tile(Sc, src, P, r1, k0, false, 0.0, nullptr, p);
                __syncthreads();
                stamp(g);
                MCol u;
                trsm_tri(Tc, Sc, u);
                put_col(a.A, P, r1, k0, u);
#pragma unroll
                for (int I = 0; I < 4; ++I)
#pragma unroll
                    for (int r = 0; r < 4; ++r) Sc[16 * I + kr + 4 * r][16 * wave + cc] = u.v[I][r];
                __syncthreads();  // all of U in S; T has been read
                syrk_block(Sc, Tc, 0, wave, dg[0]);
                // U_{k-1,k} is published once its stores are complete; the
                // product above hid their latency
                publish(&vU[km * nt + kb], kb);
                swapped = !swapped;
            }
            {
                Tile& Sd = swapped ? T : S;
                Tile& Td = swapped ? S : T;
                diag_factor(a, kb, Sd, Td, fact_flag, rec, [&] {
                    if (type == kTaskPanel) {
                        syrk_block(Td, Sd, I1, J1, dg[1]);
                        syrk_block(Td, Sd, I2, J2, dg[2]);
                    }
                });
            }
            if (threadIdx.x == 0 &&
                (__hip_atomic_load(&a.ctrl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrNotPD))
                *flag = 1.0;
            __syncthreads();
            if (*flag != 0.0) return false;
            out = &vU[kb * nt + kb];
            val = kb + 1;
            out2 = &vL[kb * nt + kb];
        } else if (type == kTaskTrsm) {
            // X_kj = L^-1_kk X_kj, L^-1_kk from Linv
            const uint32_t j0 = jb * kTile;
            load_tiles(S, a.Linv, k0, k0, T, part == 0 ? (kb == 0 ? a.Gp : a.A) : a.Linv, k0, j0, P);
            __syncthreads();
            stamp(g);
            MCol x;
            trsm_tri(S, T, x);
            put_col(part == 0 ? a.A : a.Linv, P, k0, j0, x);
            out = part == 0 ? &vU[kb * nt + jb] : &vL[kb * nt + jb];
            val = part == 0 ? kb + 1 : kb - jb + 1;
        } else if (len > 1) {
            // A_ij -= sum over the run's steps of U_ki^T U_kj: the tile is read and
            // stored once, and each step's tiles are on their way during the
            // products of the step before.  (One task per step, each with its own
            // wait, three loads and a store, kept the FP64 matrix cores 40 % busy:
            // p = 7003, 8.5 us per task on each of two blocks per unit.)
            MTile old;
            load_tile_m(old, kb == 0 ? a.Gp : a.A, P, ib * kTile, jb * kTile, kb == 0 && ib == jb, tau, a.lam_m2, p);
            TilePair next;
            fetch_tiles(next, a.A, k0, ib * kTile, a.A, k0, jb * kTile, P);
            put_tiles(next, S, T);
            __syncthreads();
            stamp(g);
            MAcc acc;
            zero_acc(acc);
            for (uint32_t s = 0; s < len; ++s) {
                const bool more = s + 1 < len;
                const uint32_t ks = (kb + s + 1) * kTile;
                if (more) fetch_tiles(next, a.A, ks, ib * kTile, a.A, ks, jb * kTile, P);
                // claim the next item while the last products run
                if (!more && queue && threadIdx.x == 0) reserved = atomicAdd(&a.ctrl->task_next, 1u);
                gemm_tn(S, T, acc);
                if (more) {
                    __syncthreads();  // every wave has read S and T
                    put_tiles(next, S, T);
                    __syncthreads();
                }
            }
            put_tile_m(a.A, P, ib * kTile, jb * kTile, acc, -1.0, old);
            out = &vU[ib * nt + jb];
            val = kb + len;
        } else {
            // A_ij -= U_ki^T U_kj  or  L^-1_ij -= U_ki^T L^-1_kj; the three
            // tiles' loads are in flight together
            MTile old;
            if (part == 0)
                load_tile_m(old, kb == 0 ? a.Gp : a.A, P, ib * kTile, jb * kTile, kb == 0 && ib == jb, tau,
                            a.lam_m2, p);
            else
                load_tile_m(old, jb == kb ? nullptr : a.Linv, P, ib * kTile, jb * kTile, false, 0.0, nullptr, p);
            load_tiles(S, a.A, k0, ib * kTile, T, part == 0 ? a.A : a.Linv, k0, jb * kTile, P);
            __syncthreads();
            stamp(g);
            MAcc acc;
            zero_acc(acc);
            gemm_tn(S, T, acc);
            put_tile_m(part == 0 ? a.A : a.Linv, P, ib * kTile, jb * kTile, acc, -1.0, old);
            out = part == 0 ? &vU[ib * nt + jb] : &vL[ib * nt + jb];
            val = part == 0 ? kb + 1 : kb - jb + 1;
        }
        if (threadIdx.x == 0 && queue) {
            if (by_runs && len == 1) reserved = atomicAdd(&a.ctrl->task_next, 1u);
            *next_lds = (double)reserved;
        }
        publish(out, val, out2, 1u);
        stamp(g);
        x = queue ? (uint32_t)*next_lds : x + 1;
        n = queue ? n0 + x : n + 1;
        __syncthreads();
    }
    return true;
}

// Values handed from row to row of the substitution: two P-vectors after the
// 2 p + 8 scratch doubles, on a 128-byte boundary, which hold kNotReady (a NaN
// no arithmetic produces) until the value is stored and again between launches.
// A reader polls the values themselves, so a hand-off is one store and one load.
__device__ __forceinline__ double* handoff(Args& a) { return (double*)(a.vec + handoff_offset(a.x.p)); }

// One wave: hand[idx] of every lane once all are there.  After a failure of the
// group (or a time-out, which sets one) it returns what is there.
__device__ __forceinline__ double take(const double* hand, int idx, Ctrl* ctrl, uint64_t timeout, uint32_t cap) {
    uint64_t t0 = 0;
    uint32_t nap = 1;
    for (int it = 0;; ++it) {
        const double v = ldc(hand + idx);
        const uint32_t err = __hip_atomic_load(&ctrl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__ballot((unsigned long long)__double_as_longlong(v) == kNotReady) == 0ull) return v;
        if (err & (kErrTimeout | kErrNotPD)) return v;
        if (it == 0) t0 = wall_clock64();
        if (wall_clock64() - t0 > timeout) {
            if ((threadIdx.x & 63) == 0) atomicOr(&ctrl->err, kErrTimeout);
            return v;
        }
        backoff(nap, cap);
    }
}

// beta = U^-1 (U^-T b + s) by blocked substitution (where the factorisation
// leaves L^-1 out beyond its diagonal tiles, half of its flops).  Block r of the
// group owns tile rows r, r + gp, ...  Forward, its rows in increasing order:
// w_i = L^-1_ii (b_i - sum_{k < i} U_ki^T w_k); backward, in decreasing order:
// beta_i = (L^-1_ii)^T (w_i + s_i - sum_{k > i} U_ik beta_k).  A row waits only on
// rows finished before it in the same direction, so the solve cannot deadlock.
//
// Bound by the hand-off from row to row, so all that does not depend on the
// last w_k (beta_k) is done before it arrives: the next tile and L^-1_ii are in
// registers, the sums stay in each wave's registers (forward, wave q sums rows
// 16 q .. of the tile, broadcast from the 16 lanes that polled them; backward,
// rows 16 q .. of the output, one column per lane) and meet in LDS once per row,
// and each wave then multiplies 16 rows of the diagonal tile.  Per row step: 1.45 us,
// against 5.2-5.8 with flags beside the data, tiles loaded after the flag and
// three barriers (p = 4096: 640 -> 184 us; p = 7003: 1270 -> 326 us).
__device__ __forceinline__ void subst_solve(Args& a, Group& g, uint32_t rank, uint32_t k, double* lds, bool from_sum) {
    const uint32_t p = a.x.p, P = padded(p), nt = P / kTile;
    double* hw = handoff(a);  // w
    double* hb = hw + P;      // beta
    const double* s_noise = a.vec + p;
    double* part = lds;  // 4 x 64
    const int lane = threadIdx.x & 63, c = lane & 15, grp = lane >> 4;
    const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // sum over the four groups of 16 lanes
    auto over_groups = [](double v) {
        v += __shfl_xor(v, 16);
        return v + __shfl_xor(v, 32);
    };
    for (uint32_t i = rank; i < nt; i += g.size) {
        const uint32_t i0 = i * kTile, j0 = i0 + lane;
        const double b = j0 < p ? (from_sum ? ldc(&a.bsum[j0]) * a.xscale[j0] : a.b[j0]) : 0.0;
        if (from_sum && q == 0 && j0 < p) a.b[j0] = b;
        double l[16], t[16];  // L^-1_ii: row 16 q + c, columns 16 grp ..
        const double* lp = a.Linv + (size_t)(i0 + 16 * q + c) * P + i0 + 16 * grp;
#pragma unroll
        for (int j = 0; j < 16; ++j) l[j] = ldc(lp + j);
        const double* up = a.A + (size_t)(16 * q) * P + j0;  // U_0i: rows 16 q .., column `lane`
#pragma unroll
        for (int j = 0; j < 16; ++j) t[j] = i > 0 ? ldc(up + (size_t)j * P) : 0.0;
        double acc = 0.0;  // minus this wave's share of sum_k (U_ki^T w_k)_lane
        for (uint32_t kk = 0; kk < i; ++kk) {
            double nx[16];
            up += (size_t)kTile * P;
            if (kk + 1 < i) {
#pragma unroll
                for (int j = 0; j < 16; ++j) nx[j] = ldc(up + (size_t)j * P);
            } else {
#pragma unroll
                for (int j = 0; j < 16; ++j) nx[j] = 0.0;
            }
            double w = take(hw + kk * kTile + 16 * q, c, a.ctrl, g.timeout, min(i - kk, 8u));
            dot_bcast(acc, w, t);
#pragma unroll
            for (int j = 0; j < 16; ++j) t[j] = nx[j];
        }
        part[q * kTile + lane] = acc;
        __syncthreads();
        double r = -(b + ((part[lane] + part[kTile + lane]) + (part[2 * kTile + lane] + part[3 * kTile + lane])));
        double w = 0.0;
        dot_bcast(w, r, l);
        w = over_groups(w);
        if (grp == 0) stc(hw + i0 + 16 * q + c, w);
        __syncthreads();  // part is free again
    }
    bool keep;
    const uint32_t slot = record_slot(a, k, &keep);
    bool nonfinite = false;
    const uint32_t nown = rank < nt ? (nt - 1 - rank) / g.size + 1 : 0u;
    for (uint32_t o = nown; o-- > 0;) {
        const uint32_t i = rank + o * g.size, i0 = i * kTile, j0 = i0 + lane;
        const double ws = ldc(hw + j0) + (j0 < p ? ldc(&s_noise[j0]) : 0.0);
        double l[16], t[16], acc[16];  // L^-1_ii: rows 16 grp .., column 16 q + c
        const double* lp = a.Linv + (size_t)(i0 + 16 * grp) * P + i0 + 16 * q + c;
#pragma unroll
        for (int j = 0; j < 16; ++j) l[j] = ldc(lp + (size_t)j * P);
        const double* row = a.A + (size_t)(i0 + 16 * q) * P + lane;  // U_ik: rows 16 q .., column `lane`
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            t[j] = i + 1 < nt ? ldc(row + (size_t)j * P + (nt - 1) * kTile) : 0.0;
            acc[j] = 0.0;
        }
        for (uint32_t kk = nt - 1; kk > i; --kk) {
            double nx[16];
            if (kk - 1 > i) {
#pragma unroll
                for (int j = 0; j < 16; ++j) nx[j] = ldc(row + (size_t)j * P + (kk - 1) * kTile);
            } else {
#pragma unroll
                for (int j = 0; j < 16; ++j) nx[j] = 0.0;
            }
            const double bv = take(hb + kk * kTile, lane, a.ctrl, g.timeout, min(kk - i, 8u));
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                acc[j] = fma(t[j], bv, acc[j]);
                t[j] = nx[j];
            }
        }
        // acc[j] summed over the lanes: each exchange halves the rows a lane keeps,
        // so lane l ends with row l >> 2 of the wave's 16
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            const int off = 32 >> st, h = 8 >> st;
            const bool up = (lane & off) != 0;
#pragma unroll
            for (int j = 0; j < h; ++j) {
                const double send = up ? acc[j] : acc[j + h];
                const double kept = up ? acc[j + h] : acc[j];
                acc[j] = kept + __shfl_xor(send, off);
            }
        }
        acc[0] += __shfl_xor(acc[0], 2);
        acc[0] += __shfl_xor(acc[0], 1);
        if ((lane & 3) == 0) part[16 * q + (lane >> 2)] = acc[0];
        __syncthreads();
        double r = part[lane] - ws;  // minus the right-hand side
        double bi = 0.0;
        dot_bcast(bi, r, l);
        bi = over_groups(bi);
        const uint32_t col = i0 + 16 * q + c;
        if (grp == 0) stc(hb + col, bi);
        if (grp == 0 && col < p) {
            a.beta[col] = bi;
            a.beta32[col] = (float)(bi * a.xscale[col]);
            if (!isfinite(bi)) nonfinite = true;
            if (keep) {
                a.ring_beta[(size_t)slot * p + col] = bi;
                if (a.ring_lam) a.ring_lam[(size_t)slot * p + col] = ldc(&a.lam_m2[col]);
            }
        }
        __syncthreads();  // part is free again
    }
    if (nonfinite) atomicOr(&a.ctrl->err, kErrNonFinite);
    if (keep && rank == 0 && threadIdx.x == 0) a.ring_tau[slot] = current_tau(a);
    // no block leaves before every value it may wait on is there: the launch's
    // closing block clears them after this barrier
    group_sync(g);
}

// ---- one-block path, p <= 16 -----------------------------------------------------
// LDS (doubles, after hyper_lambda_tau's): the noise of beta (16), F (16 rows of
// 17) and the failed pivot (0: none).
constexpr int kSmallNoise = 32, kSmallF = 48, kSmallFail = kSmallF + 16 * 17, kSmallLds = 384;
static_assert(kSmallFail < kSmallLds, "one-block path LDS layout");

// acc -= (lane C of acc's row of 16 lanes) * y.
template <int C>
__device__ __forceinline__ void eliminate(double& acc, double y) {
    asm("s_nop 1\n\t" HSP_FMSUB(0, 0, 1, 2) : "+v"(acc) : "v"(y), "n"(C));
}

// Q = F^T D F, F unit upper triangular, by the pivots of D one after another: d
// holds Q (column l % 16 in lane l, a copy in each row of 16 lanes), and on return
// d[i] row i of F right of the diagonal; piv is D's entry l % 16.  Row I (or rows I
// and I + 1) of v loses x_I y, x_I being lane I of x's row of 16 lanes.
template <int I>
__device__ __forceinline__ void fmsub1(double (&v)[16], double x, double y) {
    asm("s_nop 1\n\t" HSP_FMSUB(0, 1, 2, 3) : "+v"(v[I]) : "v"(x), "v"(y), "n"(I));
}
template <int I>
__device__ __forceinline__ void fmsub2(double (&v)[16], double x, double y) {
    asm("s_nop 1\n\t" HSP_FMSUB(0, 2, 3, 4) HSP_FMSUB(1, 2, 3, 5)
        : "+&v"(v[I]), "+&v"(v[I + 1])
        : "v"(x), "v"(y), "n"(I), "n"(I + 1));
}
template <int C, int I>
__device__ __forceinline__ void ldl_rows(double (&d)[16], double f) {
    if constexpr (I < 16) {
        if constexpr (I > C + 1 && I < 15) fmsub2<I>(d, f, d[C]);
        else fmsub1<I>(d, f, d[C]);
        ldl_rows<C, I + (I > C + 1 && I < 15 ? 2 : 1)>(d, f);
    }
}
template <int C = 0>
__device__ __forceinline__ void ldl_pivots(double (&d)[16], double& piv) {
    if constexpr (C < 16) {
        const int c = threadIdx.x & 15;
        settle(d[C]);
        const double f = d[C] / row_bcast<C>(d[C]);
        ldl_rows<C, C + 1>(d, f);
        piv = c == C ? d[C] : piv;
        d[C] = c > C ? f : 0.0;
        ldl_pivots<C + 1>(d, piv);
    }
}

// v becomes F^-T v (entry l % 16 in lane l, d as ldl_pivots leaves it), and x
// becomes F^-1 x (row[k]: entry k of row l % 16 of F, zero up to the diagonal).
template <int I = 0>
__device__ __forceinline__ void solve_forward(double& v, const double (&d)[16]) {
    if constexpr (I < 15) {
        eliminate<I>(v, d[I]);
        solve_forward<I + 1>(v, d);
    }
}
template <int K = 15>
__device__ __forceinline__ void solve_backward(double& x, const double (&row)[16]) {
    if constexpr (K > 0) {
        eliminate<K>(x, row[K]);
        solve_backward<K - 1>(x, row);
    }
}

// While the z pass runs, wave 0 factors Q (padded to 16 with the identity) as
// F^T D F, wave 1 draws nu and xi, wave 2 the noise s; then wave 0 takes b and
// solves U beta = U^-T b + s, U = D^1/2 F, on its lanes, one entry per lane of a
// row of 16: F beta = D^-1 F^-T b + D^-1/2 s, two triangular solves of one
// multiply-add a step.  Divisions and square roots are correctly rounded (the
// hardware's reciprocal square root after one Newton step is off by up to 38
// 2^-53).  Bound by latencies; after b arrives it takes 15 + 15 steps and a
// division, where solves with a division per row took ~4 us.  N = 1000, p = 10,
// 8 sweeps: 89 us, as with two products by an explicit U^-T from such roots (88).
__device__ __forceinline__ void small_path(Args& a, Group& g, uint32_t k, double* lds) {
    const uint32_t p = a.x.p;
    const int lane = threadIdx.x & 63, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool beta = (a.mode & kModeBeta) != 0, in = (uint32_t)c < p;
    const uint32_t cj = min((uint32_t)c, p - 1u);
    double d[16], piv = 1.0, root = 1.0;
    if (wave == 0 && beta) {
#pragma unroll
        for (int i = 0; i < 16; ++i) d[i] = a.G[(size_t)min((uint32_t)i, p - 1u) * p + cj];
    }
    const double scale = a.xscale[cj];
    const double tau = hyper_lambda_tau(a, k, true, lds);
    __syncthreads();
    stamp(g);
    if (wave == 1 && (a.mode & kModeNuXi)) {
        if ((uint32_t)lane < p) {
            const Words4 w = draw_words(a.seed, lane, k, kTagNu, 0, a.chain);
            a.nu_m1[lane] = -log(u01d(w.w0)) / (1.0 + lds[kRedLambda + lane]);
        } else if (lane == kSmallP) {
            const Words4 w = draw_words(a.seed, 0, k, kTagXi, 0, a.chain);
            *a.xi_m1 = -log(u01d(w.w0)) / (1.0 + tau);
        }
    }
    if (wave == 2 && beta && lane < kSmallP) {
        const Words4 w = draw_words(a.seed, lane, k, kTagBetaS, 0, a.chain);
        lds[kSmallNoise + lane] = in ? box_muller_d(u01d(w.w0), u01d(w.w1)) : 0.0;
    }
    if (wave == 0 && beta) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const double q = i == c ? fma(tau, lds[kRedLambda + cj], d[i]) : d[i];
            d[i] = in && (uint32_t)i < p ? q : (i == c ? 1.0 : 0.0);
        }
        ldl_pivots(d, piv);
        const unsigned long long fail = __ballot(lane < 16 && !(piv > 0.0));
        if (lane == 0) lds[kSmallFail] = fail ? (double)__ffsll((long long)fail) : 0.0;
        root = sqrt(piv);
        if (lane < 16) {
#pragma unroll
            for (int i = 0; i < 16; ++i) lds[kSmallF + i * 17 + lane] = d[i];
        }
    }
    __syncthreads();
    const bool bad = beta && lds[kSmallFail] != 0.0;
    if (wave != 0) return;
    const bool from_sum = (a.mode & (kModeZ | kModeBsum)) != 0;
    double b = 0.0;
    double row[16], noise = 0.0;  // row c of F; entry c of D^-1/2 s
    if (beta) {
#pragma unroll
        for (int j = 0; j < 16; ++j) row[j] = lds[kSmallF + c * 17 + j];
        noise = lds[kSmallNoise + c] / root;
    }
    if (from_sum) {
        if ((a.mode & kModeZ) && lane == 0) wait_count(&a.ctrl->z_count, g.zbase + a.zgroups, a.ctrl, a.timeout_ticks, 8);
        // b as the z blocks (of this launch, or of an earlier pass) accumulated it,
        // in the units of the stored X, unscaled exactly
        b = ldc(&a.bsum[cj]) * scale;
        if (lane < 16 && in) a.b[c] = b;
    } else if (beta) {
        b = a.b[cj];
    }
    bool keep;
    const uint32_t slot = record_slot(a, k, &keep);
    if (beta && !bad) {
        double v = in ? b : 0.0;
        solve_forward(v, d);
        double bj = v / piv + noise;
        solve_backward(bj, row);
        if (lane < 16 && in) {
            a.beta[c] = bj;
            a.beta32[c] = (float)(bj * scale);
            if (keep) a.ring_beta[(size_t)slot * p + c] = bj;
        }
        if (__ballot(lane < 16 && in && !isfinite(bj)) && lane == 0) atomicOr(&a.ctrl->err, kErrNonFinite);
    }
    if (bad && lane == 0) {
        atomicOr(&a.ctrl->err, kErrNotPD);
        atomicCAS(&a.ctrl->chol_info, 0, (int)lds[kSmallFail]);
    }
    if (keep) {
        if (a.ring_lam && lane < 16 && in) a.ring_lam[(size_t)slot * p + c] = lds[kRedLambda + c];
        if (lane == 0) a.ring_tau[slot] = tau;
    }
}

// The part of the tile path before b is needed: lambda, tau, nu, xi, the noise of
// beta and the factorisation's tasks.  False if the factorisation failed.
__device__ __forceinline__ bool tile_factor(Args& a, Group& g, uint32_t rank, uint32_t k, double* lds) {
    const uint32_t p = a.x.p;
    Tile& S = *reinterpret_cast<Tile*>(lds);
    Tile& T = *reinterpret_cast<Tile*>(lds + kTile * kTileLd);
    double* flag = lds + 2 * kTile * kTileLd - 1;  // T's unused padding corner
    double* s_noise = a.vec + p;
    // with kModePost an earlier launch of this sweep did all this
    if (a.mode & kModePost) return true;
    const double tau = hyper_lambda_tau(a, k, rank == 0, lds);
    // No block waits here for block 0's lambda^-2 in memory: whoever reads it in
    // the factorisation has waited for a tile that follows from block 0's first,
    // stored later.  nu and xi wait until every block has read the old ones.
    // (A launch without the factorisation has no later barrier: all wait.)
    if (a.mode & kModeBeta) {
        hyper_arrive(g);
        if (rank == g.size - 1) hyper_wait(g);
    } else {
        group_sync(g);
    }
    if (rank == g.size - 1) {
        if (a.mode & kModeNuXi) hyper_nu_xi(a, k);
        if (a.mode & kModeBeta)
            for (uint32_t i = threadIdx.x; i < p; i += kThreads) {
                const Words4 w = draw_words(a.seed, i, k, kTagBetaS, 0, a.chain);
                stc(&s_noise[i], box_muller_d(u01d(w.w0), u01d(w.w1)));
            }
    }
    if (!(a.mode & kModeBeta)) return true;
    // Factorisation of [Q | I]: U in A (upper), L^-1 = U^-T in Linv (lower), as
    // this block's list of tile tasks.
    return run_tasks(a, g, rank, tau, S, T, flag);
}

// The rest of the tile path, from the factorisation (ok: this block's part of
// it succeeded) and b to beta.
__device__ __forceinline__ void tile_beta(Args& a, Group& g, uint32_t rank, uint32_t k, double* lds, bool ok) {
    const uint32_t p = a.x.p, P = padded(p);
    double* flag = lds + 2 * kTile * kTileLd - 1;
    double* s_noise = a.vec + p;
    const unsigned long long ztarget = (a.mode & kModeZ) ? g.zbase + a.zgroups : 0ull;
    if ((a.mode & kModeBeta) && !(a.mode & kModePost)) {
        group_sync_z(g, ztarget);
    } else {
        if (ztarget && threadIdx.x == 0) wait_count(&a.ctrl->z_count, ztarget, a.ctrl, a.timeout_ticks, 64);
        __syncthreads();
    }
    if (a.mode & kModePre) return;  // b is taken by a later launch of this sweep

    // b = X^T z into LDS (zero on the padding), as the z groups accumulated
    // it; block 0 also stores it.  A vector too long for the LDS (big) is
    // read from memory where it is used instead.
    const bool big = P + 16 * 17 > (uint32_t)kLdsDoubles;
    const bool from_sum = (a.mode & (kModeZ | kModeBsum)) != 0;
    auto b_at = [&](uint32_t j) -> double {
        if (j >= p) return 0.0;
        return from_sum ? ldc(&a.bsum[j]) * a.xscale[j] : a.b[j];  // unscaled exactly
    };
    double* bl = lds;
    // (the failure flags of this launch's factorisation, or with kModePost of the
    // earlier one's, come with b)
    uint32_t err = 0;
    if (threadIdx.x == 0) err = __hip_atomic_load(&g.ctrl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool by_rows = (a.mode & kModeBeta) && a.subst;  // the owner of a row takes its b
    for (uint32_t j = threadIdx.x; !by_rows && j < P; j += kThreads) {
        const double s = b_at(j);
        if (from_sum && rank == 0 && j < p) a.b[j] = s;
        if (!big) bl[j] = s;
    }
    if (threadIdx.x == 0) *flag = (err & (kErrNotPD | kErrTimeout)) ? 1.0 : 0.0;
    __syncthreads();
    ok = ok && *flag == 0.0;

    if (by_rows && ok) {
        subst_solve(a, g, rank, k, lds, from_sum);
    } else if ((a.mode & kModeBeta) && !by_rows && ok) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        // y = L^-1 b + s, four rows per wave at a time.  L^-1 is zero above the
        // diagonal and the identity on the padding, and b is zero there, so
        // the sums need no bounds: row i runs over every column up to the
        // group's last row.  Rows are dealt so that each wave gets short and
        // long ones.
        double* yv = a.vec;
        for (uint32_t i0 = (rank * 4 + wave) * 4; i0 < p; i0 += g.size * 16) {
            double acc[4] = {0.0, 0.0, 0.0, 0.0};
            const double* L0 = a.Linv + (size_t)i0 * P;
            const uint32_t jn = i0 + 4;
            uint32_t j = lane;
            for (; j + 192 < jn; j += 256) {
                double x[4][4], bj[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    bj[u] = big ? b_at(j + 64 * u) : bl[j + 64 * u];
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[u][r] = ldc(L0 + (size_t)r * P + j + 64 * u);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[r] = fma(x[u][r], bj[u], acc[r]);
            }
            for (; j < jn; j += 64) {
                const double bj = big ? b_at(j) : bl[j];
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r] = fma(ldc(L0 + (size_t)r * P + j), bj, acc[r]);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) acc[r] += __shfl_xor(acc[r], off);
            if (lane < 4 && i0 + lane < p) {
                double yi = acc[0];
#pragma unroll
                for (int r = 1; r < 4; ++r) yi = lane == r ? acc[r] : yi;
                stc(&yv[i0 + lane], yi + ldc(&s_noise[i0 + lane]));
            }
        }
        group_sync(g);
        // beta = L^-T y, y from LDS (zero on the padding); column j sums rows
        // i >= j, the rest of L^-1 being zero.  Block r takes two 16-column
        // blocks, one from each end (columns 16 r and P - 16 (r + 1) on), so
        // every block reads about the same number of rows; 16 row groups per
        // column, four rows of loads in flight each.
        double* yl = lds;
        if (!big)
            for (uint32_t j = threadIdx.x; j < P; j += kThreads) yl[j] = j < p ? ldc(&yv[j]) : 0.0;
        auto y_at = [&](uint32_t i) -> double { return big ? (i < p ? ldc(&yv[i]) : 0.0) : yl[i]; };
        double* red = big ? lds : lds + P;
        __syncthreads();
        bool keep;
        const uint32_t slot = record_slot(a, k, &keep);
        const int tc = threadIdx.x & 15, tr = threadIdx.x >> 4;
        bool nonfinite = false;
        for (uint32_t cb0 = rank * 16; cb0 < P / 2; cb0 += g.size * 16) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const uint32_t cb = half == 0 ? cb0 : P - 16 - cb0;
                const uint32_t col = cb + tc;
                const double* Lc = a.Linv + col;
                double acc[4] = {0.0, 0.0, 0.0, 0.0};
                uint32_t i = cb + tr;
                // sixteen loads in flight; the same accumulation order as
                // the four-row loop below
                for (; i + 240 < P; i += 256) {
                    double x[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) x[u] = ldc(Lc + (size_t)(i + 16 * u) * P);
#pragma unroll
                    for (int u = 0; u < 16; ++u) acc[u & 3] = fma(x[u], y_at(i + 16 * u), acc[u & 3]);
                }
                for (; i + 48 < P; i += 64)
#pragma unroll
                    for (int u = 0; u < 4; ++u) acc[u] = fma(ldc(Lc + (size_t)(i + 16 * u) * P), y_at(i + 16 * u), acc[u]);
                for (; i < P; i += 16) acc[0] = fma(ldc(Lc + (size_t)i * P), y_at(i), acc[0]);
                red[tr * 17 + tc] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
                __syncthreads();
                if (tr == 0 && col < p) {
                    double bi = 0.0;
                    for (int q = 0; q < 16; ++q) bi += red[q * 17 + tc];
                    a.beta[col] = bi;
                    a.beta32[col] = (float)(bi * a.xscale[col]);
                    if (!isfinite(bi)) nonfinite = true;
                    if (keep) {
                        a.ring_beta[(size_t)slot * p + col] = bi;
                        if (a.ring_lam) a.ring_lam[(size_t)slot * p + col] = ldc(&a.lam_m2[col]);
                    }
                }
                __syncthreads();
            }
        }
        if (nonfinite) atomicOr(&a.ctrl->err, kErrNonFinite);
        if (keep && rank == 0 && threadIdx.x == 0) a.ring_tau[slot] = current_tau(a);
    }
}

// The p-side role of block `rank` of the group, in two parts: all that comes
// before b, and the rest.  Between them the block may take units of the z pass.
// pside_begin returns false if the factorisation failed.  SMALL: a kernel for
// p <= 16 alone, without the tile path.
template <bool SMALL>
__device__ __forceinline__ bool pside_begin(Args& a, Group& g, uint32_t rank, uint32_t k, double* lds) {
    g.trace = a.trace ? a.trace + (size_t)rank * kTraceSlots : nullptr;
    if (g.trace && threadIdx.x == 0) g.trace[0] = wall_clock64();
    g.ctrl = a.ctrl;
    g.base = a.ctrl->bar_epoch;
    g.zbase = a.ctrl->z_epoch;
    g.size = a.gp;
    g.n = 0;
    g.slot = 0;
    g.npotrf = 0;
    g.timeout = a.timeout_ticks;
    // the two-launch split is for the tile path; a launch never asks the
    // one-block path for half a sweep
    if constexpr (!SMALL) {
        if (a.x.p > (uint32_t)kSmallP) return tile_factor(a, g, rank, k, lds);
    }
    if (!(a.mode & (kModePre | kModePost))) small_path(a, g, k, lds);
    return true;
}

template <bool SMALL>
__device__ __forceinline__ void pside_end(Args& a, Group& g, uint32_t rank, uint32_t k, double* lds, bool ok) {
    if constexpr (!SMALL) {
        if (a.x.p > (uint32_t)kSmallP) tile_beta(a, g, rank, k, lds, ok);
    }
    // the last barrier above was passed by every block of the group, and the
    // z-pass blocks have all finished if they ran: close the launch
    if (rank == 0) {
        __syncthreads();
        if (threadIdx.x == 0) {
            a.ctrl->bar_epoch = g.base + (unsigned long long)g.n * g.size;
            if (a.mode & kModeZ) a.ctrl->z_epoch = g.zbase + a.zgroups;
            if (a.mode & kModeTau) *a.tau_m2 = current_tau(a);
            if (a.mode & kModeAdvance) a.ctrl->sweep = k;
        }
        if (a.x.p > (uint32_t)kSmallP && (a.mode & kModeBeta) && !(a.mode & kModePost)) {
            const uint32_t nt = padded(a.x.p) / kTile;
            for (uint32_t e = threadIdx.x; e < 2 * nt * nt; e += kThreads) a.ver[e] = 0u;
            if (threadIdx.x == 0) {
                a.ctrl->task_next = 0u;
                a.ctrl->hyper_count = 0ull;
            }
        }
        if (a.subst && (a.mode & kModeBeta) && !(a.mode & kModePre)) {
            const uint32_t P = padded(a.x.p);
            for (uint32_t e = threadIdx.x; e < 2 * P; e += kThreads)
                stc(handoff(a) + e, __longlong_as_double((long long)kNotReady));
        }
        if (a.mode & (kModeZ | kModeBsum)) {
            // every block of the group has read b's accumulator (before the
            // barrier that follows y): clear it for the next launch
            if (threadIdx.x == 0) a.ctrl->z_next = 0u;
            for (uint32_t j = threadIdx.x; j < a.x.ld; j += kThreads) stc(&a.bsum[j], 0.0);
        }
    }
}

}  // namespace hsp
