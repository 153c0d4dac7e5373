// One Gibbs sweep as one kernel launch.
//
// The grid has two roles.  Blocks [0, gp) form the p-side group: lambda^-2,
// tau^-2, nu^-1, xi^-1 and the Cholesky factorisation of Q need only the
// previous sweep, so they run while blocks [gp, gp + gz) stream X through the
// z pass (z | beta and the partial sums of X^T z).  The group then waits for
// the z pass, reduces X^T z and draws beta.  This is the schedule of
// Section 5 -- (i) z in parallel with lambda, then tau; (ii) beta with nu and
// xi -- inside a single launch, and the p-side work hides under the
// bandwidth-bound pass over X.
//
// The group blocks come first in the grid: they are dispatched before any
// z-pass block and stay resident, so their barriers only ever wait on
// blocks that are running.  The z-pass blocks never wait on anything.
#include <algorithm>
#include <utility>

#include "mc_dev.hpp"
#include "pside_dev.hpp"
#include "zpass_dev.hpp"

namespace hsp {
namespace {

// The launch's description lives in device memory (read through the scalar
// cache as needed) rather than in kernel arguments, which would otherwise stay
// pinned in scalar registers for the whole kernel.
// A launch may serve several independent chains (a batch): block b belongs
// to chain chain_of_block[b] (chain 0 for all when the map is null) and runs
// that chain's role at position b - block0 of its blocks, or, marked with
// kWorkerBit, is a worker of the pack's shared z queue.
template <int XT, int KC, int R, bool WIDE, bool SMALL = false>
__device__ __forceinline__ void run_block(Args& a, double* lds) {
    constexpr int RC = SMALL ? 64 : kRedCols;  // columns of an LDS reduction segment
    uint32_t b = blockIdx.x - a.block0;
    const uint32_t k = a.ctrl->sweep + 1u;
    if (a.idle) {
        if (b == a.idle) return;
        if (b > a.idle) --b;
    }
    const bool pside = b < a.gp;
    if (!pside && b - a.gp >= a.gz) return;  // no z-pass work in this launch
    Group g;
    bool ok = true, z = !pside;
    if (pside) {
        ok = pside_begin<SMALL>(a, g, b, k, lds);
        // a block whose factorisation work is done may take units of the z pass:
        // the group's next barrier, which every reader of b passes, covers its
        // additions, and the z-pass blocks' own count is not touched
        z = a.help && b > 0 && (a.mode & kModeZ) && (a.mode & kModeBeta);
        __syncthreads();
    }
    if (z) {
        ZSums<XT, KC> sums;
        const bool any = z_take<XT, KC, R, WIDE, SMALL ? kWave / R : 1>(a, b - a.gp, a.gz, pside, k, lds, sums);
        if (!pside) {
            z_finish<XT, KC, WIDE, RC>(a, b - a.gp, a.gz, lds, sums, any);
            return;
        }
        if (any) z_flush<XT, KC, WIDE, RC>(a, sums.b, sums.maxatt, sums.capped, lds);
    }
    pside_end<SMALL>(a, g, b, k, lds, ok);
}

// KC: 16-byte chunks per lane of a wave (of the whole row, or with WIDE of
// the wave's quarter of it); R: rows per tile.
template <int XT, int KC, int R, bool WIDE>
__global__ __launch_bounds__(kThreads, 2) void sweep_kernel(const SweepArgs* const* __restrict__ args,
                                                            const uint16_t* __restrict__ chain_of_block) {
    __shared__ double lds[kLdsDoubles];
    const uint32_t c = chain_of_block ? chain_of_block[blockIdx.x] : 0u;
    if constexpr (!WIDE) {
        if (c & kWorkerBit) {
            zqueue_role<XT, KC, R>(args, c & ~(uint32_t)kWorkerBit, lds);
            return;
        }
    }
    run_block<XT, KC, R, WIDE>(*(Args*)args[c], lds);
}



// A lone chain with p <= 16 (rows of one chunk): without the tile path, its LDS
// and its registers, so that a sweep of tens of microseconds starts and fetches
// its code sooner.
template <int XT>
__global__ __launch_bounds__(kThreads, 2) void small_sweep_kernel(const SweepArgs* const* __restrict__ args,
                                                                  const uint16_t* __restrict__) {
    __shared__ double lds[kSmallLds];
    run_block<XT, 1, rows_for(XT, 1), false, true>(*(Args*)args[0], lds);
}

// The multi-chain z pass for chains sharing one bfloat16 design (KS
// 32-column steps per wave); no block waits for another.
template <int KS>
__global__ __launch_bounds__(kThreads, 2) void mc_zpass_kernel(const McArgs* __restrict__ mc) {
    __shared__ double lds[kMcLdsDoubles];
    McView& m = *(McView*)mc;
    mc_role<KS>(m, blockIdx.x, lds);
}

__global__ __launch_bounds__(256) void mc_sum_kernel(const McArgs* __restrict__ mc) {
    __shared__ double lds[256];
    McView& m = *(McView*)mc;
    mc_sum_role(m, lds);
}

using KernelFn = void (*)(const SweepArgs* const*, const uint16_t*);

template <int XT, int... KCs>
KernelFn pick(int kc, std::integer_sequence<int, KCs...>) {
    KernelFn f = nullptr;
    ((kc == KCs + 1 ? (f = &sweep_kernel<XT, KCs + 1, rows_for(XT, KCs + 1), false>, 0) : 0), ...);
    return f;
}

// wide rows: kcw chunks per lane of each wave's quarter
template <int XT, int... KCs>
KernelFn pick_wide(int kcw, std::integer_sequence<int, KCs...>) {
    KernelFn f = nullptr;
    ((kcw == KCs + 1 ? (f = &sweep_kernel<XT, KCs + 1, rows_for(XT, 4 * (KCs + 1)), true>, 0) : 0), ...);
    return f;
}

KernelFn kernel_for(int xtype, int chunks) {
    if (!wide_chunks(xtype, chunks)) {
        if (xtype == 0) return pick<0>(chunks, std::make_integer_sequence<int, 6>{});
        return pick<1>(chunks, std::make_integer_sequence<int, 2>{});
    }
    const int kcw = (chunks + 3) / 4;
    if (xtype == 0) return pick_wide<0>(kcw, std::make_integer_sequence<int, kMaxP / (kWave * 4 * 4)>{});
    return pick_wide<1>(kcw, std::make_integer_sequence<int, kMaxP / (kWave * 8 * 4)>{});
}

// The kernel of a lone chain's launches.
KernelFn lone_kernel(const XLayout& x, int chunks) {
    if (x.p > (uint32_t)kSmallP) return kernel_for(x.xtype, chunks);
    return x.xtype == 0 ? &small_sweep_kernel<0> : &small_sweep_kernel<1>;
}

}  // namespace

uint32_t max_group(const XLayout& x, int capacity) {
    const uint32_t nt = (x.p + kTile - 1) / kTile;
    // (few tiles: block 0's chain has most of the tasks, and the substitution a
    // block per row)
    uint32_t gp = x.p <= (uint32_t)kSmallP ? 1u : nt < kFewTiles ? std::max(nt, nt * (nt - 1) / 2) : nt * (nt + 1) / 2;
    // the factorisation's tile tasks (each ~6 us on one block) against the
    // pass over X (~6 TB/s) on the other three quarters of the device
    double tasks = 0.0;
    for (uint32_t k = 0; x.p > (uint32_t)kSmallP && k < nt; ++k) {
        const double m = nt - k - 1;
        tasks += 1.0 + m + m * (m + 1.0) / 2.0 + (chain_inverse(nt) ? k + m * (k + 1.0) : 0.0);
    }
    const double z_us = (double)x.N * x.ld * (x.xtype == 0 ? 4 : 2) / 6.0e6;
    const bool factor_bound = tasks * 6.0 / (kMaxGroup - 1) > z_us;
    if (x.p <= kLargeP && !factor_bound) {
        // the factorisation hides under the z pass: a quarter of the device at most
        if (gp > (uint32_t)kMaxGroup) gp = kMaxGroup;
        if (gp > (uint32_t)capacity / 4) gp = capacity / 4 > 0 ? capacity / 4 : 1;
    } else if (with_inverse(nt)) {
        // the factorisation outweighs the pass over X: three quarters
        const uint32_t cap = (uint32_t)capacity * 3 / 4;
        if (gp > cap) gp = cap > 0 ? cap : 1;
    } else {
        // Without L^-1 the updates run at ~4.2 us a task and block, and block 0's
        // chain at ~17 us a step: more than tasks / (2 nt) blocks would only wait for
        // the chain.  The pass over X keeps its share of the time, which is the
        // chain's or that of all the work on all blocks, and a sixteenth.  us per sweep
        // at 128 / 192 / 256 / 320 / 384 / 448 / 480 blocks:
        // p = 2000, N = 2e4 float32 525 / 528 / 536 / - / 576 (96: 522, 64: 607);
        // p = 3000, N = 1e4 float32 902 / 783 / 796 / - / 891; p = 4096, N = 2e5
        // float32 1870 / 1448 / 1390 / 1503 / 1589 / 2097; p = 7003, N = 6e4 bfloat16
        // - / - / 4186 / 3980 / 3773 / 3620 / 3645; p = 10000, N = 5e4 bfloat16
        // - / - / 11284 / - / 9818 / 9313 / 9047.
        const double share = 1.0 - z_us / std::max(17.0 * nt, z_us + tasks * 4.2 / capacity);
        const uint32_t want = std::max((uint32_t)kMaxGroup, (uint32_t)std::min(tasks / (2.0 * nt), share * capacity));
        gp = std::max(1u, std::min({gp, want, (uint32_t)capacity * 15 / 16}));
    }
    return gp;
}

hipError_t sweep_plan(const XLayout& x, int num_cus, SweepPlan* plan, uint32_t gp_req) {
    const int vec = x.xtype == 0 ? 4 : 8;
    plan->chunks = (int)((x.ld + kWave * vec - 1) / (kWave * vec));
    plan->rows = rows_for(x.xtype, plan->chunks);
    const bool wide = wide_chunks(x.xtype, plan->chunks);
    KernelFn f = lone_kernel(x, plan->chunks);
    if (!f) return hipErrorInvalidValue;
    int per_cu = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(f),
                                                                kThreads, 0);
    if (e != hipSuccess) return e;
    if (per_cu < 1) return hipErrorInvalidConfiguration;
    plan->capacity = per_cu * num_cus;
    plan->cus = (uint32_t)num_cus;
    uint32_t gp = max_group(x, plan->capacity);
    if (gp_req > 0 && gp_req < gp) gp = gp_req;
    plan->gp = gp;
    const uint64_t tiles = (x.N + plan->rows - 1) / plan->rows;
    // a wave takes a tile (a block, for wide rows)
    uint64_t gz = wide ? tiles : (tiles + kWPB - 1) / kWPB;
    const uint64_t room = (uint64_t)plan->capacity - gp;
    if (gz > room) gz = room;
    if (gz < 1) gz = 1;
    plan->gz = (uint32_t)gz;
    // a short pass (fewer than four tiles per taker) goes out one tile per wave at
    // a time: with units of 8 tiles N = 1e5, p = 100 had 391 units for 509 blocks
    const uint64_t takers = wide ? gz : gz * kWPB;
    if (tiles < 4 * takers) plan->unit = wide ? 1u : (uint32_t)kWPB;
    return hipSuccess;
}

// Blocks b and b + (compute units) of a full grid share a compute unit (the
// dispatcher deals blocks out to the units in order, twice round).  When a
// launch fills the device at two blocks per unit, block 0 (the p-side's
// critical chain) would share its unit with a z-pass block; that block is
// left idle instead, and the z pass takes one block fewer: the chain then
// has its unit to itself (N = 1e6, p = 1000 bfloat16, while that chain was its bound:
// 0.415 -> 0.402 ms per sweep; float32, bound by its z pass, unchanged).
void sweep_finish_args(SweepArgs* a, const SweepPlan& plan) {
    a->gp = plan.gp;
    a->gz = (a->mode & kModeZ) ? plan.gz : 0u;
    a->idle = 0u;
    if (a->gp > 0u && a->gz > plan.cus && plan.capacity == 2 * (int)plan.cus &&
        a->gp + a->gz == (uint32_t)plan.capacity) {
        a->gz -= 1u;
        a->idle = plan.cus;
    }
    // A group of more than a quarter of the device leaves the z pass too few blocks
    // to end with it: its blocks (but not block 0, which finishes last) then take
    // z-pass units when the factorisation has no task left for them.  N = 2e5,
    // p = 4096 float32 (384 of 512 blocks): the z pass ends at 1622 instead of
    // 2329 us, 2.51 -> 1.82 ms per sweep.  Smaller groups stay out: they would find
    // little left, and looking costs a short sweep 2 % (N = 1e5, p = 100).
    a->help = 4u * a->gp > (uint32_t)plan.capacity ? 1u : 0u;
    a->zgroups = z_groups(a->gz);
    a->z_static_pct = plan.static_pct;
    a->z_unit = plan.unit;
}

hipError_t sweep_launch(const SweepArgs& host, const SweepArgs* const* table, const SweepPlan& plan,
                        hipStream_t st) {
    KernelFn f = lone_kernel(host.x, plan.chunks);
    if (!f) return hipErrorInvalidValue;
    const uint16_t* none = nullptr;
    void* args[] = {&table, &none};
    return hipLaunchKernel(reinterpret_cast<const void*>(f), dim3(host.gp + host.gz + (host.idle ? 1u : 0u)),
                           dim3(kThreads),
                           args, 0, st);
}

int pack_capacity(int xtype, int chunks, int num_cus) {
    KernelFn f = kernel_for(xtype, chunks);
    int per_cu = 0;
    if (!f || hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(f),
                                                           kThreads, 0) != hipSuccess)
        return 0;
    return per_cu * num_cus;
}

hipError_t mc_launch(const McArgs* mc, uint32_t ld, uint32_t gz, uint32_t nchains, hipStream_t st) {
    if (ld > kMcMaxLd || nchains < 1 || nchains > (uint32_t)kMcChains) return hipErrorInvalidValue;
    void* args[] = {&mc};
    const void* f = mc_steps(ld) == 4u ? reinterpret_cast<const void*>(&mc_zpass_kernel<4>)
                                       : reinterpret_cast<const void*>(&mc_zpass_kernel<kMcKs>);
    if (hipError_t e = hipLaunchKernel(f, dim3(gz), dim3(kThreads), args, 0, st)) return e;
    return hipLaunchKernel(reinterpret_cast<const void*>(&mc_sum_kernel), dim3((ld + 63) / 64, nchains), dim3(256),
                           args, 0, st);
}

hipError_t pack_launch(int xtype, int chunks, const SweepArgs* const* table, const uint16_t* chain_of_block,
                       uint32_t blocks, hipStream_t st) {
    KernelFn f = kernel_for(xtype, chunks);
    if (!f) return hipErrorInvalidValue;
    void* args[] = {&table, &chain_of_block};
    return hipLaunchKernel(reinterpret_cast<const void*>(f), dim3(blocks), dim3(kThreads), args, 0, st);
}

}  // namespace hsp
