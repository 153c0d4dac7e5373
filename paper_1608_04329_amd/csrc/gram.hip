// One-time work at creation: the column scales of X, X packed into the
// library layout, input validation, and G = X^T X in float64 (Section 5,
// beta step i).  Also small kernels outside the sweep: the sorting of rows, the
// gathering of a few draws, the device Philox test hook and the read-ceiling probe.
#include <mutex>
#include <type_traits>

#include "hsp_internal.hpp"
#include "philox.hpp"

namespace hsp {
namespace {

__device__ __forceinline__ float load_x(const XLayout& x, size_t row, uint32_t col) {
    if (x.xtype == 0) return static_cast<const float*>(x.X)[row * x.ld + col];
    const uint32_t bits = (uint32_t) static_cast<const uint16_t*>(x.X)[row * x.ld + col] << 16;
    return __uint_as_float(bits);
}

// float32 -> bfloat16, round to nearest, ties to even (finite inputs).
__device__ __forceinline__ uint16_t to_bf16(float f) {
    const uint32_t u = __float_as_uint(f);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// Column maxima of |x|: block (bx, by) scans rows [bx R, bx R + R) of the 256
// columns at by * 256, one column per thread (a row's columns are adjacent
// threads, so every load instruction reads one contiguous row segment), and
// merges its maximum into out[col] by an atomic maximum on the bit pattern
// (non-negative floats order as unsigned integers; NaN sorts above infinity).
constexpr uint32_t kColmaxRows = 512;
__global__ __launch_bounds__(256) void colmax_kernel(const float* __restrict__ src, uint32_t N, uint32_t p,
                                                     uint32_t* __restrict__ out) {
    const uint32_t col = blockIdx.y * 256u + threadIdx.x;
    if (col >= p) return;
    const size_t r0 = (size_t)blockIdx.x * kColmaxRows;
    const size_t r1 = min((size_t)N, r0 + kColmaxRows);
    uint32_t m = 0;
    for (size_t r = r0; r < r1; ++r) m = max(m, __float_as_uint(src[r * p + col]) & 0x7FFFFFFFu);
    atomicMax(&out[col], m);
}

// The library's copy: column j multiplied by 2^-e[j] (exact), rounded to
// bfloat16 if asked (rounding commutes with the power-of-two scale).  Each
// element is read and written by the same thread, so src may alias dst when
// the two layouts coincide.
__global__ void pack_kernel(const float* src, XLayout dst, const int32_t* __restrict__ e) {
    const size_t n = (size_t)dst.N * dst.ld;
    for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < n;
         idx += (size_t)gridDim.x * blockDim.x) {
        const size_t row = idx / dst.ld;
        const uint32_t col = (uint32_t)(idx % dst.ld);
        const float v = col < dst.p ? ldexpf(src[row * dst.p + col], -e[col]) : 0.0f;
        if (dst.xtype == 0) const_cast<float*>(static_cast<const float*>(dst.X))[idx] = v;
        else const_cast<uint16_t*>(static_cast<const uint16_t*>(dst.X))[idx] = to_bf16(v);
    }
}

__global__ void validate_kernel(XLayout x, const uint8_t* __restrict__ y, Ctrl* ctrl) {
    const size_t n = (size_t)x.N * x.ld;
    bool bad = false;
    for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < n;
         idx += (size_t)gridDim.x * blockDim.x) {
        if (!isfinite(load_x(x, idx / x.ld, (uint32_t)(idx % x.ld)))) bad = true;
    }
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < x.N;
         i += (size_t)gridDim.x * blockDim.x)
        if (y[i] > 1) bad = true;
    if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(&ctrl->err, kErrInput);
}

// ---- G = X^T X on the FP64 matrix cores ---------------------------------------
// The upper triangle of G is cut into T x T tiles (ti <= tj, "pairs"), T = 32
// NB, and the rows of X into splits.  Block (pair, split) stages kGramK rows of
// X's column tiles ti and tj in LDS as float32 (two buffers, one barrier per
// stage, the next stage's loads in flight during the products) and accumulates
// X_ti^T X_tj with v_mfma_f64_16x16x4f64, widening each element exactly as it
// leaves LDS.  Wave (wr, wc) owns the 16 x 16 blocks (2 i + wr, 2 j + wc),
// i, j < NB: interleaved, so that in the last tile column and on the diagonal,
// where blocks beyond p and below the diagonal are left out, the four waves
// keep equal shares.  Lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16],
// i.e. rows of the stage are the contraction index, and holds D[l / 16 + 4 r]
// [l % 16] in its r-th result.  Every split writes its partial tile (its blocks
// inside the matrix and not below its diagonal); a second kernel sums the splits
// of each entry in split order, so G does not depend on timing.
//
// Bound by the matrix cores: one operation takes 64 cycles of a SIMD, and with
// NB = 4 a wave reads and widens 8 fragments per 16 operations (NB = 2: 4 per
// 4), so LDS, conversions and the loads of X mostly hide behind them.  N = 1e6,
// p = 1000 float32: 16.9 ms (64 TFLOP/s of the blocks computed; a large library
// product reaches 73), against 80 ms with 64-wide tiles staged as float64 by
// 4-byte loads; N = 3e5, p = 777 bfloat16: 14.3 -> 3.4 ms.
constexpr int kGramK = 32;  // rows of X per stage
typedef double GAcc __attribute__((ext_vector_type(4)));

// A tile's LDS row: T floats and 16 more, so that the four rows one fragment
// read touches lie in different quarters of the 64 banks.
template <int NB>
constexpr int gram_stride() { return 32 * NB + 16; }

// VN consecutive columns from col of one row, as 16 bytes of X.  ALIGNED (rows
// start on 16-byte boundaries): one load with no branch; columns past p are
// read only inside the 16 bytes that hold column p - 1, and whole groups past p
// read that group again (what they hold only enters products of columns past p,
// which are dropped).  Otherwise elements past p are zeros, loaded one by one.
template <int XT, int VN, bool ALIGNED>
__device__ __forceinline__ uint4 gram_fetch(const XLayout& x, size_t row, uint32_t col) {
    if constexpr (ALIGNED) {
        const uint32_t c = min(col, (x.p - 1u) / VN * VN);
        return *reinterpret_cast<const uint4*>(static_cast<const char*>(x.X) + (row * x.ld + c) * (XT == 0 ? 4 : 2));
    } else {
        uint32_t u[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < VN; ++e)
            if (col + e < x.p) {
                if constexpr (XT == 0) u[e & 3] = static_cast<const uint32_t*>(x.X)[row * x.ld + col + e];
                else u[(e >> 1) & 3] |= (uint32_t) static_cast<const uint16_t*>(x.X)[row * x.ld + col + e] << (16 * (e & 1));
            }
        return make_uint4(u[0], u[1], u[2], u[3]);
    }
}

// The products of one stage: acc(i, j) += S(:, block 2 i + wr)^T B(:, block
// 2 j + wc) for j < JL, and only i <= j on a diagonal tile (which for wave
// (1, 0) includes blocks (2 i + 1, 2 i) just below the diagonal: dropped when
// the tile is written, rather than branched around).
template <int NB, int JL, bool DIAG>
__device__ __forceinline__ void gram_products(const float* __restrict__ S, const float* __restrict__ B, int wr, int wc,
                                              GAcc (&acc)[NB][NB]) {
    constexpr int LD = gram_stride<NB>(), IL = DIAG ? JL : NB;
    const int lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
    const float* sp = S + kr * LD + 16 * wr + cc;
    const float* bp = B + kr * LD + 16 * wc + cc;
#pragma unroll 2
    for (int q0 = 0; q0 < kGramK; q0 += 4) {
        double a[IL], b[JL];
#pragma unroll
        for (int i = 0; i < IL; ++i) a[i] = (double)sp[q0 * LD + 32 * i];
#pragma unroll
        for (int j = 0; j < JL; ++j) b[j] = (double)bp[q0 * LD + 32 * j];
#pragma unroll
        for (int i = 0; i < IL; ++i)
#pragma unroll
            for (int j = DIAG ? i : 0; j < JL; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
}

// Pair idx of a class (GramGeometry): tile column tj, tile row ti.
__device__ __forceinline__ void pair_of(uint32_t cls, uint32_t idx, uint32_t nt, uint32_t& ti, uint32_t& tj) {
    ti = idx;
    tj = cls == kGramDiag ? idx : nt - 1;
    if (cls == kGramLastDiag) ti = tj;
    if (cls != kGramFull) return;
    uint32_t r = 0;
    while (idx >= nt - 2 - r) { idx -= nt - 2 - r; ++r; }
    ti = r;
    tj = r + 1 + idx;
}

// Item w of a launch's (split, pair) list.  The classes have different numbers of
// splits; their items are merged by where in the rows they start, (i + 1/2) / n of
// a class's n items, ties to the lower class.  Sixteen lanes try the items of a
// class around the expected one (gram_guess), each counting the items ahead of its
// own (gram_rank); the lane whose count is w knows its class and item (each w has
// one: merging is a bijection, and the expected item is at most three off).
__host__ __device__ __forceinline__ int64_t gram_guess(uint64_t own, uint64_t sum, uint32_t w) {
    return (int64_t)((2ull * w + 1ull) * own / (2ull * sum));
}
__host__ __device__ __forceinline__ uint64_t gram_rank(const uint64_t (&n)[kGramClasses], uint64_t own, uint32_t c, uint64_t j) {
    uint64_t rank = j;
#pragma unroll
    for (int k = 0; k < kGramClasses; ++k)
        if ((uint32_t)k != c && n[k] > 0) {
            const uint64_t at = (2ull * j + 1ull) * n[k];
            rank += (((uint32_t)k < c ? at : at - 1ull) / own + 1ull) / 2ull;
        }
    return rank;
}
__device__ __forceinline__ void gram_item(const GramGeometry& g, const GramPart& part, uint32_t w, uint32_t& cls,
                                          uint32_t& item) {
    const uint32_t lane = threadIdx.x & 63u, c = lane >> 4;
    uint64_t n[kGramClasses], sum = 0, own = 0;
#pragma unroll
    for (int k = 0; k < kGramClasses; ++k) {
        n[k] = (uint64_t)part.count[k] * g.nsplit[k];
        sum += n[k];
        if (c == (uint32_t)k) own = n[k];
    }
    const int64_t j = gram_guess(own, sum, w) + (int64_t)(lane & 15u) - 8;
    const bool in = j >= 0 && j < (int64_t)own;
    const uint64_t rank = in ? gram_rank(n, own, c, (uint64_t)j) : 0ull;
    const int who = __builtin_ctzll(__ballot(in && rank == w));
    cls = (uint32_t)who >> 4;
    item = (uint32_t)__builtin_amdgcn_readlane((int)j, who);
}

// The pairs of part over the rows of x.  CHUNK: these are rows row0, row0 + 1, ...
// of the N rows that the splits cut up, and a split that began before row0 goes on
// from its partial tile (else row0 = 0, N = x.N).  work holds, class after class, a
// tile per (split, pair of the part), split-major.  Blocks are dealt to the eight
// XCDs in turn; each XCD takes a contiguous eighth of the list, so the pairs of one
// range of rows mostly run on one XCD, whose L2 serves the rows they share.  Not so
// with CHUNK: the items with rows of the chunk are next to each other in the list,
// and go to all XCDs (as eighths of the list they ran on one or two of them: the
// first of those creations 252 -> 217 ms, the second 283 -> 211).
//
// QUARTER (with CHUNK): blocks of a 64-wide quarter of a 128-wide tile each, four
// times as many.  An entry's products are added in the same order, so G is the same
// bit for bit.  For chunks that lie in one or a few splits: whole tiles are then
// about npairs blocks, fewer than there are compute units (gram_chunk_launch).
template <int XT, int NB, bool ALIGNED, bool CHUNK, bool QUARTER = false>
__global__ __launch_bounds__(256, 2) void gram_tile_kernel(XLayout x, double* __restrict__ work, GramGeometry g,
                                                           GramPart part, uint32_t items, uint64_t row0, uint64_t N) {
    constexpr int T = 32 * NB, LD = gram_stride<NB>(), WT = QUARTER ? 2 * T : T;  // WT: width of work's tiles
    constexpr int VN = XT == 0 ? 4 : 8, TPR = T / VN, RPP = 256 / TPR, PASSES = kGramK / RPP;
    static_assert(RPP * PASSES == kGramK, "whole passes per stage");
    __shared__ __align__(16) float lds[2][2][kGramK * LD];
    constexpr uint32_t kParts = QUARTER ? 4u : 1u;
    const uint32_t per_xcd = (kParts * items + 7u) / 8u;
    const uint32_t b = CHUNK ? blockIdx.x : (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if (b >= kParts * items) return;
    const uint32_t w = b / kParts, qi = b % kParts >> 1, qj = b % kParts & 1u;
    uint32_t cls, item, ti, tj, count = 1, first = 0, rows_per_split = 0;
    gram_item(g, part, w, cls, item);
    size_t tile = item;
#pragma unroll
    for (uint32_t k = 0; k < kGramClasses; ++k) {
        if (k < cls) tile += (size_t)part.count[k] * g.nsplit[k];
        if (k == cls) {
            count = part.count[k];
            first = part.first[k];
            rows_per_split = g.rows[k];
        }
    }
    const uint32_t nt = g.nt, split = item / count;
    pair_of(cls, first + item % count, nt, ti, tj);
    size_t r_begin = (size_t)split * rows_per_split;
    size_t r_end = min((size_t)(CHUNK ? N : x.N), r_begin + rows_per_split);
    bool resume = false;
    if constexpr (CHUNK) {
        if (r_begin >= row0 + x.N || r_end <= row0) return;
        resume = r_begin < row0;
        r_begin = resume ? 0 : r_begin - row0;
        r_end = min((size_t)x.N, r_end - row0);
    }
    double* out = work + tile * (WT * WT) + (qi * WT + qj) * T;
    if constexpr (QUARTER) {
        ti = 2 * ti + qi;
        tj = 2 * tj + qj;
        if (ti > tj || tj * T >= x.p) return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave >> 1, wc = wave & 1;
    const bool diag = ti == tj;
    // 16-wide blocks of the two column tiles inside the matrix (tile ti is whole
    // unless the pair is diagonal)
    const int nI = (int)min(2u * NB, (x.p - ti * T + 15u) / 16u), nJ = (int)min(2u * NB, (x.p - tj * T + 15u) / 16u);
    GAcc acc[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = GAcc{0.0, 0.0, 0.0, 0.0};
    const int lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
    // block (2 i + wr, 2 j + wc) is inside the matrix and not below its diagonal
    auto held = [&](int i, int j) { return 2 * i + wr < nI && 2 * j + wc < nJ && (!diag || 2 * i + wr <= 2 * j + wc); };
    if (CHUNK && resume) {
        uint32_t at = kr * WT + cc;
        asm volatile("" : "+v"(at));  // the addresses are not kept for the stores at the end
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
                if (held(i, j)) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        acc[i][j][r] = out[(16 * (2 * i + wr) + 4 * r) * WT + 16 * (2 * j + wc) + at];
                }
    }
    // staging: thread t takes VN columns of stage rows t / TPR + RPP s
    const uint32_t c = threadIdx.x % TPR * VN, rb = threadIdx.x / TPR;
    uint4 va[PASSES], vb[PASSES];
    auto fetch = [&](size_t r0) {  // rows past the split's end: its last row again
#pragma unroll
        for (int s = 0; s < PASSES; ++s) {
            const size_t row = min(r0 + rb + RPP * s, r_end - 1);
            va[s] = gram_fetch<XT, VN, ALIGNED>(x, row, ti * T + c);
            if (!diag) vb[s] = gram_fetch<XT, VN, ALIGNED>(x, row, tj * T + c);
        }
    };
    auto widen = [&](const uint4& w, bool in, float* dst) {
        const uint32_t u[4] = {w.x, w.y, w.z, w.w};
        float v[VN];
#pragma unroll
        for (int e = 0; e < VN; ++e) {
            const uint32_t bits = XT == 0 ? u[e & 3] : (e & 1) ? u[(e >> 1) & 3] & 0xFFFF0000u : u[(e >> 1) & 3] << 16;
            v[e] = in ? __uint_as_float(bits) : 0.0f;
        }
#pragma unroll
        for (int e = 0; e < VN; e += 4) *reinterpret_cast<float4*>(dst + e) = make_float4(v[e], v[e + 1], v[e + 2], v[e + 3]);
    };
    auto put = [&](int buf, size_t r0) {
#pragma unroll
        for (int s = 0; s < PASSES; ++s) {
            const uint32_t row = rb + RPP * s;
            const bool in = r0 + row < r_end;
            widen(va[s], in, &lds[buf][0][row * LD + c]);
            if (!diag) widen(vb[s], in, &lds[buf][1][row * LD + c]);
        }
    };
    fetch(r_begin);
    put(0, r_begin);
    __syncthreads();
    auto rows = [&](auto jl, auto dg) {
        int buf = 0;
        for (size_t r0 = r_begin; r0 < r_end; r0 += kGramK, buf ^= 1) {
            const bool more = r0 + kGramK < r_end;
            if (more) fetch(r0 + kGramK);
            const float* S = lds[buf][0];
            gram_products<NB, decltype(jl)::value, decltype(dg)::value>(S, diag ? S : lds[buf][1], wr, wc, acc);
            if (more) put(buf ^ 1, r0 + kGramK);
            __syncthreads();
        }
    };
    auto columns = [&](auto dg) {  // the last tile column: only as wide as the matrix
        const int jl = (nJ + 1) / 2;
        if (jl == NB) rows(std::integral_constant<int, NB>{}, dg);
        else if (NB == 4 && jl == 3) rows(std::integral_constant<int, NB == 4 ? 3 : 1>{}, dg);
        else if (NB == 4 && jl == 2) rows(std::integral_constant<int, NB == 4 ? 2 : 1>{}, dg);
        else rows(std::integral_constant<int, 1>{}, dg);
    };
    if (diag) columns(std::true_type{});
    else columns(std::false_type{});
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
            if (held(i, j)) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    out[(16 * (2 * i + wr) + kr + 4 * r) * WT + 16 * (2 * j + wc) + cc] = acc[i][j][r];
            }
}

// G from the partial tiles of part, mirrored, and unscaled
// by 2^(e_i + e_j) (exact) if e.  A block takes 64 entries; wave w sums the
// splits of the w-th quarter in order, eight loads in flight, and the four sums
// are added in wave order: a fixed order, and four times the loads in flight of
// one thread per entry (N = 1e5, p = 100, 342 splits: 80 -> 8 us).  FEW (at most four
// splits of any pair, so that a quarter is one): 256 entries per block, one thread
// sums all of an entry's, which is the same sum (hsp_gram, N = 3, p = 2100: 107 -> 72 us).
template <bool FEW>
__global__ __launch_bounds__(256) void gram_reduce_kernel(const double* __restrict__ work, GramGeometry g, GramPart part,
                                                          uint32_t p, const int32_t* __restrict__ e,
                                                          double* __restrict__ G) {
    __shared__ double part_sum[4][64];
    const uint32_t T = g.tile, tt = T * T, lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    constexpr uint32_t E = FEW ? 256u : 64u;  // entries of a block; E divides T * T: they share a pair
    const size_t idx = blockIdx.x * (size_t)E + (FEW ? threadIdx.x : lane);
    uint32_t pc = (uint32_t)(blockIdx.x * (size_t)E / tt), cls = 0, count = 0, first = 0, nsplit = 1, ti, tj;
    const uint32_t local = (uint32_t)(idx % tt);
    size_t base = 0;
    bool found = false;
#pragma unroll
    for (uint32_t k = 0; k < kGramClasses; ++k) {
        if (found) continue;
        if (pc < part.count[k]) {
            found = true;
            cls = k;
            count = part.count[k];
            first = part.first[k];
            nsplit = g.nsplit[k];
        } else {
            pc -= part.count[k];
            base += (size_t)part.count[k] * g.nsplit[k];
        }
    }
    pair_of(cls, first + pc, g.nt, ti, tj);
    const uint32_t i = ti * T + local / T, j = tj * T + local % T;
    const bool live = i < p && j < p && !(ti == tj && j < i);
    const uint32_t per = (nsplit + 3u) / 4u, s0 = FEW ? 0u : min(wave * per, nsplit), s1 = FEW ? nsplit : min(s0 + per, nsplit);
    const double* src = work + (base + pc) * tt + local;
    const size_t step = (size_t)count * tt;
    double s = 0.0;
    if (live) {
#pragma unroll 8
        for (uint32_t sp = s0; sp < s1; ++sp) s += src[sp * step];
    }
    if constexpr (!FEW) {
        part_sum[wave][lane] = s;
        __syncthreads();
        if (wave != 0) return;
        s = ((part_sum[0][lane] + part_sum[1][lane]) + part_sum[2][lane]) + part_sum[3][lane];
    }
    if (!live) return;
    if (e) s = ldexp(s, e[i] + e[j]);
    G[(size_t)i * p + j] = s;
    G[(size_t)j * p + i] = s;
}

__global__ void philox_test_kernel(uint64_t seed, const uint32_t* ctr, uint32_t n, uint32_t* out) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const Words4 w = philox4x32_10(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3],
                                   (uint32_t)seed, (uint32_t)(seed >> 32));
    out[4 * i] = w.w0;
    out[4 * i + 1] = w.w1;
    out[4 * i + 2] = w.w2;
    out[4 * i + 3] = w.w3;
}

__global__ void pad_gram_kernel(const double* __restrict__ G, uint32_t p, uint32_t P,
                                double* __restrict__ Gp) {
    const size_t n = (size_t)P * P;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n;
         e += (size_t)gridDim.x * blockDim.x) {
        const uint32_t i = (uint32_t)(e / P), j = (uint32_t)(e % P);
        Gp[e] = (i < p && j < p) ? G[(size_t)i * p + j] : (i == j ? 1.0 : 0.0);
    }
}

}  // namespace

namespace {
bool gram_aligned(const XLayout& x) {
    return (size_t)x.ld * (x.xtype == 0 ? 4 : 2) % 16 == 0 && (uintptr_t)x.X % 16 == 0;
}
}  // namespace

// Tile width: 64 up to p = 128, where 128-wide tiles would be mostly padding, and
// for short designs, which are too few blocks of 128-wide tiles (us with 128- and
// 64-wide tiles, float32: N = 500, p = 130 31 / 22, p = 333 70 / 59, p = 2100 162 /
// 148; N = 2000, p = 130 68 / 58, p = 1000 135 / 115, but p = 2100 277 / 281;
// N = 3000, p = 1000 167 / 137, p = 700 99 / 100, p = 2100 359 / 370).  These take as
// many splits of up to 256 rows as 2 MB of partials hold, if that many: a larger
// workspace is not one that the runtime has at hand (about 30 us; N = 800, p = 130
// 54 -> 25 us, N = 500, p = 200 52 -> 25).
// Row splits: at least four 64-wide-tile blocks per compute unit in all.  With
// 128-wide tiles a class takes splits in proportion to the products of a row of
// its tiles (16 per wave for a whole tile, 10 on the diagonal, fewer in a narrow
// last tile column) plus a stage's loads and barrier, which cost about as much as
// 2 products (24 where rows of bfloat16 are off 16-byte boundaries and loaded one
// by one, 4 float32): the blocks on the device at one time then end together.
// Their number is the one with the shortest modelled time: the blocks of the
// busiest unit one after another (its FP64 matrix cores do 64 multiply-adds a
// cycle at 2.4 GHz; a block alone on its unit keeps them a little less busy) plus,
// per block, its 128 KB of partials written and read at 4 TB/s and allocated and
// freed (about 1.6 us per MB).  With as many splits for every pair, blocks of the
// diagonal and of a narrow last column left their units early: N = 1e6, p = 1000
// float32 18.3 ms, N = 3e5, p = 777 bfloat16 (9 columns in the last tile) 4.35 ms,
// N = 1e5, p = 129 float32 0.46 ms; now 16.9, 3.4 and 0.13 ms.
GramGeometry gram_geometry(const XLayout& x, int num_cus) {
    GramGeometry g{};
    const uint64_t nt64 = (x.p + 63) / 64, np64 = nt64 * (nt64 + 1) / 2;
    const uint64_t max_split = ((uint64_t)x.N + 63) / 64;
    const uint64_t lo = std::max<uint64_t>(1, std::min(max_split, ((uint64_t)num_cus * 4 + np64 - 1) / np64));
    g.tile = x.p <= 128u || x.N <= 1024u || (x.N <= 2048u && x.p <= 1024u) ? 64u : 128u;
    g.nt = (x.p + g.tile - 1) / g.tile;
    const uint32_t inner = g.nt - 1;
    g.npairs[kGramFull] = inner > 0 ? inner * (inner - 1) / 2 : 0u;
    g.npairs[kGramDiag] = g.npairs[kGramLast] = inner;
    g.npairs[kGramLastDiag] = 1;
    const uint32_t jl = (std::min(8u, (x.p - inner * g.tile + 15) / 16) + 1) / 2;
    const uint32_t stage = gram_aligned(x) ? 2 : x.xtype == 0 ? 4 : 24;
    const uint32_t cost[kGramClasses] = {16 + stage, 10 + stage, 4 * jl + stage, jl * (jl + 1) / 2 + stage};
    auto cut = [&](uint64_t n, GramGeometry* h) {  // n splits of a whole pair
        for (int c = 0; c < kGramClasses; ++c) {
            const uint64_t nc = g.tile == 64u ? n : (n * cost[c] + cost[0] - 1) / cost[0];
            const uint64_t rows = (((uint64_t)x.N + nc - 1) / nc + 63) / 64 * 64;
            h->rows[c] = (uint32_t)rows;
            h->nsplit[c] = (uint32_t)(((uint64_t)x.N + rows - 1) / rows);
        }
    };
    if (g.tile == 64u) {
        const uint64_t fit = ((2u << 20) - 1u) / (np64 * 64 * 64 * sizeof(double));
        cut(x.p > 128u && x.N <= 256u * fit ? std::min(lo, fit) : lo, &g);
        return g;
    }
    cut(lo, &g);
    // one pair's partials over every split fit the fixed workspace
    const uint64_t np = (uint64_t)g.nt * (g.nt + 1) / 2;
    const uint64_t hi = std::min({max_split, ((uint64_t)num_cus * 16 + np - 1) / np,
                                  (uint64_t)kGramScratchDoubles / (128 * 128)});
    GramGeometry best = g;
    double best_us = 1e300;
    for (uint64_t n = lo; n <= std::max(lo, hi); n += std::max<uint64_t>(1, n / 64)) {
        cut(n, &g);
        double rows = 0.0;
        uint64_t blocks = 0;
        for (int c = 0; c < kGramClasses; ++c) {
            if (g.npairs[c] > 0) rows = std::max(rows, g.rows[c] * cost[c] / 16.0);
            blocks += (uint64_t)g.npairs[c] * g.nsplit[c];
        }
        const uint64_t q = (blocks + num_cus - 1) / num_cus;
        const double us = ((double)q + (q & 1 ? 0.15 : 0.0)) * rows * (128.0 * 128 / (64 * 2400.0)) + (double)blocks * 0.265;
        if (us < best_us) {
            best_us = us;
            best = g;
        }
    }
    return best;
}

bool gram_item_host(const uint64_t (&n)[kGramClasses], uint32_t w, uint32_t* cls, uint64_t* item) {
    uint64_t sum = 0;
    for (uint64_t v : n) sum += v;
    int found = 0;
    for (uint32_t c = 0; c < kGramClasses; ++c)
        for (int64_t j = gram_guess(n[c], sum, w) - 8, e = j + 16; j < e; ++j)
            if (j >= 0 && j < (int64_t)n[c] && gram_rank(n, n[c], c, (uint64_t)j) == w) {
                *cls = c;
                *item = (uint64_t)j;
                ++found;
            }
    return found == 1;
}

size_t gram_work_doubles(const GramGeometry& g) {
    size_t tiles = 0;
    for (int c = 0; c < kGramClasses; ++c) tiles += (size_t)g.npairs[c] * g.nsplit[c];
    return tiles * g.tile * g.tile;
}

namespace {

template <int XT, int NB>
void gram_tiles(const XLayout& x, double* work, const GramGeometry& g, const GramPart& part, uint64_t row0, uint64_t N,
                hipStream_t st) {
    const bool aligned = gram_aligned(x);
    uint32_t items = 0;
    for (int c = 0; c < kGramClasses; ++c) items += part.count[c] * g.nsplit[c];
    const dim3 grid((items + 7u) / 8u * 8u);
    auto f = x.N < N ? &gram_tile_kernel<XT, NB, true, true> : aligned ? &gram_tile_kernel<XT, NB, true, false>
                                                                       : &gram_tile_kernel<XT, NB, false, false>;
    hipLaunchKernelGGL(f, grid, dim3(256), 0, st, x, work, g, part, items, row0, N);
}

// The partial tiles of part over x, rows row0 ... of N.
void gram_tiles_launch(const XLayout& x, double* work, const GramGeometry& g, const GramPart& part, uint64_t row0,
                       uint64_t N, hipStream_t st) {
    if (x.xtype == 0 && g.tile == 64) gram_tiles<0, 2>(x, work, g, part, row0, N, st);
    else if (x.xtype == 0) gram_tiles<0, 4>(x, work, g, part, row0, N, st);
    else if (g.tile == 64) gram_tiles<1, 2>(x, work, g, part, row0, N, st);
    else gram_tiles<1, 4>(x, work, g, part, row0, N, st);
}

hipError_t gram_sum_launch(const double* work, const GramGeometry& g, const GramPart& part, uint32_t p,
                           const int32_t* e, double* G, hipStream_t st) {
    size_t pairs = 0;
    for (int c = 0; c < kGramClasses; ++c) pairs += part.count[c];
    const bool few = *std::max_element(g.nsplit, g.nsplit + kGramClasses) <= 4;
    hipLaunchKernelGGL(few ? &gram_reduce_kernel<true> : &gram_reduce_kernel<false>,
                       dim3((unsigned)(pairs * g.tile * g.tile / (few ? 256 : 64))), dim3(256), 0, st, work, g, part, p, e, G);
    return hipGetLastError();
}

GramPart whole(const GramGeometry& g) {
    GramPart part{};
    for (int c = 0; c < kGramClasses; ++c) part.count[c] = g.npairs[c];
    return part;
}

}  // namespace

hipError_t gram_launch(const XLayout& x, const GramGeometry& g, const int32_t* e, double* G, double* work,
                       size_t work_doubles, hipStream_t st) {
    // (the sum launches 4 threads per entry of a tile, and a launch takes fewer than
    // 2^32: 65535 pairs of 128-wide tiles, which G has from p = 46209 on)
    const size_t most = std::min<size_t>(work_doubles / ((size_t)g.tile * g.tile), 65535);
    GramPart part{};
    while (true) {
        size_t room = most, taken = 0;
        bool left = false;
        for (int c = 0; c < kGramClasses; ++c) {
            part.first[c] += part.count[c];
            part.count[c] = (uint32_t)std::min<size_t>(g.npairs[c] - part.first[c], room / g.nsplit[c]);
            room -= (size_t)part.count[c] * g.nsplit[c];
            taken += part.count[c];
            left |= part.first[c] < g.npairs[c];
        }
        if (!left) return hipSuccess;
        if (taken == 0) return hipErrorInvalidValue;
        gram_tiles_launch(x, work, g, part, 0, x.N, st);
        if (hipError_t err = gram_sum_launch(work, g, part, x.p, e, G, st)) return err;
    }
}

// A fixed device workspace for callers that cannot allocate: gram_scratch()
// returns its device address on the current device (found once per device
// with hipGetSymbolAddress; the array's name is not a device address in host
// code).  Every call on one device shares it.
namespace {
__device__ __align__(256) double scratch[kGramScratchDoubles];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t gram_scratch(double** ptr) {
    *ptr = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = static_cast<double*>(p);
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

size_t gram_pair_doubles(const GramGeometry& g) {
    uint32_t ns = 0;
    for (int c = 0; c < kGramClasses; ++c)
        if (g.npairs[c] > 0) ns = std::max(ns, g.nsplit[c]);
    return (size_t)ns * g.tile * g.tile;
}

hipError_t gram_chunk_launch(const XLayout& chunk, const GramGeometry& g, uint64_t row0, uint64_t N, int num_cus,
                             double* work, hipStream_t st) {
    if (chunk.N == 0) return hipSuccess;
    if (row0 % 64 != 0 || row0 + chunk.N > N || !gram_aligned(chunk)) return hipErrorInvalidValue;
    // Blocks with rows of this chunk.  Up to one per compute unit, quarters of tiles:
    // creation from N = 4e5, p = 1000 float32 in chunks of 4096 rows (36 pairs) 217
    // -> 189 ms, from N = 2e5, p = 2000 in chunks of 2048 (136 pairs) 211 -> 191;
    // with more, whole tiles read X fewer times.
    uint64_t live = 0, items = 0;
    for (int c = 0; c < kGramClasses; ++c) {
        live += g.npairs[c] * ((row0 + chunk.N - 1) / g.rows[c] - row0 / g.rows[c] + 1);
        items += (uint64_t)g.npairs[c] * g.nsplit[c];
    }
    if (g.tile == 128 && chunk.N < N && live <= (uint64_t)num_cus) {
        const dim3 grid((unsigned)((4 * items + 7) / 8 * 8));
        auto f = chunk.xtype == 0 ? &gram_tile_kernel<0, 2, true, true, true> : &gram_tile_kernel<1, 2, true, true, true>;
        hipLaunchKernelGGL(f, grid, dim3(256), 0, st, chunk, work, g, whole(g), (uint32_t)items, row0, N);
    } else {
        gram_tiles_launch(chunk, work, g, whole(g), row0, N, st);
    }
    return hipGetLastError();
}

hipError_t gram_reduce_launch(const double* work, const GramGeometry& g, uint32_t p, const int32_t* e, double* G,
                              hipStream_t st) {
    return gram_sum_launch(work, g, whole(g), p, e, G, st);
}

hipError_t pad_gram_launch(const double* G, uint32_t p, uint32_t P, double* Gp, hipStream_t st) {
    hipLaunchKernelGGL(pad_gram_kernel, dim3(1024), dim3(256), 0, st, G, p, P, Gp);
    return hipGetLastError();
}

// key[i] = (2 y_i - 1) sum_j x_ij beta32_j: one wave per row (lanes over
// columns, a wave-wide sum), float32, over the stored column-scaled X.
__global__ __launch_bounds__(256) void row_key_kernel(XLayout x, const float* __restrict__ b32,
                                                      const uint8_t* __restrict__ y, float* __restrict__ key) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t waves = gridDim.x * (blockDim.x / 64u);
    for (uint32_t i = blockIdx.x * (blockDim.x / 64u) + threadIdx.x / 64u; i < x.N; i += waves) {
        float acc = 0.0f;
        for (uint32_t j = lane; j < x.p; j += 64u) acc = fmaf(load_x(x, i, j), b32[j], acc);
        for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
        if (lane == 0) key[i] = y[i] ? acc : -acc;
    }
}

// Row i of Xo is row perm[i] of X (16-byte vectors; a row is ld elements,
// a multiple of 16 bytes), with y and the original row indices alongside.
__global__ __launch_bounds__(256) void gather_rows_kernel(XLayout x, const uint32_t* __restrict__ perm,
                                                          uint4* __restrict__ Xo, const uint8_t* __restrict__ y,
                                                          uint8_t* __restrict__ yo, const uint32_t* __restrict__ id,
                                                          uint32_t* __restrict__ ido) {
    const size_t vpr = (size_t)x.ld * (x.xtype == 0 ? 4 : 2) / 16;  // 16-byte vectors per row
    const uint4* X = static_cast<const uint4*>(x.X);
    for (uint32_t i = blockIdx.x; i < x.N; i += gridDim.x) {
        const uint32_t src = perm[i];
        for (size_t v = threadIdx.x; v < vpr; v += blockDim.x) Xo[(size_t)i * vpr + v] = X[(size_t)src * vpr + v];
        if (threadIdx.x == 0) {
            yo[i] = y[src];
            ido[i] = id ? id[src] : src;
        }
    }
}

__global__ __launch_bounds__(256) void fetch_draws_kernel(const Ctrl* __restrict__ ctrl, const double* __restrict__ rb,
                                                          const double* __restrict__ rt, const double* __restrict__ rl,
                                                          uint32_t p, uint32_t first, uint32_t cap, uint32_t count,
                                                          double* __restrict__ out) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x, nb = rb ? count * p : 0u, nt = rt ? count : 0u;
    if (i == 0) {
        out[0] = (double)ctrl->err;
        out[1] = (double)ctrl->chol_info;
        out[2] = (double)ctrl->sweep;
    }
    if (i >= nb + nt + (rl ? count * p : 0u)) return;
    const bool tau = i >= nb && i < nb + nt;
    const uint32_t e = i < nb ? i : tau ? (i - nb) * p : i - nb - nt;  // draw e / p, coordinate e % p
    const size_t slot = (first + e / p) % cap;
    out[kFetchHead + i] = tau ? rt[slot] : (i < nb ? rb : rl)[slot * p + e % p];
}

// Read ceiling: stream `bytes` (a multiple of 16) with eight 16-byte
// non-temporal loads in flight per lane, grid-stride, the same kind of load
// as the z pass, and nothing else.
typedef unsigned int RdVec __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void stream_read_kernel(const RdVec* __restrict__ x, size_t n16,
                                                          float* __restrict__ sink) {
    constexpr int kUnroll = 8;
    float s = 0.0f;
    size_t i = (size_t)blockIdx.x * 256 * kUnroll + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * 256 * kUnroll;
    for (; i + 256 * (kUnroll - 1) < n16; i += stride) {
        RdVec v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) v[u] = __builtin_nontemporal_load(x + i + 256 * u);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) s += __uint_as_float(v[u].x ^ v[u].y ^ v[u].z ^ v[u].w);
    }
    for (; i < n16; i += 256) {  // the ragged end, one load at a time
        const RdVec v = __builtin_nontemporal_load(x + i);
        s += __uint_as_float(v.x ^ v.y ^ v.z ^ v.w);
    }
    if (s == -1.0f) sink[0] = s;  // never true for the sums of finite data; keeps the loads
}

hipError_t fetch_draws_launch(const Ctrl* ctrl, const double* ring_beta, const double* ring_tau, const double* ring_lam,
                              uint32_t p, uint32_t first, uint32_t capacity, uint32_t count, double* out,
                              hipStream_t st) {
    const uint32_t n = (ring_beta ? count * p : 0u) + (ring_tau ? count : 0u) + (ring_lam ? count * p : 0u);
    hipLaunchKernelGGL(fetch_draws_kernel, dim3(n / 256 + 1), dim3(256), 0, st, ctrl, ring_beta, ring_tau, ring_lam, p,
                       first, capacity, count, out);
    return hipGetLastError();
}

hipError_t stream_read_launch(const void* x, size_t bytes, int num_cus, float* sink, hipStream_t st) {
    const size_t n16 = bytes / 16;
    const unsigned blocks = (unsigned)(2 * num_cus);
    hipLaunchKernelGGL(stream_read_kernel, dim3(blocks), dim3(256), 0, st,
                       static_cast<const RdVec*>(x), n16, sink);
    return hipGetLastError();
}

hipError_t row_key_launch(const XLayout& x, const float* beta32, const uint8_t* y, float* key, hipStream_t st) {
    hipLaunchKernelGGL(row_key_kernel, dim3(4096), dim3(256), 0, st, x, beta32, y, key);
    return hipGetLastError();
}

hipError_t gather_rows_launch(const XLayout& x, const uint32_t* perm, void* Xo, const uint8_t* y, uint8_t* yo,
                              const uint32_t* id, uint32_t* ido, hipStream_t st) {
    hipLaunchKernelGGL(gather_rows_kernel, dim3(8192), dim3(256), 0, st, x, perm, static_cast<uint4*>(Xo), y, yo,
                       id, ido);
    return hipGetLastError();
}

hipError_t philox_test_launch(uint64_t seed, const uint32_t* ctr, uint32_t n, uint32_t* out,
                              hipStream_t st) {
    hipLaunchKernelGGL(philox_test_kernel, dim3((n + 255) / 256), dim3(256), 0, st, seed, ctr, n, out);
    return hipGetLastError();
}

hipError_t colmax_launch(const float* src, uint32_t N, uint32_t p, uint32_t* colmax_bits, hipStream_t st) {
    const dim3 grid((N + kColmaxRows - 1) / kColmaxRows, (p + 255) / 256);
    hipLaunchKernelGGL(colmax_kernel, grid, dim3(256), 0, st, src, N, p, colmax_bits);
    return hipGetLastError();
}

hipError_t pack_x_launch(const float* src, const XLayout& dst, const int32_t* e, hipStream_t st) {
    hipLaunchKernelGGL(pack_kernel, dim3(4096), dim3(256), 0, st, src, dst, e);
    return hipGetLastError();
}

hipError_t validate_launch(const XLayout& x, const uint8_t* y, Ctrl* ctrl, hipStream_t st) {
    hipLaunchKernelGGL(validate_kernel, dim3(4096), dim3(256), 0, st, x, y, ctrl);
    return hipGetLastError();
}

}  // namespace hsp
