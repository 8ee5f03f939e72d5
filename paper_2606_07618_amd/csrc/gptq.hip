// GPTQ with fixed NVFP4 block scales on AMD Instinct MI355X (gfx950), in its LDLQ form
// (implementation details, GPTQ paragraph): the block scales are chosen before the pass (by
// any of the quantizers), the input channels are visited in descending order of the Hessian
// diagonal, the Hessian is damped by 0.01 x its mean diagonal, and
//   x_a = w_a + sum_{b < a} (w_b - w^_b) U_ba,     w^_a = Q(x_a)
// with Hp = (U + I) D (U + I)^T the factorization of the damped, reordered Hessian (U strictly
// upper triangular).  LDLQ and GPTQ give the same result.  Everything is binary64 with a
// fixed order of correctly rounded operations per value:
//   * factor: Hp is factored in place (column-major) in 64-column blocks from the last: the
//     block's own columns right-looking from its last column (rows in registers, each
//     column's updates to the block's remaining triangle in parallel); then the rows above
//     it, each a 64-column triangular solve, also right-looking; then the block's
//     contribution (U_ik U_jk) D_k, k walked downwards, is subtracted from the rest of the
//     upper triangle in tiles, first the column of tiles the next block needs, then the rest
//     beside the next block's own factor (look-ahead).  So each element receives its terms
//     k = n-1, ..., j+1 in that order.
//   * quantize: columns are taken in tiles of 64, the values kept by columns.  A launch takes one
//     tile: each row's lanes add the terms of the tile or two before it, then walk the columns:
//     column b's value is quantized and its error times U added to the tile's later columns, b =
//     a0, a0 + 1, ... in order.  Beside it the same launch adds earlier tiles' errors times U to the
//     columns past the tile, term by term in tile order (look-ahead).  Every x_a therefore
//     receives its terms b = 0, 1, ... in ascending order, as the sequential definition adds them.
//   The sequential kernels (diagonal block, panel, tile) hold no branch per step: the columns
//   are interleaved over a row's lanes, so a step's updates need at most one select, and its
//   operands that do not depend on the running values are formed ahead of the dependent chain.
// Q(x) is the quantizers' rounding: y = RN32(RN32(x) / S), nibble sign(y) << 3 | RNE_FP4(|y| /
// s), w^ = +-E2M1 * s * S (exact in binary64).
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include <utility>

#include "exact_fp.h"
#include "nvfp4ss.h"

namespace {

using namespace nvfp4_exact;

constexpr int kTile = 64;

template <typename In>
__device__ __forceinline__ float load_w(const In* w, int64_t i);

template <>
__device__ __forceinline__ float load_w<float>(const float* w, int64_t i) { return w[i]; }

template <>
__device__ __forceinline__ float load_w<uint16_t>(const uint16_t* w, int64_t i) {
    return __uint_as_float((uint32_t)w[i] << 16);
}

// f(integral_constant<int, B>) for B = 0, 1, ... in order (the calls unrolled at compile time).
template <typename F, int... B>
__device__ __forceinline__ void for_each_index(F&& f, std::integer_sequence<int, B...>) {
    (f(std::integral_constant<int, B>()), ...);
}

// Lane l of each 16-lane row broadcasts v to the row's lanes (DPP row_newbcast).
template <int L>
__device__ __forceinline__ double row_bcast(double v) {
    constexpr int ctrl = 0x150 + L;
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, ctrl, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), ctrl, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Four consecutive values (16-byte aligned).
__device__ __forceinline__ void read_row(double (&t)[4], const double* p) {
    const double2 a = reinterpret_cast<const double2*>(p)[0], b = reinterpret_cast<const double2*>(p)[1];
    t[0] = a.x;
    t[1] = a.y;
    t[2] = b.x;
    t[3] = b.y;
}

// ---- column order and damping ------------------------------------------------------------

__global__ __launch_bounds__(256) void diag_kernel(const double* __restrict__ H, int64_t n,
                                                   double* __restrict__ diag) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) diag[i] = H[i * n + i];
}

// perm[rank(i)] = i, inv[i] = rank(i), rank = number of columns with a larger diagonal, or an equal one
// and a smaller index (a stable descending order).  A NaN counts as -infinity: it would compare false with
// every value and share a rank, and a rank that no column has leaves perm unwritten there, an index out of
// range.  (The sum keeps it, so the factor reports it.)  64 columns i per workgroup; each of its 16 waves
// counts over a sixteenth of every 1024-value chunk of the diagonal staged in LDS (one value per
// step, read by the wave's lanes alike), and the sixteen counts are added.
// Beside them, the last workgroup: lambda = damp * (sum of the diagonal in index order) / n, one lane
// adding the staged chunks.  At n = 4096 the two take 25 us side by side.
constexpr int kOrderParts = 16;
__global__ __launch_bounds__(64 * kOrderParts) void order_kernel(const double* __restrict__ diag, int64_t n,
                                                                 int* __restrict__ perm, int* __restrict__ inv,
                                                                 double damp, double* __restrict__ lambda) {
    constexpr int kChunk = 1024, kPer = kChunk / kOrderParts;
    __shared__ double chunk[kChunk];
    __shared__ int part_rank[kOrderParts][64];
    const bool sum = blockIdx.x == gridDim.x - 1;
    const int il = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + il;
    auto order_key = [](double v) { return v == v ? v : -(double)INFINITY; };
    const double d = i < n ? order_key(diag[i]) : 0.0;
    int rank = 0;
    double tr = 0.0;
    for (int64_t c0 = 0; c0 < n; c0 += kChunk) {
        __syncthreads();                                          // the previous chunk is used
        const double v = c0 + threadIdx.x < n ? diag[c0 + threadIdx.x] : 0.0;
        chunk[threadIdx.x] = sum ? v : order_key(v);
        __syncthreads();
        if (sum) {
            if (threadIdx.x == 0) {
                const int m = (int)(n - c0 < kChunk ? n - c0 : kChunk);
#pragma unroll 16
                for (int k = 0; k < m; ++k) tr += chunk[k];
            }
            continue;
        }
        const int64_t jb = c0 + part * kPer;
        const int m = (int)(n - jb < kPer ? (n - jb > 0 ? n - jb : 0) : kPer);
#pragma unroll 8
        for (int jj = 0; jj < m; ++jj) {
            const double e = chunk[part * kPer + jj];
            rank += (e > d || (e == d && jb + jj < i)) ? 1 : 0;
        }
    }
    if (sum) {
        if (threadIdx.x == 0) lambda[0] = damp * (tr / (double)n);
        return;
    }
    part_rank[part][il] = rank;
    __syncthreads();
    if (part == 0 && i < n) {
        int r = 0;
        for (int k = 0; k < kOrderParts; ++k) r += part_rank[k][il];
        perm[r] = (int)i;
        inv[i] = r;
    }
}

// ---- factor: blocked, from the last 64-column block backwards ---------------------------
// Uc holds A = Hp column-major (Uc[j n + i] = A_ij for i <= j) and is overwritten in place by U.
// Below the diagonal blocks it receives U by rows as well (Uc[i n + j] = U_ij for j > i in a later
// block: factor_panel_kernel writes it, the quantization reads it); inside them the lower triangle
// is never written, and the values read from it feed only results that are discarded.  Element
// (i, j) must receive its terms k = n-1, n-2, ..., j+1 in that order; the blocks are finished
// last-first and every kernel walks k downwards, so it does.

// The damped, reordered Hessian, its upper triangle only (only that is read as A), 64 x 64 values per
// workgroup through LDS: read along the rows of H (64 values scattered over one row of 8 n bytes),
// written along the columns of Uc.  An XCD (workgroup index mod 8) takes the tiles of one row block
// after another, so that the block's 64 rows of H come from memory once and then from its L2:
// [4096, 4096] 157 -> 73 us (each value's line of H was fetched for it alone).
__global__ __launch_bounds__(256) void init_a_kernel(const double* __restrict__ H,
                                                     const int* __restrict__ perm,
                                                     const double* __restrict__ lambda, int64_t n,
                                                     double* __restrict__ Uc) {
    __shared__ double v[kTile][kTile + 1];
    __shared__ int pr[kTile];
    const int64_t tiles = n / kTile, seq = blockIdx.x / 8;
    const int64_t ti = seq / tiles * 8 + blockIdx.x % 8, tj = seq % tiles;
    if (ti > tj) return;                               // also past the last row block: tj < tiles
    const int64_t i0 = ti * kTile, j0 = tj * kTile;
    const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
    if (part == 0) pr[lane] = perm[i0 + lane];
    const int pc = perm[j0 + lane];
    __syncthreads();
#pragma unroll 8
    for (int a = part; a < kTile; a += 4) v[a][lane] = H[(int64_t)pr[a] * n + pc];
    __syncthreads();
    const int64_t i = i0 + lane;
    for (int b = part; b < kTile; b += 4) {
        const int64_t j = j0 + b;
        double x = v[lane][b];
        if (i == j) x = x + lambda[0];
        if (i <= j) Uc[j * n + i] = x;
    }
}

// The diagonal block [k0, k0 + 64): its D and its U, column by column from the last.  The
// block's own 64 columns, right-looking: at step kk (from the last) D_kk is the updated
// diagonal, U_i,kk = A_i,kk / D_kk for i < kk, and every A_ij (i <= j < kk) then loses
// (U_ik U_jk) D_k, so each element receives its terms k = 63, 62, ... in the order the
// column-by-column definition sums them.  A quad of threads per row, thread q holding the
// row's values of columns 4m + q in registers; column kk of U goes through LDS.  One barrier
// per step: after its updates every thread forms D_(kk-1) itself from the value its owner
// published before the step (the owner's own update, the same operations), so the threads
// holding column kk - 1 can divide at once and publish that column for the next step.
struct alignas(16) DiagLds {
    double col[2][kTile];          // col[kk & 1][16 (i & 3) + (i >> 2)] = U_{k0+i, k0+kk}
    double pre[2];                 // pre[kk & 1]: A_(kk-1),(kk-1) before step kk
    double Db[kTile];
};

__device__ __forceinline__ int quad_slot(int j) { return 16 * (j & 3) + (j >> 2); }

__device__ __forceinline__ void factor_diag_body(double* __restrict__ Uc, double* __restrict__ D,
                                                 int64_t n, int64_t k0, int* __restrict__ status,
                                                 DiagLds& L) {
    const int tid = threadIdx.x;
    const int i = tid >> 2, q = tid & 3;
    double v[16];                            // A (then U) of (k0 + i, k0 + 4m + q)
#pragma unroll
    for (int m = 0; m < 16; ++m) v[m] = Uc[(k0 + 4 * m + q) * n + k0 + i];
    // the column buffers start at zero: a step reads slots of rows it does not update (their
    // results are discarded by the selects)
    if (tid < 2 * kTile) L.col[tid / kTile][tid % kTile] = 0.0;
    // column 63: its diagonal, then its U, and A_62,62 for step 63
    if (i == kTile - 1 && q == 3) L.Db[kTile - 1] = v[15];
    __syncthreads();
    {
        const double d = L.Db[kTile - 1];
        const double u = v[15] / d;
        if (q == 3 && i < kTile - 1) {
            v[15] = u;
            L.col[1][quad_slot(i)] = u;
        }
        if (i == kTile - 2 && q == 2) L.pre[1] = v[15];
    }
    __syncthreads();
    auto step = [&](auto kc) {
        constexpr int kk = kTile - 1 - decltype(kc)::value, par = kk & 1;
        const double d = L.Db[kk];
        const double* c = &L.col[par][0];
        const double ui = c[quad_slot(i)];
        const double* cq = c + 16 * q;
        // the updates of this step: A_ij, i <= j = 4m + q < kk, in two halves of eight columns
        // (U values read together first).  Values left of the diagonal (j < i) are updated too:
        // they feed nothing (no diagonal, division, published value or store reads them), so
        // only the column bound j < kk needs a select, in one register per step.
#pragma unroll
        for (int h = 0; h < 16; h += 8) {
            double uj[8];
#pragma unroll
            for (int m = 0; m < 8; ++m) uj[m] = 4 * (h + m) < kk ? cq[h + m] : 0.0;
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const int mm = h + m;
                if (4 * mm < kk) {
                    double nv = v[mm] - (ui * uj[m]) * d;
                    asm volatile("" : "+v"(nv));     // formed in every lane, then selected (no
                                                     // branch around the update and its reads)
                    v[mm] = (4 * mm + 3 < kk || q < kk - 4 * mm) ? nv : v[mm];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (kk >= 1) {
            constexpr int k1 = kk - 1, q1 = k1 & 3, m1 = k1 >> 2;
            // D_(kk-1): its owner's update of this step, formed by every thread alike
            const double u1 = c[quad_slot(k1)];
            const double d1 = L.pre[par] - (u1 * u1) * d;
            const double u = v[m1] / d1;
            if (q == q1 && i < k1) {
                v[m1] = u;
                L.col[par ^ 1][quad_slot(i)] = u;
            }
            if (tid == 0) L.Db[k1] = d1;
            if constexpr (kk >= 2) {
                constexpr int k2 = kk - 2, q2 = k2 & 3, m2 = k2 >> 2;
                if (i == k2 && q == q2) L.pre[par ^ 1] = v[m2];
            }
            __syncthreads();
        }
    };
    for_each_index(step, std::make_integer_sequence<int, kTile>());
#pragma unroll
    for (int m = 0; m < 16; ++m) {
        const int j = 4 * m + q;
        if (i < j) Uc[(k0 + j) * n + k0 + i] = v[m];
    }
    if (tid < kTile) {
        const double d = L.Db[tid];
        D[k0 + tid] = d;
        if (!(d > 0.0) || !isfinite(d)) status[0] = 1;           // not positive definite
    }
}

__global__ __launch_bounds__(4 * kTile) void factor_diag_kernel(double* __restrict__ Uc, double* __restrict__ D,
                                                                int64_t n, int64_t k0, int* __restrict__ status) {
    __shared__ DiagLds L;
    factor_diag_body(Uc, D, n, k0, status, L);
}

// Rows above the block (i < k0), 16 per workgroup, a 16-lane row of lanes per matrix row: lane
// q holds the row's values of block columns 16m + q (m = 0..3) in registers.  Each row is a
// triangular solve from the block's last column, right-looking: at step kk the row's value of
// column kk is final, U_i,kk = A_i,kk / D_kk (broadcast in the lane row), and each of the
// row's columns j < kk loses (U_i,kk U_j,kk) D_kk.  So each value receives its terms kk = 63,
// 62, ... in the order the column-by-column definition sums them.  A step holds no branch and
// at most four updates per lane; the block's U and D are staged in LDS (each lane's columns of
// a U row contiguous) and read a step ahead: 13.2 -> 12.6 us a launch.
constexpr int kPanelRows = 16;
__device__ __forceinline__ int row16_slot(int j) { return 4 * (j & 15) + (j >> 4); }

__global__ __launch_bounds__(256) void factor_panel_kernel(double* __restrict__ Uc,
                                                           const double* __restrict__ D, int64_t n,
                                                           int64_t k0) {
    __shared__ double Ub[kTile][kTile];       // Ub[kk][4 q + m] = U_{k0+16m+q, k0+kk}
    __shared__ double Db[kTile];
    const int tid = threadIdx.x;
    const int64_t i0 = (int64_t)blockIdx.x * kPanelRows;
    for (int t = tid; t < kTile * kTile; t += 256) {
        const int kk = t / kTile, jj = t % kTile;                 // coalesced over jj
        Ub[kk][row16_slot(jj)] = Uc[(k0 + kk) * n + k0 + jj];
    }
    if (tid < kTile) Db[tid] = D[k0 + tid];
    const int rr = tid >> 4, q = tid & 15;
    const int64_t i = i0 + rr;
    double v[4], uf[4];                      // uf: the lane's columns of U
    if (i < k0) {
#pragma unroll
        for (int m = 0; m < 4; ++m) v[m] = Uc[(k0 + 16 * m + q) * n + i];
    }
    __syncthreads();
    if (i >= k0) return;                     // whole lane rows; rows share nothing
    const double* Up = &Ub[0][4 * q];
    double dc = Db[kTile - 1], tc[4];
    read_row(tc, Up + (kTile - 1) * kTile);
    auto step = [&](auto kc) {
        constexpr int kk = kTile - 1 - decltype(kc)::value, qk = kk & 15, mk = kk >> 4;
        // the next step's row of U and D, read a step ahead
        constexpr int kn = kk >= 1 ? kk - 1 : 0;
        const double dk = dc;
        double tn[4];
        read_row(tn, Up + kn * kTile);
        dc = Db[kn];
        __builtin_amdgcn_sched_barrier(0);
        const double u = row_bcast<qk>(v[mk]) / dk;
        Uc[(k0 + kk) * n + i] = u;           // the row's lanes store the same value
        if (q == qk) uf[mk] = u;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            if (16 * m < kk) {               // some lane of the row holds a column before kk
                const double nv = v[m] - (u * tc[m]) * dk;
                v[m] = (16 * m + 15 < kk || q < kk - 16 * m) ? nv : v[m];
            }
            tc[m] = tn[m];
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    for_each_index(step, std::make_integer_sequence<int, kTile>());
    // the row's U once more by rows, in the lower triangle (nothing of A is there): the
    // quantization reads U_{i,k} over consecutive k
#pragma unroll
    for (int m = 0; m < 4; ++m) Uc[i * n + k0 + 16 * m + q] = uf[m];
}

// A_ij -= sum over the block's k, downwards, of (U_ik U_jk) D_k for i <= j < k0: one
// 16R x 16R tile of the upper triangle (rows i0.., columns j0..) per workgroup (tiles wholly
// below it exit), R x R values per lane; the block's 64 k in two halves of 32 (the upper
// first), so that four workgroups of the 64 x 64 tiles fit a CU's LDS: four waves per SIMD to
// issue the binary64 chains.  The 32 x 32 tiles (R = 2) serve the column of tiles the next
// block needs, which is on the critical path: four times the workgroups, a quarter of the
// chain per lane.
constexpr int kHalf = kTile / 2;
template <int R>
struct alignas(16) FTrailLdsT {
    double Ui[kHalf][16 * R + 2];  // Ui[kk][ii] = U_{i0+ii, k0+h+kk} (rows padded: 16-byte rows)
    double Uj[kHalf][16 * R + 2];
    double Dk[kTile];
};
using FTrailLds = FTrailLdsT<4>;

// Lane (tr, tc) owns rows i0 + R tr .. + R - 1 and columns j0 + R tc .. + R - 1, so that its
// values of a column and its operands of a step sit in 16-byte pairs.
template <int R>
__device__ __forceinline__ void factor_trailing_body(double* __restrict__ Uc, const double* __restrict__ D,
                                                     int64_t n, int64_t k0, int64_t i0, int64_t j0,
                                                     FTrailLdsT<R>& L) {
    static_assert(R % 2 == 0, "pairs of values");
    constexpr int B = 16 * R;
    if (i0 > j0 + B - 1) return;
    if (threadIdx.x < kTile) L.Dk[threadIdx.x] = D[k0 + threadIdx.x];
    const int tr = threadIdx.x / 16, tc = threadIdx.x % 16;
    const int64_t ir = i0 + R * tr, jc = j0 + R * tc;
    double acc[R][R];                        // acc[a][b]: (ir + a, jc + b)
#pragma unroll
    for (int b = 0; b < R; ++b) {
        const double2* src = reinterpret_cast<const double2*>(Uc + (jc + b) * n + ir);
#pragma unroll
        for (int a = 0; a < R; a += 2) {
            const double2 v = src[a / 2];
            acc[a][b] = v.x;
            acc[a + 1][b] = v.y;
        }
    }
    // each half's operands are loaded into registers while the previous half is computed
    constexpr int kPer = B * kHalf / 256;
    double pi[kPer], pj[kPer];
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
        const int t = threadIdx.x + 256 * e, kk = t / B, r = t % B;      // coalesced over r
        pi[e] = Uc[(k0 + kHalf + kk) * n + i0 + r];
        pj[e] = Uc[(k0 + kHalf + kk) * n + j0 + r];
    }
    for (int h = kHalf; h >= 0; h -= kHalf) {
        __syncthreads();                                          // the previous half is used
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const int t = threadIdx.x + 256 * e, kk = t / B, r = t % B;
            L.Ui[kk][r] = pi[e];
            L.Uj[kk][r] = pj[e];
        }
        __syncthreads();
        if (h > 0) {
#pragma unroll
            for (int e = 0; e < kPer; ++e) {
                const int t = threadIdx.x + 256 * e, kk = t / B, r = t % B;
                pi[e] = Uc[(k0 + kk) * n + i0 + r];
                pj[e] = Uc[(k0 + kk) * n + j0 + r];
            }
        }
#pragma unroll(R == 2 ? 4 : 2)
        for (int kk = kHalf - 1; kk >= 0; --kk) {
            double ua[R], ub[R];
            const double2* ap = reinterpret_cast<const double2*>(&L.Ui[kk][R * tr]);
            const double2* bp = reinterpret_cast<const double2*>(&L.Uj[kk][R * tc]);
#pragma unroll
            for (int a = 0; a < R; a += 2) {
                const double2 av = ap[a / 2], bv = bp[a / 2];
                ua[a] = av.x;
                ua[a + 1] = av.y;
                ub[a] = bv.x;
                ub[a + 1] = bv.y;
            }
            const double dk = L.Dk[h + kk];
#pragma unroll
            for (int a = 0; a < R; ++a)
#pragma unroll
                for (int b = 0; b < R; ++b) acc[a][b] = acc[a][b] - (ua[a] * ub[b]) * dk;
        }
    }
#pragma unroll
    for (int b = 0; b < R; ++b)
#pragma unroll
        for (int a = 0; a < R; ++a) {
            const int64_t i = ir + a, j = jc + b;
            if (i <= j) Uc[j * n + i] = acc[a][b];
        }
}

// Tiles (blockIdx.y, blockIdx.x) of 16R x 16R in the columns from j0.
template <int R>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void factor_trailing_kernel(
        double* __restrict__ Uc, const double* __restrict__ D, int64_t n, int64_t k0, int64_t j0) {
    __shared__ FTrailLdsT<R> L;
    factor_trailing_body<R>(Uc, D, n, k0, (int64_t)blockIdx.y * 16 * R, j0 + (int64_t)blockIdx.x * 16 * R, L);
}

// Look-ahead: the next diagonal block [kd, kd + 64) (workgroup 0, once the column of tiles it
// needs has been updated) beside the rest of the current block's trailing update, tiles with
// bj < nb (the other workgroups, nb x nb of them).  The two touch disjoint elements.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void factor_lookahead_kernel(
        double* __restrict__ Uc, double* __restrict__ D, int64_t n, int64_t k0, int64_t nb, int64_t kd,
        int* __restrict__ status) {
    __shared__ union {
        DiagLds d;
        FTrailLds t;
    } L;
    if (blockIdx.x == 0) {
        factor_diag_body(Uc, D, n, kd, status, L.d);
    } else {
        const int64_t idx = blockIdx.x - 1;
        factor_trailing_body<4>(Uc, D, n, k0, idx / nb * kTile, idx % nb * kTile, L.t);
    }
}

// ---- quantize -----------------------------------------------------------------------------

// X[inv[c]][r] = w[r][c]: the weights by columns, in the visiting order.  64 x 64 values per
// workgroup through LDS, so that both sides move whole lines: [4096, 4096] bf16 46 us (gathered
// row by row in the visiting order 64).  One dimension of workgroups (a row block's column tiles
// after another): the second of a grid is limited to 65535 by some runtimes, 4.2 million rows.
template <typename In>
__global__ __launch_bounds__(256) void init_x_kernel(const In* __restrict__ w, const int* __restrict__ inv,
                                                     int64_t rows, int64_t n, double* __restrict__ X) {
    __shared__ float v[kTile][kTile + 1];
    __shared__ int to[kTile];
    const uint32_t tiles = (uint32_t)(n / kTile);
    const int64_t c0 = (int64_t)(blockIdx.x % tiles) * kTile, r0 = (int64_t)(blockIdx.x / tiles) * kTile;
    const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
    for (int k = part; k < kTile; k += 4)
        if (r0 + k < rows) v[k][lane] = load_w<In>(w, (r0 + k) * n + c0 + lane);
    if (part == 0) to[lane] = inv[c0 + lane];
    __syncthreads();
    if (r0 + lane < rows)
        for (int k = part; k < kTile; k += 4) X[(int64_t)to[k] * rows + r0 + lane] = (double)v[lane][k];
}

// One tile of 64 columns, right-looking, a 16-lane row of lanes per matrix row and 16 rows per
// workgroup: lane q holds the running values of tile columns 16m + q, m = 0..3.  The tile's values
// first receive the terms of the one or two tiles before it (the lane row's errors broadcast in it
// with DPP, U in LDS), then column b is taken: every lane quantizes its own value of the group m =
// b / 16 (only lane b % 16's is final), that lane's error is broadcast, and each lane adds error *
// U_b,a to its columns a > b.  A column's values stay as they are once it is taken, so the group's
// last step leaves every lane its own error and code.  Every value thus receives its terms in
// ascending order, as the sequential definition adds them.
// Bound by the instructions of the walk: a wave alone on its SIMD issues one in about 8 cycles, so
// a column costs what it holds, about 25 (two exact quotients by reciprocal and remainder, the
// conversion to E2M1 and back, two broadcasts, at most four updates): 15 us a tile with the terms of
// one before.  A quad of lanes per row, with an IEEE division and seven binary64 comparisons by
// every lane, took 35 us and a launch of 7 us for those terms.
constexpr int kTileRows = 16;
struct alignas(16) TileLds {
    double T[kTile][kTile + 2];    // T[b][4q + m] = U_{b, 16m + q} of one 64 x 64 block of U (rows padded:
                                   // the staging writes of a wave, one per row, spread over the banks)
    int pc[kTile];
};

// What quantizing a value of one column and row takes.
struct ColumnScale {
    double w, sS;                  // the weight; s S
    float M, rM, cvs;              // s = M 2^E, RN32(1 / M), s (1 for the zero code: M = rM = 0)
    int code;
};

// Q(x) as in the definition: the error w - Q(x) and the nibble.  k is the number of midpoints passed,
// a tie counting only toward an even index; none for a zero scale.
__device__ __forceinline__ void quantize_any(double x, float S, const ColumnScale& c, double* e, uint32_t* nibble) {
    const float y = __fdiv_rn(__double2float_rn(x), S);
    const double ay = fabs((double)y), s = e4m3_f64(c.code);
    int k = 0;
#pragma unroll
    for (int j = 0; j < 7; ++j) k += ((j & 1) ? ay >= e2m1_mid(j) * s : ay > e2m1_mid(j) * s) ? 1 : 0;
    k = c.code == 0 ? 0 : k;
    const bool neg = signbit(y);
    const double wq = (double)((0xC8643210u >> (4 * k)) & 15u) * (s * (0.5 * (double)S));
    *e = c.w - (neg ? -wq : wq);
    *nibble = (neg ? 8u : 0u) | (uint32_t)k;
}

typedef float float2v __attribute__((ext_vector_type(2)));

// v / d from r = RN32(1 / d) and one remainder (Markstein), correctly rounded where nothing under- or
// overflows; in this form a zero keeps its sign.
__device__ __forceinline__ float div_recip(float v, float d, float r) {
    const float u = v * r;
    return fmaf(-fmaf(u, d, -v), r, u);
}

// The same for S in [2^-26, 2^26] and |RN32(x)| < 2^100 (*ok is cleared otherwise).  A quotient that
// is inexact because it underflows is below 2^-20 and gives a zero of its sign either way.  RN32(y / M)
// rounds to the same E2M1 value as y / s: a midpoint times M has at most 7 significant bits, so y is at
// least an ulp away from one that it misses.
__device__ __forceinline__ void quantize_fast(double x, float S, float rS, const ColumnScale& c, double* e,
                                              uint32_t* nibble, bool* ok) {
    const float xf = __double2float_rn(x);
    *ok = *ok && fabsf(xf) < 0x1p100f;
    const float u = div_recip(div_recip(xf, S, rS), c.M, c.rM);
    uint32_t any;                        // the conversion writes one byte and keeps the others
    asm volatile("" : "=v"(any));
    const uint32_t p = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(any, u, u, c.cvs, 0);
    const float2v g = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(p, 1.0f, 0);
    *e = c.w - (double)g.x * c.sS;       // +-E2M1 * (s S), exact
    *nibble = p & 15u;
}

__device__ __forceinline__ double lane_row_value(double v, int lane) {
    return __shfl(v, (int)(threadIdx.x & 48) | lane, 64);
}

template <typename In>
__device__ __forceinline__ void tile_body(const In* __restrict__ w, const int* __restrict__ perm,
                                          const double* __restrict__ Uc, const uint8_t* __restrict__ scales,
                                          const float* __restrict__ tensor_scale, int64_t rows, int64_t n,
                                          int block, int64_t a0, int nprev, double* __restrict__ X,
                                          uint8_t* __restrict__ codes, int64_t rblock, TileLds& L) {
    const int tid = threadIdx.x;
    const int rr = tid >> 4, q = tid & 15;
    const int64_t r = rblock * kTileRows + rr;
    const bool live = r < rows;
    const int64_t rc = live ? r : rows - 1;            // the loads of rows past the end
    if (tid < kTile) L.pc[tid] = perm[a0 + tid];
    double x[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) x[m] = X[(a0 + 16 * m + q) * rows + rc];
    // the block of U that the walk needs, fetched ahead of the earlier tiles' terms
    double own[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) own[k] = Uc[(a0 + (tid >> 6) + 4 * k) * n + a0 + (tid & 63)];   // U_{a0 + b, a0 + a}
    const double* Tp = &L.T[0][4 * q];
    constexpr int kTRow = kTile + 2;
    for (int64_t ap = a0 - (int64_t)nprev * kTile; ap < a0; ap += kTile) {
        double ev[4];                                  // this lane's errors: columns 16m + q of the tile
#pragma unroll
        for (int m = 0; m < 4; ++m) ev[m] = X[(ap + 16 * m + q) * rows + rc];
        double t[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) t[k] = Uc[(ap + (tid >> 6) + 4 * k) * n + a0 + (tid & 63)];   // by rows
        __syncthreads();                               // the previous block is used
#pragma unroll
        for (int k = 0; k < 16; ++k) L.T[(tid >> 6) + 4 * k][row16_slot(tid & 63)] = t[k];
        __syncthreads();
        double tc[4];
        read_row(tc, Tp);
        auto term = [&](auto bc) {
            constexpr int b = decltype(bc)::value;
            double tn[4];                              // the next row of U: read a step ahead, no further
            read_row(tn, Tp + (b + 1 < kTile ? b + 1 : b) * kTRow);
            __builtin_amdgcn_sched_barrier(0);
            const double e = row_bcast<(b & 15)>(ev[b >> 4]);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                x[m] = x[m] + e * tc[m];
                tc[m] = tn[m];
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        for_each_index(term, std::make_integer_sequence<int, kTile>());
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) L.T[tid & 63][row16_slot((tid >> 6) + 4 * k)] = own[k];   // own[k] = U_{b, a}: b = tid & 63
    __syncthreads();
    const float S = tensor_scale[0];
    const float rS = __fdiv_rn(1.0f, S);
    const int64_t nb = n / block;
    ColumnScale cs[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int c = L.pc[16 * m + q];
        const int code = scales[rc * nb + c / block];
        const double s = e4m3_f64(code);
        const float sf = (float)s;
        cs[m].w = (double)load_w<In>(w, rc * n + c);
        cs[m].sS = s * (double)S;
        cs[m].M = code == 0 ? 0.f : __uint_as_float((__float_as_uint(sf) & 0x007FFFFFu) | 0x3F800000u);
        cs[m].rM = code == 0 ? 0.f : __fdiv_rn(1.0f, cs[m].M);
        cs[m].cvs = code == 0 ? 1.0f : sf;
        cs[m].code = code;
    }
    double xs[4], e[4];
    uint32_t nib[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) xs[m] = x[m];
    bool ok = S >= 0x1p-26f && S <= 0x1p26f;
    double tc[4];
    read_row(tc, Tp);
    auto column = [&](auto bc) {
        constexpr int b = decltype(bc)::value, qb = b & 15, mb = b >> 4;
        double tn[4];
        read_row(tn, Tp + (b + 1 < kTile ? b + 1 : b) * kTRow);
        __builtin_amdgcn_sched_barrier(0);
        quantize_fast(x[mb], S, rS, cs[mb], &e[mb], &nib[mb], &ok);
        const double eb = row_bcast<qb>(e[mb]);
#pragma unroll
        for (int m = mb; m < 4; ++m) {
            const double v = x[m] + eb * tc[m];
            x[m] = m > mb || q > qb ? v : x[m];
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) tc[m] = tn[m];
        __builtin_amdgcn_sched_barrier(0);
    };
    for_each_index(column, std::make_integer_sequence<int, kTile>());
    if (__any(!ok)) {                                  // the wave's rows once more, by the definition
#pragma unroll
        for (int m = 0; m < 4; ++m) x[m] = xs[m];
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll 1
            for (int qb = 0; qb < 16; ++qb) {
                quantize_any(x[mb], S, cs[mb], &e[mb], &nib[mb]);
                const double eb = lane_row_value(e[mb], qb);
#pragma unroll
                for (int m = mb; m < 4; ++m) {
                    const double v = x[m] + eb * Tp[(16 * mb + qb) * kTRow + m];
                    x[m] = m > mb || q > qb ? v : x[m];
                }
            }
    }
    if (live) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            X[(a0 + 16 * m + q) * rows + r] = e[m];    // the tile's errors take its values' place
            codes[r * n + L.pc[16 * m + q]] = (uint8_t)nib[m];
        }
    }
}

// X[k][r] += sum over nterms errors b = a0, a0 + 1, ... in order of E[b][r] * U_{b, k}, for 128 rows (two
// to a lane, 64 apart) and 8 columns k0 .. k0 + 7 of each wave.  E is read over consecutive rows;
// U_{b, k..k+7} is the same for all lanes and comes through the scalar cache into scalar registers, an
// operand of the binary64 instructions as it is: no LDS, no barrier, 32 arithmetic instructions for
// two loads of a lane and one scalar load.  Scalar loads return out of order, so they are waited for
// all at once, some 700 cycles after their issue: two steps' are fetched a pair of steps ahead (16
// columns and one step ahead left a wave waiting for them, 300 ns a step).  Bound by binary64 issue:
// a SIMD with four such waves takes 5.7 cycles an instruction (4.9 with eight, 12.5 with one; a
// multiply and an addition each, as the definition rounds them), and the launches of [4096, 4096]
// take 3.76 ms in all, of which the terms are 2.5.  (4 x 4 values per lane with both operands in
// LDS, the tile's chain of 35 us beside them: 4.4 ms.)
typedef double double8 __attribute__((ext_vector_type(8)));
constexpr int kTermRows = 128, kTermCols = 8;

__device__ __forceinline__ void add_terms(const double* __restrict__ Uc, int64_t rows, int64_t n, int64_t a0,
                                          int nterms, int64_t k0, int64_t r0, double* __restrict__ X) {
    constexpr int H = kTermRows / 64;                  // rows of a lane
    constexpr int kAhead = 4;                          // steps of E in flight
    const int lane = threadIdx.x & 63;
    int64_t rr[H], rc[H];
    double acc[H][kTermCols];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        rr[h] = r0 + lane + 64 * h;
        rc[h] = rr[h] < rows ? rr[h] : rows - 1;
#pragma unroll
        for (int c = 0; c < kTermCols; ++c) acc[h][c] = X[(k0 + c) * rows + rc[h]];
    }
    const double* ep = X + a0 * rows;
    const double* up = Uc + a0 * n + k0;
    // the wave's lines of U, touched once so that the scalar loads find them in the XCD's L2
    const double t0 = up[(int64_t)lane * n], t1 = up[(int64_t)(nterms - 64 + lane) * n];
    double e[H][kAhead], en[H][kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
#pragma unroll
        for (int h = 0; h < H; ++h) e[h][i] = ep[(int64_t)i * rows + rc[h]];
    asm volatile("" ::"v"(t0), "v"(t1) : "memory");
    auto urow = [&](int b) { return *reinterpret_cast<const double8*>(up + (int64_t)b * n); };
    double8 u0 = urow(0), u1 = urow(1);
    for (int b0 = 0; b0 < nterms; b0 += kAhead) {      // nterms: a multiple of 64
        const int bn = b0 + kAhead < nterms ? b0 + kAhead : b0;
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
#pragma unroll
            for (int h = 0; h < H; ++h) en[h][i] = ep[(int64_t)(bn + i) * rows + rc[h]];
#pragma unroll
        for (int i = 0; i < kAhead; i += 2) {
            const int b2 = i + 2 < kAhead ? b0 + i + 2 : bn;
            const double8 n0 = urow(b2), n1 = urow(b2 + 1);
            __builtin_amdgcn_sched_barrier(0);
            double p[H][kTermCols];                    // all products, then all sums: no instruction waits
#pragma unroll
            for (int half = 0; half < 2; ++half) {
#pragma unroll
                for (int c = 0; c < kTermCols; ++c)
#pragma unroll
                    for (int h = 0; h < H; ++h) p[h][c] = e[h][i + half] * (half ? u1[c] : u0[c]);
#pragma unroll
                for (int c = 0; c < kTermCols; ++c)
#pragma unroll
                    for (int h = 0; h < H; ++h) acc[h][c] = acc[h][c] + p[h][c];
            }
            __builtin_amdgcn_sched_barrier(0);
            u0 = n0;
            u1 = n1;
        }
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
#pragma unroll
            for (int h = 0; h < H; ++h) e[h][i] = en[h][i];
    }
#pragma unroll
    for (int c = 0; c < kTermCols; ++c)
#pragma unroll
        for (int h = 0; h < H; ++h)
            if (rr[h] < rows) X[(k0 + c) * rows + rr[h]] = acc[h][c];
}
// Launch t: tile t (workgroups 0 .. ntile-1; nprev tiles' terms first) beside the terms of nterms
// errors from ap on ncb blocks of 32 columns from kstart (the other workgroups, 128 rows each).  While
// many columns are left they are read and written once per pair of tiles: pair (2j-2, 2j-1) goes to
// the columns past tile 2j in the launches 2j and 2j+1, half of them each, the first with tile 2j+1
// among them, so tile 2j adds the pair's terms itself and tile 2j+1 only tile 2j's.  For the last
// columns, where the tile's own chain is the longer role, every launch adds the tile before.
// Every column has its terms in ascending order, and the two roles touch disjoint values.
template <typename In>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void quantize_kernel(
        const In* __restrict__ w, const int* __restrict__ perm, const double* __restrict__ Uc,
        const uint8_t* __restrict__ scales, const float* __restrict__ tensor_scale, int64_t rows,
        int64_t n, int block, int64_t a0, int nprev, double* __restrict__ X, uint8_t* __restrict__ codes,
        int64_t ntile, int64_t ap, int nterms, int64_t kstart, int64_t ncb) {
    __shared__ TileLds L;
    if ((int64_t)blockIdx.x < ntile) {
        tile_body<In>(w, perm, Uc, scales, tensor_scale, rows, n, block, a0, nprev, X, codes, blockIdx.x, L);
    } else {
        const int64_t idx = blockIdx.x - ntile;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        add_terms(Uc, rows, n, ap, nterms, kstart + (idx % ncb * 4 + wave) * kTermCols, idx / ncb * kTermRows, X);
    }
}

__global__ __launch_bounds__(256) void pack_kernel(const uint8_t* __restrict__ codes, int64_t npairs,
                                                   uint8_t* __restrict__ q) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t < npairs) q[t] = (uint8_t)(codes[2 * t] | (codes[2 * t + 1] << 4));
}

__global__ void clear_status_kernel(int* status) { status[0] = 0; }

// ---- workspace ---------------------------------------------------------------------------

struct Layout {
    size_t perm, diag, lambda, D, Uc, X, codes, total;
};

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

Layout layout_of(int64_t rows, int64_t n) {
    Layout l;
    size_t o = 0;
    l.perm = o;   o = align256(o + (size_t)n * sizeof(int));
    l.diag = o;   o = align256(o + (size_t)n * sizeof(double));
    l.lambda = o; o = align256(o + sizeof(double));
    l.D = o;      o = align256(o + (size_t)n * sizeof(double));
    l.Uc = o;     o = align256(o + (size_t)n * n * sizeof(double));
    l.X = o;      o = align256(o + (size_t)rows * n * sizeof(double));
    // unused room of 128 values a row: the size stays what callers have been told, at 64 columns no less
    // than the interface's 8 (cols^2 + 2 rows cols) bytes
    o = align256(o + (size_t)2 * rows * kTile * sizeof(double));
    l.codes = o;  o = align256(o + (size_t)rows * n);
    l.total = o;
    return l;
}

// The last tiles, whose terms go tile by tile: their launches are as long as a tile's own chain, and 64
// terms are half the work of a wave beside it.  8, 16 and 32 of them, whole calls: [4096, 4096] 7.51, 7.50,
// 7.48 ms, [4096, 2048] 2.60, 2.59, 2.59, [4096, 8192] 30.2, 30.1, 30.0, [14336, 4096] 16.94, 16.96, 17.27,
// [14336, 2048] 5.10, 5.08, 5.28.  With few rows the chain is the longer role for longer, and more would be
// the better: [128, 4096] 4.93, 4.87, 4.72.
constexpr int64_t kSingleTiles = 16;

unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

template <typename In>
int run_ldlq(const void* wv, int64_t rows, int64_t n, int block, const double* H,
             const uint8_t* scales, const float* S, double damp, uint8_t* q, int* status,
             char* ws, hipStream_t st) {
    const In* w = static_cast<const In*>(wv);
    const Layout l = layout_of(rows, n);
    int* perm = reinterpret_cast<int*>(ws + l.perm);
    int* inv = reinterpret_cast<int*>(ws + l.D);        // read before the factor writes D
    double* diag = reinterpret_cast<double*>(ws + l.diag);
    double* lambda = reinterpret_cast<double*>(ws + l.lambda);
    double* D = reinterpret_cast<double*>(ws + l.D);
    double* Uc = reinterpret_cast<double*>(ws + l.Uc);
    double* X = reinterpret_cast<double*>(ws + l.X);
    uint8_t* codes = reinterpret_cast<uint8_t*>(ws + l.codes);

    hipLaunchKernelGGL(clear_status_kernel, dim3(1), dim3(1), 0, st, status);
    hipLaunchKernelGGL(diag_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, H, n, diag);
    hipLaunchKernelGGL(order_kernel, dim3(blocks_for(n, 64) + 1), dim3(64 * kOrderParts), 0, st, diag, n, perm, inv,
                       damp, lambda);
    if (hipGetLastError() != hipSuccess) return NVFP4_ERR_HIP;
    const int64_t tiles = n / kTile;
    hipLaunchKernelGGL(init_a_kernel, dim3((unsigned)((tiles + 7) / 8 * 8 * tiles)), dim3(256), 0, st, H, perm, lambda,
                       n, Uc);
    hipLaunchKernelGGL(init_x_kernel<In>, dim3((unsigned)(tiles * blocks_for(rows, kTile))), dim3(256), 0, st, w, inv,
                       rows, n, X);
    // factor, from the last block: its diagonal block, then per block the panel above it, the
    // column of tiles the next diagonal block and panel need, and then the next diagonal block
    // beside the rest of the trailing update (look-ahead)
    hipLaunchKernelGGL(factor_diag_kernel, dim3(1), dim3(4 * kTile), 0, st, Uc, D, n, n - kTile, status);
    for (int64_t k0 = n - kTile; k0 > 0; k0 -= kTile) {
        hipLaunchKernelGGL(factor_panel_kernel, dim3(blocks_for(k0, kPanelRows)), dim3(256), 0, st, Uc, D,
                           n, k0);
        const int64_t nb = k0 / kTile - 1;                         // the next block's tile column
        hipLaunchKernelGGL(factor_trailing_kernel<2>, dim3(2, (unsigned)(2 * (nb + 1))), dim3(256), 0, st, Uc,
                           D, n, k0, nb * kTile);
        hipLaunchKernelGGL(factor_lookahead_kernel, dim3((unsigned)(1 + nb * nb)), dim3(256), 0, st, Uc, D,
                           n, k0, nb > 0 ? nb : 1, k0 - kTile, status);
        if (hipGetLastError() != hipSuccess) return NVFP4_ERR_HIP;
    }
    // quantize: tile t beside the terms of earlier tiles on the later columns (quantize_kernel)
    const int64_t ntiles = n / kTile;
    const unsigned tile_wgs = blocks_for(rows, kTileRows), row_wgs = blocks_for(rows, kTermRows);
    const int64_t t0 = ntiles > kSingleTiles ? (ntiles - kSingleTiles) & ~(int64_t)1 : 0;   // the last pair's launch
    for (int64_t t = 0; t < ntiles; ++t) {
        const int64_t even = t & ~(int64_t)1;               // the launches even, even + 1 share a pair
        const bool pairs = t < t0 || (t == t0 && t > 0);
        int64_t c0 = t + 1, c1 = ntiles;                    // the tiles that receive terms
        int nprev = t > 0 ? 1 : 0, nterms = nprev * kTile;
        int64_t ap = (t - 1) * kTile;
        if (pairs) {
            const int64_t mid = t == t0 ? ntiles : even + 1 + (ntiles - even) / 2;
            if (t == even) c1 = mid;
            else c0 = mid;
            ap = (even - 2) * kTile;
            nterms = even >= 2 ? 2 * kTile : 0;
            if (t == even && t >= 2) nprev = 2;
        }
        const int64_t ncb = nterms > 0 && c1 > c0 ? (c1 - c0) * (kTile / (4 * kTermCols)) : 0;
        hipLaunchKernelGGL(quantize_kernel<In>, dim3((unsigned)(tile_wgs + ncb * row_wgs)), dim3(256), 0, st, w, perm,
                           Uc, scales, S, rows, n, block, t * kTile, nprev, X, codes, (int64_t)tile_wgs, ap, nterms,
                           c0 * kTile, ncb > 0 ? ncb : 1);
        if (hipGetLastError() != hipSuccess) return NVFP4_ERR_HIP;
    }
    hipLaunchKernelGGL(pack_kernel, dim3(blocks_for(rows * n / 2, 256)), dim3(256), 0, st, codes,
                       rows * n / 2, q);
    return hipGetLastError() == hipSuccess ? NVFP4_OK : NVFP4_ERR_HIP;
}

}  // namespace

extern "C" {

size_t nvfp4_ldlq_workspace_bytes(int64_t rows, int64_t cols) {
    if (rows < 0 || cols < 0) return 0;
    return layout_of(rows, cols).total;
}

int nvfp4_ldlq(const void* w, int dtype, int64_t rows, int64_t cols, int block, const double* hessian,
               const uint8_t* scales, const float* tensor_scale, double damp, uint8_t* q, int* status,
               void* workspace, size_t workspace_bytes, void* stream) {
    if (dtype != NVFP4_IN_F32 && dtype != NVFP4_IN_BF16) return NVFP4_ERR_DTYPE;
    if (block != 16 && block != 32 && block != 64 && block != 128) return NVFP4_ERR_BLOCK;
    if (rows < 0 || cols < 0 || cols % kTile != 0) return NVFP4_ERR_SHAPE;
    if (cols > 0x7FFFFFFF || rows * cols > ((int64_t)1 << 40)) return NVFP4_ERR_SHAPE;
    if (!(damp >= 0.0) || !isfinite(damp)) return NVFP4_ERR_ARG;
    if (!status || !tensor_scale) return NVFP4_ERR_NULL;
    if (rows * cols > 0 && (!w || !hessian || !scales || !q)) return NVFP4_ERR_NULL;
    if (((uintptr_t)hessian & 7) || ((uintptr_t)status & 3)) return NVFP4_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    if (rows * cols == 0) {
        hipLaunchKernelGGL(clear_status_kernel, dim3(1), dim3(1), 0, st, status);
        return hipGetLastError() == hipSuccess ? NVFP4_OK : NVFP4_ERR_HIP;
    }
    if (!workspace || workspace_bytes < layout_of(rows, cols).total) return NVFP4_ERR_WORKSPACE;
    if ((uintptr_t)workspace & 255) return NVFP4_ERR_ALIGN;
    char* ws = static_cast<char*>(workspace);
    return dtype == NVFP4_IN_F32
        ? run_ldlq<float>(w, rows, cols, block, hessian, scales, tensor_scale, damp, q, status, ws, st)
        : run_ldlq<uint16_t>(w, rows, cols, block, hessian, scales, tensor_scale, damp, q, status, ws, st);
}

}  // extern "C"
