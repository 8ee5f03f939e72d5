// Reference block scales for NVFP4 gap reports, on AMD Instinct MI355X (gfx950):
//   * the optimal real (FP32) block scale and its loss (appendix "Optimal FP32 Scale for FP4
//     Quantization", first paragraph);
//   * the FP8-quantized optimal scale (same appendix, second paragraph);
//   * the exact loss of given E4M3 block scales, and a deterministic binary64 sum,
// for the relative gaps of AbsMax, 4/6 and ScaleSweep to the optimum (Figures 1 and 4).
//
// The loss of one block, L(s) = sum_i w_i (|y_i| - RNE_FP4(|y_i| / s) s)^2, is piecewise
// quadratic in s; it changes pieces where |y_i| / s crosses a midpoint between neighbouring
// E2M1 values, i.e. at the 7 breakpoints |y_i| / m_k of every non-zero element.  Between two
// consecutive breakpoints the rounding of every element is fixed, so L = A - 2 B s + C s^2
// there and its minimum on the closed piece is at B / C clamped to the piece.
//
// Work layout: one wavefront per micro-block (two at n = 64, four at n = 128).  It sorts the
// block's 7 n breakpoints (padded with +inf to 8 n) with a bitonic network, and then every lane
// scores every 64th piece: the roundings on the piece follow from which breakpoints lie below
// it, its coefficients are summed in element order, and its minimum formed as above.  A
// lexicographic minimum (loss, piece index) picks the optimum, the lowest piece on
// a tie, and the all-zero reconstruction (s -> infinity) ahead of any piece of equal loss.
// Everything is binary64 with correctly rounded division and no contraction, so each
// value is a fixed sequence of IEEE operations.  This is analysis work, bound by binary64
// ALU throughput, not part of the quantizers' hot path.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "exact_fp.h"
#include "nvfp4ss.h"

namespace {

constexpr int kWave = 64;

using namespace nvfp4_exact;

template <typename In>
__device__ __forceinline__ float load_elem(const In* x, int64_t i);

template <>
__device__ __forceinline__ float load_elem<float>(const float* x, int64_t i) { return x[i]; }

template <>
__device__ __forceinline__ float load_elem<uint16_t>(const uint16_t* x, int64_t i) {
    return __uint_as_float((uint32_t)x[i] << 16);        // bfloat16 -> binary32, exact
}

struct Best {
    double val, s;
    int seg;                 // -1: the all-zero reconstruction
};

__device__ __forceinline__ bool better(const Best& a, const Best& b) {
    return a.val < b.val || (a.val == b.val && a.seg < b.seg);
}

// How a block of N elements is spread over a workgroup.  Its 7 N breakpoints, padded to 8 N, sit
// kPer to a thread; one wave up to N = 32, more above, so that a CU holds at least five waves per
// SIMD whatever the block's LDS (binary64 chains and LDS reads need them to overlap).
template <int N>
struct Spread {
    static constexpr int kWaves = N <= 32 ? 1 : N / 32;
    static constexpr int kThreads = kWaves * kWave;
    static constexpr int kBreaks = 8 * N;
    static constexpr int kPer = kBreaks / kThreads;            // 2 at N = 16, else 4
    // Most blocks that a workgroup takes together: their elements are loaded, and their FP8 neighbours
    // scored, by full waves.
    // (At N = 32 the extra registers cost the fifth wave per SIMD and 5 % of the time.)
    static constexpr int kBatch = N == 16 ? 4 : 1;
};

// v of lane (lane ^ D), D < 16 (DPP: quad permutations, a half-row mirror, a row rotation).
template <int D>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
    static_assert(D == 1 || D == 2 || D == 4 || D == 8, "inside a row of 16 lanes");
    auto dpp = [](uint32_t t, auto ctrl) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)t, decltype(ctrl)::value, 0xF, 0xF, true);
    };
    if constexpr (D == 1) return dpp(v, std::integral_constant<int, 0xB1>());      // quad_perm 1 0 3 2
    if constexpr (D == 2) return dpp(v, std::integral_constant<int, 0x4E>());      // quad_perm 2 3 0 1
    if constexpr (D == 4)                                                          // 7 - l, then 3 - l
        return dpp(dpp(v, std::integral_constant<int, 0x141>()), std::integral_constant<int, 0x1B>());
    return dpp(v, std::integral_constant<int, 0x128>());                           // row_ror 8
}

template <int D>
__device__ __forceinline__ double exchange_other(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    return __longlong_as_double(
        (long long)(((uint64_t)lane_xor<D>((uint32_t)(b >> 32)) << 32) | lane_xor<D>((uint32_t)b)));
}

// One compare-exchange between lanes D apart: the lane keeps the smaller of the two keys, or the
// larger.  (Equal keys are only the +inf padding.)
template <int D>
__device__ __forceinline__ double exchange(double v, bool keep_min) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    double lo_lane = v, other;
    if constexpr (D < 16) {
        other = exchange_other<D>(v);
    } else {                   // rows (16) or halves (32) of the two operands swap: both lanes of a
                               // pair see the lower lane's key, then the upper lane's
        const auto h = D == 16 ? __builtin_amdgcn_permlane16_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false)
                               : __builtin_amdgcn_permlane32_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);
        const auto l = D == 16 ? __builtin_amdgcn_permlane16_swap((uint32_t)b, (uint32_t)b, false, false)
                               : __builtin_amdgcn_permlane32_swap((uint32_t)b, (uint32_t)b, false, false);
        lo_lane = __longlong_as_double((long long)(((uint64_t)h[0] << 32) | l[0]));
        other = __longlong_as_double((long long)(((uint64_t)h[1] << 32) | l[1]));
    }
    return (lo_lane < other) == keep_min ? lo_lane : other;
}

// Ascending bitonic sort of the kBreaks keys, thread t holding positions kPer t + r; the runs of
// eight (one element's breakpoints) come in sorted, alternately up and down.  Strides inside a
// thread and inside a wave stay in registers; the few across waves go through LDS.
template <int N>
__device__ __forceinline__ void sort_keys(double (&k)[Spread<N>::kPer], double* lds) {
    using Sp = Spread<N>;
    constexpr int R = Sp::kPer;
    const int tid = threadIdx.x;
    auto stage = [&](auto size_c, auto stride_c) {
        constexpr int size = decltype(size_c)::value, stride = decltype(stride_c)::value;
        const bool asc = size >= Sp::kBreaks || (tid & (size / R)) == 0;
        if constexpr (stride < R) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (r & stride) continue;
                const double u = k[r], v = k[r + stride];
                const bool keep = (u < v) == asc;
                k[r] = keep ? u : v;
                k[r + stride] = keep ? v : u;
            }
        } else {
            constexpr int d = stride / R;                      // threads apart
            const bool keep_min = ((tid & d) == 0) == asc;
            if constexpr (d < kWave) {
#pragma unroll
                for (int r = 0; r < R; ++r) k[r] = exchange<d>(k[r], keep_min);
            } else {
                __syncthreads();
#pragma unroll
                for (int r = 0; r < R; ++r) lds[r * Sp::kThreads + tid] = k[r];
                __syncthreads();
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const double o = lds[r * Sp::kThreads + (tid ^ d)];
                    k[r] = (k[r] < o) == keep_min ? k[r] : o;
                }
            }
        }
    };
    auto merge = [&](auto size_c) {
        constexpr int size = decltype(size_c)::value;
        if constexpr (size <= Sp::kBreaks) {
            auto down = [&](auto self, auto stride_c) {
                constexpr int stride = decltype(stride_c)::value;
                stage(size_c, stride_c);
                if constexpr (stride > 1) self(self, std::integral_constant<int, stride / 2>());
            };
            down(down, std::integral_constant<int, size / 2>());
        }
    };
    merge(std::integral_constant<int, 16>());
    merge(std::integral_constant<int, 32>());
    merge(std::integral_constant<int, 64>());
    merge(std::integral_constant<int, 128>());
    merge(std::integral_constant<int, 256>());
    merge(std::integral_constant<int, 512>());
    merge(std::integral_constant<int, 1024>());
}

// 420 / (4 m_j) for the midpoints 4 m_j = 1, 3, 5, 7, 10, 14, 20: nine bits each.
__device__ __forceinline__ double break_factor(int j) {
    constexpr uint64_t packed = 420ull | 140ull << 9 | 84ull << 18 | 60ull << 27 | 42ull << 36 |
                                30ull << 45 | 21ull << 54;
    return (double)(int)((packed >> (9 * j)) & 511u);
}

// RN(k / 105) for a key k (24 + 9 bits): a multiply by the rounded reciprocal and one exact
// remainder's correction (Markstein).  NaN for the padding, whose quotient nothing reads.
__device__ __forceinline__ double div_105(double k) {
    constexpr double r = 1.0 / 105.0;
    const double q = k * r;
    return fma(fma(-q, 105.0, k), r, q);
}

// The least value of a wave, in every lane.
__device__ __forceinline__ double wave_min(double v) {
    v = fmin(v, exchange_other<1>(v));
    v = fmin(v, exchange_other<2>(v));
    v = fmin(v, exchange_other<4>(v));
    v = fmin(v, exchange_other<8>(v));
    v = fmin(v, exchange<16>(v, true));
    return fmin(v, exchange<32>(v, true));
}

__device__ __forceinline__ int wave_min(int v) {
    v = min(v, (int)lane_xor<1>((uint32_t)v));
    v = min(v, (int)lane_xor<2>((uint32_t)v));
    v = min(v, (int)lane_xor<4>((uint32_t)v));
    v = min(v, (int)lane_xor<8>((uint32_t)v));
    const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
    v = min((int)h[0], (int)h[1]);
    const auto q = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
    return min((int)q[0], (int)q[1]);
}

__device__ __forceinline__ double read_lane(double v, int lane) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(
        (long long)(((uint64_t)hi << 32) | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane)));
}

// The breakpoints |y| / m are sorted by the key |y| (420 / 4m), which is exact in binary64 (24 + 9
// bits) and orders and ties them as the quotients do: two different quotients of 24-bit values by
// these midpoints are at least 2^-29 apart, so their roundings neither meet nor cross, and a
// piece's midpoint is never within rounding of a breakpoint.  The key's low bits are free and
// carry the element.  So on the piece above the first `seg` breakpoints, an element has passed 7
// minus as many midpoints as it has breakpoints among those: a count of its positions below seg
// (a compare, and a bit count below the lane), instead of comparisons with seven products per
// element and piece, and the terms it adds to B and C come from a table of its eight roundings,
// formed once.  VALU issue bounds the kernel (784 instructions a block at N = 16, of
// which the sort and the pieces take 300 each): [4096, 4096] bfloat16 with weights 1.20 ms (a
// comparison with each product, breakpoints sorted in LDS, the FP8 losses on one lane: 4.19 ms);
// at N = 32, 64, 128 0.83, 0.71 and 0.61 ms for half, a quarter and an eighth of the rows (2.92,
// 2.23, 2.46).  Five waves per SIMD: four cost 6 % at N = 64 and 128.
template <typename In, int N>
__global__ __launch_bounds__(Spread<N>::kThreads, 5) void optimum_kernel(const In* __restrict__ x,
                                                                     const float* __restrict__ colw,
                                                                     const float* __restrict__ tensor_scale,
                                                                     int64_t nblocks, int64_t bpr, int batch,
                                                                     double* __restrict__ opt_loss,
                                                                     double* __restrict__ opt_scale,
                                                                     uint8_t* __restrict__ fp8_code,
                                                                     double* __restrict__ fp8_loss) {
    using Sp = Spread<N>;
    constexpr int R = Sp::kPer, W = Sp::kWaves, P = Sp::kBreaks;
    const int KB = Sp::kBatch == 1 ? 1 : batch;
    __shared__ alignas(16) double key[P];     // sorted keys, then breakpoints, then FP8 loss terms
    __shared__ alignas(16) double2 tab[P];    // tab[8 i + c]: element i's terms of B and C with c
                                              // of its breakpoints passed
    __shared__ alignas(16) double ads[Sp::kBatch][N], wds[Sp::kBatch][N], aas[Sp::kBatch][N];   // |y|, w, w y^2
    __shared__ uint32_t first[W > 1 ? W : 1][W > 1 ? N : 1];   // breakpoints below a wave's pieces
    __shared__ Best wave_best[W];
    __shared__ double scale_of[Sp::kBatch];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const float S = tensor_scale[0];
    const bool weighted = colw != nullptr;

    const int64_t kb_step = (int64_t)gridDim.x * KB % bpr;
    int64_t kb = ((int64_t)blockIdx.x * KB + tid / N) % bpr;   // column of this thread's block
    for (int64_t blk0 = (int64_t)blockIdx.x * KB; blk0 < nblocks; blk0 += (int64_t)gridDim.x * KB) {
        if (tid < N * KB) {
            double a = 0.0, wi = 1.0;
            if (blk0 + tid / N < nblocks) {
                const float y = __fdiv_rn(load_elem<In>(x, blk0 * N + tid), S);   // y = RN32(x / S)
                a = fabs((double)y);
                if (weighted) wi = (double)colw[kb * N + tid % N];
            }
            ads[0][tid] = a;
            wds[0][tid] = wi;
            aas[0][tid] = wi * a * a;
        }
        __syncthreads();
        for (int b = 0; b < KB && blk0 + b < nblocks; ++b) {
            const double *ad = ads[b], *wd = wds[b], *aa = aas[b];
            // Breakpoints: 7 for each non-zero finite element.  An infinity or a NaN has none (its keys
            // would not be ordered, and an element must not have more than 7 positions): the loss is
            // infinite or NaN whatever the scale.
            int nb = 0;
            bool zero = true;
#pragma unroll
            for (int i = 0; i < N; i += kWave) {
                const double a = ad[(i + lane) & (N - 1)];
                const uint64_t nonzero = __ballot(i + lane < N && a != 0.0);
                zero = zero && nonzero == 0;
                nb += 7 * __popcll(nonzero & __ballot(a < INFINITY));
            }
            double k[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int p = tid * R + r, e = p >> 3, h = p & 7;
                // even elements rise (m from the largest), odd ones fall; the padding is +inf
                const bool up = (e & 1) == 0, pad = h == (up ? 7 : 0);
                const double a = ad[e];
                const double v = a * break_factor(pad ? 0 : up ? 6 - h : h - 1);
                k[r] = pad || a == 0.0 || !(a < INFINITY)
                           ? INFINITY
                           : __longlong_as_double(__double_as_longlong(v) | (long long)e);
                // the element's terms with h breakpoints passed: rounded to value 7 - h
                const double g = e2m1_value(7 - h), w = wd[e];
                tab[p] = a == 0.0 ? make_double2(0.0, 0.0) : make_double2(w * a * g, w * g * g);
            }
            sort_keys<N>(k, key);
            __syncthreads();
#pragma unroll
            for (int r = 0; r < R; ++r) key[tid * R + r] = k[r];
            __syncthreads();
            // wave v's pieces are seg = 64 (R v + t) + lane; the breakpoint above each, its element
            const int seg0 = kWave * R * wave;
            uint32_t id[R];
            double hi_bp[R];
#pragma unroll
            for (int t = 0; t < R; ++t) {
                const uint64_t b = (uint64_t)__double_as_longlong(key[seg0 + kWave * t + lane]);
                id[t] = seg0 + kWave * t + lane < nb ? (uint32_t)b & 127u : 128u;      // padding: none
                hi_bp[t] = div_105(__longlong_as_double((long long)(b & ~127ull)));    // RN(|y| / m)
            }
            if constexpr (W > 1) {
                const double from = key[seg0];
                for (int i = lane; i < N; i += kWave) {
                    uint32_t c = 0;
#pragma unroll
                    for (int j = 0; j < 7; ++j)
                        c += __longlong_as_double(__double_as_longlong(ad[i] * break_factor(j)) | (long long)i) < from ? 1u : 0u;
                    first[wave][i] = ad[i] != 0.0 ? c : 0u;
                }
            }
            __syncthreads();                       // the keys are used
#pragma unroll
            for (int t = 0; t < R; ++t) key[seg0 + kWave * t + lane] = hi_bp[t];
            __syncthreads();

            double A = 0.0;                        // sum w y^2: the loss of the all-zero reconstruction
            double B[R], C[R];
#pragma unroll
            for (int t = 0; t < R; ++t) B[t] = C[t] = 0.0;
#pragma unroll 4
            for (int i = 0; i < N; ++i) {
                uint32_t below = W > 1 ? first[wave][i] : 0u;
                A += aa[i];
#pragma unroll
                for (int t = 0; t < R; ++t) {
                    const uint64_t m = __ballot(id[t] == (uint32_t)i);
                    const uint32_t c = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)m, below));
                    const double2 v = tab[8 * i + c];              // c <= 7: an element has 7
                    B[t] += v.x;
                    C[t] += v.y;
                    if (t + 1 < R) below += (uint32_t)__popcll(m);
                }
            }
            Best best{A, INFINITY, -1};
#pragma unroll
            for (int t = 0; t < R; ++t) {
                const int seg = seg0 + kWave * t + lane;
                const double lo = seg == 0 ? 0.0 : key[seg == 0 ? 0 : seg - 1];
                const double hi = seg == nb ? INFINITY : hi_bp[t];
                if (seg > nb || !(hi > lo)) continue;
                const double s_ref = seg == 0 ? 0.5 * hi : seg == nb ? 2.0 * lo : 0.5 * (lo + hi);
                Best cand{0.0, 0.0, seg};
                if (C[t] <= 0.0) {
                    cand.val = A;
                    cand.s = s_ref;
                } else {
                    double s = B[t] / C[t];
                    if (s < lo) s = lo;
                    if (s > hi) s = hi;
                    if (s <= 0.0) continue;
                    double val = A - 2.0 * B[t] * s + C[t] * s * s;
                    if (val < 0.0) val = 0.0;
                    cand.val = val;
                    cand.s = s;
                }
                if (better(cand, best)) best = cand;
            }
            // the wave's least loss, the lowest piece on a tie (every lane holds at least the all-zero
            // reconstruction)
            {
                const double least = wave_min(best.val);
                const int seg = wave_min(best.val == least ? best.seg : INT32_MAX);
                const uint64_t m = __ballot(best.val == least && best.seg == seg);
                const int from = m ? (int)__builtin_ctzll(m) : 0;          // m = 0 only with NaN
                best = Best{read_lane(best.val, from), read_lane(best.s, from), __builtin_amdgcn_readlane(best.seg, from)};
            }
            if constexpr (W > 1) {
                if (lane == 0) wave_best[wave] = best;
                __syncthreads();
                best = wave_best[0];
#pragma unroll
                for (int v = 1; v < W; ++v)
                    if (better(wave_best[v], best)) best = wave_best[v];
            }
            double J = best.val, s_opt = best.s;
            if (zero) {                             // all-zero block: zero loss at any scale
                J = 0.0;
                s_opt = 1.0;
            }
            if (tid == 0) {
                opt_loss[blk0 + b] = J;
                if (opt_scale) opt_scale[blk0 + b] = s_opt;
                scale_of[b] = s_opt;
            }
            __syncthreads();                        // key and tab are reused
        }
        if (fp8_code || fp8_loss) {
            // the FP8 values just below and just above s_opt; the lower-loss one (the lower value
            // on a tie); positive codes only.  One thread per term, then one lane per sum adds its
            // N terms in element order.
            auto neighbours = [&](double s, int& cf, int& cc) {
                cf = floor_e4m3(s);
                cc = (e4m3_f64(cf) < s && cf < 126) ? cf + 1 : cf;
                cf = cf < 1 ? 1 : cf;
                cc = cc < 1 ? 1 : cc;
            };
            int cf, cc;
            for (int t = tid; t < 2 * N * KB; t += Sp::kThreads) {
                const int b = t / (2 * N), i = t & (N - 1);
                if (blk0 + b < nblocks) {
                    neighbours(scale_of[b], cf, cc);
                    const double s = e4m3_f64(t & N ? cc : cf);
                    const double a = ads[b][i];
                    const double g = e2m1_value(round_fp4_index(a, s));
                    const double e = a - g * s;
                    key[t] = wds[b][i] * (e * e);
                }
            }
            __syncthreads();
            const int b = tid / 2;
            if (b < KB && blk0 + b < nblocks) {
                double j = 0.0;
                const double* term = key + tid * N;
#pragma unroll 16
                for (int i = 0; i < N; ++i) j = j + term[i];
                const double jc = exchange_other<1>(j);
                if ((tid & 1) == 0) {
                    neighbours(scale_of[b], cf, cc);
                    if (fp8_code) fp8_code[blk0 + b] = (uint8_t)(jc < j ? cc : cf);
                    if (fp8_loss) fp8_loss[blk0 + b] = jc < j ? jc : j;
                }
            }
        }
        __syncthreads();                        // LDS is reused by the next blocks
        kb += kb_step;
        if (kb >= bpr) kb -= bpr;
    }
}

// Exact loss of each block at its given E4M3 scale code: one lane per block.
template <typename In, int N>
__global__ __launch_bounds__(256) void block_loss_kernel(const In* __restrict__ x,
                                                         const float* __restrict__ colw,
                                                         const float* __restrict__ tensor_scale,
                                                         const uint8_t* __restrict__ scales,
                                                         int64_t nblocks, int64_t bpr,
                                                         double* __restrict__ loss) {
    const int64_t blk = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (blk >= nblocks) return;
    const float S = tensor_scale[0];
    const int64_t kb = blk % bpr;
    const int code = scales[blk] > 126 ? 126 : scales[blk];
    const double s = e4m3_f64(code);
    double J = 0.0;
    for (int i = 0; i < N; ++i) {
        const float y = __fdiv_rn(load_elem<In>(x, blk * N + i), S);
        const double a = fabs((double)y);
        const double g = e2m1_value(round_fp4_index(a, s));
        const double e = a - g * s;
        double t = e * e;
        if (colw) t = (double)colw[kb * N + i] * t;
        J = J + t;
    }
    loss[blk] = J;
}

// Deterministic binary64 sum: each of G <= 256 workgroups sums a fixed slice (a strided
// per-thread sum, then a fixed tree), and one wave adds the G partials in a fixed tree.
constexpr int kSumThreads = 256, kSumParts = 256;

__global__ __launch_bounds__(kSumThreads) void sum_partial_kernel(const double* __restrict__ v,
                                                                  int64_t n, double* __restrict__ part) {
    __shared__ double sh[kSumThreads];
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kSumThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kSumThreads)
        acc += v[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int h = kSumThreads / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(kWave) void sum_final_kernel(const double* __restrict__ part, int g,
                                                          double* __restrict__ out) {
    double acc = 0.0;
    for (int i = threadIdx.x; i < g; i += kWave) acc += part[i];
    for (int off = kWave / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
    if (threadIdx.x == 0) out[0] = acc;
}

bool aligned_to(const void* p, uintptr_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

int check_tensor(const void* x, int dtype, int64_t rows, int64_t cols, int block,
                 const float* col_weight, const float* tensor_scale) {
    if (!tensor_scale) return NVFP4_ERR_NULL;
    if (dtype != NVFP4_IN_F32 && dtype != NVFP4_IN_BF16) return NVFP4_ERR_DTYPE;
    if (block != 16 && block != 32 && block != 64 && block != 128) return NVFP4_ERR_BLOCK;
    if (rows < 0 || cols < 0 || cols % block != 0) return NVFP4_ERR_SHAPE;
    if (rows * cols > 0 && !x) return NVFP4_ERR_NULL;
    if (x && !aligned_to(x, dtype == NVFP4_IN_F32 ? 4 : 2)) return NVFP4_ERR_ALIGN;
    if (col_weight && !aligned_to(col_weight, 4)) return NVFP4_ERR_ALIGN;
    return NVFP4_OK;
}

// Up to this many blocks of 16 take a workgroup each instead of sharing one by fours: until the CUs have
// had their 20 waves twice, a batch is a chain of four.  Alone and by fours, bfloat16 with weights: 256
// blocks 6.9 / 16.4 us (binary32 unweighted 6.8 / 16.3), 4096 11.1 / 17.3, 10240 20.4 / 23.3, 16384
// 29.2 / 28.4, 262144 361 / 316.
constexpr int64_t kSingleBlocks = 10240;

template <typename In, int N>
hipError_t launch_optimum(const void* x, const float* colw, const float* S, int64_t nblocks,
                          int64_t bpr, double* opt_loss, double* opt_scale, uint8_t* code,
                          double* fp8_loss, hipStream_t st) {
    const int batch = nblocks <= kSingleBlocks ? 1 : Spread<N>::kBatch;
    const int64_t groups = (nblocks + batch - 1) / batch;
    const int64_t grid = groups < 65536 ? groups : 65536;      // grid-stride over blocks
    hipLaunchKernelGGL((optimum_kernel<In, N>), dim3((unsigned)grid), dim3(Spread<N>::kThreads), 0, st,
                       static_cast<const In*>(x), colw, S, nblocks, bpr, batch, opt_loss, opt_scale,
                       code, fp8_loss);
    return hipGetLastError();
}

template <typename In, int N>
hipError_t launch_loss(const void* x, const float* colw, const float* S, const uint8_t* scales,
                       int64_t nblocks, int64_t bpr, double* loss, hipStream_t st) {
    const int64_t grid = (nblocks + 255) / 256;
    hipLaunchKernelGGL((block_loss_kernel<In, N>), dim3((unsigned)grid), dim3(256), 0, st,
                       static_cast<const In*>(x), colw, S, scales, nblocks, bpr, loss);
    return hipGetLastError();
}

template <typename In>
hipError_t dispatch_optimum(int block, const void* x, const float* colw, const float* S,
                            int64_t nblocks, int64_t bpr, double* l, double* s, uint8_t* c,
                            double* f, hipStream_t st) {
    switch (block) {
        case 16: return launch_optimum<In, 16>(x, colw, S, nblocks, bpr, l, s, c, f, st);
        case 32: return launch_optimum<In, 32>(x, colw, S, nblocks, bpr, l, s, c, f, st);
        case 64: return launch_optimum<In, 64>(x, colw, S, nblocks, bpr, l, s, c, f, st);
        default: return launch_optimum<In, 128>(x, colw, S, nblocks, bpr, l, s, c, f, st);
    }
}

template <typename In>
hipError_t dispatch_loss(int block, const void* x, const float* colw, const float* S,
                         const uint8_t* scales, int64_t nblocks, int64_t bpr, double* loss,
                         hipStream_t st) {
    switch (block) {
        case 16: return launch_loss<In, 16>(x, colw, S, scales, nblocks, bpr, loss, st);
        case 32: return launch_loss<In, 32>(x, colw, S, scales, nblocks, bpr, loss, st);
        case 64: return launch_loss<In, 64>(x, colw, S, scales, nblocks, bpr, loss, st);
        default: return launch_loss<In, 128>(x, colw, S, scales, nblocks, bpr, loss, st);
    }
}

}  // namespace

extern "C" {

int nvfp4_block_optimum(const void* x, int dtype, int64_t rows, int64_t cols, int block,
                        const float* col_weight, const float* tensor_scale, double* opt_loss,
                        double* opt_scale, uint8_t* fp8_code, double* fp8_loss, void* stream) {
    const int rc = check_tensor(x, dtype, rows, cols, block, col_weight, tensor_scale);
    if (rc != NVFP4_OK) return rc;
    const int64_t nblocks = rows * cols / block;
    if (nblocks == 0) return NVFP4_OK;
    if (!opt_loss) return NVFP4_ERR_NULL;
    if (!aligned_to(opt_loss, 8) || (opt_scale && !aligned_to(opt_scale, 8)) ||
        (fp8_loss && !aligned_to(fp8_loss, 8)))
        return NVFP4_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    const hipError_t e = dtype == NVFP4_IN_F32
        ? dispatch_optimum<float>(block, x, col_weight, tensor_scale, nblocks, cols / block,
                                  opt_loss, opt_scale, fp8_code, fp8_loss, st)
        : dispatch_optimum<uint16_t>(block, x, col_weight, tensor_scale, nblocks, cols / block,
                                     opt_loss, opt_scale, fp8_code, fp8_loss, st);
    return e == hipSuccess ? NVFP4_OK : NVFP4_ERR_HIP;
}

int nvfp4_block_loss(const void* x, int dtype, int64_t rows, int64_t cols, int block,
                     const float* col_weight, const float* tensor_scale, const uint8_t* scales,
                     double* loss, void* stream) {
    const int rc = check_tensor(x, dtype, rows, cols, block, col_weight, tensor_scale);
    if (rc != NVFP4_OK) return rc;
    const int64_t nblocks = rows * cols / block;
    if (nblocks == 0) return NVFP4_OK;
    if (!scales || !loss) return NVFP4_ERR_NULL;
    if (!aligned_to(loss, 8)) return NVFP4_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    const hipError_t e = dtype == NVFP4_IN_F32
        ? dispatch_loss<float>(block, x, col_weight, tensor_scale, scales, nblocks, cols / block, loss, st)
        : dispatch_loss<uint16_t>(block, x, col_weight, tensor_scale, scales, nblocks, cols / block, loss, st);
    return e == hipSuccess ? NVFP4_OK : NVFP4_ERR_HIP;
}

size_t nvfp4_sum_workspace_bytes(void) { return kSumParts * sizeof(double); }

int nvfp4_sum_f64(const double* v, int64_t n, double* out, void* workspace,
                  size_t workspace_bytes, void* stream) {
    if (!out) return NVFP4_ERR_NULL;
    if (n < 0) return NVFP4_ERR_SHAPE;
    if (n > 0 && !v) return NVFP4_ERR_NULL;
    if (!workspace || workspace_bytes < kSumParts * sizeof(double)) return NVFP4_ERR_WORKSPACE;
    if (!aligned_to(workspace, 8) || !aligned_to(out, 8) || (v && !aligned_to(v, 8)))
        return NVFP4_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    int64_t g = (n + kSumThreads * 8 - 1) / (kSumThreads * 8);
    if (g < 1) g = 1;
    if (g > kSumParts) g = kSumParts;
    double* part = static_cast<double*>(workspace);
    hipLaunchKernelGGL(sum_partial_kernel, dim3((unsigned)g), dim3(kSumThreads), 0, st, v, n, part);
    if (hipGetLastError() != hipSuccess) return NVFP4_ERR_HIP;
    hipLaunchKernelGGL(sum_final_kernel, dim3(1), dim3(kWave), 0, st, part, (int)g, out);
    return hipGetLastError() == hipSuccess ? NVFP4_OK : NVFP4_ERR_HIP;
}

}  // extern "C"
