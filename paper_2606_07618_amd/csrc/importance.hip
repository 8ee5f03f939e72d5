// Importance vectors for the WMSE objective on AMD Instinct MI355X (gfx950): squared norms
// of input channels (WMSE section; "Quantization" paragraph of the implementation details).
//   * weights W [d_out, d_in]: Imp_j = ||W[:, j]||^2 over the calibration activations X of
//     the layer -- here any matrix whose column norms are wanted;
//   * activations: the squared norms of the consuming weight's input channels;
//   * query states, key cache, value cache: the input-channel squared norms of K, Q and W^O.
// A matrix x [rows, cols] is reduced column-wise into groups of rows: row r belongs to group
// ((r / group_rows) mod groups) / group_div, so attention tensors laid out as
// [batch * heads * tokens, head_dim] reduce per head (group_rows = tokens, groups = heads),
// and group_div merges the query heads that share a KV head.
//
// Pass 1: a wavefront owns 64 adjacent columns of a chunk of rows (256 or more, at most 2048
// chunks); each lane walks its column down the chunk in runs of rows of one group,
// accumulating in binary64 into an LDS accumulator per group, then writes the chunk's
// per-group partial sums.  Pass 2 adds the partials of each
// (group, column) in a fixed order (sixteen contiguous runs of chunks, then the sixteen run
// sums) and rounds once to binary32.  The order is fixed, so results are deterministic.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "nvfp4ss.h"

namespace {

constexpr int kLanes = 64;
constexpr int64_t kMinChunkRows = 256;
constexpr int64_t kMaxChunks = 2048;

// Rows per chunk: at least 256, and few enough chunks that the final pass stays short.
int64_t chunk_rows_for(int64_t rows) {
    const int64_t c = (rows + kMaxChunks - 1) / kMaxChunks;
    return c <= kMinChunkRows ? kMinChunkRows : (c + 7) / 8 * 8;
}
constexpr int kMaxGroups = 64;

// One wavefront per (64 columns, chunk of rows).  The order of the sums is fixed: every column is
// added row by row down its chunk, so one lane walks one column.  What bounds the pass is memory
// (2 or 4 bytes and two binary64 instructions an element), so the loads are kept apart from the
// walk: the wave fetches a tile of 64 (bfloat16) or 32 rows x 64 columns as eight 16-byte loads per lane (a
// row's 64 values are 8 lanes wide in bfloat16, 16 in binary32), always one tile ahead in
// registers, and hands it to the walk through LDS, where runs of any length cost no load latency.
// WIDE needs rows that start on 16 bytes; otherwise each lane loads its own column's values.
// [14336, 4096] bfloat16: 23.9 us, 4.9 TB/s, the rate of a large copy (2-byte loads eight rows at
// a time into the walk, every run's sum added through LDS: 125 us).
constexpr int kTileLoads = 8;
template <typename In>
struct Tile {
    static constexpr int kPer = 16 / sizeof(In);                 // values of a 16-byte load
    static constexpr int kLanesPerRow = kLanes / kPer;
    static constexpr int kRowsPerLoad = kLanes / kLanesPerRow;
    static constexpr int kRows = kTileLoads * kRowsPerLoad;      // 64 bfloat16, 32 binary32
};

__device__ __forceinline__ double widen(float v) { return (double)v; }
__device__ __forceinline__ double widen(uint16_t v) { return (double)__uint_as_float((uint32_t)v << 16); }

template <typename In, bool WIDE>
__global__ __launch_bounds__(kLanes) void norms_partial_kernel(const In* __restrict__ x, int64_t rows,
                                                               int64_t cols, int64_t group_rows,
                                                               int64_t groups, int64_t group_div,
                                                               int gout, int64_t chunk_rows,
                                                               double* __restrict__ part) {
    using T = Tile<In>;
    extern __shared__ double acc_lds[];          // [gout][64]: sized at launch
    double (*acc_g)[kLanes] = reinterpret_cast<double (*)[kLanes]>(acc_lds);
    __shared__ alignas(16) In tile[T::kRows][kLanes];
    const int lane = threadIdx.x;
    const int64_t c0 = (int64_t)blockIdx.x * kLanes;
    const int64_t c = c0 + lane;
    const int64_t r0 = (int64_t)blockIdx.y * chunk_rows;
    const int64_t r1 = r0 + chunk_rows < rows ? r0 + chunk_rows : rows;
    for (int g = 0; g < gout; ++g) acc_g[g][lane] = 0.0;
    // the tile of rows from rt, into registers; rows past r1 and columns past cols read as zero
    const int seg = lane % T::kLanesPerRow, sub = lane / T::kLanesPerRow;
    uint4 wide[kTileLoads];
    In narrow[WIDE ? 1 : T::kRows];
    auto fetch = [&](int64_t rt) {
        if constexpr (WIDE) {                    // cols is a multiple of kPer: a load is in or out
            const int64_t cs = c0 + seg * T::kPer;
#pragma unroll
            for (int k = 0; k < kTileLoads; ++k) {
                const int64_t r = rt + k * T::kRowsPerLoad + sub;
                wide[k] = r < r1 && cs < cols ? *reinterpret_cast<const uint4*>(x + r * cols + cs)
                                              : make_uint4(0u, 0u, 0u, 0u);
            }
        } else {
#pragma unroll
            for (int k = 0; k < T::kRows; ++k) narrow[k] = rt + k < r1 && c < cols ? x[(rt + k) * cols + c] : In(0);
        }
    };
    // rows are walked in runs of one group: r = q * group_rows + rem, and q mod groups =
    // gd * group_div + gm, so a run ends after (group_div - gm) * group_rows - rem rows.  Runs of
    // one row into one group are one run: every square is exact, so adding them to the run or to
    // the group's sum is the same sequence of roundings.
    fetch(r0);
    const int64_t gi = (r0 / group_rows) % groups;
    int gd = (int)(gi / group_div);
    int64_t run_end = r0 + ((group_div - gi % group_div) * group_rows - r0 % group_rows);
    if (gout == 1 && group_div * group_rows == 1) run_end = r1;
    double acc = 0.0, sum_g = 0.0;               // the run's sum; its group's sum before the run
    for (int64_t rt = r0; rt < r1; rt += T::kRows) {
        __syncthreads();                         // one wave: the previous tile is walked
        if constexpr (WIDE) {
#pragma unroll
            for (int k = 0; k < kTileLoads; ++k)
                *reinterpret_cast<uint4*>(&tile[k * T::kRowsPerLoad + sub][seg * T::kPer]) = wide[k];
        } else {
#pragma unroll
            for (int k = 0; k < T::kRows; ++k) tile[k][lane] = narrow[k];
        }
        __syncthreads();
        if (rt + T::kRows < r1) fetch(rt + T::kRows);
        const int m = (int)(r1 - rt < T::kRows ? r1 - rt : T::kRows);
        for (int k = 0; k < m;) {
            const int e = run_end - rt < m ? (int)(run_end - rt) : m;
            for (; k + 8 <= e; k += 8) {
                double v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = widen(tile[k + j][lane]);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc = fma(v[j], v[j], acc);   // v v is exact in binary64
            }
            for (; k < e; ++k) {
                const double v = widen(tile[k][lane]);
                acc = fma(v, v, acc);
            }
            if (rt + k == run_end) {
                acc_g[gd][lane] = sum_g + acc;
                acc = 0.0;
                run_end += group_div * group_rows;
                gd = gd + 1 == gout ? 0 : gd + 1;
                sum_g = acc_g[gd][lane];         // read here, needed at the end of the next run
            }
        }
    }
    acc_g[gd][lane] = sum_g + acc;               // the run that the chunk's end cuts off
    if (c < cols)
        for (int g = 0; g < gout; ++g)
            part[((int64_t)blockIdx.y * gout + g) * cols + c] = acc_g[g][lane];
}

template <typename In>
__device__ __forceinline__ float load_value(const In* x, int64_t i);

template <>
__device__ __forceinline__ float load_value<float>(const float* x, int64_t i) { return x[i]; }

template <>
__device__ __forceinline__ float load_value<uint16_t>(const uint16_t* x, int64_t i) {
    return __uint_as_float((uint32_t)x[i] << 16);
}

// The same sums straight from memory, eight rows of a run at a time: no tile in LDS, so more waves of a
// CU, and a run's additions wait for no second pass through LDS.  prefer_runs says where it is the faster
// form.
template <typename In>
__global__ __launch_bounds__(kLanes) void norms_runs_kernel(const In* __restrict__ x, int64_t rows,
                                                            int64_t cols, int64_t group_rows,
                                                            int64_t groups, int64_t group_div, int gout,
                                                            int64_t chunk_rows, double* __restrict__ part) {
    extern __shared__ double acc_lds[];          // [gout][64]: sized at launch
    double (*acc_g)[kLanes] = reinterpret_cast<double (*)[kLanes]>(acc_lds);
    const int lane = threadIdx.x;
    const int64_t c = (int64_t)blockIdx.x * kLanes + lane;
    const int64_t r0 = (int64_t)blockIdx.y * chunk_rows;
    const int64_t r1 = r0 + chunk_rows < rows ? r0 + chunk_rows : rows;
    for (int g = 0; g < gout; ++g) acc_g[g][lane] = 0.0;
    // rows are walked in runs of one group: r = q * group_rows + rem, and q mod groups =
    // gd * group_div + gm, so a run ends after (group_div - gm) * group_rows - rem rows
    int64_t rem = r0 % group_rows;
    const int64_t gi = (r0 / group_rows) % groups;
    int64_t gm = gi % group_div;
    int gd = (int)(gi / group_div);
    const bool col_ok = c < cols;
    const In* xc = x + (col_ok ? c : 0);
    for (int64_t r = r0; r < r1;) {
        const int64_t run = (group_div - gm) * group_rows - rem;
        const int64_t end = r + run < r1 ? r + run : r1;
        double acc = 0.0;
        int64_t rr = r;
        for (; rr + 8 <= end; rr += 8) {          // eight independent loads in flight
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = load_value<In>(xc, (rr + j) * cols);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc += (double)v[j] * (double)v[j];
        }
        for (; rr < end; ++rr) {
            const double v = (double)load_value<In>(xc, rr * cols);
            acc += v * v;
        }
        if (col_ok) acc_g[gd][lane] += acc;
        r = end;
        rem = 0;
        gm = 0;
        gd = gd + 1 == gout ? 0 : gd + 1;
    }
    if (c < cols)
        for (int g = 0; g < gout; ++g)
            part[((int64_t)blockIdx.y * gout + g) * cols + c] = acc_g[g][lane];
}

// Whether runs straight from memory are the faster form (waves: the grid; run: rows of a run; wide: rows
// start on 16 bytes).  A run takes its rows eight loads at a time and the rest singly, so what it waits for
// is run / 8 + run % 8 latencies; up to a fifth of its rows (8, 16, 17, 25, 33, 40, ...) is few.  So the
// answer also turns on where the input lies: figures are the tiles' time over the runs', cold (inputs that
// no cache holds) and warm (one that the L2s or the memory-side cache hold).
//  * runs of less than eight rows or many loads: 0.36 to 1.0 cold, 0.38 to 1.04 warm;
//  * rows that do not start on 16 bytes, few loads: the tiles' narrow loads take as long as the walk.  16
//    waves 0.96 to 1.3 cold, 1.5 to 1.95 warm; 4096 and more 1.03 to 1.5 and 1.0 to 1.6 (a quarter of the
//    rows, runs of 9, 1.09 to 1.19 and 0.94 to 1.4); a grid whose tiles a CU cannot hold at once 1.2 to
//    1.46; between them 0.74 to 1.0 cold, 1.0 to 1.9 warm, which stays with the tiles;
//  * otherwise 0.37 to 0.98 cold up to 2048 waves, 0.6 to 1.2 warm; 16 waves a CU, which keep the memory
//    busy by themselves, 0.87 to 1.09 and 0.87 to 1.13, of it runs of a smallest chunk and more.
bool prefer_runs(int64_t waves, int64_t run, int64_t gout, bool wide) {
    constexpr int64_t kCus = 256;
    const bool full = waves >= 16 * kCus;
    if (wide) return gout > 1 && run >= kMinChunkRows && full;
    const int64_t loads = run / 8 + run % 8;
    if (run < 8 || (full ? 4 : 5) * loads > run) return false;
    const int64_t tile_bytes = (waves + kCus - 1) / kCus * (8192 + gout * kLanes * (int64_t)sizeof(double));   // a CU's
    return waves <= 64 || full || tile_bytes > 160 * 1024;
}

// One workgroup per (group, 64 columns): 16 waves each add a contiguous sixteenth of the chunk
// partials in order (eight loads in flight), then the sixteen sums are added in order.
constexpr int kFinalSubs = 16;

__global__ __launch_bounds__(kLanes * kFinalSubs) void norms_final_kernel(
        const double* __restrict__ part, int64_t nchunks, int64_t cols, int gout, int64_t rep_out,
        float* __restrict__ out) {
    __shared__ double sub_sum[kFinalSubs][kLanes];
    const int lane = threadIdx.x % kLanes, sub = threadIdx.x / kLanes;
    const int64_t tiles = (cols + kLanes - 1) / kLanes;
    const int64_t g = blockIdx.x / tiles;
    const int64_t c = (blockIdx.x % tiles) * kLanes + lane;
    const int64_t per = (nchunks + kFinalSubs - 1) / kFinalSubs;
    const int64_t k0 = sub * per, k1 = k0 + per < nchunks ? k0 + per : nchunks;
    double s = 0.0;
    if (c < cols) {
        const double* p = part + g * cols + c;
        const int64_t stride = (int64_t)gout * cols;
        int64_t k = k0;
        for (; k + 8 <= k1; k += 8) {
            double v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = p[(k + j) * stride];
#pragma unroll
            for (int j = 0; j < 8; ++j) s += v[j];
        }
        for (; k < k1; ++k) s += p[k * stride];
    }
    sub_sum[sub][lane] = s;
    __syncthreads();
    if (sub == 0 && c < cols) {
        double t = 0.0;
        for (int j = 0; j < kFinalSubs; ++j) t += sub_sum[j][lane];
        const float v = (float)t;
        for (int64_t j = 0; j < rep_out; ++j) out[(g * rep_out + j) * cols + c] = v;
    }
}

int64_t workspace_bytes(int64_t rows, int64_t cols, int64_t groups, int64_t group_div) {
    if (rows < 0 || cols < 0) return NVFP4_ERR_SHAPE;
    if (groups < 1 || group_div < 1 || groups % group_div) return NVFP4_ERR_ARG;
    const int64_t gout = groups / group_div;
    if (gout > kMaxGroups) return NVFP4_ERR_ARG;
    const int64_t cr = chunk_rows_for(rows);
    const int64_t nchunks = (rows + cr - 1) / cr;
    return nchunks * gout * cols * (int64_t)sizeof(double);
}

}  // namespace

extern "C" {

int64_t nvfp4_channel_sq_norms_workspace_bytes(int64_t rows, int64_t cols, int64_t groups,
                                               int64_t group_div) {
    return workspace_bytes(rows, cols, groups, group_div);
}

int nvfp4_channel_sq_norms(const void* x, int dtype, int64_t rows, int64_t cols, int64_t group_rows,
                           int64_t groups, int64_t group_div, int64_t rep_out, float* out,
                           void* workspace, size_t ws_bytes, void* stream) {
    if (dtype != NVFP4_IN_F32 && dtype != NVFP4_IN_BF16) return NVFP4_ERR_DTYPE;
    const int64_t need = workspace_bytes(rows, cols, groups, group_div);
    if (need < 0) return (int)need;
    if (group_rows < 1 || rep_out < 1) return NVFP4_ERR_ARG;
    if (!out) return NVFP4_ERR_NULL;
    const int64_t gout = groups / group_div;
    const int64_t cr = chunk_rows_for(rows);
    const int64_t nchunks = (rows + cr - 1) / cr;
    if ((cols + kLanes - 1) / kLanes > 0x7FFFFFFF) return NVFP4_ERR_SHAPE;
    if (cols == 0) return NVFP4_OK;
    hipStream_t st = (hipStream_t)stream;
    if (rows > 0 && !x) return NVFP4_ERR_NULL;
    if (rows > 0 && (!workspace || (int64_t)ws_bytes < need)) return NVFP4_ERR_WORKSPACE;
    if (((uintptr_t)workspace & 7) || ((uintptr_t)out & 3)) return NVFP4_ERR_ALIGN;
    double* part = static_cast<double*>(workspace);
    const dim3 grid((unsigned)((cols + kLanes - 1) / kLanes), (unsigned)nchunks);
    const size_t lds = (size_t)gout * kLanes * sizeof(double);
    // rows == 0: the final pass alone writes zeros (it reads no partials)
    auto launch = [&](auto kernel, auto* xt) {
        hipLaunchKernelGGL(kernel, grid, dim3(kLanes), lds, st, xt, rows, cols, group_rows, groups, group_div,
                           (int)gout, cr, part);
    };
    const bool wide = ((uintptr_t)x & 15) == 0 && cols * (dtype == NVFP4_IN_F32 ? 4 : 2) % 16 == 0;
    // rows of a run (kMinChunkRows and more: some large number)
    const int64_t run = (group_div < kMinChunkRows ? group_div : kMinChunkRows) *
                        (group_rows < kMinChunkRows ? group_rows : kMinChunkRows);
    const bool runs = prefer_runs((int64_t)grid.x * grid.y, run, gout, wide);
    if (rows > 0 && runs && dtype == NVFP4_IN_F32)
        launch(norms_runs_kernel<float>, static_cast<const float*>(x));
    else if (rows > 0 && runs)
        launch(norms_runs_kernel<uint16_t>, static_cast<const uint16_t*>(x));
    else if (rows > 0 && dtype == NVFP4_IN_F32)
        launch(wide ? norms_partial_kernel<float, true> : norms_partial_kernel<float, false>,
               static_cast<const float*>(x));
    else if (rows > 0)
        launch(wide ? norms_partial_kernel<uint16_t, true> : norms_partial_kernel<uint16_t, false>,
               static_cast<const uint16_t*>(x));
    if (rows > 0 && hipGetLastError() != hipSuccess) return NVFP4_ERR_HIP;
    const int64_t nwg = gout * ((cols + kLanes - 1) / kLanes);
    hipLaunchKernelGGL(norms_final_kernel, dim3((unsigned)nwg), dim3(kLanes * kFinalSubs), 0, st, part,
                       rows > 0 ? nchunks : 0, cols, (int)gout, rep_out, out);
    return hipGetLastError() == hipSuccess ? NVFP4_OK : NVFP4_ERR_HIP;
}

}  // extern "C"
