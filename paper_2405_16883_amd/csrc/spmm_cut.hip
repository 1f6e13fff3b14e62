// Long rows cut by columns, a range of columns per XCD.
//
// The gathers of a graph's long rows reference all of B, and every XCD has its own L2 of 4 MB: with rows dealt to the XCDs
// whole, each of them reads the often used rows of B for itself and keeps few.  Here XCD x takes, of every long row, the
// entries whose columns lie in the x-th of 8 ranges of columns, so that the 8 L2s hold 8 different parts of B; with B far
// beyond that, a range is divided further (up to 16 parts) and the XCD goes through the parts one after the other, each time over all
// rows that are long enough to have a few entries in one.  Every piece leaves a partial row; a second launch adds them in column order.
//
// The ranges hold equal shares of the stored entries (column histogram).  A piece is a range of entries [p0, p1) found by binary
// search over the row's columns; the pieces of a row cover each of its entries once whatever the columns are (columns out of order or
// other columns at execution only cost reuse).  What bounds it: L2 misses, as without; 2.4 M nodes, 122 M entries, n = 100: 58.3 -> 44.4 GB
// fetched (and 0.9 GB of partial rows written and 1.0 read), 7.95 -> 6.65 ms; an LRU model of the L2s with 512 wavefronts per XCD gives
// 58.4 -> 42.6 GB.  Rows of B are read with the default policy here: with the hot/cold split the cut rows take 4.26 instead of 3.23 ms.
// Pieces of 8 / 16 / 32 entries in the mean: equal / best / 2 % slower.
#include "device_util.h"
#include "spmm_internal.h"

#include <algorithm>
#include <type_traits>

namespace scorch {

struct CutPlanArgs {
    const int32_t *rowptr, *colidx;
    int32_t m, k, nnz;
    int32_t tiles_per_block;
    int32_t finest;  // see cut_class
    int32_t shift;   // columns per histogram bin (log2)
    int64_t cap_pieces;  // room for so many
    int32_t *counts;  // [kCutBuckets][workgroups]
    int32_t *hist;
    CutInfo *info;
    int32_t *rows;
    int2 *spans;
    int32_t max_rows;
    int32_t max_len;  // every row that the plan cuts into pieces of entries is to be cut by columns, or none is
};

// Rows per bucket and workgroup, and the histogram of the columns of the long rows (64 evenly spaced entries of each stand for all).
__global__ __launch_bounds__(kBlock) void cut_count_kernel(const CutPlanArgs a) {
    __shared__ int s_rows[kCutBuckets];
    __shared__ int s_hist[kCutBins];
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i < kCutBins; i += kBlock) s_hist[i] = 0;
    if (tid < kCutBuckets) s_rows[tid] = 0;
    __syncthreads();
    for (int t = 0; t < a.tiles_per_block; ++t) {
        const int64_t i = ((int64_t)blockIdx.x * a.tiles_per_block + t) * kBlock + tid;
        int p0 = 0, len = 0;
        if (i < a.m) {
            p0 = a.rowptr[i];
            len = a.rowptr[i + 1] - p0;
        }
        const bool is_long = len >= kCutMinLen;
        if (is_long) atomicAdd(&s_rows[cut_bucket(len)], 1);
        for (unsigned long long todo = __ballot(is_long); todo != 0ull; todo &= todo - 1ull) {
            const int src = __builtin_ctzll(todo);
            const int q0 = __shfl(p0, src, kWave), n = __shfl(len, src, kWave);
            const int c = a.colidx[q0 + (int)(((int64_t)lane * n) >> 6)];
            if ((uint32_t)c < (uint32_t)a.k) atomicAdd(&s_hist[c >> a.shift], n >> 6);
        }
    }
    __syncthreads();
    if (tid < kCutBuckets) a.counts[tid * (int)gridDim.x + (int)blockIdx.x] = s_rows[tid];
    for (int i = tid; i < kCutBins; i += kBlock)
        if (s_hist[i]) atomicAdd(&a.hist[i], s_hist[i]);
}

// One workgroup: which rows are cut, where their pieces stand, and the ranges of columns.
__global__ __launch_bounds__(kBlock) void cut_layout_kernel(const CutPlanArgs a, int nblk) {
    __shared__ int s_rows[kCutBuckets];
    __shared__ int64_t s_pre[kCutBins + 1];
    __shared__ int64_t s_wave[kWavesPerBlock];
    constexpr int kPer = kCutBins / kBlock;
    const int tid = threadIdx.x;
    if (tid < kCutBuckets) s_rows[tid] = 0;
    __syncthreads();
    for (int i = tid; i < kCutBuckets * nblk; i += kBlock) {
        const int v = a.counts[i];
        if (v) atomicAdd(&s_rows[i / nblk], v);
    }
    int h[kPer];
    int64_t sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        h[i] = a.hist[tid * kPer + i];
        sum += h[i];
    }
    int64_t run = sum;  // of the bins up to and with this thread's
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int64_t o = __shfl_up((long long)run, off, kWave);
        if ((tid & 63) >= off) run += o;
    }
    if ((tid & 63) == kWave - 1) s_wave[tid >> 6] = run;
    __syncthreads();
    int64_t total = 0;
    run -= sum;
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w) {
        if (w < (tid >> 6)) run += s_wave[w];
        total += s_wave[w];
    }
    if (tid == 0) {
        CutInfo c{};
        int rows[kCutBuckets];
        for (int b = 0; b < kCutBuckets; ++b) rows[b] = s_rows[b];
        cut_layout(rows, a.finest, a.cap_pieces, c);
        int64_t entries = 0;  // of the rows that are cut, about
        for (int b = 0; b < kCutBuckets; ++b)
            if (cut_bucket_len(b) >= c.len) entries += (int64_t)rows[b] * cut_bucket_len(b) * 5 / 4;
        if (entries * 20 < a.nnz || c.len > a.max_len) c.len = INT32_MAX;
        if (c.len == INT32_MAX) c.n_rows = c.pieces = 0;
        a.info->len = c.len;
        a.info->pieces = c.pieces;
        a.info->n_rows = c.n_rows;
        a.info->longest = 0;
        a.info->limit = min(4096, max(512, a.nnz / 4096));
        for (int j = 0; j < kCutClasses; ++j) {
            a.info->rows[j] = c.rows[j];
            a.info->row_off[j] = c.row_off[j];
            a.info->piece_off[j] = c.piece_off[j];
        }
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        s_pre[tid * kPer + i] = run;
        run += h[i];
    }
    if (tid == kBlock - 1) s_pre[kCutBins] = run;
    __syncthreads();
    if (tid < kCutBounds) {
        const int64_t target = total * tid / kCutBounds;
        int lo = 0, hi = kCutBins - 1;  // the last bin that starts at or before the target
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_pre[mid] <= target) lo = mid;
            else hi = mid - 1;
        }
        const int64_t in_bin = max((int64_t)1, s_pre[lo + 1] - s_pre[lo]);
        a.info->bound[tid] = tid == 0 ? 0 : (int)(((int64_t)lo << a.shift) + (((target - s_pre[lo]) << a.shift) / in_bin));
    }
}

// Ids of the rows that are cut, class by class, ascending within a class.
__global__ __launch_bounds__(kBlock) void cut_list_kernel(const CutPlanArgs a) {
    __shared__ int s_run[kCutClasses];
    __shared__ int s_wave[kCutClasses][kWavesPerBlock];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int nblk = (int)gridDim.x, blk = (int)blockIdx.x;
    const int32_t cut_len = a.info->len;
    if (cut_len == INT32_MAX) return;
    if (tid < kCutClasses) s_run[tid] = a.info->row_off[tid];
    __syncthreads();
    for (int b = 0; b < kCutBuckets; ++b) {
        if (cut_bucket_len(b) < cut_len) continue;
        int v = 0;
        for (int i = tid; i < blk; i += kBlock) v += a.counts[b * nblk + i];
        if (v) atomicAdd(&s_run[cut_class(b, a.finest)], v);
    }
    __syncthreads();
    for (int t = 0; t < a.tiles_per_block; ++t) {
        const int64_t i = ((int64_t)blk * a.tiles_per_block + t) * kBlock + tid;
        const int len = i < a.m ? a.rowptr[i + 1] - a.rowptr[i] : 0;
        const int cls = len >= cut_len ? cut_class(cut_bucket(len), a.finest) : -1;
        if (!__syncthreads_or(cls >= 0)) continue;
        int rank = 0;
#pragma unroll
        for (int j = 0; j < kCutClasses; ++j) {
            const unsigned long long mask = __ballot(cls == j);
            if (cls == j) rank = (int)__builtin_popcountll(mask & ((1ull << lane) - 1ull));
            if (lane == 0) s_wave[j][wv] = (int)__builtin_popcountll(mask);
        }
        __syncthreads();
        if (cls >= 0) {
            int pos = s_run[cls] + rank;
            for (int w = 0; w < wv; ++w) pos += s_wave[cls][w];
            if (pos < a.max_rows) a.rows[pos] = (int)i;
        }
        __syncthreads();
        if (tid < kCutClasses) s_run[tid] += s_wave[tid][0] + s_wave[tid][1] + s_wave[tid][2] + s_wave[tid][3];
    }
}

// Class of the r-th row that is cut, and its place among the rows of the class.
__device__ __forceinline__ int class_of_row(const CutInfo &c, int r, int &i) {
    int j = kCutClasses - 1;
    while (j > 0 && r >= c.rows[j]) r -= c.rows[j--];
    i = r;
    return j;
}

// Entry ranges of the pieces, one wavefront per row.
__global__ __launch_bounds__(kBlock) void cut_span_kernel(const CutPlanArgs a) {
    const CutInfo &c = *a.info;
    const int lane = threadIdx.x & 63;
    const int n_rows = c.n_rows;
    int longest = 0;
    for (int r = (int)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6); r < n_rows; r += (int)gridDim.x * kWavesPerBlock) {
        int i;
        const int j = class_of_row(c, r, i);
        const int row = a.rows[c.row_off[j] + i];
        const int p0 = a.rowptr[row], p1 = a.rowptr[row + 1];
        const int parts = 1 << j;
        int before = p0;  // end of the pieces so far: the row's entries are covered once even if the columns are in no order
        for (int q0 = 0; q0 < kXcds * parts; q0 += kWave) {
            const int q = q0 + lane;
            int end = p1;
            if (q + 1 < kXcds * parts) {
                const int bound = c.bound[(q + 1) << (kCutClasses - 1 - j)];
                int lo = p0, hi = p1;
                while (lo < hi) {
                    const int mid = lo + ((hi - lo) >> 1);
                    if (a.colidx[mid] < bound) lo = mid + 1;
                    else hi = mid;
                }
                end = lo;
            }
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const int o = __shfl_up(end, off, kWave);
                if (lane >= off) end = max(end, o);
            }
            end = max(end, before);
            int beg = __shfl_up(end, 1, kWave);
            if (lane == 0) beg = before;
            before = __shfl(end, kWave - 1, kWave);
            if (q < kXcds * parts) {
                const int x = q >> j, s = q & (parts - 1);
                const int64_t idx = (int64_t)x * c.pieces + c.piece_off[j] + (int64_t)s * c.rows[j] + i;
                if (idx < a.cap_pieces) a.spans[idx] = make_int2(beg, end);
                longest = max(longest, end - beg);
            }
        }
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) longest = max(longest, __shfl_xor(longest, off, kWave));
    if (lane == 0 && longest > 0) atomicMax(&a.info->longest, longest);
}

scorch_status_t launch_plan_cut(const scorch_spmm_plan_t *plan, const int32_t *rowptr, const int32_t *colidx, PlanResult *result,
                                hipStream_t stream) {
    const WorkspaceLayout &L = plan->layout;
    char *ws = plan->workspace;
    const int64_t tiles = ((int64_t)plan->m + kBlock - 1) / kBlock;
    CutPlanArgs a{};
    a.rowptr = rowptr;
    a.colidx = colidx;
    a.m = plan->m;
    a.k = plan->k;
    a.nnz = (int32_t)plan->nnz;
    a.tiles_per_block = (int32_t)((tiles + kPlanBlocksMax - 1) / kPlanBlocksMax);
    a.finest = plan->params.CUTJ;
    while (((int64_t)(plan->k - 1) >> a.shift) >= kCutBins) ++a.shift;
    a.cap_pieces = L.cap_cut;
    a.counts = reinterpret_cast<int32_t *>(ws + L.off_cut_counts);
    a.hist = reinterpret_cast<int32_t *>(ws + L.off_cut_hist);
    a.info = reinterpret_cast<CutInfo *>(ws + L.off_cut_info);
    a.rows = reinterpret_cast<int32_t *>(ws + L.off_cut_rows);
    a.spans = reinterpret_cast<int2 *>(ws + L.off_cut_spans);
    a.max_len = plan->params.CH + 1;
    a.max_rows = (int32_t)(L.cap_cut / kXcds);
    const uint32_t nblk = (uint32_t)((tiles + a.tiles_per_block - 1) / a.tiles_per_block);
    const uint32_t g = (uint32_t)std::min<int64_t>(std::max<int64_t>(1, (a.max_rows + kWavesPerBlock - 1) / kWavesPerBlock), 256 * 8);
    hipError_t e = hipMemsetAsync(a.hist, 0, kCutBins * 4, stream);
    if (e != hipSuccess) return hip_fail(e, "clear the column histogram");
    hipLaunchKernelGGL(cut_count_kernel, dim3(nblk), dim3(kBlock), 0, stream, a);
    hipLaunchKernelGGL(cut_layout_kernel, dim3(1), dim3(kBlock), 0, stream, a, (int)nblk);
    hipLaunchKernelGGL(cut_list_kernel, dim3(nblk), dim3(kBlock), 0, stream, a);
    hipLaunchKernelGGL(cut_span_kernel, dim3(g), dim3(kBlock), 0, stream, a);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(&result->cut, a.info, sizeof(result->cut), hipMemcpyDeviceToHost, stream);
    if (e != hipSuccess) return hip_fail(e, "launch the kernels that cut rows");
    return SCORCH_OK;
}

// Adds the partial rows of every row that is cut, in column order.  A team of lanes takes a row, up to 16 pieces in flight.
struct CutSumArgs {
    const CutInfo *cut;
    const int32_t *rows;
    const float *partials;
    float *C;
    int64_t ldc;
    int32_t n, stride;
    int32_t team;  // lanes per row, a power of two up to 64
    const float *bias;
    int32_t act;
    bool aligned;
};

__global__ __launch_bounds__(kBlock) void cut_sum_kernel(const CutSumArgs a) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const CutInfo &c = *a.cut;
    const int per_block = kBlock / a.team;
    const int r = (int)blockIdx.x * per_block + (int)threadIdx.x / a.team;
    if (r >= c.n_rows) return;
    int i;
    const int j = class_of_row(c, r, i);
    const int parts = 1 << j;
    const int64_t part_stride = (int64_t)c.rows[j] * a.stride, xcd_stride = (int64_t)c.pieces * a.stride;
    const float *src = a.partials + ((int64_t)c.piece_off[j] + i) * a.stride;
    float *dst = a.C + (int64_t)a.rows[c.row_off[j] + i] * a.ldc;
    for (int col = ((int)threadIdx.x % a.team) * 4; col < a.n; col += a.team * 4) {
        f4 sum = {0.f, 0.f, 0.f, 0.f};
        auto add = [&](auto count, int q0) {
            constexpr int kCount = decltype(count)::value;
            f4 v[kCount];
#pragma unroll
            for (int u = 0; u < kCount; ++u) {
                const int q = q0 + u;
                v[u] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(src + (q >> j) * xcd_stride + (q & (parts - 1)) * part_stride + col));
            }
#pragma unroll
            for (int u = 0; u < kCount; ++u) sum += v[u];
        };
        if (j == 0) add(std::integral_constant<int, kXcds>(), 0);
        else
            for (int q0 = 0; q0 < kXcds * parts; q0 += 2 * kXcds) add(std::integral_constant<int, 2 * kXcds>(), q0);
        if (a.aligned) {
            if (a.bias)
#pragma unroll
                for (int t = 0; t < 4; ++t) sum[t] += a.bias[col + t];
            if (a.act == 1)
#pragma unroll
                for (int t = 0; t < 4; ++t) sum[t] = fmaxf(sum[t], 0.f);
            __builtin_nontemporal_store(sum, reinterpret_cast<f4 *>(dst + col));
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (col + t >= a.n) break;
                float x = sum[t];
                if (a.bias) x += a.bias[col + t];
                if (a.act == 1) x = fmaxf(x, 0.f);
                dst[col + t] = x;
            }
        }
    }
}

scorch_status_t launch_cut_sum(const scorch_spmm_plan_t *plan, float *C, int64_t ldc, const float *bias, int32_t act, hipStream_t stream) {
    const char *ws = plan->workspace;
    CutSumArgs a{};
    a.cut = reinterpret_cast<const CutInfo *>(ws + plan->layout.off_cut_info);
    a.rows = reinterpret_cast<const int32_t *>(ws + plan->layout.off_cut_rows);
    a.partials = reinterpret_cast<const float *>(ws + plan->layout.off_cut_partials);
    a.C = C;
    a.ldc = ldc;
    a.n = plan->n;
    a.stride = plan->layout.partial_stride;
    a.team = 1;
    while (a.team < 64 && a.team * 4 < plan->n) a.team *= 2;
    a.bias = bias;
    a.act = act;
    a.aligned = plan->n % 4 == 0 && ldc % 4 == 0 && reinterpret_cast<uintptr_t>(C) % 16 == 0;
    const int per_block = kBlock / a.team;
    const uint32_t grid = (uint32_t)((plan->cut_rows + per_block - 1) / per_block);
    hipLaunchKernelGGL(cut_sum_kernel, dim3(grid), dim3(kBlock), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "launch cut_sum_kernel");
    return SCORCH_OK;
}

}  // namespace scorch
