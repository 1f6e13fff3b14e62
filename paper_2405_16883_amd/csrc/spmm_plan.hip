// Planner: one-time analysis of a CSR sparsity pattern on the device.
//
// The paper's remedy for SpMM cost is CPU-side loop ordering and tiling (Sections 4.1, 4.2); it
// names load balance and irregular access as the open problems of sparse kernels (related-work
// section).  On a GPU the skew of row lengths decides everything, so rows are classed by length
// and handed to different execution paths (see spmm_exec.hip):
//   short  len <= LW       -> windows of consecutive rows, cut along the merge path
//                             key_i = rowptr[i] + ALPHA*i every BN key units
//   wave   LW < len <= CH  -> ascending list of row ids, one wavefront each
//   block  len > CH        -> pieces of at most BCH entries; a row with several pieces gets
//                             consecutive partial-row slots and an entry in the split list
// All lists come out in ascending row order (stable compaction), so the plan is a pure function
// of rowptr and the parameters.
#include "spmm_internal.h"
#include "rowptr_keys.h"

#include <algorithm>
#include <cstdlib>
#include <mutex>

namespace scorch {

constexpr int kQ = 5;  // counted quantities: wave rows, items, split rows, slots, short rows

// Arguments of the two planning kernels.  The number of stored entries is not known on the host when they are launched:
// every workgroup reads it from rowptr[m] and works out the parameters and the workspace layout itself
// (choose_params and layout_workspace are the same code on both sides; what stands behind the lists only the host knows, see
// choose_plan), so that the host waits once, at the end.
struct PlanArgs {
    const int32_t *rowptr;
    int32_t m, k, n;
    Tuning tuning;
    char *workspace;
    uint64_t workspace_bytes;
    int32_t tiles_per_block;  // a workgroup takes this many tiles of kBlock rows
    int32_t counted;          // 1: plan_count_kernel has run; 0: every workgroup counts the rows before its own
    int32_t one_shot;         // see build_plan
    PlanResult *result;       // host memory
};

// a / b for a >= 0, b > 0.  The planning kernels divide 64-bit numbers only where they have to: a division takes a
// wavefront a third of a microsecond.
__host__ __device__ static inline int64_t div_pos(int64_t a, int64_t b) {
    if ((b & (b - 1)) == 0) return a >> __builtin_ctzll((unsigned long long)b);
    if ((((uint64_t)a | (uint64_t)b) >> 32) == 0) return (uint32_t)a / (uint32_t)b;
    return a / b;
}

__host__ __device__ static uint64_t bytes_needed(const WorkspaceLayout &L, bool one_shot);

struct RowClass {
    int wave, items, split, slots, is_short;
};

__device__ __forceinline__ RowClass classify(int len, int LW, int CH, int BCH) {
    RowClass r{0, 0, 0, 0, 0};
    if (len < 0) return r;  // of no class: the host finds a row missing
    if (len <= LW) r.is_short = 1;
    else if (len <= CH) r.wave = 1;
    else {
        r.items = (len + BCH - 1) / BCH;
        if (r.items > 1) {
            r.split = 1;
            r.slots = r.items;
        }
    }
    return r;
}

// Exclusive prefix sum over the 256 threads of a workgroup; `total` is the workgroup sum.
__device__ __forceinline__ int block_exclusive_scan(int v, int &total, int *s_wave /*[4]*/) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int o = __shfl_up(inc, off, kWave);
        if (lane >= off) inc += o;
    }
    __syncthreads();
    if (lane == kWave - 1) s_wave[wv] = inc;
    __syncthreads();
    int base = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w) {
        const int t = s_wave[w];
        if (w < wv) base += t;
        total += t;
    }
    return base + inc - v;
}

// Sums of kQ quantities over the workgroup, returned in every thread.
__device__ __forceinline__ void block_sums(int (&v)[kQ], int (*s_sum)[kQ] /*[4]*/) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1)
#pragma unroll
        for (int k = 0; k < kQ; ++k) v[k] += __shfl_xor(v[k], off, kWave);
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < kQ; ++k) s_sum[threadIdx.x >> 6][k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kQ; ++k) v[k] = s_sum[0][k] + s_sum[1][k] + s_sum[2][k] + s_sum[3][k];
}

// Exclusive prefix sum of a truth value over the workgroup.
__device__ __forceinline__ int block_rank(bool v, int &total, int *s_wave /*[4]*/) {
    const unsigned long long mask = __ballot(v);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) s_wave[wv] = (int)__builtin_popcountll(mask);
    __syncthreads();
    int base = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w) {
        if (w < wv) base += s_wave[w];
        total += s_wave[w];
    }
    return base + (int)__builtin_popcountll(mask & ((1ull << lane) - 1ull));
}

__device__ __forceinline__ void count_row(int (&q)[kQ], int len, const PlanParams &p) {
    const RowClass rc = classify(len, p.LW, p.CH, p.BCH);
    q[0] += rc.wave;
    q[1] += rc.items;
    q[2] += rc.split;
    q[3] += rc.slots;
    q[4] += rc.is_short;
}

// counts[q][b] = quantity q over the rows of workgroup b.
__global__ __launch_bounds__(kBlock) void plan_count_kernel(const PlanArgs a) {
    __shared__ int s_sum[kWavesPerBlock][kQ];
    const int32_t nnz = a.rowptr[a.m];
    if (nnz < 0) return;
    const PlanParams p = choose_params(a.m, a.k, nnz, a.n, a.tuning);
    if (bytes_needed(layout_workspace(a.m, a.k, nnz, a.n, p), a.one_shot) > a.workspace_bytes) return;  // the host reports it
    int32_t *counts = reinterpret_cast<int32_t *>(a.workspace);  // the first section of the layout
    int q[kQ] = {0, 0, 0, 0, 0};
    const int64_t row0 = (int64_t)blockIdx.x * a.tiles_per_block * kBlock + threadIdx.x;
    for (int t = 0; t < a.tiles_per_block; ++t) {
        const int64_t i = row0 + (int64_t)t * kBlock;
        if (i < a.m) count_row(q, a.rowptr[i + 1] - a.rowptr[i], p);
    }
    block_sums(q, s_sum);
    if (threadIdx.x < kQ) {
        int v = q[0];
#pragma unroll
        for (int k = 1; k < kQ; ++k) v = (int)threadIdx.x == k ? q[k] : v;
        counts[(int)threadIdx.x * (int)gridDim.x + (int)blockIdx.x] = v;
    }
}

// Writes every list of the plan, tile of kBlock rows by tile.
//   lists    stable compaction of the row classes (ascending row order): what precedes the workgroup's rows comes from
//            the counts of the workgroups before it, or is counted here when there are few of them
//   windows  win_row_start[w] = number of rows whose key rowptr[i] + ALPHA*i is below w*BN.  A tile owns the windows
//            that start in it; it keeps the row pointers of its rows and of the 64 after them in LDS, and every thread
//            finds the first and the last row of a window there.
//   stages   what a window's wavefront stages in LDS: the entries from the first to the last short row of the window
//            (rows of up to LW entries), at most kStageMax of them, so that the execution kernel can fetch colidx/vals at
//            once instead of waiting for the row pointers first.  (first entry, number of entries), or (0, -1)
//            for a window without short rows.
// Bound by launch and memory latency, hence one kernel for all of it with its first loads issued together.  Lists,
// windows and stages took a launch each before, with a scan in between and for every window a binary search over rowptr
// in global memory: 19 717 rows, 108 000 entries: five kernels of 21 us in all, now two of 12; a coordinate list of that size
// through scorch_coo_to_csr_rowptr and scorch_spmm_csr_static, with two waits before and one now: 80.7 -> 32.1 us.
__global__ __launch_bounds__(kBlock) void plan_build_kernel(const PlanArgs a) {
    __shared__ int s_wave[kWavesPerBlock];
    __shared__ int s_sum[kWavesPerBlock][kQ];
    __shared__ int s_rp[kBlock + kWindowRowsMax + 1];
    const int tid = threadIdx.x;
    const int nblk = (int)gridDim.x, blk = (int)blockIdx.x;
    const bool last_block = blk == nblk - 1;
    const int row_first = blk * a.tiles_per_block * kBlock;  // below m < 2^31 for every workgroup of the grid
    const int32_t *counts = reinterpret_cast<const int32_t *>(a.workspace);
    // everything that does not depend on the parameters is requested at once: the number of entries, the counts of the
    // workgroups before this one, the row pointers of the first tile
    const int32_t nnz = a.m > 0 ? a.rowptr[a.m] : 0;
    int run[kQ] = {0, 0, 0, 0, 0};
    // a workspace that does not even hold the counts is not read; that nothing fits it is found below
    if (a.counted && a.workspace_bytes >= (uint64_t)kQ * nblk * sizeof(int32_t))
        for (int j = tid; j < blk; j += kBlock)
#pragma unroll
            for (int k = 0; k < kQ; ++k) run[k] += counts[k * nblk + j];
    const int32_t rp_first = a.m > 0 ? a.rowptr[min((int64_t)row_first + tid, (int64_t)a.m)] : 0;
    const int32_t rp_first2 = a.m > 0 && tid <= kWindowRowsMax ? a.rowptr[min((int64_t)row_first + kBlock + tid, (int64_t)a.m)] : 0;
    PlanParams p{};
    WorkspaceLayout L{};
    bool fits = nnz >= 0;
    if (fits) {
        p = choose_params(a.m, a.k, nnz, a.n, a.tuning);
        L = layout_workspace(a.m, a.k, nnz, a.n, p);
        fits = bytes_needed(L, a.one_shot) <= a.workspace_bytes;
    }
    if (fits) {
        int32_t *win_row_start = reinterpret_cast<int32_t *>(a.workspace + L.off_win);
        int2 *stage = reinterpret_cast<int2 *>(a.workspace + L.off_stage);
        int32_t *wave_rows = reinterpret_cast<int32_t *>(a.workspace + L.off_wave);
        int2 *wave_span = reinterpret_cast<int2 *>(a.workspace + L.off_wave_span);
        int4 *items = reinterpret_cast<int4 *>(a.workspace + L.off_items);
        int4 *split = reinterpret_cast<int4 *>(a.workspace + L.off_split);
        if (!a.counted) {
#pragma unroll 4
            for (int i = tid; i < row_first; i += kBlock) count_row(run, a.rowptr[i + 1] - a.rowptr[i], p);
        }
        block_sums(run, s_sum);
        for (int t = 0; t < a.tiles_per_block; ++t) {
            const int64_t t0 = (int64_t)row_first + (int64_t)t * kBlock;
            if (t0 >= a.m && !(a.m == 0 && t == 0)) break;
            const int rows = (int)min((int64_t)kBlock, a.m - t0);  // 0 only for an empty matrix
            __syncthreads();  // s_rp of the previous tile has been read
            if (t == 0) {
                s_rp[tid] = rp_first;
                if (tid <= kWindowRowsMax) s_rp[kBlock + tid] = rp_first2;
            } else {
                for (int i = tid; i < kBlock + kWindowRowsMax + 1; i += kBlock) s_rp[i] = a.rowptr[min(t0 + i, (int64_t)a.m)];
            }
            const int before = t0 > 0 ? a.rowptr[t0 - 1] : 0;
            __syncthreads();
            // ---- lists ----
            RowClass rc{0, 0, 0, 0, 0};
            int p0 = 0, p1 = 0;
            if (tid < rows) {
                p0 = s_rp[tid];
                p1 = s_rp[tid + 1];
                rc = classify(p1 - p0, p.LW, p.CH, p.BCH);
            }
            int total;
            const int pos_wave = run[0] + block_rank(rc.wave, total, s_wave);
            run[0] += total;
            int pos_item = 0, pos_split = 0, pos_slot = 0;
            if (__syncthreads_or(rc.items)) {  // few tiles hold a long row
                pos_item = run[1] + block_exclusive_scan(rc.items, total, s_wave);
                run[1] += total;
                pos_split = run[2] + block_rank(rc.split, total, s_wave);
                run[2] += total;
                pos_slot = run[3] + block_exclusive_scan(rc.slots, total, s_wave);
                run[3] += total;
            }
            (void)block_rank(rc.is_short, total, s_wave);
            run[4] += total;
            // The capacities hold for every valid rowptr; the guards only keep a malformed one in bounds
            // (the host then reports the overflow from the totals).
            if (rc.wave && pos_wave < L.cap_wave) {
                wave_rows[pos_wave] = (int)t0 + tid;
                wave_span[pos_wave] = make_int2(p0, p1);
            }
            for (int c = 0; c < rc.items && (int64_t)pos_item + c < L.cap_items; ++c) {
                const int b = p0 + c * p.BCH;
                items[pos_item + c] = make_int4((int)t0 + tid, b, min(p1, b + p.BCH), rc.split ? pos_slot + c : -1);
            }
            if (rc.split && pos_split < L.cap_split) split[pos_split] = make_int4((int)t0 + tid, pos_slot, rc.items, 0);
            // ---- windows that start in this tile (the last tile also owns those that start past the last row) ----
            auto key = [&](int j) { return (int64_t)s_rp[j] + (int64_t)p.ALPHA * (t0 + j); };
            const bool last_tile = t0 + rows >= a.m;
            const int own = last_tile ? rows : rows - 1;  // index of the last row (or of the end) that this tile owns
            const int64_t w_lo = t0 > 0 ? max((int64_t)0, div_pos(max((int64_t)0, (int64_t)before + (int64_t)p.ALPHA * (t0 - 1)), p.BN) + 1) : 0;
            const int64_t w_hi = min(L.n_windows - 1, div_pos(max((int64_t)0, key(own)), p.BN));
            for (int64_t w = w_lo + tid; w <= w_hi; w += kBlock) {
                int lo = 0, hi = own;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (key(mid) < w * p.BN) lo = mid + 1;
                    else hi = mid;
                }
                const int r0 = lo;
                win_row_start[w] = (int)(t0 + r0);
                hi = (int)min((int64_t)r0 + kWindowRowsMax, a.m - t0);  // a window holds at most kWindowRowsMax rows
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (key(mid) < (w + 1) * p.BN) lo = mid + 1;
                    else hi = mid;
                }
                int sbeg = 0, send = -1;
                for (int r = r0, prev = s_rp[r0]; r < lo; ++r) {
                    const int next = s_rp[r + 1];
                    if (next - prev <= p.LW) {
                        if (send < 0) sbeg = prev;
                        send = next;
                    }
                    prev = next;
                }
                stage[w] = send < 0 ? make_int2(0, -1) : make_int2(sbeg, min(send - sbeg, kStageMax));
            }
            if (last_tile && tid == 0) win_row_start[L.n_windows] = a.m;
        }
    }
    if (last_block && tid == 0) {
        if (fits) *reinterpret_cast<int32_t *>(a.workspace + L.off_totals) = 0;  // for the kernels that look at the columns
        a.result->nnz = nnz;
#pragma unroll
        for (int k = 0; k < kQ; ++k) a.result->totals[k] = run[k];
        __hip_atomic_store(&a.result->done, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Sets *unsorted (host memory) when some row's column indices are not strictly increasing (one wavefront per row).
__global__ __launch_bounds__(kBlock) void plan_sorted_kernel(const int32_t *rowptr, const int32_t *colidx, int32_t m,
                                                             int32_t *seen, int32_t *unsorted) {
    const int lane = threadIdx.x & 63;
    for (int64_t row = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6); row < m;
         row += (int64_t)gridDim.x * kWavesPerBlock) {
        const int p0 = rowptr[row], p1 = rowptr[row + 1];
        bool bad = false;
        for (int p = p0 + 1 + lane; p < p1; p += kWave) bad |= colidx[p] <= colidx[p - 1];
        if (report_unsorted(bad, seen, unsorted)) break;
    }
}

// ---- hot columns ------------------------------------------------------------------------------------------
// When B is larger than the memory-side cache, the gathers of the rarely referenced rows of B stream through that
// cache and evict the often referenced ones.  The planner therefore counts how often every column of A occurs,
// marks the most referenced columns up to a byte budget as hot (one bit per column), and the kernels read only
// those rows of B with the default cache policy and all others with the streaming (nt) policy, which on this
// hardware leaves the memory-side cache alone.

// deg[c] = number of sampled stored entries with column c.  One entry is taken out of every `stride` consecutive
// ones (stride a power of two; 1 = all entries), at a position that varies from one group of entries to the next:
// a fixed position would always pick the same rank within rows of a regular length, i.e. always low or always high
// columns.  The count only ranks the columns for a cache policy, so a sample serves; the atomic additions (one
// 32-byte memory transaction each) are what the planner spends most of its time on for a large matrix.
__global__ __launch_bounds__(kBlock) void plan_coldeg_kernel(const int32_t *colidx, int64_t nnz, int32_t k,
                                                             int32_t stride, int32_t *deg) {
    const int64_t groups = (nnz + stride - 1) / stride;
    for (int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x; g < groups; g += (int64_t)gridDim.x * kBlock) {
        const int64_t p = g * stride + (int64_t)((((uint32_t)g * 2654435761u) >> 16) & (uint32_t)(stride - 1));
        if (p >= nnz) continue;
        const int c = colidx[p];
        if ((uint32_t)c < (uint32_t)k) atomicAdd(&deg[c], 1);
    }
}

// Histogram bin of a degree: 16 bins per power of two, monotone in d; bin 0 holds d = 0.
__host__ __device__ __forceinline__ int degree_bin(int d) {
    if (d <= 0) return 0;
    const int e = 31 - __builtin_clz((unsigned)d);
    const int frac = e >= 4 ? (d >> (e - 4)) & 15 : (d << (4 - e)) & 15;
    return e * 16 + frac + 1;
}

// bins[b] = (number of columns, number of stored entries) whose degree falls into bin b.  Counted per workgroup
// in LDS first: nearly all columns of a graph fall into a handful of bins.
__global__ __launch_bounds__(kBlock) void plan_degbins_kernel(const int32_t *deg, int32_t k, unsigned long long *bins) {
    __shared__ unsigned int s_cnt[kDegBins], s_sum[kDegBins];  // a workgroup sees fewer than 2^31 entries in total
    for (int b = threadIdx.x; b < kDegBins; b += kBlock) {
        s_cnt[b] = 0;
        s_sum[b] = 0;
    }
    __syncthreads();
    for (int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x; c < k; c += (int64_t)gridDim.x * kBlock) {
        const int d = deg[c];
        const int b = degree_bin(d);
        atomicAdd(&s_cnt[b], 1u);
        atomicAdd(&s_sum[b], (unsigned int)d);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kDegBins; b += kBlock) {
        if (s_cnt[b]) {
            atomicAdd(&bins[2 * b], (unsigned long long)s_cnt[b]);
            atomicAdd(&bins[2 * b + 1], (unsigned long long)s_sum[b]);
        }
    }
}

// mask word w holds the hot bits of columns 32w .. 32w+31: hot = degree bin >= min_bin.
__global__ __launch_bounds__(kBlock) void plan_hotmask_kernel(const int32_t *deg, int32_t k, int min_bin, int64_t nwords,
                                                              uint32_t *mask) {
    for (int64_t w = (int64_t)blockIdx.x * kBlock + threadIdx.x; w < nwords; w += (int64_t)gridDim.x * kBlock) {
        uint32_t bits = 0;
        for (int i = 0; i < 32; ++i) {
            const int64_t c = w * 32 + i;
            if (c < k && degree_bin(deg[c]) >= min_bin) bits |= 1u << i;
        }
        mask[w] = bits;
    }
}

static scorch_status_t mark_hot_columns(scorch_spmm_plan_t *plan, const int32_t *colidx, bool forced, bool one_shot,
                                        hipStream_t stream) {
    const WorkspaceLayout &L = plan->layout;
    char *ws = plan->workspace;
    int32_t *deg = reinterpret_cast<int32_t *>(ws + L.off_coldeg);
    uint32_t *mask = reinterpret_cast<uint32_t *>(ws + L.off_hotmask);
    unsigned long long *bins = reinterpret_cast<unsigned long long *>(ws + L.off_degbins);
    hipError_t e = hipMemsetAsync(deg, 0, (size_t)plan->k * 4, stream);
    if (e == hipSuccess) e = hipMemsetAsync(bins, 0, (size_t)kDegBins * 16, stream);
    if (e != hipSuccess) return hip_fail(e, "clear column degrees");
    // every entry up to 2^24 of them, beyond that every 2nd, 4th, ... so that at most 2^24 are counted
    int32_t stride = 1;
    while ((plan->nnz + stride - 1) / stride > kHotSampleMax) stride *= 2;
    const int64_t groups = (plan->nnz + stride - 1) / stride;
    const uint32_t g1 = (uint32_t)std::min<int64_t>((groups + kBlock - 1) / kBlock, 256 * 64);
    const uint32_t g2 = (uint32_t)std::min<int64_t>(((int64_t)plan->k + kBlock - 1) / kBlock, 256 * 4);
    hipLaunchKernelGGL(plan_coldeg_kernel, dim3(g1), dim3(kBlock), 0, stream, colidx, plan->nnz, plan->k, stride, deg);
    hipLaunchKernelGGL(plan_degbins_kernel, dim3(g2), dim3(kBlock), 0, stream, deg, plan->k, bins);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "launch column-degree kernels");
    static_assert(sizeof(unsigned long long) == 8, "bin layout");
    unsigned long long host_bins[2 * kDegBins];
    e = hipMemcpyAsync(host_bins, bins, sizeof(host_bins), hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return hip_fail(e, "read the column-degree histogram");
    // a row of B occupies whole 128-byte lines in the caches
    const int64_t row_bytes = ((int64_t)plan->n * 4 + 127) / 128 * 128;
    const int64_t max_rows = std::max<int64_t>(1, (int64_t)plan->params.HOT * 1024 / row_bytes);
    int64_t rows = 0, entries = 0;
    int min_bin = kDegBins;
    for (int b = kDegBins - 1; b >= 1; --b) {  // bin 0: columns that never occur
        if (rows + (int64_t)host_bins[2 * b] > max_rows) break;
        rows += (int64_t)host_bins[2 * b];
        entries += (int64_t)host_bins[2 * b + 1];
        min_bin = b;
    }
    plan->n_hot = 0;
    plan->hot_share = groups > 0 ? (float)std::min(1.0, (double)entries / (double)groups) : 0.f;  // of the sampled entries
    // Worth it only when a small part of B takes a large part of the gathers (measured on the large power-law
    // workload: 5 % of the rows of B, 54 % of the gathers, 6.5 % less time).
    if (rows == 0 || (!forced && plan->hot_share < 0.25f)) return SCORCH_OK;
    const int64_t nwords = (int64_t)plan->k / 32 + 1;
    const uint32_t g3 = (uint32_t)std::min<int64_t>((nwords + kBlock - 1) / kBlock, 256 * 16);
    hipLaunchKernelGGL(plan_hotmask_kernel, dim3(g3), dim3(kBlock), 0, stream, deg, plan->k, min_bin, nwords, mask);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "launch plan_hotmask_kernel");
    if (!one_shot && (e = hipStreamSynchronize(stream)) != hipSuccess) return hip_fail(e, "wait for plan_hotmask_kernel");
    plan->n_hot = (int32_t)std::min<int64_t>(rows, 0x7fffffff);
    return SCORCH_OK;
}

// Row pointers from a sorted list of row keys.  Coordinate list: keys are the row coordinates of the entries and
// position p itself is the pointer (pos == nullptr).  Doubly compressed rows: keys are the ids of the stored rows
// and pos[p] is where row keys[p] starts (pos[count] = nnz).  Key p closes the rows between its predecessor and
// itself: rowptr[r] = pos[p] for keys[p-1] < r <= keys[p]; the sentinel p = count closes the rows up to m.
__global__ __launch_bounds__(kBlock) void rowptr_from_keys_kernel(const int32_t *keys, const int32_t *pos, int64_t count,
                                                                  int32_t m, bool strictly_increasing, int32_t *rowptr,
                                                                  int32_t *bad_flag) {
    for (int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x; p <= count; p += (int64_t)gridDim.x * kBlock) {
        const int prev = p > 0 ? keys[p - 1] : -1;
        const int cur = p < count ? keys[p] : m;
        int32_t lo, hi;
        if (!rowptr_fill_range(p, count, prev, cur, m, strictly_increasing, lo, hi)) {
            if (bad_flag) *bad_flag = 1;
            continue;
        }
        const int32_t value = pos ? pos[p] : (int32_t)p;
        for (int r = lo; r <= hi; ++r) rowptr[r] = value;  // 0 <= lo, hi <= m
    }
}

scorch_status_t launch_rowptr_from_keys(int32_t m, int64_t count, const int32_t *keys, const int32_t *pos,
                                        bool strictly_increasing, int32_t *rowptr, int32_t *bad_flag,
                                        hipStream_t stream) {
    const uint32_t grid = (uint32_t)std::min<int64_t>((count + 1 + kBlock - 1) / kBlock, 256 * 32);
    hipLaunchKernelGGL(rowptr_from_keys_kernel, dim3(grid), dim3(kBlock), 0, stream, keys, pos, count, m,
                       strictly_increasing, rowptr, bad_flag);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "launch rowptr_from_keys_kernel");
    return SCORCH_OK;
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
Tuning read_tuning_from_env() { return parse_tuning(std::getenv("SCORCH_SPMM_TUNE")); }

// largest power of two that is at most x (1 <= x), 2^30 at most
__host__ __device__ static int32_t pow2_floor(int64_t x) {
    return 1 << (63 - __builtin_clzll((unsigned long long)(x < (1ll << 30) ? x : (1ll << 30))));
}

// XCD-sliced execution pays when B as a whole overflows an XCD's 4 MB L2 at least twice over but a 128-byte-wide
// column slice of it fits, and rows are long enough that re-reading colidx/vals and walking the row once per slice
// is cheap next to the gathers (8 bytes of A against 128 bytes of B per entry and slice).  Measured on uniform random
// patterns: 164 entries per row, B 8-32 MB: 1.3-2.1x faster than the plain gather; 82 entries, B 8-33 MB: 1.0-1.5x;
// 65 entries: even; 33-41 entries: 1.2-1.4x slower; B of 4 MB (mostly L2-resident anyway): 1.1-1.3x slower.
// Beyond that: the 128-byte slices still win over whole rows when a slice is a few times larger than an XCD's L2
// (uniform patterns and a power-law graph with 100-164 entries per row, slices of 4-13 MB: 1.1-2.3x faster; a
// 17 MB slice: 1.1x slower), and with shorter rows 256-byte slices do (an XCD's L2 then keeps twice to sixteen times
// as many rows of B as with whole rows, and a wavefront has 4 rows of B in flight per load): power-law graphs of
// 50 k to 1 M nodes, 5 to 100 entries per row, n = 128 to 1024 in multiples of 64: 5-30 % less time than whole rows
// (one case of 21: 1 %); uniform and pruned patterns outside the 128-byte rule: 0-43 % less; n = 160: 0-16 % less;
// n = 96, 100, 132: 4-30 % more, hence the multiple of 64.  Returns the columns per slice (0 = whole rows).
__host__ __device__ static int32_t want_sliced(int32_t m, int32_t k, int64_t nnz, int32_t n, bool hot_candidate) {
    if (m <= 0 || n % 4 != 0 || n < 2 * kSliceCols) return 0;
    const int64_t slice_bytes = (int64_t)k * kSliceCols * 4;
    const int64_t b_bytes = (int64_t)k * n * 4;
    const bool long_rows = nnz >= 64 * (int64_t)m && b_bytes >= 8ll << 20;
    if (long_rows && slice_bytes <= kL2SliceBudget) return kSliceCols;
    if (hot_candidate) return 0;  // the hot/cold split needs whole rows
    if (long_rows && slice_bytes <= 13ll << 20 && n >= 128) return kSliceCols;  // n = 64 with a 13 MB slice: 2-6 % more time
    // B of 6 MB (1.5 L2s), 410 entries per row, n = 384: 19 % less time with 256-byte slices; B of 4 MB: 23 % more
    return (n >= 128 && n % 64 == 0 && b_bytes >= 6ll << 20) ? 64 : 0;
}

// The panel kernel (spmm_panel.hip) streams all of B through LDS once per block of 64 rows of A, a cost that does
// not depend on nnz, and then pays per entry less than the gather kernels.  It needs a workgroup (64 rows x 512 or
// 256 columns) for every CU.  From sweeps over unstructured-pruned shapes (4096..65536 rows, k 2048..16384):
//   wide tiles (n >= 512): ahead of the gather kernels from 3 % stored entries upwards (3 %: 0.70 against 0.73 ms,
//     4 %: 0.39 against 0.47, 6 %: 0.48 against 0.70, 10 %: 0.65 against 1.12), behind with fewer than 256 workgroups;
//   narrow tiles: about even with the gather kernels at 10 % (0.50 against 0.52 ms, 0.54 against 0.62), behind at
//     4-8 %; used from 10 % upwards when only they give 256 workgroups.
// Returns the kernel shape (0 = do not use, 1 = 256-column tiles, 2 = 512-column tiles).
__host__ __device__ static int32_t want_panel(int32_t m, int32_t k, int64_t nnz, int32_t n) {
    if (m <= 0 || k < 1024 || n % 4 != 0 || n < kPanelCols || nnz < 128 * (int64_t)m) return 0;
    const double density = (double)nnz / ((double)m * (double)k);
    const int64_t row_blocks = ((int64_t)m + 63) / 64;
    if (n >= 2 * kPanelCols && density >= 0.03 && row_blocks * ((n + 2 * kPanelCols - 1) / (2 * kPanelCols)) >= 256) return 2;
    // 256-column tiles: from 7.5 % stored entries upwards, counted per tile column actually used (a last tile that is
    // half empty costs as much as a full one).  Measured on pruned-weight shapes with n = 256, 384, 4096: at 8 % the
    // panel kernel is 0-23 % faster than the gathers, at 10 % 0-30 %, at 6 % between 10 % faster and 20 % slower.
    const int64_t tiles1 = (n + kPanelCols - 1) / kPanelCols;
    if (density * (double)n / (double)(tiles1 * kPanelCols) >= 0.075 && row_blocks * tiles1 >= 256) return 1;
    return 0;
}

// Columns a row of B is padded to in LDS by the resident kernel (spmm_resident.hip).
__host__ __device__ static int32_t resident_width(int32_t n) {
    return n <= 4 ? 4 : 1 << (32 - __builtin_clz((unsigned)(n - 1)));
}

// The resident kernel against the gather kernels, for at most 64 columns: both times as fitted to sweeps over m = 1024 ...
// 16 384, k = 1024 ... 16 384, 1 ... 50 % stored, n = 1 ... 64, in units of 0.1 ps (integers: host and device have to
// decide alike).  Gathers: 2.3 ps (n = 1) to 11 ps (n = 64) per entry.  Resident: 2 to 3 ps per entry, but at least
// 1.2 us per row and chunk that a wavefront goes through (4096 wavefronts), 4 us to fill LDS, and the second launch over the partial
// rows.  Measured, gather / resident in us, 4096 x 16 384 with 10 % stored: n = 4 25.0 / 19.8, 8 38.8 / 21.6, 16 42.0 / 21.5,
// 32 45.9 / 33.4, 64 78.4 / 53.0; with 1 %: 5.0 / 7.6, 5.3 / 9.7, 5.6 / 13.0, 5.9 / 24.8, 10.8 / 34.1; 16 384 x 4096 with 26 %: n = 16
// 72.3 / 43.3, n = 64 153 / 80.
__host__ __device__ static int32_t want_resident(int32_t m, int32_t k, int64_t nnz, int32_t n) {
    if (m <= 0 || k <= 0 || n < 3 || n > 64) return 0;
    const int32_t W = resident_width(n);
    // as below, without a division: the planning kernels evaluate this, and most matrices end here (both sides alike in float64)
    if ((double)m * k * W > (double)nnz * kResidentFloats) return 0;
    const int64_t chunks = resident_chunks(k, W);
    if ((int64_t)m * chunks > nnz) return 0;  // never pays: a row of a chunk costs 2930, an entry saves 110 at most (and the rest fits 64 bits)
    const int64_t per_entry = n > 32 ? 110 : n % 4 != 0 ? 75 : n > 8 ? 57 : n > 4 ? 50 : 35;
    const int64_t entries = nnz * (W > 32 ? 30 : W > 16 ? 26 : 20), rows = (int64_t)m * chunks * 2930;
    int64_t resident = 40000000 + (entries > rows ? entries : rows);
    if (chunks > 1) resident += 30000000 + (int64_t)m * chunks * W * 27;
    return resident * 10 < nnz * per_entry * 9 ? W : 0;
}

// Chunks of the resident kernel: no fewer than B needs, and as many as make the longest wavefront's work shortest.  Every chunk has as many
// blocks of rows as let all workgroups run at once, and a wavefront of a block takes whole rows, so a few rows more than a multiple
// of 16 cost as much as 16.  In ns, as fitted for want_resident: 8 per entry of a row's chunk and 400 per row and chunk of a wavefront; 2.7 per
// 1000 floats of partial rows.  4096 x 16 384 with 10 % stored, n = 16: seven chunks, the last half full, 8 rows of 253 entries per wavefront;
// eight even ones, 8 rows of 205.
static int32_t resident_balance(int32_t m, int32_t k, int64_t nnz, int32_t W) {
    const int32_t fewest = resident_chunks(k, W);
    if (fewest == 1) return 1;  // no partial rows, no second launch
    int32_t best = fewest;
    int64_t best_cost = INT64_MAX;
    for (int32_t c = fewest; c <= fewest + 8; ++c) {
        const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>(kCus / c, ((int64_t)m + 15) / 16));
        const int64_t rows = (((int64_t)m + blocks - 1) / blocks + 15) / 16;
        const int64_t rounds = (blocks * c + kCus - 1) / kCus;
        const int64_t cost = rounds * rows * (8 * (nnz / ((int64_t)m * c)) + 400) + (int64_t)m * c * W / 1000 * 27 / 10;
        if (cost < best_cost) {
            best_cost = cost;
            best = c;
        }
    }
    return best;
}

constexpr int64_t kCutNnzMin = 1 << 20;

// Cutting long rows by columns (spmm_cut.hip) pays where B is as large as the 8 L2s (32 MB) together, a row of it is more than one
// 128-byte line, and the gathers are more than the second launch's 4 us.  Not where a smaller plan would do (see layout_workspace).
// Measured whole / cut, us, and what the plan takes longer: graph of 2.4 M nodes, degree 50, n = 100 7954 / 6673 (0.6 ms); 1 M, 50, n = 64
// 1687 / 1345 (0.4); 300 000, 50, n = 100 952 / 708 (0.35); 600 000, 30, n = 100 1178 / 970 (0.35); 2.4 M, 20, n = 33 1556 / 1341 (0.4); 2.4 M, 10,
// n = 64 849 / 794 (0.35); no row of 128 entries 0.06 ms for nothing.  Rows that are all long, where neither slices (n not a multiple of 4) nor
// panels serve: 4096 x 16 384, 10 % stored, n = 1001 3026 / 1124 (0.13); 10 000 x 40 000, 3 %, n = 229 1678 / 501 (0.3); from 8 MB on where the mean
// row leaves 40 entries for a piece: 8000 x 16 384, 5 %, n = 333 975 / 415 (0.27); 16 384 x 2000, 30 %, n = 1501 2411 / 2210 (0.3); 1500 x 8000, 30 %,
// n = 1001 1561 / 541 (0.07); with less, rows of 164, n = 129 (8 MB) 95 / 109.  B below 8 MB can gain too (3000 x 12 000, 10 %, n = 101, 4.8 MB 122 / 73) but is
// left alone: such plans are small.  Not: n = 32, 169 343 rows (21 MB) 39.8 / 46.2, 2.4 M nodes of degree 3 212 / 225; 1.3 M entries, n = 64 41.1 / 43.7;
// with 32-column slices (SLICED = 32) 121 / 145.
static bool want_cut(int32_t m, int32_t k, int64_t nnz, int32_t n, int32_t sliced) {
    const int64_t b_bytes = (int64_t)k * n * 4;
    return n > 32 && nnz * n >= 100000000 && (sliced == 0 || sliced == 64) &&
           (b_bytes >= 32ll << 20 || (b_bytes >= 8ll << 20 && nnz >= kCutAllLong * (int64_t)m));
}

// Bytes that a plan cannot do without.
__host__ __device__ static uint64_t bytes_needed(const WorkspaceLayout &L, bool one_shot) {
    return one_shot ? L.one_shot : L.without_cut;
}

// Rows of A whose partial rows fit at a time, and where they stand (`off`), in a workspace of `bytes` that only a one-shot plan
// uses: behind everything else, or over the lists of the gather kernels, which the resident kernel does not read.
static int32_t partial_rows_in(const WorkspaceLayout &L, int32_t m, uint64_t bytes, uint64_t &off) {
    off = L.off_res_partials;
    uint64_t room = bytes - off;
    if (room < L.res_row_bytes * m && room < L.off_res_ptr) {
        off = 0;
        room = L.off_res_ptr;
    }
    return room >= L.res_row_bytes * m ? m : (int32_t)(room / L.res_row_bytes);
}

__host__ __device__ PlanParams choose_params(int32_t m, int32_t k, int64_t nnz, int32_t n, const Tuning &t) {
    PlanParams p;
    p.ALPHA = 4;
    // Windows of 128 key units, but small problems get smaller windows so that there are a few thousand
    // wavefronts' worth of them (a lane group walks its rows one after the other, each a full memory latency).
    // Narrow B (n <= 32) means 8 or more lane groups per wavefront, each walking one row of the window (for n <= 4
    // the lanes split the window's entries): larger windows keep more of them busy.
    const int32_t bn_cap = n <= 32 ? kBNMax : 128;
    p.BN = std::min<int32_t>(bn_cap, std::max<int32_t>(16, pow2_floor(std::max<int64_t>(1, (nnz + (int64_t)p.ALPHA * m) / 4096))));
    p.LW = 32;
    // B several times larger than the memory-side cache: see build_plan (hot columns).
    const bool hot_candidate = (int64_t)k * n * 4 > 3 * kMallBytes && n >= 96 && nnz >= 4 * (int64_t)k;
    p.SLICED = want_sliced(m, k, nnz, n, hot_candidate);
    if (t.sliced >= 0) {  // 0: off, 1: the default width, 32 / 64 / 128: that many columns per slice
        const int32_t cols = t.sliced == 1 ? kSliceCols : t.sliced;
        p.SLICED = ((cols == 32 || cols == 64 || cols == 128) && n % 4 == 0) ? cols : 0;
    }
    // A row stride of B above 512 bytes scatters a 128-byte column slice over few L2 sets; gather from a
    // dense slice-major copy instead (costs one read and one write of B per call).
    p.PACK = (p.SLICED == kSliceCols && n > 128) ? 1 : 0;
    if (t.pack >= 0) p.PACK = (p.SLICED == kSliceCols && t.pack != 0) ? 1 : 0;
    p.PANEL = want_panel(m, k, nnz, n);
    if (t.panel >= 0) p.PANEL = (t.panel > 0 && t.panel <= 3 && n % 4 == 0 && k > 0) ? t.panel : 0;
    // The panel kernel fetches its panels straight from the caller's row-major B (pruned-FFN workload, row stride 8 KB:
    // 1.10 against 1.13 ms with a tile-major copy made at every call, which costs one read and one write of B; the
    // workgroups of a tile column walk the same panels at the same time, so only a few panels per die have to stay in
    // L2 and the set conflicts of a power-of-two stride do not matter); pack=1 brings the copy back.
    p.PDIRECT = (p.PANEL && (t.pack != 1 || p.PANEL == 3)) ? 1 : 0;
    p.RES = p.PANEL == 0 ? want_resident(m, k, nnz, n) : 0;
    if (t.res >= 0) p.RES = (t.res > 0 && n <= 64 && k > 0 && m > 0 && p.PANEL == 0) ? resident_width(n) : 0;
    // Enough independent wavefront tasks to fill 256 CUs several times over, but pieces long
    // enough that the per-piece overhead stays small.
    const int64_t coltiles = p.SLICED ? (n + p.SLICED - 1) / p.SLICED : std::max<int64_t>(1, (n + 511) / 512);
    const int32_t ch_cap = p.SLICED ? 4096 : 1024;
    p.CH = std::min<int32_t>(ch_cap, std::max<int32_t>(256, pow2_floor(std::max<int64_t>(1, nnz * coltiles / 32768))));
    p.U = 8;
    p.NT = 1;
    // B several times larger than the memory-side cache: see build_plan (hot columns).  Budget: a quarter of that
    // cache.  Measured on the large power-law pattern: B 3.8x / 4.9x / 9.8x the cache: 5-6 % less time; 2.4x: 4 % more;
    // 1.2x: 57 % more (the cache then holds most of B anyway and the streaming policy forfeits that).
    // Rows of B narrower than three cache lines lose with it on every pattern tried (n = 64: 4-18 % more time).
    p.HOT = (hot_candidate && p.SLICED == 0) ? (int32_t)(kMallBytes / 4 / 1024) : 0;
    if (t.hot >= 0) p.HOT = t.hot;
    if (t.bn > 0) p.BN = t.bn;
    if (t.alpha > 0) p.ALPHA = t.alpha;
    if (t.lw > 0) p.LW = t.lw;
    if (t.ch > 0) p.CH = t.ch;
    // One-lane groups (n <= 4): a workgroup takes 256 entries per step, so much longer pieces are still short chains,
    // and rows that are not cut need no second launch (mid-size graph pattern, n = 1: 21.2 -> 18.1 us).
    p.BCH = (n <= 4 ? 64 : 4) * p.CH;
    if (t.bch > 0) p.BCH = t.bch;
    if (t.u > 0) p.U = t.u;
    if (t.nt >= 0) p.NT = t.nt;
    // Hard limits the kernels rely on.
    p.BN = std::min(std::max(p.BN, 16), kBNMax);
    p.LW = std::min(std::max(p.LW, 0), kLWMax);
    p.ALPHA = std::max(p.ALPHA, (p.BN + kWindowRowsMax - 1) / kWindowRowsMax);  // <= 64 rows per window
    p.CH = std::max(p.CH, p.LW);
    p.BCH = std::max(p.BCH, 64);
    p.U = p.U >= 8 ? 8 : 4;
    p.NT &= 1;
    p.RESC = p.CUT = p.CUTJ = 0;  // see choose_plan
    return p;
}

__host__ __device__ static uint64_t align_up(uint64_t x, uint64_t a) { return (x + a - 1) & ~(a - 1); }  // a: a power of two

__host__ __device__ WorkspaceLayout layout_workspace(int32_t m, int32_t k, int64_t nnz, int32_t n, const PlanParams &p) {
    WorkspaceLayout L{};
    L.nblk = ((int64_t)m + kBlock - 1) / kBlock;
    L.n_windows = div_pos(nnz + (int64_t)p.ALPHA * m, p.BN) + 1;
    L.cap_wave = std::min<int64_t>(m, div_pos(nnz, p.LW + 1));
    const int64_t long_rows = std::min<int64_t>(m, div_pos(nnz, (int64_t)p.CH + 1));
    L.cap_items = div_pos(nnz, p.BCH) + long_rows;
    L.cap_split = std::min<int64_t>(m, div_pos(nnz, (int64_t)p.BCH + 1));
    L.cap_slots = div_pos(nnz, p.BCH) + L.cap_split;
    L.partial_stride = (n + 3) / 4 * 4;
    uint64_t off = 0;
    L.off_counts = off;
    off = align_up(off + (uint64_t)kQ * L.nblk * 4, 256);
    L.off_totals = off;
    off = align_up(off + kQ * 4, 256);
    L.off_win = off;
    off = align_up(off + (uint64_t)(L.n_windows + 1) * 4, 256);
    L.off_stage = off;
    off = align_up(off + (uint64_t)L.n_windows * 8, 256);
    L.off_wave = off;
    off = align_up(off + (uint64_t)L.cap_wave * 4, 256);
    L.off_wave_span = off;
    off = align_up(off + (uint64_t)L.cap_wave * 8, 256);
    L.off_items = off;
    off = align_up(off + (uint64_t)L.cap_items * 16, 256);
    L.off_split = off;
    off = align_up(off + (uint64_t)L.cap_split * 16, 256);
    L.off_partials = off;
    off = align_up(off + (uint64_t)L.cap_slots * L.partial_stride * 4, 256);
    // arrival counters: a split row has one per column tile of the launch; the narrowest tile any mapping uses is 16 columns
    L.ticket_tiles = std::max<int64_t>(1, ((int64_t)n + 15) / 16);
    L.off_tickets = off;
    off = align_up(off + (uint64_t)L.cap_slots * L.ticket_tiles * 4, 256);  // indexed by a split row's first slot
    L.off_bpack = off;
    if (p.PACK || (p.PANEL && !p.PDIRECT)) off = align_up(off + (uint64_t)k * ((n + 2 * kPanelCols - 1) / (2 * kPanelCols)) * (2 * kPanelCols) * 4, 256);
    L.off_res_ptr = off;
    if (p.RES) {
        const int64_t chunks = p.RESC;
        off = align_up(off + (uint64_t)(chunks + 1) * m * 4, 256);
        if (chunks > 1) L.res_row_bytes = (uint64_t)chunks * p.RES * 4;
    }
    L.off_coldeg = off;
    if (p.HOT) off = align_up(off + (uint64_t)k * 4, 256);
    L.off_hotmask = off;
    if (p.HOT) off = align_up(off + ((uint64_t)k / 32 + 2) * 4, 256);
    L.off_degbins = off;
    if (p.HOT) off = align_up(off + (uint64_t)kDegBins * 16, 256);
    L.off_res_partials = off;  // a one-shot plan has fewer of them
    off = align_up(off + L.res_row_bytes * m, 256);
    L.without_cut = std::max<uint64_t>(off, 256);
    L.off_cut_info = off;
    // scorch_spmm_csr_static gives the planned call's bits and analyses at every call, so that no rows are cut where it serves.  One call, us,
    // whole / cut: 169 343 rows of 15, n = 128 142 / 298; 100 000 of 50, n = 100 265 / 674; 4000 x 8000, 5 %, n = 333 200 / 390; 10 000 x 40 000, 3 %,
    // n = 61 402 / 696 (the product alone 120 / 113, 246 / 194, 180 / 115, 377 / 158).
    if (p.CUT == 2 || (p.CUT == 1 && off > SCORCH_STATIC_SCRATCH_BYTES)) L.cap_cut = cut_capacity(m, k, nnz, p.CUTJ);
    if (L.cap_cut > 0) {
        off = align_up(off + sizeof(CutInfo), 256);
        L.off_cut_counts = off;
        off = align_up(off + (uint64_t)kCutBuckets * kPlanBlocksMax * 4, 256);
        L.off_cut_hist = off;
        off = align_up(off + (uint64_t)kCutBins * 4, 256);
        L.off_cut_rows = off;
        off = align_up(off + (uint64_t)L.cap_cut / kXcds * 4, 256);
        L.off_cut_spans = off;
        off = align_up(off + (uint64_t)L.cap_cut * 8, 256);
        L.off_cut_partials = off;
        off = align_up(off + (uint64_t)L.cap_cut * L.partial_stride * 4, 256);
    }
    L.total = std::max<uint64_t>(off, 256);
    L.one_shot = L.cap_cut > 0 ? L.total : L.off_res_partials;
    return L;
}

// Whether a one-shot plan of the resident kernel runs in so many bytes.
static bool resident_runs_in(uint64_t bytes, int32_t m, int32_t k, int64_t nnz, int32_t n, const PlanParams &p) {
    const WorkspaceLayout L = layout_workspace(m, k, nnz, n, p);
    uint64_t off;
    return L.off_res_partials <= bytes && partial_rows_in(L, m, bytes, off) >= std::min(m, 64);
}

// The parameters of a plan.  The planning kernels go by choose_params alone: what they write stands before everything that the chunks of the
// resident kernel and the pieces of cut rows move, and working these out there (64-bit divisions) took 13 us per plan (pruned
// 4096 x 16 384, n = 16).  What does not fit the workspace on account of them, the host finds.
PlanParams choose_plan(int32_t m, int32_t k, int64_t nnz, int32_t n, const Tuning &t) {
    PlanParams p = choose_params(m, k, nnz, n, t);
    if ((nnz >= kCutNnzMin && t.cut != 0) || t.cut > 0) {
        // the kernel for it is compiled for the default unroll depth and cache policies
        const bool possible = m > 0 && k > 0 && n > 16 && p.PANEL == 0 && p.RES == 0 && p.PACK == 0 && t.fix <= 0 && t.u <= 0 && t.nt < 0 && t.cold == 0;
        p.CUT = !possible ? 0 : t.cut > 0 ? 2 : want_cut(m, k, nnz, n, p.SLICED) ? 1 : 0;
        // parts of the columns of an XCD, up to 16 MB of B each: 122 MB in 1 / 4 / 8 / 16 parts 7100 / 6690 / 6600 / 6720 us,
        // 32 MB in 1 / 2 / 4 / 8 1356 / 1336 / 1356 / 1391, 5 MB in 1 / 2 / 4 212 / 226 / 237
        const int64_t xcd_bytes = (int64_t)k * (p.SLICED ? p.SLICED : n) * 4 / kXcds;
        while (p.CUTJ < kCutClasses - 1 && (xcd_bytes >> p.CUTJ) > (16ll << 20)) ++p.CUTJ;
        if (t.cutj >= 0) p.CUTJ = std::min(t.cutj, kCutClasses - 1);
    }
    if (!p.RES) return p;
    p.RESC = resident_balance(m, k, nnz, p.RES);
    // scorch_spmm_csr_static takes what the gather kernels need no more than its scratch for, and gives the planned call's
    // bits: where the resident kernel does not run in the scratch either, with as many chunks as are best or with the fewest (whose
    // table of row pointers is smaller), it runs nowhere.
    PlanParams gather = p;
    gather.RES = 0;
    if (layout_workspace(m, k, nnz, n, gather).total <= SCORCH_STATIC_SCRATCH_BYTES && !resident_runs_in(SCORCH_STATIC_SCRATCH_BYTES, m, k, nnz, n, p)) {
        p.RESC = resident_chunks(k, p.RES);
        if (!resident_runs_in(SCORCH_STATIC_SCRATCH_BYTES, m, k, nnz, n, p)) p.RES = 0;
    }
    return p;
}

// How the rows are dealt to the workgroups of the planning kernels: at most kPlanBlocksMax workgroups, so that the
// counts of all workgroups before one are few enough to be added up by each.  Up to kPlanRecount workgroups the counting launch
// is left out and every workgroup counts the rows before its own, 8 batches of row pointers at most; with 78 of them the
// build kernel took 30 us instead of 7.7 + 4.3 for the counts.
constexpr int32_t kPlanRecount = 8;

// Slots of host memory that the planning kernels write their result to: taken for the length of one call and given back
// (as many as calls were in flight at once, under a kilobyte each).
static std::mutex g_result_mutex;
static PlanResult *g_result_free;  // linked through the slots themselves: nothing here can throw

static scorch_status_t take_result(PlanResult **out) {
    std::lock_guard<std::mutex> lock(g_result_mutex);
    if (!g_result_free) {
        constexpr size_t kSlots = 4096 / sizeof(PlanResult);
        void *page = nullptr;
        hipError_t e = hipHostMalloc(&page, kSlots * sizeof(PlanResult), hipHostMallocPortable | hipHostMallocMapped);
        if (e != hipSuccess) return hip_fail(e, "allocate host memory for the plan's result");
        PlanResult *slots = static_cast<PlanResult *>(page);
        for (size_t i = 0; i < kSlots; ++i) {
            slots[i].next = g_result_free;
            g_result_free = slots + i;
        }
    }
    *out = g_result_free;
    g_result_free = g_result_free->next;
    return SCORCH_OK;
}

static void give_result_back(PlanResult *r) {
    std::lock_guard<std::mutex> lock(g_result_mutex);
    r->next = g_result_free;
    g_result_free = r;
}

// The result once it has arrived.  Everything enqueued on the stream so far has finished as well, except for a one-shot plan: there
// the host only watches for the result itself, which arrives some microseconds before a wait on the stream returns; after
// about a millisecond (the stream was busy with something else) it waits for the stream.
static scorch_status_t wait_for_result(PlanResult *r, bool one_shot, hipStream_t stream) {
    if (one_shot) {
        for (int i = 0; i < 20000; ++i) {
            if (__atomic_load_n(&r->done, __ATOMIC_ACQUIRE)) return SCORCH_OK;
            __builtin_ia32_pause();
        }
    }
    const hipError_t e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return hip_fail(e, "wait for plan kernels");
    if (!__atomic_load_n(&r->done, __ATOMIC_ACQUIRE)) {
        set_error("plan kernels ended without a result");
        return SCORCH_ERR_HIP;
    }
    return SCORCH_OK;
}

// build_plan once a slot for the result has been taken.  `lost`: a wait failed, so a kernel may still write to the slot.
static scorch_status_t build_plan_in(PlanResult *result, bool *lost, scorch_spmm_plan_t *plan, const int32_t *rowptr, const int32_t *colidx,
                                     uint64_t workspace_bytes, bool one_shot, hipStream_t stream) {
    result->done = 0;
    result->unsorted = 0;
    const int64_t tiles = std::max<int64_t>(1, ((int64_t)plan->m + kBlock - 1) / kBlock);
    PlanArgs a{};
    a.rowptr = rowptr;
    a.m = plan->m;
    a.k = plan->k;
    a.n = plan->n;
    a.tuning = plan->tuning;
    a.workspace = plan->workspace;
    a.workspace_bytes = workspace_bytes;
    a.tiles_per_block = (int32_t)((tiles + kPlanBlocksMax - 1) / kPlanBlocksMax);
    const uint32_t nblk = (uint32_t)((tiles + a.tiles_per_block - 1) / a.tiles_per_block);
    a.counted = nblk > (uint32_t)kPlanRecount;
    a.one_shot = one_shot;
    a.result = result;
    if (a.counted) hipLaunchKernelGGL(plan_count_kernel, dim3(nblk), dim3(kBlock), 0, stream, a);
    hipLaunchKernelGGL(plan_build_kernel, dim3(nblk), dim3(kBlock), 0, stream, a);
    hipError_t e = hipGetLastError();
    scorch_status_t st = e != hipSuccess ? hip_fail(e, "launch plan kernels") : wait_for_result(result, one_shot, stream);
    const PlanResult got = *result;
    if (st != SCORCH_OK) {
        *lost = true;
        return st;
    }
    if (got.nnz < 0) {
        set_error("rowptr[m] = %d is negative", got.nnz);
        return SCORCH_ERR_INVALID_ARG;
    }
    plan->nnz = got.nnz;
    plan->params = choose_plan(plan->m, plan->k, plan->nnz, plan->n, plan->tuning);
    plan->layout = layout_workspace(plan->m, plan->k, plan->nnz, plan->n, plan->params);
    if (plan->params.RES && !one_shot && plan->layout.total > workspace_bytes) {  // what B needs at least, then
        plan->params.RESC = resident_chunks(plan->k, plan->params.RES);
        plan->layout = layout_workspace(plan->m, plan->k, plan->nnz, plan->n, plan->params);
    }
    const WorkspaceLayout &L = plan->layout;
    if (bytes_needed(L, one_shot) > workspace_bytes) return SCORCH_ERR_WORKSPACE_TOO_SMALL;  // the caller words the message
    char *ws = plan->workspace;
    plan->n_wave = got.totals[0];
    plan->n_items = got.totals[1];
    plan->n_split = got.totals[2];
    plan->n_slots = got.totals[3];
    plan->n_short = got.totals[4];
    // Every row is of one class.  Where one is not, its pointers decrease, and windows may be missing from the table.
    if ((int64_t)plan->n_wave + plan->n_short + plan->n_split + (plan->n_items - plan->n_slots) != plan->m) {
        set_error("rowptr decreases (or changed while it was read)");
        return SCORCH_ERR_INVALID_ARG;
    }
    if (plan->n_wave > L.cap_wave || plan->n_items > L.cap_items || plan->n_split > L.cap_split ||
        plan->n_slots > L.cap_slots) {
        set_error("plan lists exceed the workspace bound (rowptr changed while it was read?)");
        return SCORCH_ERR_INVALID_ARG;
    }
    // The panel and resident kernels need every row's columns in strictly increasing order; without colidx this cannot be
    // verified, so the mode is dropped.
    if (!colidx || plan->m == 0 || plan->nnz == 0) plan->params.PANEL = plan->params.RES = plan->params.CUT = 0;
    if (L.cap_cut > 0 && L.total > workspace_bytes) {  // no room for the pieces
        plan->params.CUT = 0;
        plan->layout.total = L.without_cut;
    }
    if (plan->params.PANEL || plan->params.RES) {
        int32_t *seen = reinterpret_cast<int32_t *>(ws + L.off_totals);  // cleared by plan_build_kernel
        const uint32_t g = (uint32_t)std::min<int64_t>(((int64_t)plan->m + kWavesPerBlock - 1) / kWavesPerBlock, 256 * 16);
        if (plan->params.RES) {
            st = launch_plan_resident(plan, rowptr, colidx, seen, &result->unsorted, stream);
            if (st != SCORCH_OK) return st;
        } else {
            hipLaunchKernelGGL(plan_sorted_kernel, dim3(g), dim3(kBlock), 0, stream, rowptr, colidx, plan->m, seen, &result->unsorted);
        }
        e = hipStreamSynchronize(stream);
        if (e != hipSuccess) {
            *lost = true;
            return hip_fail(e, "wait for the look at the columns");
        }
        if (__atomic_load_n(&result->unsorted, __ATOMIC_ACQUIRE)) plan->params.PANEL = plan->params.RES = 0;
    }
    if (plan->params.RES) {
        plan->off_res_partials = L.off_res_partials;
        plan->res_rows = one_shot ? partial_rows_in(L, plan->m, workspace_bytes, plan->off_res_partials) : plan->m;
    }
    plan->cut_pieces = plan->cut_rows = 0;
    plan->cut_len = 0;
    if (plan->params.CUT && L.cap_cut > 0) {  // there is room for the pieces
        st = launch_plan_cut(plan, rowptr, colidx, result, stream);
        if (st != SCORCH_OK) return st;
        e = hipStreamSynchronize(stream);
        if (e != hipSuccess) {
            *lost = true;
            return hip_fail(e, "wait for the kernels that cut rows");
        }
        // where a piece came out too long to be one wavefront's work, no row is cut
        const CutInfo &c = result->cut;
        if (c.len != INT32_MAX && c.longest <= c.limit) {
            plan->cut_pieces = c.pieces;
            plan->cut_rows = c.n_rows;
            plan->cut_len = c.len;
        }
    }
    plan->n_hot = 0;
    plan->hot_share = 0.f;
    if (plan->params.HOT && colidx && plan->nnz > 0 && plan->k > 0) {
        st = mark_hot_columns(plan, colidx, plan->tuning.hot > 0, one_shot, stream);
        if (st != SCORCH_OK) return st;
    }
    // the arrival counters of split rows (only used with fix=1) start at zero; every launch leaves them at zero again
    if (L.cap_slots > 0 && plan->tuning.fix > 0) {
        e = hipMemsetAsync(ws + L.off_tickets, 0, (size_t)L.cap_slots * L.ticket_tiles * 4, stream);
        if (e == hipSuccess && !one_shot) e = hipStreamSynchronize(stream);
        if (e != hipSuccess) return hip_fail(e, "clear arrival counters");
    }
    return SCORCH_OK;
}

scorch_status_t build_plan(scorch_spmm_plan_t *plan, const int32_t *rowptr, const int32_t *colidx,
                           uint64_t workspace_bytes, bool one_shot, hipStream_t stream) {
    PlanResult *result = nullptr;
    scorch_status_t st = take_result(&result);
    if (st != SCORCH_OK) return st;
    bool lost = false;
    st = build_plan_in(result, &lost, plan, rowptr, colidx, workspace_bytes, one_shot, stream);
    if (!lost) give_result_back(result);  // otherwise it is not used again
    // an error leaves nothing behind that still reads the caller's arrays
    if (st != SCORCH_OK && one_shot) (void)hipStreamSynchronize(stream);
    return st;
}

}  // namespace scorch
