// Resident kernel: CSR SpMM with a narrow B (up to 64 columns) whose rows are each wanted by many rows of A, e.g. a pruned
// weight times a small batch, C_ik = sum_j A_ij * B_jk (paper, Section 4.2).
//
// The gather kernels fetch one row of B per stored entry from L2.  For narrow rows that is bound by the number of
// requests, not by their bytes: the dies' L2s serve 226 G requests/s at most (probe of 512-byte rows), 128 bytes each, so
// 64-byte rows arrive at 14 to 16 TB/s.  Here every workgroup keeps a chunk of the rows of B in LDS for its whole life (158 KB: 158 * 256 / W
// rows of W columns) and takes, of every row of A in its block of rows, the entries that fall into the chunk.  Where
// they start is in the plan.  The plan is bound to the row pointers, not to the columns: where one of a row's entries turns
// out to lie outside the chunk, they are all gathered from B instead (resident_gather), so that other columns, in any
// order and repeated, are added up as well (4096 x 16 384, 10 % stored, n = 16: 21.5 us for the planner's columns, 51 for shuffled
// ones; the gather kernel 42).  B enters a CU once, A is read once, and each chunk leaves partial rows that a second
// launch adds in chunk order (none if B fits one chunk).
//
// Now no unit is saturated (n = 16: VALU busy 48 %, LDS 24 %, half of that bank conflicts): with LDS full a SIMD has four wavefronts.
//
//   workgroup   16 wavefronts on a CU of its own: one chunk x a block of rows
//   wavefront   one row at a time: 64 entries per window, one per lane, requested a row ahead
//   lane group  G lanes cover the W = 4 G T columns; the 64 / G groups take the window's entries in turn, an entry's
//               index and value coming from the lane that holds them by a DPP operand
// Measured on 4096 x 16 384, 10 % stored: see want_resident.
#include "device_util.h"
#include "spmm_internal.h"

#include <algorithm>

namespace scorch {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kResidentThreads = 1024;
constexpr int kResidentWaves = kResidentThreads / kWave;
constexpr int kResidentWindows = 4;  // windows of a row that are requested a row ahead

// Value of lane J of the caller's group of G lanes: quad permutation for groups of 2 and 4 lanes, row broadcast for 16.
template <int G, int J> __device__ __forceinline__ int group_lane(int x) {
    if constexpr (G == 1) return x;
    constexpr int ctrl = G == 2 ? (J == 0 ? 0xA0 : 0xF5) : (G == 4 ? J * 0x55 : 0x150 + J);
    return __builtin_amdgcn_update_dpp(0, x, ctrl, 0xF, 0xF, true);
}

// Entries J ... J + N - 1 of every group's window: the LDS reads of all of them first, then the multiply-adds.
template <int G, int T, int J, int N, int U = 0>
__device__ __forceinline__ void resident_reads(f4 (&x)[N][T], int off, const char *lds, int lig16) {
    if constexpr (U < N) {
        const uint32_t at = (uint32_t)(group_lane<G, J + U>(off) + lig16);
#pragma unroll
        for (int t = 0; t < T; ++t) x[U][t] = *reinterpret_cast<const f4 *>(lds + at + t * (16 * G));
        resident_reads<G, T, J, N, U + 1>(x, off, lds, lig16);
    }
}
template <int G, int T, int J, int N, int U = 0>
__device__ __forceinline__ void resident_fmas(f4 (&acc)[T], const f4 (&x)[N][T], int val) {
    if constexpr (U < N) {
        const float v = __int_as_float(group_lane<G, J + U>(val));
#pragma unroll
        for (int t = 0; t < T; ++t) vfma<4>(acc[t], v, x[U][t]);
        resident_fmas<G, T, J, N, U + 1>(acc, x, val);
    }
}
// The first `steps` entries of every group's window (rounded up to a multiple of N: a lane past the row's entries points
// at a row of zeros and holds a zero).  `steps` is the same for the whole wavefront.
template <int G, int T, int J = 0>
__device__ __forceinline__ void resident_window(f4 (&acc)[T], int off, int val, int steps, const char *lds, int lig16) {
    constexpr int N = G < 4 ? G : 4;
    if constexpr (J < G) {
        f4 x[N][T];
        resident_reads<G, T, J, N>(x, off, lds, lig16);
        resident_fmas<G, T, J, N>(acc, x, val);
        if (J + N < G && steps > J + N) resident_window<G, T, J + N>(acc, off, val, steps, lds, lig16);
    }
}

// Sum over the 64 / G groups of a wavefront, in every lane: rotations inside the rows of 16 lanes, then exchanges of rows
// and of halves (one vector instruction each).
template <int G> __device__ __forceinline__ float sum_groups(float x) {
    if constexpr (G <= 1) x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x121, 0xF, 0xF, true));
    if constexpr (G <= 2) x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x122, 0xF, 0xF, true));
    if constexpr (G <= 4) x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xF, 0xF, true));
    if constexpr (G <= 8) x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xF, 0xF, true));
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}

// Entry ranges of this chunk in 32 rows of a wavefront: lane i holds row i's first entry of the chunk, lane 32 + i its
// first entry after it.  They are the plan's: for the columns that the planner saw, every entry of a range lies in the
// chunk; whatever the columns of the call are, the ranges of all chunks cover each entry of the row once.
__device__ __forceinline__ int resident_bounds(const ResidentArgs &a, int64_t row0, int row_end, int chunk, int lane) {
    const int64_t row = row0 + (lane & 31) * kResidentWaves;
    return row < row_end ? a.ptr[(int64_t)(chunk + (lane >> 5)) * a.ptr_stride + row] : 0;
}

// Four columns c ... c+3 of a row of B; those past column n are never stored and may hold anything.
template <bool A16> __device__ __forceinline__ f4 resident_load_b(const ResidentArgs &a, int row, int c) {
    const float *src = a.B + (int64_t)row * a.ldb;
    if constexpr (A16) return *reinterpret_cast<const f4 *>(src + (c < a.n ? c : 0));
    f4 x;
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = src[min(c + i, a.n - 1)];
    return x;
}

template <int G, int T, bool A16, int J, int N, int U = 0>
__device__ __forceinline__ void resident_gather_batch(f4 (&acc)[T], const ResidentArgs &a, int col, int val, int lig) {
    if constexpr (U < N) {
        const int c = group_lane<G, J + U>(col);
        const float v = __int_as_float(group_lane<G, J + U>(val));
        const bool there = (uint32_t)c < (uint32_t)a.k;
        f4 x[T];
#pragma unroll
        for (int t = 0; t < T; ++t) x[t] = resident_load_b<A16>(a, there ? c : 0, t * 4 * G + lig * 4);
        resident_gather_batch<G, T, A16, J, N, U + 1>(acc, a, col, val, lig);  // the loads of the batch before its multiply-adds
#pragma unroll
        for (int t = 0; t < T; ++t) vfma<4>(acc[t], there ? v : 0.f, there ? x[t] : f4{0.f, 0.f, 0.f, 0.f});
    }
}

// The first `steps` entries of every group's window, gathered from B.  `col` is -1 in the lanes past the row's entries.
// An entry that is not there, or not a column, adds nothing, whatever row 0 of B holds.
template <int G, int T, bool A16, int J = 0>
__device__ __forceinline__ void resident_gather(f4 (&acc)[T], const ResidentArgs &a, int col, int val, int steps, int lig) {
    constexpr int N = G < 4 ? G : 4;
    if constexpr (J < G) {
        resident_gather_batch<G, T, A16, J, N>(acc, a, col, val, lig);
        if (J + N < G && steps > J + N) resident_gather<G, T, A16, J + N>(acc, a, col, val, steps, lig);
    }
}

struct ResidentWindows {
    int c[kResidentWindows];
    float v[kResidentWindows];
};

// The chunk goes straight into LDS.  A16: 16-byte vectors; otherwise (rows of B not 16-byte aligned, n not a multiple of 4)
// single floats.  Lanes past row k or column n load nothing, and what they leave only feeds columns that are never
// stored.
template <int W, bool A16>
__device__ __forceinline__ void resident_fetch(const ResidentArgs &a, int k0, int k1, float *s_b, int wv, int lane) {
    constexpr int E = A16 ? 4 : 1;
    constexpr int kPieces = kResidentFloats / (kWave * E);
    for (int i = wv; i < kPieces; i += kResidentWaves) {
        const int f = (i * kWave + lane) * E;
        const int row = f / W, col = f % W;
        if (k0 + row < k1 && col < a.n) {
            const float *src = a.B + (int64_t)(k0 + row) * a.ldb + col;
            if constexpr (A16) __builtin_amdgcn_global_load_lds(src, s_b + i * kWave * E, 16, 0, 0);
            else __builtin_amdgcn_global_load_lds(src, s_b + i * kWave * E, 4, 0, 0);
        }
    }
}

template <int G, int T, bool A16>
__global__ __launch_bounds__(kResidentThreads) void spmm_resident_kernel(const ResidentArgs a) {
    constexpr int W = 4 * G * T;
    constexpr int S = kWave / G;
    __shared__ __attribute__((aligned(16))) float s_b[kResidentFloats + W];  // the chunk and a row of zeros
    const int tid = threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int grp = lane / G, lig = lane % G;
    const int chunk = (int)(blockIdx.x % (uint32_t)a.nchunks);
    const int blk = (int)(blockIdx.x / (uint32_t)a.nchunks);
    const int k0 = chunk * a.chunk_rows;
    const int row_end = (int)min((int64_t)a.m, ((int64_t)blk + 1) * a.rows_per_block);
    const int lane_entry = S * lig + grp;  // which entry of a window this lane holds
    const char *lds = reinterpret_cast<const char *>(s_b);
    const int zero_off = kResidentFloats * 4;
    const int lig16 = lig * 16;

    resident_fetch<W, A16>(a, k0, (int)min((int64_t)a.k, (int64_t)k0 + a.chunk_rows), s_b, wv, lane);
    if (tid < W) s_b[kResidentFloats + tid] = 0.f;
    // lanes past the row's entries of the chunk read the last of them once more (no further cache lines), unused
    const auto entry = [&](uint32_t at, uint32_t end) { return min(at + (uint32_t)lane_entry, max(end, 1u) - 1u); };
    const auto request = [&](ResidentWindows &w, uint32_t s, uint32_t e) {
#pragma unroll
        for (int i = 0; i < kResidentWindows; ++i)
            if (s + i * kWave < e) {  // the same for the whole wavefront
                const uint32_t p = entry(s + i * kWave, e);
                w.c[i] = a.colidx[p];
                w.v[i] = a.vals[p];
            }
    };
    int64_t row = (int64_t)blk * a.rows_per_block + wv;
    int bounds = resident_bounds(a, row, row_end, chunk, lane);
    const auto bound = [&](int i, int which) { return (uint32_t)__builtin_amdgcn_readlane(bounds, (i & 31) + which * 32); };
    uint32_t s = bound(0, 0), e = bound(0, 1);
    ResidentWindows next{};
    request(next, s, e);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's share of the chunk has landed
    __syncthreads();
    for (int i = 1; row < row_end; row += kResidentWaves, ++i) {
        const ResidentWindows cur = next;
        if ((i & 31) == 0) bounds = resident_bounds(a, row + kResidentWaves, row_end, chunk, lane);
        const uint32_t s2 = bound(i, 0), e2 = bound(i, 1);
        request(next, s2, e2);
        f4 acc[T];
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
        const auto steps = [&](uint32_t at) { return (int)((e - at + S - 1) / S); };
        const auto valid = [&](uint32_t at) { return at + (uint32_t)lane_entry < e; };
        const auto inside = [&](int col) { return (uint32_t)(col - k0) < (uint32_t)a.chunk_rows; };
        const auto work = [&](int col, float value, uint32_t at) {
            const bool in = valid(at) && inside(col);
            const int off = in ? (col - k0) * (W * 4) : zero_off;
            resident_window<G, T>(acc, off, __float_as_int(in ? value : 0.f), steps(at), lds, lig16);
        };
        uint32_t at = s;
        bool outside = false;
#pragma unroll
        for (int i = 0; i < kResidentWindows; ++i, at += kWave)
            if (at < e) {
                outside |= valid(at) && !inside(cur.c[i]);
                work(cur.c[i], cur.v[i], at);
            }
        for (; at < e; at += kWave) {
            const uint32_t p = entry(at, e);
            const int col = a.colidx[p];
            float value = a.vals[p];
            asm volatile("" : "+v"(value));  // requested together with the index, not once it is known
            outside |= valid(at) && !inside(col);
            work(col, value, at);
        }
        if (__ballot(outside) != 0ull) {  // the row once more, wherever its columns are
#pragma unroll
            for (int t = 0; t < T; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
            for (at = s; at < e; at += kWave) {
                const uint32_t p = entry(at, e);
                resident_gather<G, T, A16>(acc, a, valid(at) ? a.colidx[p] : -1, __float_as_int(a.vals[p]), steps(at), lig);
            }
        }
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[t][i] = sum_groups<G>(acc[t][i]);
        if (grp == 0) {
            if (a.nchunks > 1) {
                float *dst = a.partials + ((int64_t)chunk * a.m + row) * W;
#pragma unroll
                for (int t = 0; t < T; ++t) *reinterpret_cast<f4 *>(dst + t * 4 * G + lig * 4) = acc[t];
            } else {
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const int c = t * 4 * G + lig * 4;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (c + i < a.n) {
                            float x = acc[t][i] + (a.bias ? a.bias[c + i] : 0.f);
                            if (a.act == 1) x = fmaxf(x, 0.f);
                            a.C[row * a.ldc + c + i] = x;
                        }
                }
            }
        }
        s = s2;
        e = e2;
    }
}

// C = act(sum of the chunks' partial rows, in chunk order, + bias): one thread per vector of four columns.
__global__ __launch_bounds__(kBlock) void spmm_resident_sum_kernel(const ResidentArgs a, int W) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t total = (int64_t)a.m * W;
    if (i * 4 >= total) return;
    const int64_t row = i * 4 / W;
    const int c = (int)(i * 4 % W);
    if (c >= a.n) return;
    const f4 *src = reinterpret_cast<const f4 *>(a.partials) + i;
    f4 sum = *src;
#pragma unroll 4
    for (int j = 1; j < a.nchunks; ++j) sum += src[(int64_t)j * (total / 4)];
#pragma unroll
    for (int x = 0; x < 4; ++x)
        if (c + x < a.n) {
            float out = sum[x] + (a.bias ? a.bias[c + x] : 0.f);
            if (a.act == 1) out = fmaxf(out, 0.f);
            a.C[row * a.ldc + c + x] = out;
        }
}

// Checks that every row's columns are strictly increasing (sets *unsorted otherwise) and writes ptr[p][row] = the row's
// first entry of chunk p or later, p = 0 ... nchunks.  One wavefront per row.
__global__ __launch_bounds__(kBlock) void plan_resident_kernel(const int32_t *rowptr, const int32_t *colidx, int32_t m,
                                                               uint32_t chunk_rows, int32_t nchunks, int32_t *ptr, int32_t *seen,
                                                               int32_t *unsorted) {
    const int lane = threadIdx.x & 63;
    for (int64_t row = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6); row < m;
         row += (int64_t)gridDim.x * kWavesPerBlock) {
        const int p0 = rowptr[row], p1 = rowptr[row + 1];
        bool bad = false;
        for (int64_t p = (int64_t)p0 + lane; p <= p1; p += kWave) {
            // entry p opens the chunks after its predecessor's up to its own; the end of the row opens the rest
            const int prev = p > p0 ? colidx[p - 1] : -1;
            const int c = p < p1 ? colidx[p] : 0;
            if (p > p0 && p < p1) bad |= c <= prev;
            const int lo = p > p0 ? (int)((uint32_t)prev / chunk_rows) + 1 : 0;
            const int hi = p < p1 ? min((int)((uint32_t)c / chunk_rows), nchunks) : nchunks;
            for (int q = lo; q <= hi; ++q) ptr[(int64_t)q * m + row] = (int)p;
        }
        if (report_unsorted(bad, seen, unsorted)) break;
    }
}

static uint32_t resident_chunk_rows(const scorch_spmm_plan_t *plan) {
    const uint32_t chunks = (uint32_t)plan->params.RESC;
    return ((uint32_t)plan->k + chunks - 1) / chunks;
}

scorch_status_t launch_plan_resident(const scorch_spmm_plan_t *plan, const int32_t *rowptr, const int32_t *colidx, int32_t *seen,
                                     int32_t *unsorted, hipStream_t stream) {
    const int W = plan->params.RES;
    const uint32_t g = (uint32_t)std::min<int64_t>(((int64_t)plan->m + kWavesPerBlock - 1) / kWavesPerBlock, 256 * 16);
    hipLaunchKernelGGL(plan_resident_kernel, dim3(g), dim3(kBlock), 0, stream, rowptr, colidx, plan->m,
                       resident_chunk_rows(plan), plan->params.RESC,
                       reinterpret_cast<int32_t *>(plan->workspace + plan->layout.off_res_ptr), seen, unsorted);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "launch plan_resident_kernel");
    return SCORCH_OK;
}

typedef void (*resident_fn)(const ResidentArgs);

template <bool A16> static resident_fn pick_resident(int W) {
    switch (W) {
        case 4: return spmm_resident_kernel<1, 1, A16>;
        case 8: return spmm_resident_kernel<2, 1, A16>;
        case 16: return spmm_resident_kernel<4, 1, A16>;
        case 32: return spmm_resident_kernel<4, 2, A16>;
        default: return spmm_resident_kernel<16, 1, A16>;
    }
}

scorch_status_t launch_resident(const scorch_spmm_plan_t *plan, const int32_t *colidx, const float *vals, const float *B, int64_t ldb,
                                float *C, int64_t ldc, const float *bias, int32_t act, hipStream_t stream) {
    const int W = plan->params.RES;
    ResidentArgs a{};
    a.colidx = colidx;
    a.vals = vals;
    a.B = B;
    a.ldb = ldb;
    a.ldc = ldc;
    a.ptr_stride = plan->m;
    a.k = plan->k;
    a.n = plan->n;
    a.partials = reinterpret_cast<float *>(plan->workspace + plan->off_res_partials);
    a.nchunks = plan->params.RESC;
    a.chunk_rows = (int32_t)resident_chunk_rows(plan);
    a.bias = bias;
    a.act = act;
    const uintptr_t pb = reinterpret_cast<uintptr_t>(B);
    const bool a16 = plan->n % 4 == 0 && ldb % 4 == 0 && pb % 16 == 0;
    const int32_t *ptr = reinterpret_cast<const int32_t *>(plan->workspace + plan->layout.off_res_ptr);
    // all rows at once, or as many as the workspace holds partial rows for (a row's sum is the same either way)
    for (int64_t row0 = 0; row0 < plan->m; row0 += plan->res_rows) {
        a.m = (int32_t)std::min<int64_t>(plan->res_rows, plan->m - row0);
        a.ptr = ptr + row0;
        a.C = C + row0 * ldc;
        // as many row blocks as let every workgroup have a CU at once
        const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>(kCus / a.nchunks, ((int64_t)a.m + kResidentWaves - 1) / kResidentWaves));
        a.rows_per_block = (int32_t)((a.m + blocks - 1) / blocks);
        const int64_t nblk = ((int64_t)a.m + a.rows_per_block - 1) / a.rows_per_block;
        hipLaunchKernelGGL(a16 ? pick_resident<true>(W) : pick_resident<false>(W), dim3((uint32_t)(nblk * a.nchunks)),
                           dim3(kResidentThreads), 0, stream, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "launch spmm_resident_kernel");
        if (a.nchunks > 1) {
            const int64_t vecs = (int64_t)a.m * W / 4;
            hipLaunchKernelGGL(spmm_resident_sum_kernel, dim3((uint32_t)((vecs + kBlock - 1) / kBlock)), dim3(kBlock), 0, stream, a, W);
            e = hipGetLastError();
            if (e != hipSuccess) return hip_fail(e, "launch spmm_resident_sum_kernel");
        }
    }
    return SCORCH_OK;
}

}  // namespace scorch
