// Dense product of a graph-convolution layer (paper, Section 5.1):  Y = act(X W + bias), X m x k with very many rows, W
// k x n small, all fp32.
//
// Bound: 4 m (k + n) bytes of X and Y against 2 m k n flops at the 157 TFLOP/s of the fp32 matrix instructions
// (v_mfma_f32_16x16x4_f32: products and sums in fp32); with k = n = 128 both take about as long.  So W is kept in LDS,
// transposed, by workgroups that stay (two per CU) and whose wavefronts walk units of 32 rows by themselves; n is cut into
// parts of up to 128 columns.  X goes straight from memory into the operand registers, a step of 16 columns ahead, once
// per part.  The product is formed as Y^T = W^T X^T: the first operand of the instruction is W^T, so that a lane ends with four
// consecutive columns of one row of Y and stores them as one vector.  Bias and activation are applied on the way out:
// left to passes of their own they read and write Y once more.  W is staged before the first rows of X are requested: the other way round,
// or with four rounds of W at a time, the start takes longer (8000 rows, 100 -> 128 10.2 / 10.9 / 10.5 us, both 11.4; many rows even).
// What is left at 169 343 rows (128 -> 128 56.5 us): one or two units per
// wavefront, so that start, product and store hardly overlap (1 M rows: 107 TFLOP/s, the dense library 96).  Column parts of 64
// instead of 128 (1 M rows 315 -> 330 us) and three or four workgroups per CU are no faster.  Scalar loads of X instead of vectors: 5-35 % more.
// Lane l of a wavefront reads, of 16 columns of X, the four from 4 (l / 16) onwards, one vector; two exchanges between the
// 16-lane rows of the wavefront (order_x) then give it columns 2 (l / 16) and the next, of each half of the 16, so that every
// instruction adds up the even or the odd columns of 8 in ascending order.  That is the order in which the dense library adds up
// (each instruction is a chain of fused multiply-adds): the same bits wherever it takes its usual kernel, so that a layer may take either.
#include "dense_tiles.h"
#include "device_util.h"
#include "spmm_internal.h"

#include <algorithm>

namespace scorch {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kDenseKMax = 144;    // columns of X: W in LDS of two workgroups per CU
constexpr int kDenseTilesMax = 8;  // 16-column tiles of Y per workgroup
constexpr int kDenseWaves = 8;
constexpr int kDenseThreads = kDenseWaves * kWave;
static_assert(16 * kDenseTilesMax * (kDenseKMax + 4 + 1) * 4 <= 80 * 1024, "two workgroups per CU");

struct DenseArgs {
    const float *X, *W, *bias;
    float *Y;
    int64_t ldx, ldw, ldy;
    int32_t m, k, n;
    int32_t parts;   // parts of n, `tiles` 16-column tiles each
    int32_t units;   // units of 16 RT rows, one wavefront each
    int32_t relu;
};

// Four columns c ... c+3 of a row of X, those past column k as zeros.
__device__ __forceinline__ f4 dense_load_x(const float *row, int c, int k) {
    if (c + 4 <= k) return *reinterpret_cast<const f4u *>(row + c);
    f4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 3; ++i)
        if (c + i < k) x[i] = row[c + i];
    return x;
}

// From columns 4 q ... 4 q + 3 of 16 in the lanes of row q to columns 2 q, 2 q + 1, 8 + 2 q, 9 + 2 q.
__device__ __forceinline__ f4 order_x(f4 x) {
    auto exchange = [](float a, float b, float &lo, float &hi) {
        const auto odd = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        const auto half = __builtin_amdgcn_permlane32_swap(odd[0], odd[1], false, false);
        lo = __uint_as_float(half[0]);
        hi = __uint_as_float(half[1]);
    };
    f4 y;
    float lo, hi;
    exchange(x[0], x[2], lo, hi);
    y[0] = lo;
    y[2] = hi;
    exchange(x[1], x[3], lo, hi);
    y[1] = lo;
    y[3] = hi;
    return y;
}

// NT: 16-column tiles of Y per workgroup.  RT: 16-row tiles per wavefront.
template <int NT, int RT>
__global__ __launch_bounds__(kDenseThreads, 4) void dense_tall_kernel(const DenseArgs a) {
    extern __shared__ __attribute__((aligned(16))) float s_w[];  // [16 NT][kpad + 4]: a row stride of 4 banks (mod 64); then the bias
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wv = tid >> 6;
    const int steps = (a.k + 15) / 16;  // 16 columns of X each
    const int stride = steps * 16 + 4;
    // workgroups go to the XCDs in turn: the parts of the same rows are 8 apart, on the same XCD
    const int part = (int)(blockIdx.x / kXcds) % a.parts;
    const int first = (int)(blockIdx.x / kXcds) / a.parts * kXcds + (int)(blockIdx.x % kXcds);
    const int nblk = (int)gridDim.x / a.parts;
    const int n0 = part * (16 * NT);
    const int q = lane >> 4, r = lane & 15;
    const float *wbase = s_w + r * stride + q * 4;
    const float *xrow[RT];
    f4 x[RT], xn[RT];
    f4 acc[NT][RT];
    auto rows_of = [&](int64_t u) {
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const int64_t row = u * (16 * RT) + t * 16 + r;
            xrow[t] = a.X + (row < a.m ? row : (int64_t)a.m - 1) * a.ldx;  // rows past the end are computed and not stored
        }
    };
    auto fetch = [&](int step) {
#pragma unroll
        for (int t = 0; t < RT; ++t) xn[t] = dense_load_x(xrow[t], step * 16 + q * 4, a.k);
    };
    // units are dealt wavefront by wavefront over the workgroups, so that a last incomplete round is spread over the chip
    const int u0 = wv * nblk + first, du = kDenseWaves * nblk;
    // four rows of W at one column per thread; neighbouring threads read neighbouring columns
    for (int i = tid; i < 16 * NT * steps * 4; i += kDenseThreads) {
        const int c = i % (16 * NT), quad = i / (16 * NT);
        const int k0 = quad / 4 * 16 + quad % 4 * 2;  // rows k0, k0 + 1, k0 + 8, k0 + 9: see order_x
        f4 w = {0.f, 0.f, 0.f, 0.f};
        if (n0 + c < a.n)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int kj = k0 + j % 2 + j / 2 * 8;
                if (kj < a.k) w[j] = a.W[(int64_t)kj * a.ldw + n0 + c];
            }
        *reinterpret_cast<f4 *>(s_w + c * stride + quad * 4) = w;
    }
    float *s_bias = s_w + 16 * NT * stride;
    if (tid < 16 * NT) s_bias[tid] = a.bias && n0 + tid < a.n ? a.bias[n0 + tid] : 0.f;
    __syncthreads();

    if (u0 >= a.units) return;
    rows_of(u0);
    fetch(0);
    for (int64_t u = u0; u < a.units; u += du) {
#pragma unroll
        for (int c = 0; c < NT; ++c)
#pragma unroll
            for (int t = 0; t < RT; ++t) acc[c][t] = f4{0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < steps; ++s) {
#pragma unroll
            for (int t = 0; t < RT; ++t) x[t] = order_x(xn[t]);
            // the next 16 columns, of the next unit at the end of this one
            if (s + 1 < steps) {
                fetch(s + 1);
            } else if (a.units - u > du) {
                rows_of(u + du);
                fetch(0);
            }
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                const f4 w = *reinterpret_cast<const f4 *>(wbase + c * 16 * stride + s * 16);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int t = 0; t < RT; ++t) acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[j], x[t][j], acc[c][t], 0, 0, 0);
            }
        }
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const int64_t row = u * (16 * RT) + t * 16 + r;
            if (row >= a.m) continue;
            float *y = a.Y + row * a.ldy + n0 + q * 4;
            int left = a.n - n0 - q * 4;
            asm("" : "+v"(left));  // compared here, block by block: kept over the loop, the results cost 80 scalar registers
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                f4 v = acc[c][t] + *reinterpret_cast<const f4 *>(s_bias + c * 16 + q * 4);
                if (a.relu)
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = v[i] < 0.f ? 0.f : v[i];  // not a number stays that
                if (left >= c * 16 + 4) {
                    *reinterpret_cast<f4u *>(y + c * 16) = v;
                } else {
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        if (c * 16 + i < left) y[c * 16 + i] = v[i];
                }
            }
        }
    }
}

typedef void (*dense_fn)(const DenseArgs);

template <int RT> static dense_fn pick_dense(int tiles) {
    switch (tiles) {
        case 1: return dense_tall_kernel<1, RT>;
        case 2: return dense_tall_kernel<2, RT>;
        case 3: return dense_tall_kernel<3, RT>;
        case 4: return dense_tall_kernel<4, RT>;
        case 5: return dense_tall_kernel<5, RT>;
        case 6: return dense_tall_kernel<6, RT>;
        case 7: return dense_tall_kernel<7, RT>;
        default: return dense_tall_kernel<8, RT>;
    }
}

scorch_status_t launch_dense_tall(int32_t m, int32_t k, int32_t n, const float *X, int64_t ldx, const float *W, int64_t ldw,
                                  const float *bias, int32_t act, float *Y, int64_t ldy, hipStream_t stream) {
    if (k > kDenseKMax) {
        set_error("dense layer: k = %d exceeds the %d rows of W that are kept in LDS", k, kDenseKMax);
        return SCORCH_ERR_UNSUPPORTED;
    }
    DenseArgs a{};
    a.X = X;
    a.W = W;
    a.bias = bias;
    a.Y = Y;
    a.ldx = ldx;
    a.ldw = ldw;
    a.ldy = ldy;
    a.m = m;
    a.k = k;
    a.n = n;
    a.relu = act == 1;
    const int32_t all_tiles = (int32_t)(((int64_t)n + 15) / 16);
    a.parts = (all_tiles + kDenseTilesMax - 1) / kDenseTilesMax;
    const int32_t tiles = (all_tiles + a.parts - 1) / a.parts;
    const int rt = dense_row_tiles(m, k, n, (int64_t)2 * kCus / a.parts * kDenseWaves);
    a.units = (int32_t)(((int64_t)m + 16 * rt - 1) / (16 * rt));
    const uint32_t lds = (uint32_t)(16 * tiles * (((k + 15) / 16) * 16 + 4 + 1) * 4);  // one more per column: the bias
    // as many workgroups as are resident at once, in whole rounds of 8 per part
    int64_t per_part = std::min<int64_t>(a.units, std::max<int64_t>(kXcds, 2 * kCus / a.parts));
    per_part = (per_part + kXcds - 1) / kXcds * kXcds;
    const int64_t grid = per_part * a.parts;
    if (grid > 0x7fffffffLL) {
        set_error("launch grid of %lld workgroups exceeds the HIP limit", (long long)grid);
        return SCORCH_ERR_UNSUPPORTED;
    }
    const dense_fn fn = rt == 2 ? pick_dense<2>(tiles) : pick_dense<1>(tiles);
    hipLaunchKernelGGL(fn, dim3((uint32_t)grid), dim3(kDenseThreads), lds, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "launch dense_tall_kernel");
    return SCORCH_OK;
}

}  // namespace scorch
