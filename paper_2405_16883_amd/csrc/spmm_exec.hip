// Execution kernels for CSR SpMM on gfx950:  C_ik = sum_j A_ij * B_jk  (paper, Section 4.2).
//
// Loop structure kept from the paper (Sections 4.1, 4.2): rows outermost, the stored entries of a
// row next, the dense column index innermost, and only that dense column loop is tiled.  On the
// GPU the column loop is laid across lanes: a group of G lanes covers G*V*T consecutive columns
// (V floats per load, T loads per lane), so every read of a B row and every write of a C row is a
// contiguous, coalesced burst.  A wavefront holds S = 64/G such groups.  V = 4 whenever n >= 4; rows
// that are not 16-byte aligned use the same loads at float alignment (template flag UA), and a row
// whose length is not a multiple of 4 ends with a vector that overlaps its neighbour.
//
// Up to four paths share one launch; the workgroup index selects the path:
//   pieces  of long rows cut by columns (large graphs; spmm_cut.hip): a few per wavefront, each to a partial row
//   items   one workgroup per piece of a long row; 4 wavefronts split the piece, partial sums are
//           combined through LDS and written to C or to a partial row
//   wave    one wavefront per medium row; the S groups take interleaved entries and are combined
//           with cross-lane shuffles
//   window  one wavefront per window of consecutive short rows; the window's colidx/vals are
//           staged in LDS with coalesced loads, then each group walks one row at a time
// No MFMA: the work is a gather, not a dense contraction.  No atomics: summation order is fixed.
#include "spmm_internal.h"
#include "device_util.h"
#include "lane_mapping.h"
#include "scouts.h"

#include <algorithm>

namespace scorch {

// Address of row c of B as seen by one lane (base = B + the lane's column offset): one 32x32->64-bit multiply
// and one shift-add (c >= 0 and the row stride fit 32 bits).
__device__ __forceinline__ const float *b_row(const float *base, int c, uint32_t ldb) {
    return base + (uint64_t)(uint32_t)c * ldb;
}

// One batch of U staged entries e, e+es, ... of a row:  acc[t] += val * B[col, boff[t] .. +V).  The U gathers
// are issued before the first multiply so that U reads of B rows are in flight per group.  PRED: entries at or
// past e_end are skipped (last batch of a row); otherwise the batch is whole and nothing is tested per entry.
// How the rows of B outside the hot set are read (hot/cold variants only).  0: streaming (non-temporal) loads, the
// default.  1..3: experiments with the other cache-policy bits of gfx950 loads, issued as buffer loads so that the
// bits can be chosen: 1 = device scope (sc1: not kept in the vector L1), 2 = system scope (sc0 sc1), 3 = sc1 + nt.
struct ColdPath {
    __amdgpu_buffer_rsrc_t rsrc;  // covers B (only used when B is smaller than 4 GB)
    uint32_t ldb_bytes;
};
template <int COLD> __device__ __forceinline__ Vec<4>::type cold_load(const ColdPath &cp, uint32_t byte_off) {
    typedef int i4 __attribute__((ext_vector_type(4)));
    constexpr int aux = COLD == 1 ? 16 : (COLD == 2 ? 17 : 18);
    const i4 raw = __builtin_amdgcn_raw_buffer_load_b128(cp.rsrc, (int)byte_off, 0, aux);
    Vec<4>::type x;
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = __int_as_float(raw[i]);
    return x;
}

template <int V, int T, int U, bool UA, bool HOT, bool PRED, int COLD = 0>
__device__ __forceinline__ void gather_batch(typename Vec<V>::type (&acc)[T], const int *lcol, const float *lval,
                                             int e, int e_end, int es, const float *const (&bbase)[T],
                                             uint32_t ldb, const ColdPath *cp = nullptr, const int *boffb = nullptr) {
    using vec = typename Vec<V>::type;
    vec x[U][T];
    float v[U];
    int c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int ee = e + u * es;
        const bool ok = !PRED || ee < e_end;
        c[u] = lcol[ok ? ee : e];
        v[u] = ok ? lval[ee] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool ok = !PRED || e + u * es < e_end;
        const bool hot = !HOT || c[u] < 0;
        const int cu = HOT ? (c[u] & 0x7fffffff) : c[u];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const float *bp = b_row(bbase[t], cu, ldb);
            if (ok) {
                if (hot) {
                    x[u][t] = vload<V, UA>(bp);
                } else {
                    // the empty statements keep this load from being merged with the one of the other branch
                    // (hoisted above or sunk below the branch, the merged load loses the streaming policy)
                    asm volatile("");
                    if constexpr (COLD == 0 || V != 4) x[u][t] = __builtin_nontemporal_load(reinterpret_cast<const vec *>(bp));
                    else x[u][t] = cold_load<COLD>(*cp, (uint32_t)cu * cp->ldb_bytes + (uint32_t)boffb[t]);
                    asm volatile("");
                }
            } else {
                x[u][t] = vzero<V>();
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int t = 0; t < T; ++t) vfma<V>(acc[t], v[u], x[u][t]);
}

// One lane group accumulates the staged entries e0, e0+es, ... (< e_end) of a row: whole batches first, then
// one partial batch.  boff[t] is a readable offset in every lane (lanes past column n point at the last
// vector of the row), so the loads carry no column test; `active` is false in the lanes whose first vector lies
// past column n: they skip the row altogether.
template <int V, int T, int U, bool UA, bool HOT = false, int COLD = 0>
__device__ __forceinline__ void gather_fma(typename Vec<V>::type (&acc)[T], const int *lcol, const float *lval,
                                           int e0, int e_end, int es, const float *Bc, uint32_t ldb, bool active,
                                           const int (&boff)[T], const ColdPath *cp = nullptr) {
    if (!active) return;
    const float *bbase[T];
    int boffb[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        bbase[t] = Bc + boff[t];
        boffb[t] = boff[t] * 4;
    }
    int e = e0;
    for (; e + (U - 1) * es < e_end; e += U * es)
        gather_batch<V, T, U, UA, HOT, false, COLD>(acc, lcol, lval, e, e_end, es, bbase, ldb, cp, boffb);
    if (e < e_end) gather_batch<V, T, U, UA, HOT, true, COLD>(acc, lcol, lval, e, e_end, es, bbase, ldb, cp, boffb);
}

// Adds up the S = 64/G lane groups of a wavefront (xor butterfly over the lane distances G..32; DPP,
// ds_swizzle or ds_bpermute depending on the distance); every lane ends with the full sum.
template <int V, int G, int T, int OFF = G>
__device__ __forceinline__ void reduce_groups(typename Vec<V>::type (&acc)[T]) {
    if constexpr (OFF < kWave) {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            auto o = vlane_xor<V, OFF>(acc[t]);
            vadd<V>(acc[t], o);
        }
        reduce_groups<V, G, T, OFF * 2>(acc);
    }
}

// A wavefront walks the entries [p0 + first, p1) of one row in chunks of 64 that are `stride`
// apart (stride = 64 for a whole wavefront-row, 256 when 4 wavefronts share a piece).  Each chunk
// is read with one coalesced load per array, parked in LDS, and broadcast from there to the lane
// groups; the next chunk is fetched into registers while the current one is consumed.
__device__ __forceinline__ int mark_hot(int c, const uint32_t *mask) {
    return c | (int)(((mask[c >> 5] >> (c & 31)) & 1u) << 31);
}

template <int V, int G, int T, int U, bool NTA, bool UA, bool HOT = false, int COLD = 0>
__device__ __forceinline__ void row_accumulate(typename Vec<V>::type (&acc)[T], int *lcol, float *lval, int lane,
                                               int grp, int pfirst, int p1, int stride, const int32_t *colidx,
                                               const float *vals, const float *Bc, uint32_t ldb,
                                               bool active, const int (&boff)[T],
                                               const uint32_t *hotmask = nullptr, const ColdPath *cp = nullptr) {
    constexpr int S = kWave / G;
    if constexpr (G == 1 && T == 1 && !HOT) {
        // One-lane groups (n <= 4): every lane owns the entries pfirst + lane + i * stride and needs no broadcast, so
        // the stage is skipped: U index/value pairs are read straight into registers, then U gathers are issued.  A row
        // of up to 64 U entries costs two memory round trips instead of two per 64 entries.  The order in which a lane
        // adds its products is the same as with the stage.
        using vec = typename Vec<V>::type;
        if (!active) return;
        const float *base = Bc + boff[0];
        for (int pb = pfirst + lane; pb - lane < p1; pb += stride * U) {
            int c[U];
            float v[U];
            vec x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int p = pb + u * stride;
                const bool ok = p < p1;
                c[u] = ok ? ld_idx<NTA>(colidx + p) : 0;
                v[u] = ok ? ld_val<NTA>(vals + p) : 0.f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = pb + u * stride < p1 ? vload<V, UA>(b_row(base, c[u], ldb)) : vzero<V>();
#pragma unroll
            for (int u = 0; u < U; ++u) vfma<V>(acc[0], v[u], x[u]);
        }
        return;
    }
    int pc = pfirst + lane;
    int cn = 0;
    float vn = 0.f;
    if (pc < p1) {
        cn = ld_idx<NTA>(colidx + pc);
        vn = ld_val<NTA>(vals + pc);
        if constexpr (HOT) cn = mark_hot(cn, hotmask);
    }
    for (int base = pfirst; base < p1; base += stride) {
        lcol[lane] = cn;
        lval[lane] = vn;
        pc = base + stride + lane;
        if (pc < p1) {
            cn = ld_idx<NTA>(colidx + pc);
            vn = ld_val<NTA>(vals + pc);
            if constexpr (HOT) cn = mark_hot(cn, hotmask);
        }
        wave_lds_sync();
        const int cnt = min(kWave, p1 - base);
        gather_fma<V, T, U, UA, HOT, COLD>(acc, lcol, lval, grp, cnt, S, Bc, ldb, active, boff, cp);
        wave_lds_sync();
    }
}

constexpr int smem_ints_per_wave() { return 2 * kStageMax + kWindowRowsMax + 2; }

template <int V, int G, int T, int U, int NT, bool UA, bool HOT = false, int COLD = 0, bool CUT = false, bool WHOLE = false>
__global__ __launch_bounds__(kBlock) void spmm_fused_kernel(const ExecArgs a) {
    using vec = typename Vec<V>::type;
    constexpr int S = kWave / G;
    constexpr int GV = G * V;
    constexpr int TW = GV * T;
    constexpr bool NTC = (NT & 1) != 0;  // streaming stores for C
    // colidx/vals are read with plain loads (a streaming hint made no difference), except in the hot/cold variants:
    // there the memory-side cache is reserved for the hot rows of B and the 8 bytes per entry of A would only
    // displace them (workload 4: another 2.7 % less time)
    constexpr bool NTA = HOT;

    constexpr bool kOneLane = G == 1 && T == 1 && !HOT;
    __shared__ int s_raw[kOneLane ? 1 : kWavesPerBlock * smem_ints_per_wave()];
    __shared__ float s_red[kWavesPerBlock * TW];
    // one-lane groups (n <= 4) only: the products of a window's entries, summed per row afterwards
    constexpr int kProducts = WHOLE ? kBNMax + kWholeMax : kStageMax;
    __shared__ __attribute__((aligned(16))) float s_prod[G == 1 ? kWavesPerBlock * kProducts * V : 1];
    __shared__ int s_flag;  // piece of a split row: this workgroup drew the row's last ticket

    const int tid = threadIdx.x;
    const int wv = tid >> 6;
    const int lane = tid & 63;
    const int grp = lane / G;
    const int lig = lane % G;

    const uint32_t per_tile = (uint32_t)a.nb_items + (uint32_t)a.nb_wave + (uint32_t)a.nb_win;
    // rows cut by columns come first: workgroup = (column tile * cut_wgs + group of pieces) * 8 + XCD
    const uint32_t cut_grid = CUT ? (uint32_t)a.cut_wgs * (uint32_t)a.ncoltiles * kXcds : 0;
    const bool cut_piece = CUT && blockIdx.x < cut_grid;
    uint32_t ct, b;
    if (cut_piece) {
        b = blockIdx.x / kXcds;
        ct = b / (uint32_t)a.cut_wgs;
        b -= ct * (uint32_t)a.cut_wgs;
        // the XCDs start at different tiles: rows of B are 256-byte blocks of different memory channels side by side, and one tile
        // at a time on all XCDs would use a part of the channels
        ct = (ct + (blockIdx.x & (kXcds - 1))) % (uint32_t)a.ncoltiles;
    } else if (!tile_of_workgroup(a.xcd_slices, a.ncoltiles, per_tile, ct, b, cut_grid)) {
        return;
    }

    // coff[t]: first column of the lane's t-th vector.  With unaligned rows (UA) n need not be a multiple of V:
    // the vector that would run past column n is moved back to end at n, so it overlaps its neighbour and both
    // lanes compute and store the same values for the shared columns.  Vectors wholly past column n (colok false)
    // point at the last vector of the row as well: they may be read, and are never stored.
    const int c0 = (int)ct * TW + lig * V;
    bool colok[T];
    int coff[T], boff[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        colok[t] = (c0 + t * GV) < a.n;
        coff[t] = min(c0 + t * GV, a.n - V);
        // packed B (XCD-sliced mode with a repacked copy): slice ct is a dense k x 32 block
        boff[t] = a.b_tile_stride ? lig * V + t * GV : coff[t];
    }
    const float *Bc = a.b_tile_stride ? a.B + (int64_t)ct * a.b_tile_stride : a.B;
    const uint32_t ldb = (uint32_t)a.ldb;
    ColdPath cold{};
    if constexpr (COLD != 0) {
        cold.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(Bc), 0, (uint32_t)a.b_bytes, 0x00020000);
        cold.ldb_bytes = ldb * 4u;
    }
    const ColdPath *cp = COLD != 0 ? &cold : nullptr;

    int *lcol = kOneLane ? s_raw : s_raw + wv * smem_ints_per_wave();
    float *lval = reinterpret_cast<float *>(lcol + kStageMax);
    int *lrp = lcol + 2 * kStageMax;

    vec acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = vzero<V>();

    if constexpr (CUT) if (cut_piece) {
        // ---- pieces of rows cut by columns: kCutRun of them per wavefront, each to its partial row ----
        // Rows of B are read with the default cache policy here whatever the variant: they are used again.
        const int x = (int)(blockIdx.x & (kXcds - 1));
        const int q0 = ((int)b * kWavesPerBlock + wv) * kCutRun;
        const int nq = min(kCutRun, a.cut_pieces - q0);
        if (nq <= 0) return;
        const int64_t first = (int64_t)x * a.cut_pieces + q0;
        const int2 span = a.cut_spans[first + min(lane, nq - 1)];
        // a piece of up to kCutShort entries is one lane group's (the sum of a piece depends on nothing but the piece)
        const int whole = lane < nq ? span.y - span.x : 0;
        const int len = whole <= kCutShort ? whole : 0;
        int end = len;  // of the piece's entries in the stage
#pragma unroll
        for (int off = 1; off < kCutRun; off <<= 1) {
            const int o = __shfl_up(end, off, kWave);
            if (lane >= off) end += o;
        }
        const int total = __shfl(end, kCutRun - 1, kWave);
        float *dst0 = a.cut_partials + first * a.partial_stride;
        {
            // short pieces: staged together, one lane group per piece
            const int shift = span.x - (end - len);  // from the place in the stage to the entry
            int ends[kCutRun], shifts[kCutRun];
#pragma unroll
            for (int i = 0; i < kCutRun; ++i) {
                ends[i] = __builtin_amdgcn_readlane(end, i);
                shifts[i] = __builtin_amdgcn_readlane(shift, i);
            }
            for (int e = lane; e < total; e += kWave) {
                int sh = shifts[0];
#pragma unroll
                for (int i = 1; i < kCutRun; ++i)
                    if (e >= ends[i - 1]) sh = shifts[i];
                lcol[e] = ld_idx<NTA>(a.colidx + e + sh);
                lval[e] = ld_val<NTA>(a.vals + e + sh);
            }
            if (lane < kCutRun) lrp[lane + 1] = end;
            if (lane == 0) lrp[0] = 0;
            wave_lds_sync();
            const unsigned long long longs = __ballot(whole > kCutShort);
            for (int i = grp; i < nq; i += S) {
                if ((longs >> i) & 1ull) continue;
#pragma unroll
                for (int t = 0; t < T; ++t) acc[t] = vzero<V>();
                gather_fma<V, T, U, UA>(acc, lcol, lval, lrp[i], lrp[i + 1], 1, Bc, ldb, colok[0], boff);
#pragma unroll
                for (int t = 0; t < T; ++t)
                    if (colok[t]) vstore<V, HOT, UA>(dst0 + (int64_t)i * a.partial_stride + coff[t], acc[t]);
            }
            if (longs == 0ull) return;
            wave_lds_sync();  // the stage is used again
        }
        for (int i = 0; i < nq; ++i) {
            const int p0 = __builtin_amdgcn_readlane(span.x, i), p1 = __builtin_amdgcn_readlane(span.y, i);
            if (p1 - p0 <= kCutShort) continue;
#pragma unroll
            for (int t = 0; t < T; ++t) acc[t] = vzero<V>();
            row_accumulate<V, G, T, U, NTA, UA>(acc, lcol, lval, lane, grp, p0, p1, kWave, a.colidx, a.vals, Bc, ldb, colok[0], boff);
            reduce_groups<V, G, T>(acc);
            if (grp == 0) {
#pragma unroll
                for (int t = 0; t < T; ++t)
                    if (colok[t]) vstore<V, HOT, UA>(dst0 + (int64_t)i * a.partial_stride + coff[t], acc[t]);
            }
        }
        return;
    }

    if (b < (uint32_t)a.nb_items) {
        // ---- piece of a long row: 4 wavefronts, LDS tree, then C or a partial row ----
        const int4 it = a.items[b];
        row_accumulate<V, G, T, U, NTA, UA, HOT, COLD>(acc, lcol, lval, lane, grp, it.y + wv * kWave, it.z, kBlock, a.colidx,
                                                       a.vals, Bc, ldb, colok[0], boff, a.hotmask, cp);
        reduce_groups<V, G, T>(acc);
        if (grp == 0) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                if constexpr (V == 1) s_red[wv * TW + t * GV + lig] = acc[t];
                else
#pragma unroll
                    for (int i = 0; i < V; ++i) s_red[wv * TW + t * GV + lig * V + i] = acc[t][i];
            }
        }
        __syncthreads();
        if (wv == 0 && grp == 0) {
            float *dst = it.w < 0 ? a.C + (int64_t)it.x * a.ldc : a.partials + (int64_t)it.w * a.partial_stride;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                if (!colok[t]) continue;
                vec r;
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const int o = t * GV + lig * V + i;
                    float s = s_red[o];
#pragma unroll
                    for (int w = 1; w < kWavesPerBlock; ++w) s += s_red[w * TW + o];
                    if constexpr (V == 1) r = s;
                    else r[i] = s;
                }
                // a partial row gets its epilogue after the pieces are added
                if (it.w < 0) r = apply_epilogue<V>(r, a.bias ? a.bias + coff[t] : nullptr, a.act);
                if (it.w < 0) vstore<V, NTC, UA>(dst + coff[t], r);
                else vstore<V, false, UA>(dst + coff[t], r);
            }
        }
        if (it.w < 0 || a.tickets == nullptr) return;  // whole row done, or the fix-up launch adds the partial rows
        // ---- piece of a split row: the workgroup that arrives last adds up the row's partial rows ----
        // Every piece publishes its partial row (device-scope release), then takes a ticket of the row (integer
        // atomic); the piece that draws the last ticket knows that all partial rows are visible (device-scope
        // acquire) and adds them in piece order, whichever piece it is: the sum does not depend on the arrival order,
        // and no floating-point atomics are involved.  The counter is left at zero for the next launch.
        const int row_p0 = a.rowptr[it.x], row_p1 = a.rowptr[it.x + 1];
        const int piece = (it.y - row_p0) / a.BCH;
        const int pieces = (row_p1 - row_p0 + a.BCH - 1) / a.BCH;
        const int first = it.w - piece;
        if (wv == 0) {
            __threadfence();  // release: this wavefront's stores of the partial row, device-wide
            if (lane == 0) {
                int32_t *tk = a.tickets + ((int64_t)first * a.ncoltiles + ct);
                const int old = atomicAdd(tk, 1);
                const int is_last = old == pieces - 1;
                if (is_last) atomicExch(tk, 0);
                s_flag = is_last;
            }
        }
        __syncthreads();
        if (!s_flag) return;
        __threadfence();  // acquire: the other pieces' partial rows
        {
            const float *src = a.partials + (int64_t)first * a.partial_stride;
            float *dst = a.C + (int64_t)it.x * a.ldc;
            const int cbeg = (int)ct * TW, cend = min(a.n, cbeg + TW);
            for (int c = cbeg + tid; c < cend; c += kBlock) {
                // read past this die's L2: the other pieces may have run on other dies
                float sum = __hip_atomic_load(src + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                for (int i = 1; i < pieces; ++i)
                    sum += __hip_atomic_load(src + (int64_t)i * a.partial_stride + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (a.bias) sum += a.bias[c];
                if (a.act == 1) sum = fmaxf(sum, 0.f);
                dst[c] = sum;
            }
        }
        return;
    }

    if (b < (uint32_t)(a.nb_items + a.nb_wave)) {
        // ---- medium row: one wavefront, groups interleave entries, shuffle reduction ----
        const int idx = (int)(b - a.nb_items) * kWavesPerBlock + wv;
        if (idx >= a.n_wave_rows) return;
        const int row = a.wave_rows[idx];
        const int2 span = a.wave_span[idx];  // the row's entry range, kept in the plan beside its id
        const int p0 = span.x, p1 = span.y;
        if (CUT && p1 - p0 >= a.cut_len) return;
        row_accumulate<V, G, T, U, NTA, UA, HOT, COLD>(acc, lcol, lval, lane, grp, p0, p1, kWave, a.colidx, a.vals, Bc, ldb,
                                                       colok[0], boff, a.hotmask, cp);
        reduce_groups<V, G, T>(acc);
        if (grp == 0) {
            float *dst = a.C + (int64_t)row * a.ldc;
#pragma unroll
            for (int t = 0; t < T; ++t)
                if (colok[t]) vstore<V, NTC, UA>(dst + coff[t], apply_epilogue<V>(acc[t], a.bias ? a.bias + coff[t] : nullptr, a.act));
        }
        return;
    }

    // ---- window of consecutive short rows ----
    const int w = (int)(b - a.nb_items - a.nb_wave) * kWavesPerBlock + wv;
    if (w >= a.n_windows) return;
    const int r0 = a.win_row_start[w];
    const int r1 = a.win_row_start[w + 1];
    const int nr = min(r1 - r0, kWindowRowsMax);
    if constexpr (WHOLE) {
        // One or two columns: a row of up to kWholeMax entries is walked here whatever its class, so that no entry between two short
        // rows is gathered in vain and medium rows need no wavefronts of their own.  A longer row can only be the last of its window
        // (rows start within kBNMax entries of each other).  A lane adds up a row of up to kLaneRow entries, the wavefront the others.
        if (nr <= 0) return;
        const int rp = a.rowptr[r0 + min(lane, nr)];
        const int next = __shfl_down(rp, 1, kWave), end = a.rowptr[r0 + nr];
        const int len = (lane == kWave - 1 ? end : next) - rp;
        const int first = __builtin_amdgcn_readlane(rp, 0);
        const int last = __builtin_amdgcn_readlane(rp, nr - 1);
        const int count = (end - last <= kWholeMax ? end : last) - first;
        vec *prod = reinterpret_cast<vec *>(s_prod) + wv * kProducts;
        constexpr int kSteps = kProducts / kWave;
        vec x[kSteps];
        float v[kSteps];
        int c[kSteps];
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
            const int e = lane + i * kWave;
            c[i] = e < count ? a.colidx[first + e] : 0;
            v[i] = e < count ? a.vals[first + e] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < kSteps; ++i) x[i] = lane + i * kWave < count ? vload<V, UA>(b_row(Bc, c[i], ldb) + boff[0]) : vzero<V>();
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
            vec pr = vzero<V>();
            vfma<V>(pr, v[i], x[i]);
            if (lane + i * kWave < count) prod[lane + i * kWave] = pr;
        }
        wave_lds_sync();
        const float *bias = a.bias ? a.bias + coff[0] : nullptr;
        if (lane < nr && len <= kLaneRow) {
            vec sum = vzero<V>();
            for (const vec *q = prod + (rp - first), *e = q + len; q < e; ++q) vadd<V>(sum, *q);
            vstore<V, NTC, UA>(a.C + (int64_t)(r0 + lane) * a.ldc + coff[0], apply_epilogue<V>(sum, bias, a.act));
        }
        for (unsigned long long todo = __ballot(lane < nr && len > kLaneRow && len <= kWholeMax); todo != 0ull; todo &= todo - 1ull) {
            const int i = __builtin_ctzll(todo);
            const int q0 = __builtin_amdgcn_readlane(rp, i) - first, n = __builtin_amdgcn_readlane(len, i);
            vec sum[1] = {vzero<V>()};
            // every lane still holds its values and gathered elements: fused multiply-adds, as everywhere for rows of this length
#pragma unroll
            for (int s = 0; s < kSteps; ++s)
                if ((uint32_t)(lane + s * kWave - q0) < (uint32_t)n) vfma<V>(sum[0], v[s], x[s]);
            reduce_groups<V, G, 1>(sum);
            if (lane == 0) vstore<V, NTC, UA>(a.C + (int64_t)(r0 + i) * a.ldc + coff[0], apply_epilogue<V>(sum[0], bias, a.act));
        }
        return;
    }
    // which entries the window stages is known from the plan, so colidx/vals are requested together with the row
    // pointers instead of after them
    const int2 stg = a.win_stage[w];
    if (stg.y < 0) return;  // no short row in this window
    const int sbeg = stg.x, cnt = stg.y;
    const int rpv = a.rowptr[r0 + min(lane, nr)];
    const int rlast = a.rowptr[r0 + nr];
    int rnext = __shfl_down(rpv, 1, kWave);
    if (lane == kWave - 1) rnext = rlast;
    const bool is_short = lane < nr && (rnext - rpv) <= a.LW;
    if constexpr (G == 1) {
        // SpMV and its neighbours (n <= 4, one lane per entry): a window has far fewer rows than the wavefront has
        // lanes, so the lanes split the window's *entries* instead of its rows: every lane reads its entries
        // (coalesced), gathers the V values of B they point at, and parks the products in LDS; then the lane of
        // each short row adds up that row's products in stored order.
        vec *prod = reinterpret_cast<vec *>(s_prod) + wv * kProducts;
        constexpr int kSteps = (kStageMax + kWave - 1) / kWave;
        vec x[kSteps];
        float v[kSteps];
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
            const int e = lane + i * kWave;
            const bool ok = e < cnt;
            const int c = ok ? a.colidx[sbeg + e] : 0;
            v[i] = ok ? a.vals[sbeg + e] : 0.f;
            x[i] = ok ? vload<V, UA>(b_row(Bc, c, ldb) + boff[0]) : vzero<V>();
        }
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
            const int e = lane + i * kWave;
            if (e < cnt) {
                vec pr = vzero<V>();
                vfma<V>(pr, v[i], x[i]);
                prod[e] = pr;
            }
        }
        wave_lds_sync();
        if (is_short) {
            for (int q = rpv - sbeg; q < rnext - sbeg; ++q) vadd<V>(acc[0], prod[q]);
            vstore<V, NTC, UA>(a.C + (int64_t)(r0 + lane) * a.ldc + coff[0],
                           apply_epilogue<V>(acc[0], a.bias ? a.bias + coff[0] : nullptr, a.act));
        }
        return;
    }
    for (int e = lane; e < cnt; e += kWave) {
        int c = ld_idx<NTA>(a.colidx + sbeg + e);
        if constexpr (HOT) c = mark_hot(c, a.hotmask);
        lcol[e] = c;
        lval[e] = ld_val<NTA>(a.vals + sbeg + e);
    }
    lrp[lane] = rpv;
    if (lane == 0) lrp[nr] = rlast;
    // the lane's bias values are the same for every row of the window: read once
    const bool has_bias = a.bias != nullptr;
    vec bias_r[T];
#pragma unroll
    for (int t = 0; t < T; ++t) bias_r[t] = (has_bias && colok[t]) ? vload<V, UA>(a.bias + coff[t]) : vzero<V>();
    wave_lds_sync();
    for (int ri = grp; ri < nr; ri += S) {
        const int q0 = lrp[ri], q1 = lrp[ri + 1];
        if (q1 - q0 > a.LW) continue;  // medium/long row: handled by another path
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] = vzero<V>();
        gather_fma<V, T, U, UA, HOT, COLD>(acc, lcol, lval, q0 - sbeg, q1 - sbeg, 1, Bc, ldb, colok[0], boff, cp);
        float *dst = a.C + (int64_t)(r0 + ri) * a.ldc;
#pragma unroll
        for (int t = 0; t < T; ++t)
            if (colok[t]) vstore<V, NTC, UA>(dst + coff[t], apply_epilogue_reg<V>(acc[t], has_bias, bias_r[t], a.act));
    }
}

// Plan-free path for matrices of few rows (a batch of sparse activations): one workgroup per row and per tile of at
// most 32 columns.  The run kernel below gives a row to one wavefront and covers as many columns as a wavefront can, so
// a matrix of 64 rows would occupy 16 compute units; here the NW wavefronts of a workgroup take interleaved chunks of
// the row, its lane groups (8 lanes, one 128-byte line of a row of B) interleaved entries, and the column tiles are
// dealt over the dies.  Bound by the latency of two dependent reads (entries, rows of B) per chunk, hence chunks of
// 128 entries, all of whose gathers are in flight at once (64 rows x 2458 entries, n = 256, operands in the memory-side cache: 62.0 -> 11.7 us).
constexpr int kRowChunk = 128;

template <int V, int G, bool UA, int NW>
__global__ __launch_bounds__(NW * kWave) void spmm_row_kernel(const ExecArgs a) {
    using vec = typename Vec<V>::type;
    constexpr int S = kWave / G;
    constexpr int TW = G * V;
    constexpr int U = kRowChunk / S >= 16 ? 16 : kRowChunk / S;
    constexpr int kPer = kRowChunk / kWave;
    __shared__ int s_col[NW][kRowChunk];
    __shared__ float s_val[NW][kRowChunk];
    __shared__ float s_red[NW * TW];
    const int tid = threadIdx.x;
    const int wv = tid >> 6;
    const int lane = tid & 63;
    const int grp = lane / G;
    const int lig = lane % G;
    uint32_t ct, row;
    if (!tile_of_workgroup(a.xcd_slices, a.ncoltiles, (uint32_t)a.m, ct, row)) return;  // the same for the whole workgroup
    const int c0 = (int)ct * TW + lig * V;
    const bool colok = c0 < a.n;
    const int coff[1] = {min(c0, a.n - V)};  // see spmm_fused_kernel
    const uint32_t ldb = (uint32_t)a.ldb;
    int *lcol = s_col[wv];
    float *lval = s_val[wv];
    // unsigned: an index past the end of a list of nearly 2^31 entries must not turn negative
    const uint32_t p0 = (uint32_t)a.rowptr[row], p1 = (uint32_t)a.rowptr[row + 1];
    constexpr uint32_t kStride = NW * kRowChunk;
    int cn[kPer];
    float vn[kPer];
    auto fetch = [&](uint32_t base) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const uint32_t p = base + i * kWave + lane;
            cn[i] = p < p1 ? a.colidx[p] : 0;
            vn[i] = p < p1 ? a.vals[p] : 0.f;
        }
    };
    vec acc[1] = {vzero<V>()};
    fetch(p0 + wv * kRowChunk);
    for (uint32_t base = p0 + wv * kRowChunk; base < p1; base += kStride) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            lcol[i * kWave + lane] = cn[i];
            lval[i * kWave + lane] = vn[i];
        }
        fetch(base + kStride);
        wave_lds_sync();
        gather_fma<V, 1, U, UA>(acc, lcol, lval, grp, (int)min((uint32_t)kRowChunk, p1 - base), S, a.B, ldb, colok, coff);
        wave_lds_sync();
    }
    reduce_groups<V, G, 1>(acc);
    if (grp == 0) {
        if constexpr (V == 1) s_red[wv * TW + lig] = acc[0];
        else
#pragma unroll
            for (int i = 0; i < V; ++i) s_red[wv * TW + lig * V + i] = acc[0][i];
    }
    __syncthreads();
    if (wv == 0 && grp == 0 && colok) {
        vec r;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            float sum = s_red[lig * V + i];
#pragma unroll
            for (int w = 1; w < NW; ++w) sum += s_red[w * TW + lig * V + i];
            if constexpr (V == 1) r = sum;
            else r[i] = sum;
        }
        vstore<V, true, UA>(a.C + (int64_t)row * a.ldc + coff[0], r);
    }
}

// Plan-free path: rows in natural order, a run of up to kNaturalRowsMax consecutive rows per wavefront (the host
// picks the run length from m alone, so that the grid still fills the chip; nothing about the row lengths is known
// before the launch).  A wavefront reads the row pointers of its run once (a lane per row) and then proceeds
// greedily: the next rows, as long as they are short (up to kNaturalShort entries) and fit the LDS stage together,
// are staged with coalesced reads and walked one row per lane group, like a window of the planned path; a longer
// row is streamed through the stage by the whole wavefront, the lane groups taking interleaved entries.
//
// Rows that are long beside the others (long_row_limit) are left to the workgroups at the front of the grid, the scouts.  A scout
// looks at rows from all over the matrix (scout_first, scout_place) and takes the long ones one after the other, all 4
// wavefronts together (interleaved 64-entry chunks, LDS tree, twice the gathers in flight), so that the longest rows
// start first and run beside everything else.  Neither the order of the rows nor how many of them are long leaves them to
// few workgroups.  Measured, us, against workgroups that each look through a stretch of 64 to 1024 neighbouring rows: graph of 169 343
// rows (longest 10 316 entries), n = 128, random order 140 -> 138, longest rows first 1149 -> 116; 16 384 rows, every
// fourth of 1000 entries, n = 64 69 -> 44; 16 000 rows of 6, n = 16 7.6 -> 7.2.
constexpr int kNaturalRowsMax = 16;
constexpr int kNaturalShort = 32;

// Position of the first bit from `from` on in the 256 bits of a workgroup (256 if there is none).
__device__ __forceinline__ int next_long(const unsigned long long *bits, int from) {
    for (int w = from / kWave; w < kWavesPerBlock; ++w) {
        unsigned long long x = bits[w];
        if (w == from / kWave) x &= ~0ull << (from % kWave);
        if (x != 0ull) return __builtin_amdgcn_readfirstlane(w * kWave + __builtin_ctzll(x));
    }
    return kBlock;
}

template <int V, int G, int T, int U, int NT, bool UA, int SU>
__global__ __launch_bounds__(kBlock) void spmm_natural_kernel(const ExecArgs a) {
    using vec = typename Vec<V>::type;
    constexpr int S = kWave / G;
    constexpr int GV = G * V;
    constexpr int TW = GV * T;
    constexpr bool NTC = (NT & 1) != 0;
    __shared__ int s_raw[kWavesPerBlock * smem_ints_per_wave()];
    __shared__ float s_red[kWavesPerBlock * TW];
    __shared__ unsigned long long s_longs[kWavesPerBlock];  // scouts: which rows are long, and their entries
    __shared__ int2 s_span[kBlock];
    const int tid = threadIdx.x;
    const int wv = tid >> 6;
    const int lane = tid & 63;
    const int grp = lane / G;
    const int lig = lane % G;
    const uint32_t per_tile = (uint32_t)a.nb_items + (uint32_t)a.nb_wave;
    uint32_t ct, b;
    if (!tile_of_workgroup(a.xcd_slices, a.ncoltiles, per_tile, ct, b)) return;  // the same for the whole workgroup
    const int NR = a.rows_per_wave;  // a power of two
    const int c0 = (int)ct * TW + lig * V;
    bool colok[T];
    int coff[T];  // see spmm_fused_kernel
#pragma unroll
    for (int t = 0; t < T; ++t) {
        colok[t] = (c0 + t * GV) < a.n;
        coff[t] = min(c0 + t * GV, a.n - V);
    }
    const uint32_t ldb = (uint32_t)a.ldb;
    int *lcol = s_raw + wv * smem_ints_per_wave();
    float *lval = reinterpret_cast<float *>(lcol + kStageMax);
    int *lrp = lcol + 2 * kStageMax;
    vec acc[T];

    const bool scout = b < (uint32_t)a.nb_items;
    const int long_limit = long_row_limit((uint32_t)a.rowptr[a.m], a.one_over_m);
    const int64_t r0 = ((int64_t)(b - (uint32_t)a.nb_items) * kWavesPerBlock + wv) * NR;
    const int nr = scout ? 0 : (int)max((int64_t)0, min((int64_t)NR, (int64_t)a.m - r0));
    const int rpv = nr > 0 ? a.rowptr[r0 + min(lane, nr)] : 0;
    const int rnext = __shfl_down(rpv, 1, kWave);  // lanes past the run hold the last pointer; lane 63 is never a row
    lrp[lane] = rpv;
    wave_lds_sync();
    int i = 0;
    while (i < nr) {
        const int base = lrp[i];
        // rows i .. j-1: the longest run of short rows (one lane group walks a row alone, so only rows of up to
        // kNaturalShort entries qualify) that fits the stage
        const bool stops = lane >= i && (lane >= nr || rnext - rpv > kNaturalShort || rnext - base > kStageMax);
        const int j = __builtin_ctzll(__ballot(stops));  // lane nr always stops
        if (j == i) {
            const int p1 = lrp[i + 1];
            if (p1 - base <= long_limit) {
#pragma unroll
                for (int t = 0; t < T; ++t) acc[t] = vzero<V>();
                row_accumulate<V, G, T, U, false, UA>(acc, lcol, lval, lane, grp, base, p1, kWave, a.colidx, a.vals,
                                                      a.B, ldb, colok[0], coff);
                reduce_groups<V, G, T>(acc);
                if (grp == 0) {
                    float *dst = a.C + (r0 + i) * a.ldc;
#pragma unroll
                    for (int t = 0; t < T; ++t)
                        if (colok[t]) vstore<V, NTC, UA>(dst + coff[t], acc[t]);
                }
            }
            ++i;
            continue;
        }
        const int cnt = min(lrp[j] - base, kStageMax);
        for (int e = lane; e < cnt; e += kWave) {
            lcol[e] = a.colidx[base + e];
            lval[e] = a.vals[base + e];
        }
        wave_lds_sync();
        for (int ri = i + grp; ri < j; ri += S) {
#pragma unroll
            for (int t = 0; t < T; ++t) acc[t] = vzero<V>();
            gather_fma<V, T, U, UA>(acc, lcol, lval, lrp[ri] - base, lrp[ri + 1] - base, 1, a.B, ldb, colok[0], coff);
            float *dst = a.C + (r0 + ri) * a.ldc;
#pragma unroll
            for (int t = 0; t < T; ++t)
                if (colok[t]) vstore<V, NTC, UA>(dst + coff[t], acc[t]);
        }
        wave_lds_sync();  // the stage is refilled next
        i = j;
    }
    if (!scout) return;

    // ---- scout: 256 rows at a time, all wavefronts on each long one ----
    for (int64_t first = scout_first(b, a.nb_items, a.scout_shift); first < a.m; first += kBlock * a.nb_items) {
        const int64_t mine = first + scout_place(tid, a.nb_items, a.scout_shift);
        int q0 = 0, q1 = 0;
        if (mine < a.m) {
            q0 = a.rowptr[mine];
            q1 = a.rowptr[mine + 1];
        }
        const unsigned long long longs = __ballot(q1 - q0 > long_limit);
        if (lane == 0) s_longs[wv] = longs;
        if (q1 - q0 > long_limit) s_span[tid] = make_int2(q0, q1);
        __syncthreads();
        for (int i = next_long(s_longs, 0); i < kBlock; i = next_long(s_longs, i + 1)) {  // the same for the whole workgroup
            const int2 span = s_span[i];
            const int p0 = span.x, p1 = span.y;
#pragma unroll
            for (int t = 0; t < T; ++t) acc[t] = vzero<V>();
            row_accumulate<V, G, T, SU, false, UA>(acc, lcol, lval, lane, grp, p0 + wv * kWave, p1, kBlock, a.colidx,
                                                      a.vals, a.B, ldb, colok[0], coff);
            reduce_groups<V, G, T>(acc);
            __syncthreads();  // s_red of the previous row has been read
            if (grp == 0) {
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    if constexpr (V == 1) s_red[wv * TW + t * GV + lig] = acc[t];
                    else
#pragma unroll
                        for (int i = 0; i < V; ++i) s_red[wv * TW + t * GV + lig * V + i] = acc[t][i];
                }
            }
            __syncthreads();
            if (wv == 0 && grp == 0) {
                float *dst = a.C + (first + scout_place(i, a.nb_items, a.scout_shift)) * a.ldc;
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    if (!colok[t]) continue;
                    vec out;
#pragma unroll
                    for (int j = 0; j < V; ++j) {
                        const int o = t * GV + lig * V + j;
                        float sum = s_red[o];
#pragma unroll
                        for (int x = 1; x < kWavesPerBlock; ++x) sum += s_red[x * TW + o];
                        if constexpr (V == 1) out = sum;
                        else out[j] = sum;
                    }
                    vstore<V, NTC, UA>(dst + coff[t], out);
                }
            }
        }
        __syncthreads();  // the list has been read
    }
}

// Copies B (k x n, row stride ldb) into slice-major order: slice s is a dense k x W block holding
// columns [W s, W s + W).  A column slice of a row-major B with a large power-of-two row stride
// lands in few L2 sets; the dense copy makes a slice a contiguous range that an XCD's L2 keeps
// (W = 32, gather kernel) or that streams as whole kilobyte rows into LDS (W = 256, panel kernel).
__global__ __launch_bounds__(kBlock) void spmm_pack_b_kernel(const float *B, int64_t ldb, int32_t k, int32_t n,
                                                             int32_t W, float *Bp) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const int quads = (n + 3) / 4;  // n % 4 == 0 is guaranteed by the caller
    const int64_t total = (int64_t)k * quads;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < total; i += (int64_t)gridDim.x * kBlock) {
        const int64_t r = i / quads;
        const int c = (int)(i - r * quads) * 4;
        const f4 v = *reinterpret_cast<const f4 *>(B + r * ldb + c);
        const int s = c / W;
        *reinterpret_cast<f4 *>(Bp + ((int64_t)s * k + r) * W + (c - s * W)) = v;
    }
}

scorch_status_t launch_pack_b(const float *B, int64_t ldb, int32_t k, int32_t n, int32_t W, float *Bp,
                              hipStream_t stream) {
    const int64_t quads = (int64_t)k * (n / 4);
    if (quads == 0) return SCORCH_OK;
    const uint32_t pgrid = (uint32_t)std::min<int64_t>((quads + kBlock - 1) / kBlock, 256 * 32);
    hipLaunchKernelGGL(spmm_pack_b_kernel, dim3(pgrid), dim3(kBlock), 0, stream, B, ldb, k, n, W, Bp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "launch spmm_pack_b_kernel");
    return SCORCH_OK;
}

// Rows cut into several pieces: add the partial rows in piece order.
__global__ __launch_bounds__(kBlock) void spmm_fixup_kernel(const FixupArgs a) {
    const int s = blockIdx.x;
    if (s >= a.n_split) return;
    const int4 d = a.split[s];
    const float *src = a.partials + (int64_t)d.y * a.partial_stride;
    float *dst = a.C + (int64_t)d.x * a.ldc;
    for (int c = threadIdx.x; c < a.n; c += kBlock) {
        float sum = src[c];
        for (int i = 1; i < d.z; ++i) sum += src[(int64_t)i * a.partial_stride + c];
        if (a.bias) sum += a.bias[c];
        if (a.act == 1) sum = fmaxf(sum, 0.f);
        dst[c] = sum;
    }
}

// ------------------------------------------------------------------------------------------
// host side: pick the lane mapping from n and the operand alignment, then launch
// ------------------------------------------------------------------------------------------

static int64_t grid_size(const Mapping &mp, int64_t per_tile) {
    return xcd_grid_size(mp.xcd_slices, mp.ncoltiles, per_tile);
}

typedef void (*kernel_fn)(const ExecArgs);

// Compiled variants: V = 4 with every group size, aligned or not; V = 2 and V = 1 only occur for n < 4, i.e. with
// groups of 1, 2 or 4 lanes.
#define SCORCH_PICK_NT(KERNEL, V, G, T, U, UA)                              \
    if (NT & 1) return KERNEL<V, G, T, U, 1, UA>;                           \
    return KERNEL<V, G, T, U, 0, UA>;
#define SCORCH_PICK_U(KERNEL, V, G, T, UA)                                  \
    if (U >= 8) { SCORCH_PICK_NT(KERNEL, V, G, T, 8, UA) } else { SCORCH_PICK_NT(KERNEL, V, G, T, 4, UA) }
#define SCORCH_PICK_G4(KERNEL, UA)                                          \
    if (T == 2) { SCORCH_PICK_U(KERNEL, 4, 64, 2, UA) }                     \
    switch (G) {                                                            \
        case 1: SCORCH_PICK_U(KERNEL, 4, 1, 1, UA)                          \
        case 2: SCORCH_PICK_U(KERNEL, 4, 2, 1, UA)                          \
        case 4: SCORCH_PICK_U(KERNEL, 4, 4, 1, UA)                          \
        case 8: SCORCH_PICK_U(KERNEL, 4, 8, 1, UA)                          \
        case 16: SCORCH_PICK_U(KERNEL, 4, 16, 1, UA)                        \
        case 32: SCORCH_PICK_U(KERNEL, 4, 32, 1, UA)                        \
        default: SCORCH_PICK_U(KERNEL, 4, 64, 1, UA)                        \
    }
#define SCORCH_PICK(KERNEL)                                                 \
    if (V == 4) {                                                           \
        if (UA) { SCORCH_PICK_G4(KERNEL, true) } else { SCORCH_PICK_G4(KERNEL, false) } \
    }                                                                       \
    if (V == 2) { SCORCH_PICK_U(KERNEL, 2, 1, 1, false) }                   \
    switch (G) {                                                            \
        case 1: SCORCH_PICK_U(KERNEL, 1, 1, 1, false)                       \
        case 2: SCORCH_PICK_U(KERNEL, 1, 2, 1, false)                       \
        default: SCORCH_PICK_U(KERNEL, 1, 4, 1, false)                      \
    }

static kernel_fn pick_fused(int V, int G, int T, int U, int NT, bool UA) { SCORCH_PICK(spmm_fused_kernel) }
// Windows that walk whole rows: one lane per group, one or two columns.
static kernel_fn pick_fused_whole(int V, int U, int NT) {
#define SCORCH_WHOLE(V)                                                                                            \
    return U >= 8 ? (NT & 1 ? spmm_fused_kernel<V, 1, 1, 8, 1, false, false, 0, false, true>                       \
                            : spmm_fused_kernel<V, 1, 1, 8, 0, false, false, 0, false, true>)                      \
                  : (NT & 1 ? spmm_fused_kernel<V, 1, 1, 4, 1, false, false, 0, false, true>                       \
                            : spmm_fused_kernel<V, 1, 1, 4, 0, false, false, 0, false, true>);
    if (V == 2) { SCORCH_WHOLE(2) }
    SCORCH_WHOLE(1)
#undef SCORCH_WHOLE
}
static kernel_fn pick_fused_hot(int G, int T, int cold) {
    // experiments with the cache policy of the cold rows: whole rows of 97..128 columns only
    if (G == 32 && T == 1 && cold == 1) return spmm_fused_kernel<4, 32, 1, 8, 1, false, true, 1>;
    if (G == 32 && T == 1 && cold == 2) return spmm_fused_kernel<4, 32, 1, 8, 1, false, true, 2>;
    if (G == 32 && T == 1 && cold == 3) return spmm_fused_kernel<4, 32, 1, 8, 1, false, true, 3>;
    if (T == 2) return spmm_fused_kernel<4, 64, 2, 8, 1, false, true>;
    switch (G) {
        case 8: return spmm_fused_kernel<4, 8, 1, 8, 1, false, true>;
        case 16: return spmm_fused_kernel<4, 16, 1, 8, 1, false, true>;
        case 32: return spmm_fused_kernel<4, 32, 1, 8, 1, false, true>;
        default: return spmm_fused_kernel<4, 64, 1, 8, 1, false, true>;
    }
}
// With rows cut by columns: groups of 8 lanes and more, one unroll depth, streaming stores, the plain hot/cold variant.
static kernel_fn pick_fused_cut(int G, int T, bool UA, bool hot) {
#define SCORCH_CUT(G, T)                                                                                                \
    return hot ? spmm_fused_kernel<4, G, T, 8, 1, false, true, 0, true>                                                 \
               : (UA ? spmm_fused_kernel<4, G, T, 8, 1, true, false, 0, true> : spmm_fused_kernel<4, G, T, 8, 1, false, false, 0, true>);
    if (T == 2) { SCORCH_CUT(64, 2) }
    switch (G) {
        case 8: SCORCH_CUT(8, 1)
        case 16: SCORCH_CUT(16, 1)
        case 32: SCORCH_CUT(32, 1)
        default: SCORCH_CUT(64, 1)
    }
#undef SCORCH_CUT
}
// The plan-free path is compiled for one unroll depth (8) and streaming stores only.
#define SCORCH_NATURAL(V, G, T, UA) return spmm_natural_kernel<V, G, T, 8, 1, UA, G == 8 ? 8 : 16>;
#define SCORCH_NATURAL_G4(UA)                                               \
    if (T == 2) { SCORCH_NATURAL(4, 64, 2, UA) }                            \
    switch (G) {                                                            \
        case 1: SCORCH_NATURAL(4, 1, 1, UA)                                 \
        case 2: SCORCH_NATURAL(4, 2, 1, UA)                                 \
        case 4: SCORCH_NATURAL(4, 4, 1, UA)                                 \
        case 8: SCORCH_NATURAL(4, 8, 1, UA)                                 \
        case 16: SCORCH_NATURAL(4, 16, 1, UA)                               \
        case 32: SCORCH_NATURAL(4, 32, 1, UA)                               \
        default: SCORCH_NATURAL(4, 64, 1, UA)                               \
    }
static kernel_fn pick_natural(int V, int G, int T, bool UA) {
    if (V == 4) {
        if (UA) { SCORCH_NATURAL_G4(true) } else { SCORCH_NATURAL_G4(false) }
    }
    if (V == 2) { SCORCH_NATURAL(2, 1, 1, false) }
    switch (G) {
        case 1: SCORCH_NATURAL(1, 1, 1, false)
        case 2: SCORCH_NATURAL(1, 2, 1, false)
        default: SCORCH_NATURAL(1, 4, 1, false)
    }
}

template <int NW> static kernel_fn pick_row(int V, int G, bool UA) {
#define SCORCH_ROW_G4(UA)                              \
    switch (G) {                                       \
        case 1: return spmm_row_kernel<4, 1, UA, NW>;  \
        case 2: return spmm_row_kernel<4, 2, UA, NW>;  \
        case 4: return spmm_row_kernel<4, 4, UA, NW>;  \
        default: return spmm_row_kernel<4, 8, UA, NW>; \
    }
    if (V == 4) {
        if (UA) { SCORCH_ROW_G4(true) } else { SCORCH_ROW_G4(false) }
    }
#undef SCORCH_ROW_G4
    if (V == 2) return spmm_row_kernel<2, 1, false, NW>;
    switch (G) {
        case 1: return spmm_row_kernel<1, 1, false, NW>;
        case 2: return spmm_row_kernel<1, 2, false, NW>;
        default: return spmm_row_kernel<1, 4, false, NW>;
    }
}

static inline int64_t ceil_div64(int64_t a, int64_t b) { return (a + b - 1) / b; }

scorch_status_t launch_planned(const scorch_spmm_plan_t *plan, const int32_t *rowptr, const int32_t *colidx,
                               const float *vals, const float *B, int64_t ldb, float *C, int64_t ldc,
                               const float *bias, int32_t act, hipStream_t stream) {
    if (plan->params.PANEL && panel_operands_ok(plan->n, B, ldb, C, ldc))
        return launch_panel(plan, rowptr, colidx, vals, B, ldb, C, ldc, bias, act, stream);
    if (plan->params.RES) return launch_resident(plan, colidx, vals, B, ldb, C, ldc, bias, act, stream);
    const Mapping mp = pick_mapping(plan->n, B, ldb, C, ldc, plan->params.SLICED);
    ExecArgs a{};
    a.rowptr = rowptr;
    a.colidx = colidx;
    a.vals = vals;
    a.B = B;
    a.C = C;
    a.ldb = ldb;
    a.ldc = ldc;
    a.m = plan->m;
    a.n = plan->n;
    char *ws = plan->workspace;
    a.win_row_start = reinterpret_cast<const int32_t *>(ws + plan->layout.off_win);
    a.win_stage = reinterpret_cast<const int2 *>(ws + plan->layout.off_stage);
    a.wave_rows = reinterpret_cast<const int32_t *>(ws + plan->layout.off_wave);
    a.wave_span = reinterpret_cast<const int2 *>(ws + plan->layout.off_wave_span);
    a.items = reinterpret_cast<const int4 *>(ws + plan->layout.off_items);
    a.partials = reinterpret_cast<float *>(ws + plan->layout.off_partials);
    // Partial rows of split rows are added by a second, small launch.  Adding them inside the fused launch, by the piece
    // that arrives last, is built and tested but off by default (fix=1 in the tuning text turns it on): with proper
    // device-scope release/acquire fences every piece makes its die write back and invalidate its L2, which cost 90 us
    // on the mid-size graph workload (213 against 123 us).  A variant with written-through atomic stores instead of
    // fences saved 3.5 us there, but the order between the partial row and the ticket then rests on when a
    // written-through store counts as complete, which the language-level memory model does not promise: not kept.
    const bool fold = plan->n_split > 0 && plan->tuning.fix > 0;
    a.tickets = fold ? reinterpret_cast<int32_t *>(ws + plan->layout.off_tickets) : nullptr;
    a.BCH = plan->params.BCH;
    a.n_windows = (int32_t)plan->layout.n_windows;
    a.n_wave_rows = plan->n_wave;
    a.n_items = plan->n_items;
    a.nb_items = plan->n_items;
    a.nb_wave = (int32_t)ceil_div64(plan->n_wave, kWavesPerBlock);
    a.nb_win = plan->n_short > 0 ? (int32_t)ceil_div64(plan->layout.n_windows, kWavesPerBlock) : 0;
    // One or two columns, mean row of up to 32 entries: medium rows stay with their windows.  Bound by L2 requests, one per entry, and the
    // chain of reads of every wavefront: fewer of both.  us before / after, n = 1: 169 343 rows, 2.5 M entries 18.9 / 16.3; 600 000 rows of 8
    // 35.2 / 29.1, of 25 95 / 76; 1.5 M rows of 4 55 / 46; 120 000 of 7 8.7 / 8.1, of 4 6.8 / 6.8.  Rows of 164 (all medium) 11.2 / 15.8, 600 000 of
    // 40 even, hence the mean.  A wavefront reads whole windows of 512 entries at once, which does not pay where windows are small (2000 rows of
    // 4, n = 2 4.2 / 4.5; 20 000 of 5 5.1 / 5.3) or where hardly a row is medium (30 000 rows of 30 6.3 / 6.8, of 10 4.7 / 5.1).
    // They have a kernel of their own: with both in one, rows of 30 took 7.6 instead of 7.1 us.  Rows beyond CH are among the items: with a smaller CH they would be a window's too.
    const bool whole_rows = mp.G == 1 && mp.V <= 2 && plan->params.CH == kWholeMax && plan->params.BN >= 128 && plan->nnz <= kLaneRow * (int64_t)plan->m &&
                   (int64_t)plan->n_wave * 256 >= plan->m;
    if (whole_rows) {
        a.nb_wave = 0;
        a.nb_win = (int32_t)ceil_div64(plan->layout.n_windows, kWavesPerBlock);
    }
    a.partial_stride = plan->layout.partial_stride;
    a.LW = plan->params.LW;
    a.ncoltiles = mp.ncoltiles;
    a.xcd_slices = mp.xcd_slices;
    a.bias = bias;
    a.act = act;
    const bool cut = plan->cut_pieces > 0;
    if (cut) {
        a.cut_spans = reinterpret_cast<const int2 *>(ws + plan->layout.off_cut_spans);
        a.cut_partials = reinterpret_cast<float *>(ws + plan->layout.off_cut_partials);
        a.cut_pieces = plan->cut_pieces;
        a.cut_len = plan->cut_len;
        a.cut_wgs = (int32_t)ceil_div64(plan->cut_pieces, kWavesPerBlock * kCutRun);
        a.nb_items = 0;  // every row among the items is cut by columns instead
    }
    const int64_t per_tile = (int64_t)a.nb_items + a.nb_wave + a.nb_win;
    const int64_t grid = grid_size(mp, per_tile) + (int64_t)a.cut_wgs * mp.ncoltiles * kXcds;
    if (grid > 0x7fffffffLL) {
        set_error("launch grid of %lld workgroups exceeds the HIP limit", (long long)grid);
        return SCORCH_ERR_UNSUPPORTED;
    }
    if (grid > 0 && mp.xcd_slices != 0 && plan->params.PACK && plan->k > 0) {
        float *Bp = reinterpret_cast<float *>(ws + plan->layout.off_bpack);
        scorch_status_t st = launch_pack_b(B, ldb, plan->k, plan->n, kSliceCols, Bp, stream);
        if (st != SCORCH_OK) return st;
        a.B = Bp;
        a.ldb = kSliceCols;
        a.b_tile_stride = (int64_t)plan->k * kSliceCols;
    }
    if (grid > 0) {
        kernel_fn fn = cut          ? pick_fused_cut(mp.G, mp.T, mp.UA, false)
                       : whole_rows ? pick_fused_whole(mp.V, plan->params.U, plan->params.NT)
                                    : pick_fused(mp.V, mp.G, mp.T, plan->params.U, plan->params.NT, mp.UA);
        if (plan->n_hot > 0 && mp.V == 4 && !mp.UA && mp.xcd_slices == 0 && mp.G >= 8 && plan->params.U >= 8 &&
            (plan->params.NT & 1)) {
            // hot/cold variant: rows of B outside the plan's hot set are read with the streaming policy
            a.hotmask = reinterpret_cast<const uint32_t *>(ws + plan->layout.off_hotmask);
            a.b_bytes = (int64_t)plan->k * ldb * 4;
            fn = cut ? pick_fused_cut(mp.G, mp.T, false, true) : pick_fused_hot(mp.G, mp.T, a.b_bytes < (1ll << 32) ? plan->tuning.cold : 0);
        }
        hipLaunchKernelGGL(fn, dim3((uint32_t)grid), dim3(kBlock), 0, stream, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "launch spmm_fused_kernel");
    }
    if (cut) return launch_cut_sum(plan, C, ldc, bias, act, stream);
    if (plan->n_split > 0 && !fold) {
        FixupArgs f{};
        f.split = reinterpret_cast<const int4 *>(ws + plan->layout.off_split);
        f.partials = a.partials;
        f.C = C;
        f.ldc = ldc;
        f.n = plan->n;
        f.n_split = plan->n_split;
        f.partial_stride = plan->layout.partial_stride;
        f.bias = bias;
        f.act = act;
        hipLaunchKernelGGL(spmm_fixup_kernel, dim3((uint32_t)plan->n_split), dim3(kBlock), 0, stream, f);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "launch spmm_fixup_kernel");
    }
    return SCORCH_OK;
}

scorch_status_t launch_natural(int32_t m, int32_t k, int32_t n, const int32_t *rowptr, const int32_t *colidx,
                               const float *vals, const float *B, int64_t ldb, float *C, int64_t ldc,
                               hipStream_t stream) {
    const NaturalMapping nm = natural_mapping(m, k, n, B, ldb, C, ldc);
    Mapping mp = nm.mp;
    ExecArgs a{};
    a.rowptr = rowptr;
    a.colidx = colidx;
    a.vals = vals;
    a.B = B;
    a.C = C;
    a.ldb = ldb;
    a.ldc = ldc;
    a.m = m;
    a.n = n;
    if (nm.row_kernel) {
        // up to 256 pairs, one per compute unit, get 16 wavefronts each (16 rows of 6000 entries, n = 32: 10.4 -> 8.6 us)
        const int waves = nm.row_units <= 256 ? 16 : kWavesPerBlock;
        mp.T = 1;
        mp.G = std::min(mp.G, 8);
        a.ncoltiles = (n + mp.G * mp.V - 1) / (mp.G * mp.V);
        a.xcd_slices = 1;
        kernel_fn fn = waves == 16 ? pick_row<16>(mp.V, mp.G, mp.UA) : pick_row<kWavesPerBlock>(mp.V, mp.G, mp.UA);
        hipLaunchKernelGGL(fn, dim3((uint32_t)xcd_grid_size(a.xcd_slices, a.ncoltiles, m)), dim3(waves * kWave), 0, stream, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "launch spmm_row_kernel");
        return SCORCH_OK;
    }
    a.xcd_slices = mp.xcd_slices;
    // Rows per wavefront (a power of two): up to 4, or up to one per lane group, as long as at least 4096 wavefronts are
    // left; more, up to 16, where the launch would have more than 12 288 workgroups, of which the chip starts one every
    // 1.9 ns at best.  Measured with 4 / 8 / 16 rows: 169 343 rows, two column slices 141 / 127 / 127 us, one 128 /
    // 134 / 139; 600 000 rows 194 / 168 / 165; 1.5 M rows, two slices 977 / 821 / 733; 30 000 rows 44 / 46 / 55.
    const int64_t rows_cap = std::max(4, std::min(kNaturalRowsMax, kWave / mp.G));
    a.rows_per_wave = 1;
    while (a.rows_per_wave < rows_cap && (int64_t)m >= 8192 * (int64_t)a.rows_per_wave) a.rows_per_wave *= 2;
    // Not where column tiles make the many workgroups out of few (long) rows: 4096 rows of 1638 entries, 16 tiles.
    while (a.rows_per_wave < kNaturalRowsMax && (int64_t)m * mp.ncoltiles > (int64_t)12288 * kWavesPerBlock * a.rows_per_wave &&
           (int64_t)m >= 8192 * (int64_t)a.rows_per_wave)
        a.rows_per_wave *= 2;
    a.nb_wave = (int32_t)ceil_div64(m, (int64_t)kWavesPerBlock * a.rows_per_wave);
    const Scouts scouts = scouts_for(m);
    a.nb_items = scouts.count;
    a.scout_shift = scouts.shift;
    a.one_over_m = 1.f / (float)m;
    a.ncoltiles = mp.ncoltiles;
    const int64_t grid = grid_size(mp, (int64_t)a.nb_items + a.nb_wave);
    if (grid > 0x7fffffffLL) {
        set_error("launch grid of %lld workgroups exceeds the HIP limit", (long long)grid);
        return SCORCH_ERR_UNSUPPORTED;
    }
    const kernel_fn fn = nm.scout_gathers == 8 && mp.G == 16 ? spmm_natural_kernel<4, 16, 1, 8, 1, false, 8>
                                                             : pick_natural(mp.V, mp.G, mp.T, mp.UA);
    hipLaunchKernelGGL(fn, dim3((uint32_t)grid), dim3(kBlock), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "launch spmm_natural_kernel");
    return SCORCH_OK;
}

}  // namespace scorch
