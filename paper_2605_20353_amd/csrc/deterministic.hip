// Deterministic sampled gradient (gcp_loss_grad with GCP_DETERMINISTIC): the
// same gradient and objective, bit for bit, on every run with the same
// samples, model, tile and device.  The default scatters add floats in an
// order that depends on timing (atomics, LDS compare-and-swap, per-workgroup
// flushes); here every sum has a fixed order:
//   1. the sampling kernel (k_loss_grad, src = 2) writes the sampled tensor
//      -- the cell's key and y = w f'(x, m) of every sample -- and each
//      wavefront's partial objective into its own slot;
//   2. k_det_pairs lists (model row, sample) for every sample and mode;
//   3. a stable radix sort by row (rocPRIM) groups each row's samples in
//      sample order;
//   4. k_det_starts finds where each row's run begins, and, where there are
//      more rows than pairs, rocPRIM's unique lists the rows whose run is not
//      empty (in row order);
//   5. k_det_reduce gives each gradient row to one lane group, which adds
//      y prod_{j != k} A_j[i_j, :] over the row's run in an order fixed by
//      the sorted run (the sampled MTTKRP of eq. gcp-gradient, Sec. 3.1.2)
//      and writes the row;
//   6. k_det_loss adds the objective partials in slot order.
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_select.hpp>

#include "det_runs.hpp"
#include "lg_kernels.hpp"

namespace gcp {
namespace {

struct DetModes {
    int d;
    uint32_t rowoff[kMaxModes + 1];
};

// (row, sample) of mode k for sample s at k * n + s.
__global__ void __launch_bounds__(256) k_det_pairs(const uint4* __restrict__ rec, int64_t n, DetModes M, KeyLayout L,
                                                   uint32_t* __restrict__ keys, uint32_t* __restrict__ vals)
{
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < n; s += (int64_t)gridDim.x * blockDim.x) {
        const uint2 w = *reinterpret_cast<const uint2*>(rec + s);
        uint32_t ci[kMaxModes];
        unpack_all<true>(L, M.d, (uint64_t)w.x | ((uint64_t)w.y << 32), ci);
#pragma unroll
        for (int k = 0; k < kMaxModes; ++k) {
            if (k < M.d) {
                keys[k * n + s] = M.rowoff[k] + ci[k];
                vals[k * n + s] = (uint32_t)s;
            }
        }
    }
}

// start[r] = first position of row r in the sorted keys (rows + 1 entries,
// start[rows] = total); every row gets a value, empty rows an empty run.
__global__ void __launch_bounds__(256) k_det_starts(const uint32_t* __restrict__ skeys, int64_t total, uint32_t rows,
                                                    uint32_t* __restrict__ start)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t lo = i == 0 ? 0 : (int64_t)skeys[i - 1] + 1;      // rows after the previous key
        const int64_t hi = i == total ? (int64_t)rows : (int64_t)skeys[i];
        for (int64_t r = lo; r <= hi; ++r) start[r] = (uint32_t)i;
    }
}

// Lanes per gradient row in k_det_reduce at VEC columns per lane: enough for R
// columns, a power of two, at most 64 and at least 8: a lane holds a pair as
// well, and a run is read in batches of that many, one after the other (2000
// samples of 60 rank-8 rows: 173 us a call with groups of 2, 77 with 8).
__host__ __device__ inline int det_group_lanes(int R, int vec)
{
    int rp = 8;
    while (rp * vec < R && rp < 64) rp <<= 1;
    return rp;
}

// Value of `v` in lane `src` of the wavefront; doubles move as two 32-bit
// halves.
__device__ __forceinline__ float lane_get(float v, int src) { return __shfl(v, src, 64); }
__device__ __forceinline__ double lane_get(double v, int src)
{
    const long long b = __double_as_longlong(v);
    const int lo = __shfl((int)(b & 0xffffffffll), src, 64);
    const int hi = __shfl((int)(b >> 32), src, 64);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

constexpr uint32_t kDetLongRun = 512;

// One lane group per gradient row: RP lanes of VEC columns (wider ranks take
// the columns RP VEC at a time), so a wavefront holds H = 64 / RP rows at once.
// A group reads its row's run of sorted (row, sample) pairs RP at a time, one
// pair per lane: the lane loads the sample's y and the model rows of the other
// modes.  Lane shuffles inside the group then hand the pairs out in run order;
// the group gathers the other modes' rows and adds y prod_{j != k} A_j[i_j, :]
// in that order.  Every sum thus has an order fixed by the sorted run alone.
// Bound by the records' random 16 bytes, a whole line out of the Infinity
// Cache each.  A batch's samples are read two batches ahead, its records one
// ahead, and U pairs' rows are in flight at once.  16 bytes per lane: a load instruction costs the
// vector memory path the same whatever its width (2^20 samples, rank 32: 142 us
// with one column per lane and no read-ahead).
// A run of kDetLongRun pairs or more is shared by a workgroup (the first
// long_wgs workgroups look for them): each lane group takes a slice whose
// bounds the run's length alone fixes, and the slices' sums are added in their
// order.  (One group walking a row's 10000 pairs is a chain of batches: 2^19
// samples of a 400x300x200x100x50 tensor at rank 32 took 5.8 ms a call, 0.37
// with shared runs; 172x25000x300 at rank 100 668 and 250 us.)
// runs: the rows to visit (those with pairs); NULL visits every row, and rows
// without pairs get 0 when the call does not accumulate.
template <typename T, int D, int VEC>
__global__ void __launch_bounds__(256) k_det_reduce(const uint32_t* __restrict__ start,
                                                    const uint32_t* __restrict__ runs,
                                                    const uint32_t* __restrict__ nruns, uint32_t rows,
                                                    const uint32_t* __restrict__ svals,
                                                    const uint4* __restrict__ rec, const T* __restrict__ A, DetModes M,
                                                    KeyLayout L, int R,
                                                    const T* __restrict__ scale, int accumulate, int long_wgs,
                                                    T* __restrict__ G)
{
    constexpr int DM = D > 0 ? D : kMaxModes;
    constexpr int DO = DM - 1;
    constexpr int U = D > 0 && DO * VEC * (int)sizeof(T) <= 48 ? 8 : 4;
    const int dd = D > 0 ? D : M.d;
    const int lane = threadIdx.x & 63;
    const int64_t wave = (((int64_t)blockIdx.x - long_wgs) * blockDim.x + threadIdx.x) >> 6;
    const int64_t nw = ((int64_t)(gridDim.x - long_wgs) * blockDim.x) >> 6;
    const T sc = scale ? *scale : T(1);
    const int RP = det_group_lanes(R, VEC);
    const int H = 64 / RP;
    const int h = lane / RP, cg = lane % RP, gl0 = h * RP;
    const int64_t nr = runs ? (int64_t)*nruns : (int64_t)rows;
    const int gi = (threadIdx.x >> 6) * H + h, groups = 4 * H;
    __shared__ T part[256 * VEC];
    __shared__ uint32_t list[256];
    __shared__ int nlist;
    // row r by this lane group, or its slice of the run where the workgroup shares the row
    auto row_sum = [&](uint32_t r, auto shared) {
        int k = 0;
        for (int kk = 1; kk < dd; ++kk)
            if (M.rowoff[kk] <= r) k = kk;
        uint32_t b = start[r], e = start[r + 1];
        if constexpr (shared.value) {
            const uint32_t rb = b, re = e;
            det_slice(rb, re, (uint32_t)groups, (uint32_t)gi, (uint32_t)RP, b, e);
        } else {
            if (e - b >= kDetLongRun || (b == e && accumulate)) return;
        }
        for (int c0 = 0; c0 < R; c0 += RP * VEC) {
            const int c = c0 + cg * VEC;
            const bool col = c < R;
            const uint64_t colL = col ? (uint32_t)c : 0u;
            T acc[VEC];
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] = T(0);
            // lane cg of the group: pair i0 + cg (past the run's end: its last pair)
            auto sample = [&](uint32_t i0) { return svals[det_lane(i0, e, (uint32_t)cg)]; };
            T yl = T(0);
            uint32_t orow[DO], s1 = 0;
            auto pair = [&](uint32_t sl) {
                const uint4 w = rec[sl];
                yl = entry_y<T>(w) * sc;
                uint32_t ci[DM];
                unpack_all<true>(L, dd, (uint64_t)w.x | ((uint64_t)w.y << 32), ci);
                // slot o holds mode o, or o + 1 from k on
#pragma unroll
                for (int o = 0; o < DO; ++o)
                    orow[o] = o >= k ? M.rowoff[o + 1] + ci[o + 1] : M.rowoff[o] + ci[o];
            };
            if (b < e) {
                pair(sample(b));
                s1 = sample(b + (uint32_t)RP);
            }
            for (uint32_t i0 = b, nv; i0 < e; i0 += nv) {
                nv = det_batch(i0, e, (uint32_t)RP);
                const T yc = yl;
                uint32_t oc[DO];
#pragma unroll
                for (int o = 0; o < DO; ++o) oc[o] = orow[o];
                for (uint32_t q0 = 0; q0 < nv; q0 += U) {
                    T yq[U], a[U][DO][VEC];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int q = gl0 + (int)min(q0 + (uint32_t)u, nv - 1);
                        yq[u] = lane_get(yc, q);
#pragma unroll
                        for (int o = 0; o < DO; ++o) {
                            if (D == 0 && o >= dd - 1) break;
                            const uint32_t row = (uint32_t)__shfl((int)oc[o], q, 64);
                            load_cols<T, VEC>(A + (uint64_t)row * (uint32_t)R + colL, a[u][o]);
                        }
                    }
                    // the next batch's loads go out behind this one's gathers:
                    // loads return in order
                    __asm__ volatile("" ::: "memory");
                    if (q0 == 0) {
                        const uint32_t s2 = s1;
                        s1 = sample(i0 + 2u * (uint32_t)RP);
                        pair(s2);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if (q0 + (uint32_t)u >= nv) continue;
#pragma unroll
                        for (int v = 0; v < VEC; ++v) {
                            T prod = T(1);
#pragma unroll
                            for (int o = 0; o < DO; ++o)
                                if (D > 0 || o < dd - 1) prod *= a[u][o][v];
                            acc[v] += yq[u] * prod;
                        }
                    }
                }
            }
            if constexpr (shared.value) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) part[threadIdx.x * VEC + v] = acc[v];
                __syncthreads();
                if (gi == 0) {
                    for (int q = 1; q < groups; ++q)
#pragma unroll
                        for (int v = 0; v < VEC; ++v) acc[v] += part[(q * RP + cg) * VEC + v];
                }
                __syncthreads();
                if (gi != 0) continue;
            }
            if (col) {
                T* g = G + (uint64_t)r * (uint32_t)R + c;
#pragma unroll
                for (int v = 0; v < VEC; ++v) g[v] = accumulate ? g[v] + acc[v] : acc[v];
            }
        }
    };
    if (blockIdx.x < (unsigned)long_wgs) {
        // rows with long runs, one by one: each thread looks at one row in turn
        for (int64_t jb = blockIdx.x; jb < nr; jb += (int64_t)long_wgs * 256) {
            if (threadIdx.x == 0) nlist = 0;
            __syncthreads();
            const int64_t j = jb + (int64_t)threadIdx.x * long_wgs;
            if (j < nr) {
                const uint32_t r = runs ? runs[j] : (uint32_t)j;
                if (start[r + 1] - start[r] >= kDetLongRun) list[atomicAdd(&nlist, 1)] = r;
            }
            __syncthreads();
            const int nl = nlist;
            for (int q = 0; q < nl; ++q) row_sum(list[q], std::true_type{});
            __syncthreads();
        }
    } else {
        // shuffles stay inside a group, so a group without a row may leave
        for (int64_t j = wave * H + h; j < nr; j += nw * H) row_sum(runs ? runs[j] : (uint32_t)j, std::false_type{});
    }
}

// The objective partials, added in an order that their number alone fixes:
// thread i takes slots i, i + 1024, ... in turn, then a tree over the threads.
// (One thread adding them all took 326 us for 6144 partials: a chain of
// dependent loads and adds.)
__global__ void __launch_bounds__(1024) k_det_loss(const double* __restrict__ parts, int64_t n, int accumulate,
                                                   double* __restrict__ out)
{
    __shared__ double sum[1024];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 1024) s += parts[i];
    sum[threadIdx.x] = s;
    for (int h = 512; h >= 1; h >>= 1) {
        __syncthreads();
        if ((int)threadIdx.x < h) sum[threadIdx.x] += sum[threadIdx.x + h];
    }
    if (threadIdx.x == 0) *out = accumulate ? *out + sum[0] : sum[0];
}

constexpr int64_t kDetLossSlots = 1 << 16;

int sort_bits(uint32_t rows)
{
    int b = 1;
    while (b < 32 && ((uint64_t)1 << b) < rows) ++b;
    return b;
}

struct DetLayout {
    int64_t rec, keys_in, vals_in, keys_out, vals_out, start, runs, nruns, parts, scratch_loss, sort_tmp, total;
    size_t sort_bytes;
};

int64_t align256(int64_t x) { return (x + 255) & ~int64_t(255); }

gcp_status det_layout(const gcp_tensor_s* t, int64_t n, DetLayout& L)
{
    const int64_t pairs = n * t->d;
    const uint32_t rows = (uint32_t)t->rowoff[t->d];
    L.sort_bytes = 0;
    hipError_t e = rocprim::radix_sort_pairs(nullptr, L.sort_bytes, (const uint32_t*)nullptr, (uint32_t*)nullptr,
                                             (const uint32_t*)nullptr, (uint32_t*)nullptr, (size_t)pairs, 0,
                                             (unsigned)sort_bits(rows + 1), (hipStream_t)0);
    if (e != hipSuccess) return hip_error(e, "rocprim::radix_sort_pairs (size query)");
    size_t unique_bytes = 0;
    e = rocprim::unique(nullptr, unique_bytes, (const uint32_t*)nullptr, (uint32_t*)nullptr, (uint32_t*)nullptr,
                        (size_t)pairs, rocprim::equal_to<uint32_t>(), (hipStream_t)0);
    if (e != hipSuccess) return hip_error(e, "rocprim::unique (size query)");
    L.sort_bytes = std::max(L.sort_bytes, unique_bytes);          // the two use the region one after the other
    int64_t off = 0;
    L.rec = off; off = align256(off + n * 16);
    L.keys_in = off; off = align256(off + pairs * 4);
    L.vals_in = off; off = align256(off + pairs * 4);
    L.keys_out = off; off = align256(off + pairs * 4);
    L.vals_out = off; off = align256(off + pairs * 4);
    L.start = off; off = align256(off + ((int64_t)rows + 1) * 4);
    L.runs = off; off = align256(off + std::min<int64_t>(rows, pairs) * 4);
    L.nruns = off; off = align256(off + 4);
    L.parts = off; off = align256(off + kDetLossSlots * 8);
    L.scratch_loss = off; off = align256(off + 8);
    L.sort_tmp = off; off = align256(off + (int64_t)L.sort_bytes);
    L.total = off;
    return GCP_OK;
}

template <typename T>
gcp_status launch_det(gcp_tensor_s* t, const gcp_sample_params* sp, const void* A, int R, gcp_loss loss,
                      unsigned flags, const void* scale_dev, void* G_out, double* loss_out, const gcp_tile* tile,
                      hipStream_t stream)
{
    if (!t->ws || !sp) return set_error(GCP_ERR_ARG, "GCP_DETERMINISTIC needs gcp_tensor_reserve first");
    if (flags & GCP_LOSS_ONLY) return set_error(GCP_ERR_ARG, "GCP_DETERMINISTIC with GCP_LOSS_ONLY");
    if (!G_out) return set_error(GCP_ERR_ARG, "G_out is NULL");
    if ((flags & GCP_SCALE_BY_DEV) && !scale_dev) return set_error(GCP_ERR_ARG, "scale_dev is NULL");
    const int64_t n = sp->p + sp->q;
    if (n < 0 || n > t->ws_max_samples)
        return set_error(GCP_ERR_ARG, "GCP_DETERMINISTIC: %lld samples exceed the reserved %lld",
                         (long long)n, (long long)t->ws_max_samples);
    // (row, sample) pairs are indexed with 32 bits (run starts, sorted values)
    if (n * t->d >= (int64_t(1) << 32))
        return set_error(GCP_ERR_ARG, "GCP_DETERMINISTIC: %lld samples x %d modes reach 2^32 (row, sample) pairs",
                         (long long)n, t->d);
    DetLayout L{};
    gcp_status st = det_layout(t, n, L);
    if (st != GCP_OK) return st;
    if (L.total > t->ws_bytes) return set_error(GCP_ERR_ARG, "the reserved workspace is too small for this call");
    char* ws = (char*)t->ws;
    const bool accumulate = (flags & GCP_ACCUMULATE) != 0;
    const uint32_t rows = (uint32_t)t->rowoff[t->d];
    // 1. the sampled tensor and the per-wavefront objective partials; the
    //    launch's own objective target is a scratch word, so that loss_out
    //    keeps its accumulate semantics
    LGOutputs xo;
    xo.rec_out = ws + L.rec;
    xo.loss_parts = loss_out ? (double*)(ws + L.parts) : nullptr;
    xo.loss_parts_cap = kDetLossSlots;
    int64_t parts = 0;
    xo.parts_used = &parts;
    gcp_tile tl = tile ? *tile : gcp_tile{};
    tl.lds_modes = 0;
    tl.bucket_modes = 0;
    st = loss_grad_with_workspace(t, sp, nullptr, A, R, loss, 0u, nullptr, nullptr,
                                  loss_out ? (double*)(ws + L.scratch_loss) : nullptr, &tl, LGWorkspace{}, stream,
                                  &xo);
    if (st != GCP_OK) return st;
    if (n == 0) {
        if (!accumulate) {
            const int64_t gn = (int64_t)rows * R;
            k_zero<T><<<zero_blocks(gn, (int)sizeof(T)), 256, 0, stream>>>((T*)G_out, gn, loss_out);
            GCP_HIP(hipGetLastError());
        }
        return GCP_OK;
    }
    DetModes M{};
    M.d = t->d;
    for (int k = 0; k <= t->d; ++k) M.rowoff[k] = (uint32_t)t->rowoff[k];
    const int cus = device_cu_count(t->device);
    const int64_t pairs = n * t->d;
    // 2. (row, sample) pairs
    const unsigned pg = (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(n, 256), (int64_t)cus * 64));
    hipLaunchKernelGGL(k_det_pairs, dim3(pg), dim3(256), 0, stream, (const uint4*)(ws + L.rec), n, M, t->layout,
                       (uint32_t*)(ws + L.keys_in), (uint32_t*)(ws + L.vals_in));
    GCP_HIP(hipGetLastError());
    // 3. stable sort by row
    size_t sort_bytes = L.sort_bytes;
    GCP_HIP(rocprim::radix_sort_pairs(ws + L.sort_tmp, sort_bytes, (const uint32_t*)(ws + L.keys_in),
                                      (uint32_t*)(ws + L.keys_out), (const uint32_t*)(ws + L.vals_in),
                                      (uint32_t*)(ws + L.vals_out), (size_t)pairs, 0,
                                      (unsigned)sort_bits(rows + 1), stream));
    // 4. run starts and the list of rows with pairs
    const unsigned sg = (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(pairs + 1, 256), (int64_t)cus * 16));
    hipLaunchKernelGGL(k_det_starts, dim3(sg), dim3(256), 0, stream, (const uint32_t*)(ws + L.keys_out), pairs, rows,
                       (uint32_t*)(ws + L.start));
    GCP_HIP(hipGetLastError());
    // 5. one lane group per gradient row: every row where there are no more
    //    rows than pairs (24000 rows, 3.1M pairs: the list alone took 35 us),
    //    else the list of those with pairs, the others staying as they are, or
    //    0 when the call does not accumulate
    const bool listed = (int64_t)rows > pairs;
    if (listed) {
        size_t unique_bytes = L.sort_bytes;
        GCP_HIP(rocprim::unique(ws + L.sort_tmp, unique_bytes, (const uint32_t*)(ws + L.keys_out),
                                (uint32_t*)(ws + L.runs), (uint32_t*)(ws + L.nruns), (size_t)pairs,
                                rocprim::equal_to<uint32_t>(), stream));
        if (!accumulate) {
            const int64_t gn = (int64_t)rows * R;
            k_zero<T><<<zero_blocks(gn, (int)sizeof(T)), 256, 0, stream>>>((T*)G_out, gn, nullptr);
            GCP_HIP(hipGetLastError());
        }
    }
    const int64_t max_runs = std::min<int64_t>(rows, pairs);
    constexpr int VW = 16 / (int)sizeof(T);
    const bool wide = R % VW == 0 && (uintptr_t)A % 16 == 0;
    const int64_t rows_per_wg = 4 * (64 / det_group_lanes(R, wide ? VW : 1));     // 4 wavefronts of 64 / RP rows
    const unsigned rg =
        (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(max_runs, rows_per_wg), (int64_t)cus * 32));
    auto reduce = wide ? (t->d == 3   ? k_det_reduce<T, 3, VW>
                          : t->d == 4 ? k_det_reduce<T, 4, VW>
                                      : k_det_reduce<T, 0, VW>)
                       : (t->d == 3   ? k_det_reduce<T, 3, 1>
                          : t->d == 4 ? k_det_reduce<T, 4, 1>
                                      : k_det_reduce<T, 0, 1>);
    // workgroups for the long runs: as many as run at once where the rows of the
    // shortest mode have long runs on average (172x25000x300, 2^19 samples: 250 us
    // a call, 295 with one per CU), else one per CU to look for the few
    // (10000x8000x6000, 2^20 samples: 246 us, 262 with four; where half of the
    // stored cells lie in 5, 50 or 1000 rows of the long mode 412, 237 and 249 us,
    // with four 420, 255 and 262)
    const int64_t shortest = *std::min_element(t->dims, t->dims + t->d);
    const int64_t lookers = pairs < (int64_t)kDetLongRun ? 0 : n / shortest >= (int64_t)kDetLongRun / 2 ? cus * 4 : cus;
    const int long_wgs = (int)std::min<int64_t>(max_runs, lookers);
    hipLaunchKernelGGL(reduce, dim3(rg + (unsigned)long_wgs), dim3(256), 0, stream, (const uint32_t*)(ws + L.start),
                       listed ? (const uint32_t*)(ws + L.runs) : nullptr, (const uint32_t*)(ws + L.nruns), rows,
                       (const uint32_t*)(ws + L.vals_out), (const uint4*)(ws + L.rec), (const T*)A, M, t->layout, R, (flags & GCP_SCALE_BY_DEV) ? (const T*)scale_dev : nullptr,
                       accumulate ? 1 : 0, long_wgs, (T*)G_out);
    GCP_HIP(hipGetLastError());
    // 6. the objective, partials in slot order
    if (loss_out) {
        hipLaunchKernelGGL(k_det_loss, dim3(1), dim3(1024), 0, stream, (const double*)(ws + L.parts), parts,
                           accumulate ? 1 : 0, loss_out);
        GCP_HIP(hipGetLastError());
    }
    return GCP_OK;
}

}  // namespace

int64_t det_workspace_bytes(const gcp_tensor_s* t, int64_t max_samples)
{
    DetLayout L{};
    if (det_layout(t, max_samples, L) != GCP_OK) return -1;
    return L.total;
}

gcp_status loss_grad_deterministic(gcp_tensor_s* t, const gcp_sample_params* sp, const gcp_samples* smp,
                                   const void* A, int R, gcp_loss loss, unsigned flags, const void* scale_dev,
                                   void* G_out, double* loss_out, const gcp_tile* tile, hipStream_t stream)
{
    if (smp) return set_error(GCP_ERR_UNSUPPORTED, "GCP_DETERMINISTIC takes drawn samples only (smp must be NULL)");
    if (!A) return set_error(GCP_ERR_ARG, "A is NULL");
    if (R < 1 || R > 256) return set_error(GCP_ERR_ARG, "R = %d outside [1, 256]", R);
    const unsigned f = flags & ~(unsigned)GCP_DETERMINISTIC;
    if (t->dt == GCP_F32) return launch_det<float>(t, sp, A, R, loss, f, scale_dev, G_out, loss_out, tile, stream);
    return launch_det<double>(t, sp, A, R, loss, f, scale_dev, G_out, loss_out, tile, stream);
}

}  // namespace gcp
