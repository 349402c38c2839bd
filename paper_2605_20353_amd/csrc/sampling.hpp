// Drawing one sample of the sampled tensor (Sec. 3.1.1) on the device.
//
// Stratified: sample s < p is a nonzero j = floor(out0 N / 2^64) of the
// Philox block (s, step, 0, 0); sample s >= p is the zero sample z = s - p,
// whose attempt a draws a cell from the block(s) (z, step, 1 | a << 8, blk)
// and is kept as soon as the cell is not in the membership table.
// Semi-stratified: the first attempt is kept without a search.
// Uniform (dense tensors): cell from (s, step, 2, blk), value read from the
// dense array.
#pragma once

#include "gcp_internal.hpp"

namespace gcp {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <typename T>
__device__ __forceinline__ T record_value(u32x4 raw);
template <>
__device__ __forceinline__ float record_value<float>(u32x4 raw) { return __uint_as_float(raw.z); }
template <>
__device__ __forceinline__ double record_value<double>(u32x4 raw)
{
    return __hiloint2double((int)raw.w, (int)raw.z);
}

template <typename T>
struct SampleCtx {
    KeyLayout L;
    int d;
    int kind;                 // gcp_sampling
    int max_attempts;
    int64_t p, q, N;
    uint64_t seed, step, client;
    T w_nz, w_z;              // N/p and (M-N)/q (uniform: M/p in w_nz)
    const Record<T>* rec;     // sparse records
    const uint64_t* table;    // membership table
    uint64_t table_mask;
    int table_log2;
    const T* dense;           // dense values (uniform sampling)
    int64_t dense_stride[kMaxModes];
    uint32_t* status;
};

// Fills the cell key, coordinates, value and weight of sample s in [0, p + q)
// of iteration `step` (the second Philox counter word).  Coordinates of drawn
// cells come straight from the draw; only a stored nonzero's are unpacked.
// The three streams share one generator call, so that the code holds its
// forty wide multiplies once.  HOIST: a loop over samples may form the
// generator's key schedule once, before it.  Its twenty 64-bit words fit the
// scalar registers of a kernel that only draws (2^21 samples, five-way 70.8
// instead of 72.6 us, four-way 64.7 and 65.9); in the gradient kernels they
// would spill, and the schedule stays with the rounds.
template <typename T, int D, bool HOIST = false>
__device__ __forceinline__ void draw_sample(const SampleCtx<T>& c, uint64_t step, int64_t s, uint64_t& key,
                                            uint32_t (&ci)[D > 0 ? D : kMaxModes], T& x, T& w)
{
    constexpr int DM = D > 0 ? D : kMaxModes;
    const int dd = D > 0 ? D : c.d;
    const bool uniform = c.kind == GCP_SAMPLE_UNIFORM;
    const bool nonzero = !uniform && s < c.p;
    const uint64_t ctr = uniform || nonzero ? (uint64_t)s : (uint64_t)(s - c.p);
    const uint64_t stream = uniform ? kStreamUniform : nonzero ? kStreamNonzero : kStreamZero;
    auto words = [&](int a, uint64_t block) {
        uint64_t k0 = c.seed, k1 = c.client;
        if constexpr (!HOIST) asm volatile("" : "+s"(k0), "+s"(k1));
        return philox4x64_10(ctr, step, stream | ((uint64_t)a << 8), block, k0, k1);
    };
    for (int a = 0;; ++a) {
        const U64x4 o = words(a, 0);
        if (nonzero) {
            const int64_t j = (int64_t)range_map(o.v[0], (uint64_t)c.N);
            // one 16-byte streaming load: records are touched once per draw
            const u32x4 raw = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(c.rec + j));
            key = (uint64_t)raw.x | ((uint64_t)raw.y << 32);
            unpack_all<true>(c.L, dd, key, ci);
            x = record_value<T>(raw);
            w = c.w_nz;
            return;
        }
#pragma unroll
        for (int k = 0; k < (DM < 4 ? DM : 4); ++k)
            if (k < dd) ci[k] = range_map32(o.v[k], (uint32_t)c.L.dims[k]);
        if constexpr (DM > 4) {
            if (dd > 4) {
                const U64x4 o2 = words(a, 1);
#pragma unroll
                for (int k = 4; k < DM; ++k)
                    if (k < dd) ci[k] = range_map32(o2.v[k - 4], (uint32_t)c.L.dims[k]);
            }
        }
        key = 0;
#pragma unroll
        for (int k = 0; k < DM; ++k)
            if (k < dd) key += pack_coord(c.L, (uint64_t)ci[k], k);
        if (uniform) {
            int64_t lin = 0;
#pragma unroll
            for (int k = 0; k < DM; ++k)
                if (k < dd) lin += (int64_t)ci[k] * c.dense_stride[k];
            x = c.dense[lin];
            w = c.w_nz;
            return;
        }
        x = T(0);
        w = c.w_z;
        if (c.kind != GCP_SAMPLE_STRATIFIED || !table_contains(c.table, c.table_mask, c.table_log2, key)) return;
        if (a + 1 >= c.max_attempts) {
            atomicOr(c.status, kStatusSampling);
            return;
        }
    }
}

}  // namespace gcp

namespace gcp {

// Host side: validate (tensor, params) and fill the device sampling context.
// n_out receives the number of samples p + q.
template <typename T>
inline gcp_status make_sample_ctx(const gcp_tensor_s* t, const gcp_sample_params* sp, SampleCtx<T>& c,
                                  int64_t& n_out)
{
    if (!t) return set_error(GCP_ERR_ARG, "tensor is NULL");
    if (!sp) return set_error(GCP_ERR_ARG, "sample params are NULL");
    if (sp->p < 0 || sp->q < 0) return set_error(GCP_ERR_ARG, "negative sample count");
    if (sp->p > (int64_t(1) << 40) || sp->q > (int64_t(1) << 40))
        return set_error(GCP_ERR_ARG, "sample count above 2^40");
    c = SampleCtx<T>{};
    c.L = t->layout;
    c.d = t->d;
    c.kind = sp->kind;
    c.max_attempts = sp->max_attempts > 0 ? sp->max_attempts : 64;
    c.p = sp->p;
    c.q = sp->q;
    c.N = t->nnz;
    c.seed = sp->seed;
    c.step = sp->step;
    c.client = sp->client;
    c.status = t->status;
    switch (sp->kind) {
    case GCP_SAMPLE_STRATIFIED:
    case GCP_SAMPLE_SEMI_STRATIFIED:
        if (t->dense) return set_error(GCP_ERR_UNSUPPORTED, "stratified sampling needs a sparse tensor");
        if (sp->kind == GCP_SAMPLE_STRATIFIED && sp->q > 0 && (uint64_t)t->nnz >= t->cells)
            return set_error(GCP_ERR_ARG, "q > 0 but the tensor has no zero cells");
        c.w_nz = sp->p > 0 ? T((double)t->nnz / (double)sp->p) : T(0);
        c.w_z = sp->q > 0 ? T((double)(t->cells - t->nnz) / (double)sp->q) : T(0);
        c.rec = (const Record<T>*)t->rec;
        c.table = t->table;
        c.table_mask = t->table_mask;
        c.table_log2 = t->table_log2;
        break;
    case GCP_SAMPLE_UNIFORM:
        if (!t->dense) return set_error(GCP_ERR_UNSUPPORTED, "uniform sampling needs a dense tensor");
        if (sp->q != 0) return set_error(GCP_ERR_ARG, "uniform sampling takes q = 0");
        c.w_nz = sp->p > 0 ? T((double)t->cells / (double)sp->p) : T(0);
        c.w_z = T(0);
        c.dense = (const T*)t->dense_vals;
        {
            int64_t st = 1;
            for (int k = t->d - 1; k >= 0; --k) {
                c.dense_stride[k] = st;
                st *= t->dims[k];
            }
        }
        break;
    default:
        return set_error(GCP_ERR_ARG, "sampling kind %d", sp->kind);
    }
    n_out = sp->p + sp->q;
    return GCP_OK;
}

}  // namespace gcp
