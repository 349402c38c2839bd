// Device core of the fused sampled loss/gradient: kernel parameters, small
// helpers and the per-chunk body shared by the HIP kernels.
#pragma once

#include <algorithm>
#include <type_traits>

#include "sampling.hpp"

namespace gcp {

template <typename T>
struct LGParams {
    SampleCtx<T> sc;
    int64_t n;            // samples p + q
    // deterministic objective: each wave's partial sum goes to its own slot
    // (workgroup * waves + wave) instead of an atomic add into loss_out.  (Here,
    // the 64-bit arrays below begin at multiples of 16 bytes: a federated round of
    // 16 four-way clients takes 4.43 ms, 4.48 with them 8 bytes further on.)
    double* loss_parts;
    const int64_t* m_coords;  // materialised list (src = 1, 3)
    const T* m_x;
    const T* m_w;
    const T* A;
    T* G;
    int R;
    int src;              // where the samples come from (lg_chunk)
    int passes;           // samples per lane group and chunk: a chunk has 64 / lanes * passes samples
    int chunk_samples;
    uint32_t stride_b;              // bytes of a model row
    uint32_t rowb[kMaxModes];       // order-specific kernels: byte offset of each mode's first row (models below 4 GiB)
    uint32_t ldsb[kMaxModes];       // the same, from a row's byte offset in A to its LDS-private copy (modulo 2^32)
    int loss;
    int semi;             // semi-stratified: samples s < p get f'(x,m) - f'(0,m)
    const T* scale;       // nullable device scalar
    double* loss_out;     // nullable
    int64_t rowoff[kMaxModes];
    uint32_t lds_mask;    // modes accumulated in LDS
    int64_t lds_off[kMaxModes];
    int64_t lds_elems;
    // bucketed scatter
    uint32_t bucket_mask;      // modes scattered through row-block buckets
    int br_shift;              // rows per bucket = 1 << br_shift
    int nb;                    // buckets over all bucketed modes
    int bucket_base[kMaxModes + 1];
    int spb;                   // samples per workgroup (tiled launch)
    int64_t nblocks;           // workgroups of the tiled launch (J)
    int64_t entry_cap;         // entries per workgroup segment list = spb * bucketed modes
    int bucket_lds;            // byte offset of the bucket staging in LDS
    uint4* entries;            // [J][entry_cap] 16-byte {key, y}
    int* start;                // [J][nb + 1] first entry of each bucket in the workgroup's list, then their number
    // owner pass: mode k's row blocks use workgroups [bwg_base[k], bwg_base[k+1]),
    // bsplits[k] per row block, each reading bsegs[k] consecutive segments
    int64_t bwg_base[kMaxModes + 1];
    int bsplits[kMaxModes];
    int bsegs[kMaxModes];
    // non-fused sampling step (src = 2): each sample's y, the sampled
    // tensor's values, and its coordinates [n x d], written instead of
    // scattering
    T* y_out;
    int64_t* c_out;
    // or, for the deterministic form, both in one 16-byte {key, y} a sample
    uint4* rec_out;
};

// Row offsets of the launch from the tensor's dims (P.lds_mask and P.lds_off
// set before): row indexes for the any-order kernels, byte offsets modulo 2^32
// for the order-specific ones.
template <typename T>
inline void set_row_offsets(LGParams<T>& P, const gcp_tensor_s* t)
{
    P.stride_b = (uint32_t)P.R * (uint32_t)sizeof(T);
    for (int k = 0; k < kMaxModes; ++k) {
        P.rowoff[k] = k < t->d ? t->rowoff[k] : t->rowoff[t->d];
        P.rowb[k] = (uint32_t)P.rowoff[k] * P.stride_b;
        P.ldsb[k] = (uint32_t)P.lds_off[k] * (uint32_t)sizeof(T) - P.rowb[k];
    }
}

template <typename T, int V>
__device__ __forceinline__ void load_cols(const T* __restrict__ p, T (&out)[V])
{
    if constexpr (V == 4 && sizeof(T) == 4) {
        float4 f = *reinterpret_cast<const float4*>(p);
        out[0] = f.x; out[1] = f.y; out[2] = f.z; out[3] = f.w;
    } else if constexpr (V == 2 && sizeof(T) == 4) {
        float2 f = *reinterpret_cast<const float2*>(p);
        out[0] = f.x; out[1] = f.y;
    } else if constexpr (V == 2 && sizeof(T) == 8) {
        double2 f = *reinterpret_cast<const double2*>(p);
        out[0] = f.x; out[1] = f.y;
    } else {
#pragma unroll
        for (int v = 0; v < V; ++v) out[v] = p[v];
    }
}

template <typename T>
__device__ __forceinline__ void global_add(T* p, T v)
{
    unsafeAtomicAdd(p, v);
}

// Float add into LDS as a compare-and-swap loop on the bit pattern.  The
// native LDS float atomic (ds_add_f32) retires about one lane per three
// clocks on gfx950, while this loop costs a few LDS integer operations per
// wave instruction when the lanes hit distinct words (one gradient row per
// lane group).  Lanes that collide are serialised by the hardware, so every
// pass of the loop completes at least one of them.
__device__ __forceinline__ void lds_add(float* p, float v)
{
    unsigned* u = reinterpret_cast<unsigned*>(p);
    unsigned old = __hip_atomic_load(u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    for (;;) {
        const unsigned nv = __float_as_uint(__uint_as_float(old) + v);
        if (__hip_atomic_compare_exchange_strong(u, &old, nv, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP))
            break;
    }
}

// Two adjacent floats (8-byte aligned) added by one 64-bit compare-and-swap
// loop: half the serial LDS round trips of two single adds.
__device__ __forceinline__ void lds_add2(float* p, float a, float b)
{
    unsigned long long* u = reinterpret_cast<unsigned long long*>(p);
    unsigned long long old = __hip_atomic_load(u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    for (;;) {
        const float lo = __uint_as_float((unsigned)old) + a;
        const float hi = __uint_as_float((unsigned)(old >> 32)) + b;
        const unsigned long long nv = (unsigned long long)__float_as_uint(lo) |
                                      ((unsigned long long)__float_as_uint(hi) << 32);
        if (__hip_atomic_compare_exchange_strong(u, &old, nv, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP))
            break;
    }
}

__device__ __forceinline__ void lds_add(double* p, double v)
{
    unsigned long long* u = reinterpret_cast<unsigned long long*>(p);
    unsigned long long old = __hip_atomic_load(u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    for (;;) {
        const unsigned long long nv =
            (unsigned long long)__double_as_longlong(__longlong_as_double((long long)old) + v);
        if (__hip_atomic_compare_exchange_strong(u, &old, nv, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP))
            break;
    }
}

// Adds VEC consecutive columns to LDS; float column pairs (8-byte aligned:
// row strides and column offsets are multiples of VEC) go through one 64-bit
// compare-and-swap each.
template <typename T, int VEC>
__device__ __forceinline__ void lds_add_cols(T* dst, const T (&c)[VEC])
{
    static_assert(VEC == 1 || VEC == 2 || VEC == 4, "columns per lane");
    if constexpr (sizeof(T) == 4 && VEC >= 2) {
        lds_add2(dst, c[0], c[1]);
        if constexpr (VEC == 4) lds_add2(dst + 2, c[2], c[3]);
    } else {
        lds_add(dst, c[0]);
        if constexpr (VEC >= 2) lds_add(dst + 1, c[1]);
        if constexpr (VEC == 4) {
            lds_add(dst + 2, c[2]);
            lds_add(dst + 3, c[3]);
        }
    }
}

// Element offset of column 0 of model row `row` (row < 2^32, checked when the
// tensor is created): one 32 x 32 -> 64-bit multiply.
__device__ __forceinline__ uint64_t row_elem(uint64_t row, int R)
{
    return (uint64_t)(uint32_t)row * (uint32_t)R;
}

template <typename T>
__device__ __forceinline__ uint4 pack_entry(uint64_t key, T y)
{
    uint4 e;
    e.x = (uint32_t)key;
    e.y = (uint32_t)(key >> 32);
    if constexpr (sizeof(T) == 4) {
        e.z = __float_as_uint(y);
        e.w = 0;
    } else {
        const uint64_t b = (uint64_t)__double_as_longlong(y);
        e.z = (uint32_t)b;
        e.w = (uint32_t)(b >> 32);
    }
    return e;
}

template <typename T>
__device__ __forceinline__ T entry_y(uint4 e)
{
    if constexpr (sizeof(T) == 4) return __uint_as_float(e.z);
    else return __longlong_as_double((long long)(((uint64_t)e.w << 32) | e.z));
}

// Butterfly exchange across lanes (lane ^ mask).  Doubles move as two 32-bit
// halves: the 64-bit form of the cross-half exchange trips a gfx950 code
// generation error in this toolchain.
__device__ __forceinline__ float xor_shfl(float v, int mask) { return __shfl_xor(v, mask, 64); }
__device__ __forceinline__ double xor_shfl(double v, int mask)
{
    const long long b = __double_as_longlong(v);
    const int lo = __shfl_xor((int)(b & 0xffffffffll), mask, 64);
    const int hi = __shfl_xor((int)(b >> 32), mask, 64);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Value of lane (at / 4) of the wavefront (at: byte address of a lane, as
// bpermute takes it).
__device__ __forceinline__ float lane_from(float v, int at)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(at, __float_as_int(v)));
}
__device__ __forceinline__ double lane_from(double v, int at)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_ds_bpermute(at, (int)(b & 0xffffffffll));
    const int hi = __builtin_amdgcn_ds_bpermute(at, (int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// DPP lane exchange of a whole wavefront (every lane has a source lane).
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum over the aligned group of LANES lanes, in every lane of it: a butterfly
// from the farthest exchange to the nearest.  From 16 lanes on, the exchanges
// 8 and 4 apart are row rotations (the row repeats with the period of the
// step before); in a group of 8, lane ^ 4 is a quad reversal then a half-row
// mirror.  All are DPP operands of VALU instructions: only the 32- and
// 64-lane groups take trips through the LDS crossbar.
template <int LANES, typename T>
__device__ __forceinline__ T group_sum(T v)
{
    if constexpr (LANES >= 64) v += xor_shfl(v, 32);
    if constexpr (LANES >= 32) v += xor_shfl(v, 16);
    if constexpr (LANES >= 16) {
        v += dpp<0x128>(v);                            // row_ror:8
        v += dpp<0x124>(v);                            // row_ror:4
    } else if constexpr (LANES == 8) {
        v += dpp<0x141>(dpp<0x1B>(v));                 // quad_perm [3,2,1,0], row_half_mirror
    }
    if constexpr (LANES >= 4) v += dpp<0x4E>(v);       // quad_perm [2,3,0,1]
    if constexpr (LANES >= 2) v += dpp<0xB1>(v);       // quad_perm [1,0,3,2]
    return v;
}

// The value of lane u (mod U) of each aligned run of U lanes, U = 1, 2 or 4.
template <int U, typename T>
__device__ __forceinline__ T quad_pick(T v, int u)
{
    if constexpr (U == 1) return v;
    else if constexpr (U == 2) return u == 0 ? dpp<0xA0>(v) : dpp<0xF5>(v);
    else return u == 0 ? dpp<0x00>(v) : u == 1 ? dpp<0x55>(v) : u == 2 ? dpp<0xAA>(v) : dpp<0xFF>(v);
}

// Derivative value of one sample (x, w, model value m); l receives its part
// of the objective when one is asked for.  nonzero: the sample is one of the
// first p.
template <typename T>
__device__ __forceinline__ T sample_y(const LGParams<T>& P, T x, T w, T m, bool nonzero, T& l)
{
    const bool semi_nz = P.semi && nonzero;
    T y = w * loss_df<T>(P.loss, x, m);
    if (semi_nz) y -= w * loss_df<T>(P.loss, T(0), m);
    if (P.loss_out) {
        l = w * loss_f<T>(P.loss, x, m);
        if (semi_nz) l -= w * loss_f<T>(P.loss, T(0), m);
    }
    return y;
}

// Exclusive prefix sum of cnt[0, n) into off[0, n] by one wavefront.
__device__ inline void wave_exclusive_scan(const int* cnt, int* off, int n, int lane)
{
    const int per = (n + 63) / 64;
    const int b0 = lane * per;
    int local = 0;
    for (int i = 0; i < per; ++i)
        if (b0 + i < n) local += cnt[b0 + i];
    int incl = local;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
    }
    int run = incl - local;
    for (int i = 0; i < per; ++i) {
        if (b0 + i < n) {
            off[b0 + i] = run;
            run += cnt[b0 + i];
        }
    }
    if (lane == 63) off[n] = incl;
}

// Samples per lane group whose factor-row gathers are issued together; divides
// LANES.  The scattering form also holds the rows until its products are out.
#ifndef GCP_UNROLL_WIDE
#define GCP_UNROLL_WIDE 2
#endif
constexpr int samples_in_flight(int order, int elem_bytes, int lanes, int vec)
{
    return (order == 0 || lanes < 4) ? 1 : elem_bytes == 8 ? 2 : vec == 4 ? GCP_UNROLL_WIDE : 4;
}

// Entries in flight per lane group in the owner pass of the bucketed scatter
// (float, four columns per lane: GCP_OWNER_UNROLL_WIDE).
#ifndef GCP_OWNER_UNROLL_WIDE
#define GCP_OWNER_UNROLL_WIDE GCP_UNROLL_WIDE
#endif
template <typename T, int D, int LANES, int VEC>
constexpr int owner_in_flight()
{
    constexpr int U = (D == 0 || LANES < 4) ? 1 : sizeof(T) == 8 ? 2 : VEC == 4 ? GCP_OWNER_UNROLL_WIDE : 4;
    static_assert(U >= 1 && LANES % U == 0, "entries in flight must divide the lanes per entry");
    return U;
}

// One chunk of up to 64 samples by one wavefront, without LDS staging.
//
// Phase 1, one lane per sample: draw or read the sample and turn its
// coordinates into the d factor rows' offsets.  Lane group g (LANES lanes)
// owns the chunk's samples g * passes + cl, cl < passes; passes is
// LANES for a full chunk of 64 and less when a call has too few samples to
// fill the GPU with full chunks.
// Phase 2, LANES lanes per sample: in pass `it` each group works on the sample
// its own lane `it` drew -- the row offsets come from that lane by bpermute,
// so the key is unpacked and the address products are formed once per sample
// instead of once per lane -- gathers the rows (every load unconditional:
// inactive samples read row 0, lanes past column R read column 0; a load under
// a branch makes the compiler wait for every load before it), and reduces the
// model value over the group by DPP adds.
//   SCATTER = false: nothing is scattered in the loop (objective only, the
//     sampled tensor is written, or every mode is bucketed): lane `it` keeps
//     its sample's model value and, after the loop, each lane evaluates the
//     loss of its own sample -- once per sample, not once per lane.
//   SCATTER = true: the U samples of a pass are evaluated by lanes cl % U and
//     y is handed back by a quad broadcast; then the leave-one-out products go
//     to the LDS-private copies or to G by atomics.
// Bound by the draw's random reads (2^21 samples of 10000x8000x6000, 5e7
// nonzeros: 66 us to draw alone, 81 us with the gathers and the objective
// where the form that unpacked keys and evaluated losses in every lane and
// staged samples through LDS took 134 us) and, with sorting, by its stores.
// P.src: 0 draw the samples (the fused sampled gradient); 1 read a
// materialised list (coordinates, x, w); 2 draw and write the sampled tensor
// (coordinates and y = w f'(x, m)): the sampling step of the non-fused
// gradient; 3 read a sampled tensor whose values are already y (w = 1 unless a
// weight list is given): the MTTKRP step of the non-fused gradient.
// GIVEN: a scattering kernel for P.src = 3 alone (the others take 0 and 1).  It
// needs no model value, so that a sample's products follow its gathers at once:
// 50000 samples of 1000x800x600x400 at rank 6 in double 23.0 us, 26.1 with P.src
// looked at in the loop of one kernel for all (208 MTTKRP calls 3% less on average,
// and the kernels without it spill fewer registers).
template <typename T, int D, int LANES, int VEC, bool SCATTER, bool WIDE = false, bool GIVEN = false>
__device__ __forceinline__ void lg_chunk(const LGParams<T>& P, int64_t s0, int passes, int lane, T* priv,
                                         uint64_t* bkey, T* by, int* bcnt, int64_t block_s0, bool tiled, T scale,
                                         double& lacc, uint64_t step)
{
    constexpr int U = samples_in_flight(D, (int)sizeof(T), LANES, VEC);
    static_assert(LANES % U == 0, "samples in flight must divide the lanes per sample");
    constexpr int DM = D > 0 ? D : kMaxModes;
    constexpr bool BYTES = D > 0 && !WIDE;   // rows by 32-bit byte offsets, else by index
    const int dd = D > 0 ? D : P.sc.d;
    const int R = P.R;
    const int g = lane / LANES, cl = lane % LANES;
    const int col0 = cl * VEC;
    const bool col_ok = col0 < R;          // VEC divides R
    const int colL = col_ok ? col0 : 0;
    const uint32_t colb = (uint32_t)colL * (uint32_t)sizeof(T);

    // phase 1
    const int64_t s = s0 + g * passes + cl;
    const bool mine = cl < passes && s < P.n;
    uint64_t key = 0;
    uint32_t off[DM];                      // BYTES: byte offset of the row in A; else its index
    T x = T(0), w = T(0);
    {
        uint32_t ci[DM];
#pragma unroll
        for (int k = 0; k < DM; ++k) ci[k] = 0;
        if (mine) {
            if (!GIVEN && (P.src == 0 || P.src == 2)) {
                draw_sample<T, D>(P.sc, step, s, key, ci, x, w);
            } else {
                bool ok = true;
#pragma unroll
                for (int k = 0; k < DM; ++k) {
                    if (k < dd) {
                        const int64_t c = P.m_coords[s * dd + k];
                        if (c < 0 || c >= P.sc.L.dims[k]) ok = false;
                        else ci[k] = (uint32_t)c;
                    }
                }
                x = P.m_x[s];
                w = P.m_w ? P.m_w[s] : T(1);
                if (!ok) {
                    atomicOr(P.sc.status, kStatusData);
#pragma unroll
                    for (int k = 0; k < DM; ++k) ci[k] = 0;
                    w = T(0);
                }
#pragma unroll
                for (int k = 0; k < DM; ++k)
                    if (k < dd) key += pack_coord(P.sc.L, (uint64_t)ci[k], k);
            }
            if (!GIVEN && P.src == 2 && P.c_out) {
#pragma unroll
                for (int k = 0; k < DM; ++k)
                    if (k < dd) P.c_out[s * dd + k] = (int64_t)ci[k];
            }
            if (tiled) {
                // stage the sample and count it for the sort, behind the draw's
                // memory latency
                bkey[s - block_s0] = key;
#pragma unroll
                for (int k = 0; k < DM; ++k)
                    if (k < dd && ((P.bucket_mask >> k) & 1u))
                        atomicAdd(bcnt + P.bucket_base[k] + (int)(ci[k] >> P.br_shift), 1);
            }
        }
#pragma unroll
        for (int k = 0; k < DM; ++k) {
            if constexpr (BYTES) off[k] = P.rowb[k] + ci[k] * P.stride_b;
            else off[k] = (uint32_t)P.rowoff[k] + ci[k];
        }
    }
    const bool given = !SCATTER && P.src == 3;
    const int from0 = (lane & ~(LANES - 1)) << 2;   // bpermute address of the group's first lane
    T mown = T(0);
    T ygiven = T(0);
    if constexpr (GIVEN) {
        ygiven = w * x * scale;
        if (tiled && mine) by[s - block_s0] = ygiven;
    }

    if (SCATTER || !given) {
        for (int it = 0; it < passes; it += U) {
            uint32_t o[U][DM];
            T a[U][DM][VEC];
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int k = 0; k < DM; ++k)
                    if (k < dd) o[u][k] = (uint32_t)__builtin_amdgcn_ds_bpermute(from0 + ((it + u) << 2), (int)off[k]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int k = 0; k < DM; ++k) {
                    if (k < dd) {
                        if constexpr (BYTES)
                            load_cols<T, VEC>(reinterpret_cast<const T*>(reinterpret_cast<const char*>(P.A) +
                                                                         (o[u][k] + colb)),
                                              a[u][k]);
                        else
                            load_cols<T, VEC>(P.A + row_elem(o[u][k], R) + colL, a[u][k]);
                    }
                }
            }
            T m[U];
            if constexpr (!GIVEN) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    T part = T(0);
#pragma unroll
                    for (int v = 0; v < VEC; ++v) {
                        T prod = a[u][0][v];
#pragma unroll
                        for (int k = 1; k < DM; ++k)
                            if (k < dd) prod *= a[u][k][v];
                        if constexpr (D == 5) {
                            // rounded after the product, as in the any-order kernel
#pragma clang fp contract(off)
                            part = part + prod;
                        } else {
                            part += prod;
                        }
                    }
                    m[u] = group_sum<LANES>(col_ok ? part : T(0));
                }
            }
            if constexpr (!SCATTER) {
#pragma unroll
                for (int u = 0; u < U; ++u) mown = cl == it + u ? m[u] : mown;
            } else {
                T yu[U];
                if constexpr (GIVEN) {
#pragma unroll
                    for (int u = 0; u < U; ++u) yu[u] = lane_from(ygiven, from0 + ((it + u) << 2));
                } else {
                    // lane cl evaluates sample it + cl % U of its group
                    const int ul = cl & (U - 1);
                    const int at = it + ul;
                    const int64_t sl = s0 + g * passes + at;
                    const T xl = lane_from(x, from0 + (at << 2));
                    const T wl = lane_from(w, from0 + (at << 2));
                    T ml = m[0];
#pragma unroll
                    for (int u = 1; u < U; ++u) ml = ul == u ? m[u] : ml;
                    const bool vl = at < passes && sl < P.n;
                    T l = T(0);
                    T y = sample_y<T>(P, xl, wl, ml, sl < P.sc.p, l);
                    if (vl && cl < U) lacc += (double)l;
                    y *= scale;
                    if (tiled && vl && cl < U) by[sl - block_s0] = y;
#pragma unroll
                    for (int u = 0; u < U; ++u) yu[u] = quad_pick<U>(y, u);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (it + u >= passes || s0 + g * passes + it + u >= P.n || !col_ok) continue;
                    // leave-one-out products y prod_{n != k} A_n[i_n, :] by
                    // prefix and suffix running products, all formed before
                    // the first goes out (each sent as it is formed: double
                    // with LDS-private modes 1-3% slower, 62.7 and 66.0 us for
                    // 2^20 samples of 300x250x200 at rank 4)
                    auto lds_row = [&](int k) -> T* {
                        if constexpr (BYTES)
                            return reinterpret_cast<T*>(reinterpret_cast<char*>(priv) + (o[u][k] + colb + P.ldsb[k]));
                        else
                            return priv + P.lds_off[k] + (o[u][k] - (uint32_t)P.rowoff[k]) * (uint32_t)R + col0;
                    };
                    auto grad_row = [&](int k) -> T* {
                        if constexpr (BYTES)
                            return reinterpret_cast<T*>(reinterpret_cast<char*>(P.G) + (o[u][k] + colb));
                        else
                            return P.G + row_elem(o[u][k], R) + col0;
                    };
                    T cv[DM][VEC];
#pragma unroll
                    for (int v = 0; v < VEC; ++v) {
                        T pre[DM];
                        pre[0] = yu[u];
#pragma unroll
                        for (int k = 1; k < DM; ++k)
                            if (k < dd) pre[k] = pre[k - 1] * a[u][k - 1][v];
                        T suf = T(1);
#pragma unroll
                        for (int k = DM - 1; k >= 0; --k) {
                            if (k < dd) {
                                cv[k][v] = pre[k] * suf;
                                suf *= a[u][k][v];
                            }
                        }
                    }
#pragma unroll
                    for (int k = DM - 1; k >= 0; --k) {
                        if (k < dd && !((P.bucket_mask >> k) & 1u)) {
                            if ((P.lds_mask >> k) & 1u) {
                                lds_add_cols<T, VEC>(lds_row(k), cv[k]);
                            } else {
                                T* dst = grad_row(k);
#pragma unroll
                                for (int v = 0; v < VEC; ++v) global_add(dst + v, cv[k][v]);
                            }
                        }
                    }
                }
            }
        }
    }
    if constexpr (!SCATTER) {
        if (mine) {
            T l = T(0);
            const T y = given ? w * x : sample_y<T>(P, x, w, mown, s < P.sc.p, l);
            lacc += (double)l;
            if (P.src == 2) {
                if (P.rec_out) P.rec_out[s] = pack_entry<T>(key, y);
                else P.y_out[s] = y;
            }
            if (tiled) by[s - block_s0] = y * scale;
        }
    }
}

// Bucketed scatter, sampling side: sorts the (key, y) of the workgroup's
// nvalid staged samples (bkey, by in LDS), counted by lg_chunk into bcnt, by
// (mode, bucket) into segment list `seg` of the bucket workspace -- scan,
// place -- and records where each bucket starts in the list.  boff is LDS
// scratch of nb + 1 ints; bcnt is zero again when it returns.  Every thread of
// the workgroup calls it.
template <typename T, int D>
__device__ __forceinline__ void bucket_write_out(const LGParams<T>& P, int64_t seg, int nvalid, const uint64_t* bkey,
                                                 const T* by, int* bcnt, int* boff)
{
    constexpr int DM = D > 0 ? D : kMaxModes;
    const int dd = D > 0 ? D : P.sc.d;
    __syncthreads();
    if ((threadIdx.x >> 6) == 0) wave_exclusive_scan(bcnt, boff, P.nb, threadIdx.x);
    __syncthreads();
    int* start = P.start + seg * (P.nb + 1);
    for (int b = threadIdx.x; b <= P.nb; b += blockDim.x) {
        start[b] = boff[b];
        if (b < P.nb) bcnt[b] = 0;
    }
    __syncthreads();
    uint4* out = P.entries + seg * P.entry_cap;
    for (int e = threadIdx.x; e < nvalid; e += blockDim.x) {
        const uint64_t key = bkey[e];
        const uint4 ent = pack_entry<T>(key, by[e]);
        uint32_t ci[DM];
        unpack_all<D == 0>(P.sc.L, dd, key, ci);
#pragma unroll
        for (int k = 0; k < DM; ++k) {
            if (k < dd && ((P.bucket_mask >> k) & 1u)) {
                const int pos = atomicAdd(boff + P.bucket_base[k] + (int)(ci[k] >> P.br_shift), 1);
                out[pos] = ent;
            }
        }
    }
    __syncthreads();
}

// LDS of the sort: the staged samples, the buckets' counts and offsets.
inline size_t sort_lds_bytes(int spb, int elem_bytes, int nb) { return (size_t)spb * (8 + elem_bytes) + (size_t)nb * 8 + 4; }

// Value that lane IT of each lane group (LANES lanes) holds, in every lane of
// the group: DPP row broadcasts, one per group of a row of 16 lanes, each
// written to its group's banks of four lanes; lane reads for groups of 32 and
// 64 (a bpermute would add to the LDS); a bpermute for groups of 2.
template <int LANES, int IT>
__device__ __forceinline__ uint32_t group_bcast(uint32_t v, int group_at)
{
    if constexpr (LANES == 16) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + IT, 0xf, 0xf, true);
    } else if constexpr (LANES == 8) {
        const int lo = __builtin_amdgcn_update_dpp(0, (int)v, 0x150 + IT, 0xf, 0xf, true);
        return (uint32_t)__builtin_amdgcn_update_dpp(lo, (int)v, 0x158 + IT, 0xf, 0xc, false);
    } else if constexpr (LANES == 4) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, IT * 0x55, 0xf, 0xf, true);    // quad_perm
    } else if constexpr (LANES == 64) {
        return (uint32_t)__builtin_amdgcn_readlane((int)v, IT);
    } else if constexpr (LANES == 32) {
        const int lo = __builtin_amdgcn_readlane((int)v, IT), hi = __builtin_amdgcn_readlane((int)v, 32 + IT);
        return (uint32_t)(group_at ? hi : lo);
    } else {
        return (uint32_t)__builtin_amdgcn_ds_bpermute(group_at + (IT << 2), (int)v);
    }
}
template <int LANES, int IT>
__device__ __forceinline__ float group_bcast(float v, int group_at)
{
    return __uint_as_float(group_bcast<LANES, IT>(__float_as_uint(v), group_at));
}
template <int LANES, int IT>
__device__ __forceinline__ double group_bcast(double v, int group_at)
{
    return __hiloint2double((int)group_bcast<LANES, IT>((uint32_t)__double2hiint(v), group_at),
                            (int)group_bcast<LANES, IT>((uint32_t)__double2loint(v), group_at));
}

template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(static_cast<F&&>(f));
    }
}

// Bucketed scatter, owner side: accumulates into `part` (LDS, rows x R) the
// contributions y prod_{n != k} A_n[i_n, :] of every entry of bucket b (rows
// [r0, r0 + rows) of mode k) in segment lists [j0, j1).  Each wavefront takes a
// run of consecutive segments and reads them as one stream of entries, 64 at a
// time, one entry per lane (a binary search over the segments' running counts
// finds a lane's entry, so that short segments fill whole batches too).  The
// lane unpacks its entry once -- the other modes' row offsets, its row's place
// in `part`, y -- and its lane group takes it by DPP broadcasts, gathers the
// rows and adds the products to LDS by compare-and-swap.  (An entry read by all
// lanes of its group costs the vector memory path as many cycles as a row
// gather, its unpacking in all of them as many instructions as the products,
// and a broadcast by bpermute adds to the LDS, which the adds fill.)  The next
// batch's entries are in flight while a batch is worked on.  Every thread of
// the workgroup calls it; part is complete when it returns.
template <typename T, int D, int LANES, int VEC, bool WIDE = false>
__device__ __forceinline__ void bucket_accumulate(const LGParams<T>& P, int k, int b, int64_t r0, int64_t rows,
                                                  int64_t j0, int64_t j1, T* part)
{
    constexpr int S = 64 / LANES;
    constexpr int U = owner_in_flight<T, D, LANES, VEC>();
    constexpr int DM = D > 0 ? D : kMaxModes;
    constexpr int DO = DM - 1;
    constexpr bool BYTES = D > 0 && !WIDE;     // rows by 32-bit byte offsets, else by index
    static_assert(D == 0 || D >= 2, "orders with their own kernels");
    const int nwaves = blockDim.x >> 6;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int g = lane / LANES, cl = lane % LANES;
    const int group_at = (lane & ~(LANES - 1)) << 2;
    const int col0 = cl * VEC;
    const int R = P.R;
    const bool col_ok = col0 < R;
    const int colL = col_ok ? col0 : 0;
    const uint32_t colb = (uint32_t)colL * (uint32_t)sizeof(T);
    const int dd = D > 0 ? D : P.sc.d;
    // entry of the batch at t this lane holds: a full batch in lane order (one
    // coalesced read, pass it works on lane it of every group), the last one
    // spread over the groups so that it takes as few passes as it can
    auto hold = [&](int t, int total) { return t + (t + 64 <= total ? lane : cl * S + g); };
    for (int64_t e = threadIdx.x; e < rows * R; e += blockDim.x) part[e] = T(0);
    __syncthreads();

    const int per = ((int)(j1 - j0) + nwaves - 1) / nwaves;
    const int64_t je = std::min<int64_t>(j0 + (wave + 1) * per, j1);
    for (int64_t jc = j0 + wave * per; jc < je; jc += 64) {
        // lane i: segment jc + i, its count, the entries before it in this
        // run, and where entry 0 of the stream would be if the stream began
        // inside this segment
        const bool has = jc + lane < je;
        const int* st = P.start + (jc + lane) * (P.nb + 1) + b;
        const int first = has ? st[0] : 0;
        const int cnt = has ? st[1] - first : 0;
        int incl = cnt;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(incl, d, 64);
            if (lane >= d) incl += o;
        }
        const int excl = incl - cnt;
        const int total = __builtin_amdgcn_readlane(incl, 63);
        if (total == 0) continue;
        const int rel = lane * (int)P.entry_cap + first - excl;
        const uint4* base = P.entries + jc * P.entry_cap;
        auto entry_of = [&](int e) -> uint4 {          // entry min(e, total - 1) of the stream
            e = min(e, total - 1);
            int sg = 0;                                // last segment that begins at or before e
#pragma unroll
            for (int step = 32; step >= 1; step >>= 1) {
                const int at = __builtin_amdgcn_ds_bpermute((sg + step) << 2, excl);
                if (at <= e) sg += step;
            }
            return base[e + __builtin_amdgcn_ds_bpermute(sg << 2, rel)];
        };
        uint4 nxt = entry_of(hold(0, total));
        for (int t = 0; t < total; t += 64) {
            const int nb = min(64, total - t);
            const uint64_t key = (uint64_t)nxt.x | ((uint64_t)nxt.y << 32);
            const T y = entry_y<T>(nxt);
            uint32_t off[DO];                          // BYTES: byte offset of the row in A; else its index
            uint32_t loc;                              // byte offset of the entry's row in part
            {
                uint32_t ci[DM];
                unpack_all<D == 0>(P.sc.L, dd, key, ci);
                uint32_t ik = ci[0];
#pragma unroll
                for (int kk = 1; kk < DM; ++kk)
                    if (kk == k) ik = ci[kk];
                loc = (ik - (uint32_t)r0) * P.stride_b;
                // slot o holds mode o, or o + 1 from k on
#pragma unroll
                for (int o = 0; o < DO; ++o) {
                    const bool after = o >= k;
                    const uint32_t i = after ? ci[o + 1] : ci[o];
                    if constexpr (BYTES) off[o] = (after ? P.rowb[o + 1] : P.rowb[o]) + i * P.stride_b;
                    else off[o] = (uint32_t)(after ? P.rowoff[o + 1] : P.rowoff[o]) + i;
                }
            }
            static_for<LANES / U>([&](auto pp) {
                constexpr int it0 = decltype(pp)::value * U;
                if (it0 * S < nb) {
                    T a[U][DO][VEC];
                    static_for<U>([&](auto uu) {
                        constexpr int u = decltype(uu)::value;
#pragma unroll
                        for (int o = 0; o < DO; ++o) {
                            if (D > 0 || o < dd - 1) {
                                const uint32_t ro = group_bcast<LANES, it0 + u>(off[o], group_at);
                                if constexpr (BYTES)
                                    load_cols<T, VEC>(reinterpret_cast<const T*>(
                                                          reinterpret_cast<const char*>(P.A) + (ro + colb)),
                                                      a[u][o]);
                                else
                                    load_cols<T, VEC>(P.A + row_elem(ro, R) + colL, a[u][o]);
                            }
                        }
                    });
                    // the next batch's entries, behind the first gathers (loads
                    // return in order)
                    if (it0 == 0 && t + 64 < total) nxt = entry_of(hold(t + 64, total));
                    static_for<U>([&](auto uu) {
                        constexpr int u = decltype(uu)::value;
                        const T yu = group_bcast<LANES, it0 + u>(y, group_at);
                        const uint32_t lu = group_bcast<LANES, it0 + u>(loc, group_at);
                        if ((nb == 64 || (it0 + u) * S + g < nb) && col_ok) {
                            T c[VEC];
#pragma unroll
                            for (int v = 0; v < VEC; ++v) {
                                c[v] = yu;
#pragma unroll
                                for (int o = 0; o < DO; ++o)
                                    if (D > 0 || o < dd - 1) c[v] *= a[u][o][v];
                            }
                            lds_add_cols<T, VEC>(reinterpret_cast<T*>(reinterpret_cast<char*>(part) + (lu + colb)), c);
                        }
                    });
                }
            });
        }
    }
    __syncthreads();
}

}  // namespace gcp
