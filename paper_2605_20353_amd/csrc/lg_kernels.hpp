// Kernel templates of the sampled loss/gradient (k_loss_grad and the row-block
// owner pass k_bucket_accum) and the table of lane shapes they are built for.
// Instantiated per dtype and order in lg_*.hip; declared here for the host
// side (loss_grad.hip, deterministic.hip).
#pragma once

#include <cmath>

#include "lg_core.hpp"

namespace gcp {

// Wavefronts per SIMD the register allocation aims at: 8 (64 VGPRs) for the
// float kernels of orders 3 and 4 that scatter nothing in their loop and for
// their owner pass, which fit them (68-76 unconstrained; four owner shapes
// spill one or two).  2^21 samples, 8 against 6 or 4: the objective of a
// 10000x8000x6000 tensor at rank 32 75.1 and 77.0 us; a 5000x5000x500x1000 one
// with every mode bucketed at rank 16 240 and 250, 32 262 and 257, 64 394 and
// 398 us.  6 (80 VGPRs) for those of order 5, where up to 14 registers spill at
// 8 (400x300x200x100x50: the objective of 2^18 samples at rank 32 23.1 us at 8,
// 19.2 at 6, 19.5 at 4; 2^20 samples at rank 20, all modes bucketed, 256, 240
// and 240 us).
template <typename T, int D, bool SCATTER, bool WIDE>
constexpr int lg_min_waves()
{
    return sizeof(T) == 4 && !SCATTER && D > 0 && !WIDE ? (D == 5 ? 6 : 8) : 4;
}

// WIDE: a model of 4 GiB or more, whose rows are found by 64-bit products.
// GIVEN: the scatter of a sampled tensor whose values are given (lg_chunk).
template <typename T, int D, int LANES, int VEC, bool SCATTER, bool WIDE, bool GIVEN>
__global__ void __launch_bounds__(1024, (lg_min_waves<T, D, SCATTER, WIDE>())) k_loss_grad(const LGParams<T> P)
{
    constexpr int DM = D > 0 ? D : kMaxModes;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // One word of each cache line of the parameter block, all at once: the loops
    // below read it phase by phase, and each phase's first read waited for a cold
    // line of its own (32768 uniform samples of a dense 400x300x200 tensor at
    // rank 32 22.7 us, 20.6 with the lines read ahead).
    {
        using Words = const __attribute__((address_space(4))) uint32_t*;
        const Words words = (Words)__builtin_amdgcn_kernarg_segment_ptr();
        uint32_t any = 0;
#pragma unroll
        for (unsigned i = 0; i < sizeof(LGParams<T>) / 4; i += 16) any |= words[i];
        asm volatile("" ::"s"(any));
    }
    const int nwaves = blockDim.x >> 6;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    T* priv = reinterpret_cast<T*>(smem);
    // bucketed scatter staging: the workgroup's samples in order
    uint64_t* bkey = reinterpret_cast<uint64_t*>(smem + P.bucket_lds);
    T* by = reinterpret_cast<T*>(smem + P.bucket_lds + (size_t)P.spb * 8);
    int* bcnt = reinterpret_cast<int*>(smem + P.bucket_lds + (size_t)P.spb * (8 + sizeof(T)));
    int* boff = bcnt + P.nb;

    if (SCATTER && P.lds_mask) {
        for (int64_t e = threadIdx.x; e < P.lds_elems; e += blockDim.x) priv[e] = T(0);
    }
    if (P.bucket_mask)
        for (int b = threadIdx.x; b < P.nb; b += blockDim.x) bcnt[b] = 0;
    if (P.bucket_mask || (SCATTER && P.lds_mask)) __syncthreads();
    const int dd = D > 0 ? D : P.sc.d;
    const int R = P.R;
    const T scale = P.scale ? *P.scale : T(1);
    const bool tiled = P.bucket_mask != 0;
    double lacc = 0.0;

    // The loops read the parameter block through a pointer that the compiler
    // cannot see through, so that it loads a phase's fields where they are used:
    // all of them loaded once before the loops do not fit the scalar registers,
    // and every use then reads a spill.
    using KernArg = const __attribute__((address_space(4))) LGParams<T>*;
    auto params = []() -> const LGParams<T>& {
        KernArg kp = (KernArg)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(kp));
        return *(const LGParams<T>*)kp;
    };
    // tiled launches sort the samples [j*spb, (j+1)*spb) together, one such
    // block after the other where there are more of them than workgroups (only
    // with LDS-private modes); else the chunks go round the wavefronts
    for (int64_t j = blockIdx.x;;) {
        const LGParams<T>& B = params();
        const int64_t b0 = tiled ? j * B.spb : 0;
        const int64_t b1 = tiled ? std::min<int64_t>(B.n, b0 + B.spb) : B.n;
        const int first = tiled ? wave : (int)blockIdx.x * nwaves + wave;
        const int64_t s_step = (int64_t)(tiled ? nwaves : nwaves * (int)gridDim.x) * B.chunk_samples;
        for (int64_t s0 = b0 + (int64_t)first * B.chunk_samples; s0 < b1; s0 += s_step) {
            const LGParams<T>& Q = params();
            lg_chunk<T, D, LANES, VEC, SCATTER, WIDE, GIVEN>(Q, s0, Q.passes, lane, priv, bkey, by, bcnt, b0, tiled, scale,
                                                lacc, Q.sc.step);
        }
        const LGParams<T>& W = params();
        if (tiled) bucket_write_out<T, D>(W, j, (int)(b1 - b0), bkey, by, bcnt, boff);
        j += gridDim.x;
        if (!SCATTER || !tiled || j >= W.nblocks) break;
    }

    if (!GIVEN && P.loss_out) {
        for (int off = 32; off >= 1; off >>= 1) lacc += xor_shfl(lacc, off);
        if (P.loss_parts) {
            if (lane == 0) P.loss_parts[(int64_t)blockIdx.x * nwaves + wave] = lacc;
        } else {
            // one add per workgroup: adds into one address are executed one
            // after the other, about 11 ns each, and one per wavefront took
            // 90 us at 8192 wavefronts
            __shared__ double wave_loss[16];
            if (lane == 0) wave_loss[wave] = lacc;
            __syncthreads();
            if (threadIdx.x == 0) {
                double l = 0.0;
                for (int i = 0; i < nwaves; ++i) l += wave_loss[i];
                if (l != 0.0) atomicAdd(P.loss_out, l);
            }
        }
    }
    if (SCATTER && P.lds_mask) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < DM; ++k) {
            if (k < dd && ((P.lds_mask >> k) & 1u)) {
                const int64_t rows = P.sc.L.dims[k];
                T* dst = P.G + P.rowoff[k] * R;
                const T* src = priv + P.lds_off[k];
                for (int64_t e = threadIdx.x; e < rows * R; e += blockDim.x) {
                    const T v = src[e];
                    if (v != T(0)) global_add(dst + e, v);
                }
            }
        }
    }
}

// Row-block owner pass of the bucketed scatter.  Workgroup (b, split) owns
// rows [r0, r0 + 2^br_shift) of bucket b's mode k and reads the segments of
// workgroups [j0, j1) of the sampling launch: per entry it gathers the other
// modes' rows, forms y prod_{n != k} A_n[i_n, :] and adds it to the LDS copy
// of its rows; the block is flushed to G once.
template <typename T, int D, int LANES, int VEC, bool WIDE>
__global__ void __launch_bounds__(1024, (lg_min_waves<T, D, false, WIDE>())) k_bucket_accum(const LGParams<T> P)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    T* part = reinterpret_cast<T*>(smem);
    const int R = P.R;
    const int dd = D > 0 ? D : P.sc.d;

    // the mode whose workgroup range holds this workgroup (ranges of modes
    // that are not bucketed are empty), then its row block and split
    int k = 0;
    for (int kk = 0; kk < dd; ++kk)
        if (P.bwg_base[kk] <= (int64_t)blockIdx.x && (int64_t)blockIdx.x < P.bwg_base[kk + 1]) k = kk;
    const uint32_t splits = (uint32_t)P.bsplits[k];
    const uint32_t local = blockIdx.x - (uint32_t)P.bwg_base[k];
    const int b = P.bucket_base[k] + (int)(local / splits);
    const int split = (int)(local % splits);
    const int64_t r0 = (int64_t)(b - P.bucket_base[k]) << P.br_shift;
    const int64_t rows = std::min<int64_t>((int64_t)1 << P.br_shift, P.sc.L.dims[k] - r0);
    // whole segments per workgroup (the host makes it a multiple of the
    // waves per workgroup); the last split takes the remainder
    const int64_t j0 = (int64_t)split * P.bsegs[k];
    const int64_t j1 = std::min<int64_t>(P.nblocks, j0 + P.bsegs[k]);
    bucket_accumulate<T, D, LANES, VEC, WIDE>(P, k, b, r0, rows, j0, j1, part);
    T* dst = P.G + (P.rowoff[k] + r0) * R;
    for (int64_t e = threadIdx.x; e < rows * R; e += blockDim.x) {
        const T v = part[e];
        if (v != T(0)) global_add(dst + e, v);
    }
}

// Zeroes p[0, n) in 16-byte stores (single ones where p is not aligned) and the
// objective.
template <typename T>
__global__ void __launch_bounds__(256) k_zero(T* __restrict__ p, int64_t n, double* __restrict__ loss_out)
{
    constexpr int V = 16 / sizeof(T);
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    if (i0 == 0 && loss_out) *loss_out = 0.0;
    const int64_t nv = (uintptr_t)p % 16 == 0 ? n / V : 0;
    for (int64_t i = i0; i < nv; i += stride) reinterpret_cast<uint4*>(p)[i] = uint4{0, 0, 0, 0};
    for (int64_t i = nv * V + i0; i < n; i += stride) p[i] = T(0);
}

// Workgroups of a k_zero launch over n elements of `bytes` bytes.
inline unsigned zero_blocks(int64_t n, int bytes) { return stream_blocks((n * bytes + 15) / 16); }

template <typename T>
using LGKernel = void (*)(const LGParams<T>);
template <typename T>
using BAKernel = void (*)(const LGParams<T>);

// (lanes, vec) shapes built for each dtype
#define GCP_LG_SHAPES_F32(X) \
    X(8, 1) X(16, 1) X(32, 1) X(64, 1) X(4, 2) X(8, 2) X(16, 2) X(32, 2) X(64, 2) X(2, 4) X(4, 4) X(8, 4) X(16, 4) X(32, 4) X(64, 4)
#define GCP_LG_SHAPES_F64(X) X(8, 1) X(16, 1) X(32, 1) X(64, 1) X(4, 2) X(8, 2) X(16, 2) X(32, 2) X(64, 2) X(64, 4)

// What a call's kernel does in its loop: no scatter (objective only, the sampled
// tensor is written, or every mode is bucketed), or the scatter of some mode
// (LDS-private or atomic), of drawn or listed samples or of given values.
enum class LGForm { no_scatter, scatter, scatter_given };

template <typename T, int D, bool WIDE>
inline LGKernel<T> pick_shape(LGForm form, int lanes, int vec)
{
#define GCP_CASE(LN, VC)                                                                        \
    if (lanes == LN && vec == VC)                                                               \
        return form == LGForm::scatter         ? k_loss_grad<T, D, LN, VC, true, WIDE, false>   \
               : form == LGForm::scatter_given ? k_loss_grad<T, D, LN, VC, true, WIDE, true>    \
                                               : k_loss_grad<T, D, LN, VC, false, WIDE, false>;
    if constexpr (sizeof(T) == 4) {
        GCP_LG_SHAPES_F32(GCP_CASE)
    } else {
        GCP_LG_SHAPES_F64(GCP_CASE)
    }
#undef GCP_CASE
    return nullptr;
}

template <typename T, int D, bool WIDE>
inline BAKernel<T> pick_bucket_shape(int lanes, int vec)
{
#define GCP_CASE(LN, VC) \
    if (lanes == LN && vec == VC) return k_bucket_accum<T, D, LN, VC, WIDE>;
    if constexpr (sizeof(T) == 4) {
        GCP_LG_SHAPES_F32(GCP_CASE)
    } else {
        GCP_LG_SHAPES_F64(GCP_CASE)
    }
#undef GCP_CASE
    return nullptr;
}

// The kernels of order D (0: any order) at a lane shape, null when the shape
// is not built.  WIDE is built for orders 3 and 4 (order 0 has 64-bit products
// anyway).
template <typename T, int D, bool WIDE>
LGKernel<T> loss_grad_kernel(LGForm form, int lanes, int vec);
template <typename T, int D, bool WIDE>
BAKernel<T> bucket_kernel(int lanes, int vec);

#define GCP_LG_INSTANTIATE(T, D, WIDE)                                         \
    template <>                                                                \
    LGKernel<T> loss_grad_kernel<T, D, WIDE>(LGForm form, int lanes, int vec) \
    {                                                                          \
        return pick_shape<T, D, WIDE>(form, lanes, vec);                    \
    }                                                                          \
    template <>                                                                \
    BAKernel<T> bucket_kernel<T, D, WIDE>(int lanes, int vec)                  \
    {                                                                          \
        return pick_bucket_shape<T, D, WIDE>(lanes, vec);                      \
    }

#define GCP_LG_DECLARE(T, D, WIDE)                                              \
    template <>                                                                 \
    LGKernel<T> loss_grad_kernel<T, D, WIDE>(LGForm form, int lanes, int vec); \
    template <>                                                                 \
    BAKernel<T> bucket_kernel<T, D, WIDE>(int lanes, int vec);

}  // namespace gcp
