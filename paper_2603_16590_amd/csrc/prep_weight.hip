// Offline weight preparation (Alg. 2, "Offline Fusion for Deployment"):
// W~ = P^-1 W per 32-row K-slab, optional block clip (Eq. 3-4, one ratio on the amax or two on min and
// max), MXFP4 along K (Sec. 2).  fp64 products and sums with the host-inverted fp64 factors or blocks, one rounding
// to fp32.  gfx950 only.
#include "batq_internal.h"
#include "mxfp4_device.h"
#include "code_layout.h"
#include "scale_layout.h"

namespace batq {
namespace {

__device__ __forceinline__ double w_value(float v) { return (double)v; }
__device__ __forceinline__ double w_value(uint16_t v) { return (double)bf16_bits_to_float(v); }

enum PrepForm { kPrepIdentity = 0, kPrepKron4 = 4, kPrepKron8 = 8, kPrepDense = 32 };

struct PrepArgs {
    const void* W;
    int64_t ldw;
    int w_is_KxN, N, N_out, il_off, nb;
    int outer_stride, inner_stride; // Kronecker forms: doubles between the inverted factors of consecutive blocks (0: shared)
};

// One thread per MX block k (blockIdx.y) and output column n (a row of the N x K storage).  Column n of W becomes row n of
// the prepared weight (N_out = N rows), or, with il_off >= 0, row 64 (n / 32) + il_off + n % 32 of a weight of
// N_out = 2 N rows: the gate (il_off 0) and up (il_off 32) projections of an MLP interleaved in groups of 32 columns for
// the GEMM's gated output.  The padding is written here too: zero codes for the rows up to a multiple of 32, zero codes
// and neutral scales for the blocks up to a multiple of 8.
//
// Bound: W in and codes out (2.53 bytes per element), beside it the fp64 pipe.  Kronecker forms multiply with the two
// inverted factors in turn (12 instead of 32 multiply-adds per element); the inner factor is read from LDS (broadcast),
// the outer one reaches the multiply-adds as scalar operands (both as scalars do not fit the scalar registers: reloads).
// 4096 x 14336 bf16, K x N: dense inverse in LDS and fills for the padding 129 + 10 us -> 43 us; without any transform 29.
// Four or eight blocks per thread, the next one's loads under a block's arithmetic, were slower (57 and 76 us): many
// short waves hide the loads better than few long ones.
template <typename WT, int FORM>
__global__ void __launch_bounds__(256, 4)
prep_weight_kernel(PrepArgs a, const double* __restrict__ outer_inv, const double* __restrict__ inner_inv,
                   const double* __restrict__ Tinv, const float* __restrict__ clip, const float* __restrict__ clip_max,
                   uint8_t* __restrict__ codes, uint8_t* __restrict__ scales) {
    // dense: the block's inverse; Kronecker: its inner factor's (broadcast reads)
    constexpr bool kKron = FORM == kPrepKron4 || FORM == kPrepKron8;
    constexpr int kInverse = FORM == kPrepDense ? 1024 : kKron ? (32 / FORM) * (32 / FORM) : 1;
    __shared__ double sT[kInverse];
    const int n = blockIdx.x * 256 + threadIdx.x;
    const int n_pad = (a.N + 31) & ~31;
    const int k = blockIdx.y;                               // includes the padding blocks of the last K group
    if constexpr (kInverse > 1) {
        const double* const src = kKron ? inner_inv + (size_t)k * a.inner_stride : Tinv + (size_t)k * 1024;
        if (k < a.nb)
            for (int i = threadIdx.x; i < kInverse; i += 256) sT[i] = src[i];
        __syncthreads();
    }
    if (n >= n_pad) return;
    const bool real = n < a.N;
    const int nc = min(n, a.N - 1);
    const WT* const col = static_cast<const WT*>(a.W) + (a.w_is_KxN ? (size_t)nc : (size_t)nc * a.ldw);
    const bool vec = !a.w_is_KxN && ((reinterpret_cast<uintptr_t>(a.W) | (uintptr_t)(a.ldw * (int64_t)sizeof(WT))) & 15u) == 0;
    auto load = [&](WT (&w)[32]) {
        if (a.w_is_KxN) {
            const WT* p = col + (size_t)(32 * k) * a.ldw;
#pragma unroll
            for (int j = 0; j < 32; ++j) w[j] = p[(size_t)j * a.ldw];
        } else if (vec) {
            const uint4* p = reinterpret_cast<const uint4*>(col + 32 * k);
            constexpr int kPer = 16 / sizeof(WT);
#pragma unroll
            for (int q = 0; q < 32 / kPer; ++q) {
                const uint4 v = p[q];
                const uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < kPer; ++e) {
                    if constexpr (sizeof(WT) == 4) w[q * kPer + e] = __uint_as_float(d[e]);
                    else w[q * kPer + e] = (WT)(d[e >> 1] >> (16 * (e & 1)));
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < 32; ++j) w[j] = col[32 * k + j];
        }
    };
    const int n_out = a.il_off >= 0 ? 64 * (n >> 5) + a.il_off + (n & 31) : n;
    uint32_t s = 127u;
    uint4 out = {0u, 0u, 0u, 0u};
    if (k < a.nb) {                                         // uniform
        double w[32];
        {
            WT raw[32];
            load(raw);
#pragma unroll
            for (int j = 0; j < 32; ++j) w[j] = w_value(raw[j]);
        }
        float y[32];
        if constexpr (FORM == kPrepKron4 || FORM == kPrepKron8) {
            constexpr int GO = FORM, GI = 32 / FORM;
            const double* const I = sT;
            const double* const O = outer_inv + (size_t)k * a.outer_stride;
            // one row of the inner factor at a time: its products with all groups, then the outer factor on them
#pragma unroll
            for (int c = 0; c < GI; ++c) {
                double row[GI];
#pragma unroll
                for (int c2 = 0; c2 < GI; ++c2) row[c2] = I[c * GI + c2];
                double v[GO];
#pragma unroll
                for (int a2 = 0; a2 < GO; ++a2) {
                    double acc = row[0] * w[a2 * GI];
#pragma unroll
                    for (int c2 = 1; c2 < GI; ++c2) acc = __builtin_fma(row[c2], w[a2 * GI + c2], acc);
                    v[a2] = acc;
                }
#pragma unroll
                for (int r = 0; r < GO; ++r) {
                    double acc = O[r * GO] * v[0];
#pragma unroll
                    for (int a2 = 1; a2 < GO; ++a2) acc = __builtin_fma(O[r * GO + a2], v[a2], acc);
                    y[r * GI + c] = (float)acc;
                }
            }
        } else if constexpr (FORM == kPrepDense) {
#pragma unroll 4
            for (int j2 = 0; j2 < 32; ++j2) {
                double acc = 0.0;
#pragma unroll
                for (int j = 0; j < 32; ++j) acc = __builtin_fma(sT[j2 * 32 + j], w[j], acc);
                y[j2] = (float)acc;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 32; ++j) y[j] = (float)w[j];
        }
        float bound;
        if (clip_max) {
            // Eq. 3-4 as printed: clamp to [r_min * min, r_max * max]; the scale comes from what is left
            float mn = y[0], mx = y[0];
#pragma unroll
            for (int j = 1; j < 32; ++j) {
                mn = __builtin_fminf(mn, y[j]);
                mx = __builtin_fmaxf(mx, y[j]);
            }
            const float lo = clip[k] * mn, hi = clip_max[k] * mx;
            bound = 0.f;
#pragma unroll
            for (int j = 0; j < 32; ++j) {
                y[j] = clamp_lo_hi(y[j], lo, hi);
                bound = __builtin_fmaxf(bound, __builtin_fabsf(y[j]));
            }
        } else {
            float m = 0.f;
#pragma unroll
            for (int j = 0; j < 32; ++j) m = __builtin_fmaxf(m, __builtin_fabsf(y[j]));
            bound = clip ? clip[k] * m : m;
        }
        if (real) {
            s = e8m0_of_bound(bound);
            const float sc = scale_operand(s);
            out.x = encode8(y, bound, sc);
            out.y = encode8(y + 8, bound, sc);
            out.z = encode8(y + 16, bound, sc);
            out.w = encode8(y + 24, bound, sc);
        }
    }
    *reinterpret_cast<uint4*>(codes + code_chunk_offset(n_out, k, a.nb)) = out;
    if (real) scales[scale_index_internal(n_out, k, a.N_out)] = (uint8_t)s;
}

template <typename WT, int FORM>
void launch_as(const batq_transform* t, const PrepArgs& a, const float* clip, const float* clip_max, uint8_t* codes,
               uint8_t* scales, dim3 grid, hipStream_t stream) {
    prep_weight_kernel<WT, FORM><<<grid, dim3(256), 0, stream>>>(a, t->d_outer_inv, t->d_inner_inv, t->d_Tinv, clip, clip_max,
                                                                 codes, scales);
}

template <typename WT>
void launch_form(const batq_transform* t, const PrepArgs& a, const float* clip, const float* clip_max, uint8_t* codes,
                 uint8_t* scales, dim3 grid, hipStream_t stream) {
    if (!t->has_transform) launch_as<WT, kPrepIdentity>(t, a, clip, clip_max, codes, scales, grid, stream);
    else if (t->form == BATQ_FORM_DENSE) launch_as<WT, kPrepDense>(t, a, clip, clip_max, codes, scales, grid, stream);
    else if (t->g_outer == 4) launch_as<WT, kPrepKron4>(t, a, clip, clip_max, codes, scales, grid, stream);
    else launch_as<WT, kPrepKron8>(t, a, clip, clip_max, codes, scales, grid, stream);
}

}  // namespace

hipError_t launch_prepare_weight(const batq_transform* t, const void* W, batq_dtype wdtype, int K, int N,
                                 int64_t ldw, int w_is_KxN, int N_out, int il_off, const float* d_clip_w,
                                 const float* d_clip_w_max, uint8_t* codes, uint8_t* scales, hipStream_t stream) {
    PrepArgs a;
    a.W = W;
    a.ldw = ldw;
    a.w_is_KxN = w_is_KxN;
    a.N = N;
    a.N_out = N_out;
    a.il_off = il_off;
    a.nb = K / 32;
    a.outer_stride = t->outer_stride;
    a.inner_stride = t->inner_stride;
    const dim3 grid((N + 255) / 256, 8 * scale_groups(a.nb));
    if (wdtype == BATQ_BF16) launch_form<uint16_t>(t, a, d_clip_w, d_clip_w_max, codes, scales, grid, stream);
    else launch_form<float>(t, a, d_clip_w, d_clip_w_max, codes, scales, grid, stream);
    return hipGetLastError();
}

}  // namespace batq
