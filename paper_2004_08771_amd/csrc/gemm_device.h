// Device helpers that the dense product kernels share.
#pragma once

#include "hb_internal.h"

namespace hb {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float sigmoidf_fast(float z)
{
    return __builtin_amdgcn_rcpf(1.0f + __expf(-z));  // v_rcp_f32: 1 ulp, no division sequence
}

template <int V>
struct IntC {
    static constexpr int value = V;
};
// calls f(IntC<activation>) with the run-time activation as a constant
template <typename F>
__device__ __forceinline__ void with_activation(int act, F &&f)
{
    if (act == ACT_SIGMOID) f(IntC<ACT_SIGMOID>());
    else if (act == ACT_RELU) f(IntC<ACT_RELU>());
    else f(IntC<ACT_NONE>());
}

// Operand rows for v_mfma_f32_32x32x2_f32 (ROWS = 32) or v_mfma_f32_16x16x4_f32 (16) straight from memory: the ROWS
// rows from `first` on (wavefront-uniform), those past `last` read as that one.  Lane (r, h) = (lane % ROWS, lane / ROWS)
// holds of row r the values k0 + QS q + lane_k(h) + c (q < NQ, c < 4) as x[4 q + c].  16-byte buffer loads at any 4-byte
// alignment where k runs along the rows, else single values of ROWS neighbouring rows.
template <bool KMAJ, int ROWS = 32, int QS = 8>
struct Fp32Rows {
    static constexpr int NQ = ROWS / 8;
    // 16 rows: four lanes to a row, two of them with the values QS / 2 further on
    static __device__ __forceinline__ int lane_k(int h) { return ROWS == 32 ? 4 * h : QS / 2 * (h >> 1) + 4 * (h & 1); }
    const float *base;
    int ld, kl;
    unsigned off;  // bytes from value k0 of row `first`
    __device__ __forceinline__ Fp32Rows(const float *P, int ld_, int first, int last, int r, int h) : ld(ld_), kl(lane_k(h))
    {
        first = min(first, last);
        const unsigned row = (unsigned)min(r, last - first);
        base = KMAJ ? P + (size_t)first * ld : P + first;
        off = 4u * (KMAJ ? row * (unsigned)ld + (unsigned)kl : row + (unsigned)kl * (unsigned)ld);
    }
    // q of a piece of 32 (16) values.  WHOLE: they are inside the contraction; else those from kend on read as zero
    template <bool WHOLE>
    __device__ __forceinline__ void load(float *x, int q, int k0, int kend) const
    {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(KMAJ ? base + k0 : base + (size_t)(k0 + QS * q) * ld), (short)0, -1, 0x00027000);
        if (KMAJ && WHOLE) {
            const v4u t = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 4 * QS * q, 0);
#pragma unroll
            for (int c = 0; c < 4; ++c) x[4 * q + c] = __uint_as_float(t[c]);
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                x[4 * q + c] = 0.f;
                if (WHOLE || k0 + QS * q + kl + c < kend)
                    x[4 * q + c] = __uint_as_float(
                        __builtin_amdgcn_raw_buffer_load_b32(rs, off, 4 * (KMAJ ? QS * q + c : c * ld), 0));
            }
        }
    }
    static constexpr int SPAN = (ROWS == 32) ? 8 : QS / 2 + 8;  // k of one q, from the first to the last
};
// n q's of both operands, side by side: where k runs along the rows, lines that several wavefronts share are asked for by all
// of them at about the same time
template <int N, typename RA, typename RB>
__device__ __forceinline__ void load_rows(const RA &ra, const RB &rb, float *xa, float *xb, int k0, int kend, int qs)
{
    if (k0 + (N - 1) * qs + RA::SPAN <= kend) {
#pragma unroll
        for (int q = 0; q < N; ++q) {
            ra.template load<true>(xa, q, k0, kend);
            rb.template load<true>(xb, q, k0, kend);
        }
    } else {
#pragma unroll
        for (int q = 0; q < N; ++q) {
            if (k0 + qs * q + RA::SPAN <= kend) {
                ra.template load<true>(xa, q, k0, kend);
                rb.template load<true>(xb, q, k0, kend);
            } else if (k0 + qs * q < kend) {
                ra.template load<false>(xa, q, k0, kend);
                rb.template load<false>(xb, q, k0, kend);
            }
        }
    }
}

// mean loss = (sum of the block partials, in index order per thread then a fixed tree) / B, by the first 256 threads
__device__ __forceinline__ void loss_finalize(const LossFinalize &f, double *dred /* 256 */)
{
    const int tid = threadIdx.x;
    if (tid < 256) {
        double s = 0.0;
        for (int i = tid; i < f.n; i += 256) s += (double)f.partials[i];
        dred[tid] = s;
    }
    __syncthreads();
#pragma unroll
    for (int st = 128; st > 0; st >>= 1) {
        if (tid < st) dred[tid] += dred[tid + st];
        __syncthreads();
    }
    if (tid == 0) {
        const float mean = (float)(dred[0] / (double)f.B);
        f.out[0] = mean;
        if (f.out2) f.out2[0] = mean;
    }
}

// XCD-aware tile order: consecutive hardware workgroup ids go round-robin over the 8 XCDs,
// so give each XCD a contiguous run of the T tiles (they share an A row panel in its L2).
__device__ __forceinline__ int xcd_tile_order(int b, int T)
{
    return ((T & 7) == 0) ? (b & 7) * (T >> 3) + (b >> 3) : b;
}

}  // namespace hb
