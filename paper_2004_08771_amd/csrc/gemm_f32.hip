// fp32 MFMA GEMM for the three dense layer products of the mini-batch step
// (Section 3 of the paper: forward Eq. (1), backward Eq. (2); on a batch the
// matrix-vector products become matrix-matrix products, the dominant cost).
//
// This file: the plan (which kernel, tile shape and split a product gets) and the kernels for
// products with few output tiles (small batches), on fp32 MFMAs.  Epilogues fuse
// bias + activation (forward), the activation derivative (backward-data) and the bias-gradient
// column sums (weight gradient).  The large products are in gemm_split.hip.
#include "gemm_device.h"

#include <algorithm>
#include <stdlib.h>

#include <type_traits>

namespace hb {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int WAVES = 8;         // wavefronts of a workgroup, which share the contraction of one output block
constexpr int NT = 64 * WAVES;
constexpr int SMALL_CHUNK = 64;  // slices of a split contraction are multiples of this

// ---- small products: one output block of 32 x 32 or 16 x 16 per workgroup, the contraction dealt to its eight wavefronts
// in groups of eight k (wavefront w has the groups w, w + 8, ..).
//
// What bounds a product of few tiles is a chain of latencies, so there is no staging through LDS and no barrier in the
// loop: a wavefront loads its share of the operands straight into the registers that its MFMAs read, two pieces of
// 256 k (of the workgroup) in flight, 16 bytes per load where k runs along the rows and else four-byte loads of
// neighbouring rows.  The eight partial blocks meet in LDS.  The sums are the same, bit for bit, for both block sizes and
// in the form of the weight gradient without a workgroup per block.
// Time stamps in a 16 x 512 x 512 forward product, 32 x 32 blocks: 1.3 us from the end of the launch before to the first
// wavefront, 1.0 to issue the loads, 1.4 until they land, 1.8 for 2 x 32 MFMAs per SIMD and the write to LDS, 0.6 to finish.
// 16 x 16 blocks (v_mfma_f32_16x16x4_f32) shorten the MFMA chain to a quarter and the loads of a workgroup to a half.
// Against four wavefronts that staged k-tiles of 64 in LDS: forward 8.3 -> 4.6 us there (64 rows 7.2 -> 4.4, 256 rows 7.5 -> 6.3),
// paired backward launch 8.9 -> 4.5 (64 rows 8.0 -> 4.7, 256 rows 9.3 -> 7.0), weight gradient 512 x 54 over 1021 rows 12.1 -> 5.3
// (its bias gradient was a chain of 512 additions per column).
constexpr int GROUPS = 8 * WAVES;  // from one group of a wavefront to its next

// Multiplies one group (ROWS = 32) or two (16) of both operands, x[4 q ..] as Fp32Rows leaves them: k in the order
// 0 4 1 5 2 6 3 7 of a group.  16 x 16: four k to an MFMA, so the lanes of the second group swap places with those of the
// first that hold the values one further on.
__device__ __forceinline__ void multiply_group(v16f &acc, const float *xa, const float *xb)
{
#pragma unroll
    for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[c], xb[c], acc, 0, 0, 0);
}
__device__ __forceinline__ void multiply_group(v4f &acc, const float *xa, const float *xb)
{
    float ya[4], yb[4];
    auto swap = [](const float *x, float *y) {  // y: 0 1 | 2 3 of the first group, then of the second
#pragma unroll
        for (int c = 0; c < 4; c += 2) {
            const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[c]), __float_as_uint(x[c + 1]), false, false);
            y[c / 2] = __uint_as_float(t[0]);
            y[2 + c / 2] = __uint_as_float(t[1]);
        }
    };
    swap(xa, ya);
    swap(xb, yb);
#pragma unroll
    for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ya[c], yb[c], acc, 0, 0, 0);
}

template <int TILE>
struct SmallLds {
    static constexpr int LD = (TILE == 32) ? 40 : 20;  // rows 4 apart: 32 (16) banks apart
    static constexpr int RED = TILE * LD;              // a partial block
    static constexpr int FLOATS = WAVES * (RED + 32);  // and the column sums of the weight gradient
};

// a finished sum -> the stored value: bias and activation (forward), the activation's derivative at o (backward-data)
template <int KIND, int ACT>
__device__ __forceinline__ float finish(float x, float bias, float o)
{
    if (KIND == GEMM_FWD) {
        x += bias;
        if (ACT == ACT_SIGMOID) x = sigmoidf_fast(x);
        else if (ACT == ACT_RELU) x = fmaxf(x, 0.f);
    } else if (KIND == GEMM_DA) {
        if (ACT == ACT_SIGMOID) x *= o * (1.f - o);
        else if (ACT == ACT_RELU) x = (o > 0.f) ? x : 0.f;
    }
    return x;
}

template <int TILE, bool A_KMAJ, bool B_KMAJ, int KIND>
__device__ __forceinline__ void gemm_f32_small_tile(const GemmArgs &a, float *smem, int id, int split)
{
    static_assert(TILE == 32 || KIND != GEMM_DW, "the weight gradient has many tiles");
    constexpr int QS = (TILE == 32) ? GROUPS : 2 * GROUPS;
    constexpr int LD = SmallLds<TILE>::LD, RED = SmallLds<TILE>::RED;
    constexpr int OUT = (TILE == 32) ? 2 : 1;                 // values that a lane finishes
    using Acc = std::conditional_t<TILE == 32, v16f, v4f>;
    constexpr int NACC = TILE * TILE / 64;
    using RA = Fp32Rows<A_KMAJ, TILE, QS>;
    using RB = Fp32Rows<B_KMAJ, TILE, QS>;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane % TILE, h = lane / TILE;

    const int tile_m = id / a.tiles_n, tile_n = id - tile_m * a.tiles_n;
    const int m0 = tile_m * TILE, n0 = tile_n * TILE;
    const int kbeg = split * a.k_chunk + 8 * wave;
    const int kend = min(a.K, split * a.k_chunk + a.k_chunk);

    const RA ra(static_cast<const float *>(a.A), a.lda, m0, a.M - 1, r, h);
    const RB rb(static_cast<const float *>(a.B), a.ldb, n0, a.N - 1, r, h);

    // the lane's values of the finished block: rows row0 + p of column r (16 x 16: the first four wavefronts have one each)
    const int row0 = (TILE == 32) ? 8 * (wave >> 1) + 4 * h + 2 * (wave & 1) : 4 * wave + h, n = n0 + r;
    const bool finishes = (TILE == 32 || wave < 4) && n < a.N;
    // what the epilogue needs is requested now
    const float bias = (KIND == GEMM_FWD && a.bias != nullptr && finishes) ? a.bias[n] : 0.f;
    float o[OUT];
#pragma unroll
    for (int p = 0; p < OUT; ++p)
        o[p] = (KIND == GEMM_DA && finishes && m0 + row0 + p < a.M)
                   ? static_cast<const float *>(a.aux)[(size_t)(m0 + row0 + p) * a.ldaux + n] : 0.f;

    Acc acc;
#pragma unroll
    for (int v = 0; v < NACC; ++v) acc[v] = 0.f;
    const bool do_colsum = (KIND == GEMM_DW) && a.colsum != nullptr && tile_n == 0;
    float colsum = 0.f;

    float xa[2][4 * RA::NQ], xb[2][4 * RB::NQ];
    auto load = [&](int set, int k0) { load_rows<RA::NQ>(ra, rb, xa[set], xb[set], k0, kend, QS); };
    auto multiply = [&](int set, int k0) {
#pragma unroll
        for (int q = 0; q < RA::NQ; ++q) {
            if (k0 + QS * q >= kend) break;  // uniform
            multiply_group(acc, &xa[set][4 * q], &xb[set][4 * q]);
            if (KIND == GEMM_DW && do_colsum)
                colsum += (xa[set][4 * q] + xa[set][4 * q + 1]) + (xa[set][4 * q + 2] + xa[set][4 * q + 3]);
        }
    };
    constexpr int STEP = 4 * GROUPS;
    if (kbeg < kend) load(0, kbeg);
    if (kbeg + STEP < kend) load(1, kbeg + STEP);
    for (int k = kbeg; k < kend; k += 2 * STEP) {
        multiply(0, k);
        if (k + 2 * STEP < kend) load(0, k + 2 * STEP);
        if (k + STEP < kend) {
            multiply(1, k + STEP);
            if (k + 3 * STEP < kend) load(1, k + 3 * STEP);
        }
    }

    // acc[v] is C(row, r) with row = 8 (v / 4) + 4 h + (v % 4) (16 x 16: v < 4)
    float *mine = smem + wave * RED;
#pragma unroll
    for (int v = 0; v < NACC; ++v) mine[(8 * (v >> 2) + 4 * h + (v & 3)) * LD + r] = acc[v];
    if (KIND == GEMM_DW && do_colsum) {  // the two halves of a wavefront hold different k
        colsum += __shfl_xor(colsum, 32, 64);
        if (h == 0) smem[WAVES * RED + wave * 32 + r] = colsum;
    }
    __syncthreads();

    float *__restrict__ C = static_cast<float *>(a.C) + (size_t)split * a.c_split_stride;
    if (TILE == 32 || wave < 4)
        with_activation(KIND == GEMM_DW ? (int)ACT_NONE : a.act, [&](auto act_c) {
            constexpr int ACT = decltype(act_c)::value;
#pragma unroll
            for (int p = 0; p < OUT; ++p) {
                const float *s = smem + (row0 + p) * LD + r;
                const float x = ((s[0] + s[4 * RED]) + (s[RED] + s[5 * RED])) + ((s[2 * RED] + s[6 * RED]) + (s[3 * RED] + s[7 * RED]));
                if (m0 + row0 + p < a.M && finishes) C[(size_t)(m0 + row0 + p) * a.ldc + n] = finish<KIND, ACT>(x, bias, o[p]);
            }
        });
    if (KIND == GEMM_DW && do_colsum) {
        const int t = threadIdx.x;
        if (t < 32 && m0 + t < a.M) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) s += smem[WAVES * RED + w * 32 + t];
            a.colsum[(size_t)split * a.M + m0 + t] = s;
        }
    }
}

// Weight gradient with a wavefront to each 32 x 32 block and a whole slice of up to NQ x 64 batch rows: no barrier and nothing
// that passes through LDS (see small_dw_wave).  It takes the shares of the eight wavefronts one after the other, in
// the order in which their sums are added.  The eight blocks of a workgroup are neighbours and read the same rows of D_l.
template <int NQ>
__device__ __forceinline__ void gemm_f32_small_dw_wave(const GemmArgs &a, int id, int split)
{
    constexpr int SETS = WAVES / NQ;  // shares in flight: 64 registers
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, h = lane >> 5;
    id = WAVES * id + wave;
    if (id >= a.tiles_m * a.tiles_n) return;
    const int tile_m = id / a.tiles_n, tile_n = id - tile_m * a.tiles_n;
    const int m0 = tile_m * 32, n0 = tile_n * 32;
    const int kbeg = split * a.k_chunk, kend = min(a.K, kbeg + a.k_chunk);
    using R = Fp32Rows<false, 32, GROUPS>;
    const R ra(static_cast<const float *>(a.A), a.lda, m0, a.M - 1, r, h);
    const R rb(static_cast<const float *>(a.B), a.ldb, n0, a.N - 1, r, h);
    const bool do_colsum = a.colsum != nullptr && tile_n == 0;
    float colsum[WAVES];
    float xa[SETS][4 * NQ], xb[SETS][4 * NQ];
    constexpr int ORDER[WAVES] = {0, 4, 1, 5, 2, 6, 3, 7};
    auto load = [&](int p) { load_rows<NQ>(ra, rb, xa[p % SETS], xb[p % SETS], kbeg + 8 * ORDER[p], kend, GROUPS); };
#pragma unroll
    for (int p = 0; p < SETS; ++p) load(p);
    v16f acc[3];  // acc[0], acc[1]: the two halves of the sum; acc[2]: an eighth
#pragma unroll
    for (int p = 0; p < WAVES; ++p) {
        const int k0 = kbeg + 8 * ORDER[p], set = p % SETS;
        v16f t;
#pragma unroll
        for (int v = 0; v < 16; ++v) t[v] = 0.f;
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if (k0 + GROUPS * q >= kend) break;  // uniform
            multiply_group(t, &xa[set][4 * q], &xb[set][4 * q]);
            if (do_colsum) s += (xa[set][4 * q] + xa[set][4 * q + 1]) + (xa[set][4 * q + 2] + xa[set][4 * q + 3]);
        }
        colsum[ORDER[p]] = s;
        if (p + SETS < WAVES) load(p + SETS);
        if ((p & 1) == 0) {
            acc[2] = t;
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) t[v] = acc[2][v] + t[v];
            if (p == 1) {
                acc[0] = t;
            } else if (p == 5) {
                acc[1] = t;
            } else {
                v16f &half = acc[p == 3 ? 0 : 1];
#pragma unroll
                for (int v = 0; v < 16; ++v) half[v] += t[v];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    float *__restrict__ C = static_cast<float *>(a.C) + (size_t)split * a.c_split_stride;
    if (n0 + r < a.N) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int m = m0 + 8 * (v >> 2) + 4 * h + (v & 3);
            if (m < a.M) C[(size_t)m * a.ldc + n0 + r] = acc[0][v] + acc[1][v];
        }
    }
    if (do_colsum) {  // the two halves of a wavefront hold different k
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) s += colsum[w] + __shfl_xor(colsum[w], 32, 64);
        if (h == 0 && m0 + r < a.M) a.colsum[(size_t)split * a.M + m0 + r] = s;
    }
}

template <int TILE, bool A_KMAJ, bool B_KMAJ, int KIND>
__global__ __launch_bounds__(NT, 4) void gemm_f32_small_kernel(GemmArgs a)
{
    __shared__ float smem[SmallLds<TILE>::FLOATS];
    gemm_f32_small_tile<TILE, A_KMAJ, B_KMAJ, KIND>(a, smem, xcd_tile_order(blockIdx.x, gridDim.x), blockIdx.y);
}

// The backward pair of one hidden layer (see launch_gemm_f32_bwd_pair) for small batches.  The product whose
// workgroups walk the longer contraction goes first: of a wide layer the backward-data product, whose few workgroups
// take most of the launch, while the many short ones of the weight gradient fill the other compute units (16 rows,
// 2048 wide: 35.2 us with the weight gradient first, 27 so; 4096 wide 99 -> 60).
// DW_NQ: a wavefront for each block of the weight gradient over up to DW_NQ x 64 batch rows (0: a workgroup)
template <int DA_TILE, int DW_NQ>
__global__ __launch_bounds__(NT, DW_NQ ? 3 : 4) void gemm_f32_small_pair_kernel(GemmArgs da, GemmArgs dw, int n_dw)
{
    __shared__ float smem[DW_NQ ? SmallLds<DA_TILE>::FLOATS : SmallLds<32>::FLOATS];
    const int n_da = (int)gridDim.x - n_dw, dw_from = (da.K > dw.k_chunk) ? n_da : 0;
    const int b = (int)blockIdx.x - dw_from;  // of the weight gradient if in [0, n_dw)
    if (b >= 0 && b < n_dw) {
        const int blocks = DW_NQ ? (dw.tiles_m * dw.tiles_n + WAVES - 1) / WAVES : dw.tiles_m * dw.tiles_n;
        const int id = xcd_tile_order(b % blocks, blocks), split = b / blocks;
        if constexpr (DW_NQ > 0) gemm_f32_small_dw_wave<DW_NQ>(dw, id, split);
        else gemm_f32_small_tile<32, false, false, GEMM_DW>(dw, smem, id, split);
    } else {
        gemm_f32_small_tile<DA_TILE, true, false, GEMM_DA>(da, smem, xcd_tile_order(dw_from ? (int)blockIdx.x : b - n_dw, n_da), 0);
    }
}
template <int NQ>
__global__ __launch_bounds__(NT, 3) void gemm_f32_small_dw_wave_kernel(GemmArgs a)
{
    gemm_f32_small_dw_wave<NQ>(a, xcd_tile_order(blockIdx.x, gridDim.x), blockIdx.y);
}

// ---- forward products of more 32 x 32 blocks than compute units.  There the loads of the kernel above, 32 bytes of each
// of 32 rows at a time, hold up each other in the L1 (1021 x 512 x 512 11.6 us, 512 x 983 x 512 12.0), so the operands pass
// through LDS (10.2, 10.7): four wavefronts, k-tiles of 64 whose rows are read 256 bytes at a time, two stages in LDS and
// one k-tile in registers.  A wavefront takes the groups of eight k that two of the kernel above take, and the sums are
// the same, bit for bit.
constexpr int STAGED_NT = 256, STAGED_BK = 64, STAGED_LD = STAGED_BK + 4;

__global__ __launch_bounds__(STAGED_NT) void gemm_f32_staged_kernel(GemmArgs a)
{
    constexpr int OPERAND = 32 * STAGED_LD, STAGE = 2 * OPERAND;  // floats
    constexpr int LD = SmallLds<32>::LD, RED = SmallLds<32>::RED;
    static_assert(2 * STAGE >= 4 * RED, "partial blocks reuse the stages");
    __shared__ __attribute__((aligned(16))) float smem[2 * STAGE];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, h = lane >> 5;
    const int id = xcd_tile_order(blockIdx.x, gridDim.x);
    const int tile_m = id / a.tiles_n, tile_n = id - tile_m * a.tiles_n;
    const int m0 = tile_m * 32, n0 = tile_n * 32;
    const int nk = (a.K + STAGED_BK - 1) / STAGED_BK;
    const float bias = (a.bias != nullptr && n0 + r < a.N) ? a.bias[n0 + r] : 0.f;

    // thread: 16 bytes at k = 4 (tid % 16) of rows tid / 16 and tid / 16 + 16 of each operand (past the end: the last row)
    const float *base[2] = {static_cast<const float *>(a.A) + (size_t)m0 * a.lda, static_cast<const float *>(a.B) + (size_t)n0 * a.ldb};
    unsigned off[2][2];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        off[0][v] = 4u * ((unsigned)min((tid >> 4) + 16 * v, a.M - 1 - m0) * (unsigned)a.lda + 4 * (tid & 15));
        off[1][v] = 4u * ((unsigned)min((tid >> 4) + 16 * v, a.N - 1 - n0) * (unsigned)a.ldb + 4 * (tid & 15));
    }
    v4f x[2][2];
    auto load = [&](int t) {
        const int k0 = t * STAGED_BK;
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base[o] + k0), (short)0, -1, 0x00027000);
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                if (k0 + STAGED_BK <= a.K) {
                    x[o][v] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rs, off[o][v], 0, 0));
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        x[o][v][c] = 0.f;
                        if (k0 + 4 * (tid & 15) + c < a.K)
                            x[o][v][c] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off[o][v], 4 * c, 0));
                    }
                }
            }
        }
    };
    auto store = [&](float *S) {
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int v = 0; v < 2; ++v)
                *reinterpret_cast<v4f *>(S + o * OPERAND + ((tid >> 4) + 16 * v) * STAGED_LD + 4 * (tid & 15)) = x[o][v];
    };
    v4f fa[2], fb[2];  // groups wave and wave + 4 of a k-tile
    auto read = [&](const float *S) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            fa[q] = *reinterpret_cast<const v4f *>(S + r * STAGED_LD + 8 * (wave + 4 * q) + 4 * h);
            fb[q] = *reinterpret_cast<const v4f *>(S + OPERAND + r * STAGED_LD + 8 * (wave + 4 * q) + 4 * h);
        }
    };
    v16f acc[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[q][v] = 0.f;

    // global loads run two k-tiles ahead, the write to LDS one; the fragments of tile kt + 1 are read right behind the barrier
    // of tile kt, under its last MFMAs
    load(0);
    store(smem);
    if (nk > 1) load(1);
    __syncthreads();
    read(smem);
    for (int kt = 0; kt < nk; ++kt) {
        float *next = smem + ((kt + 1) & 1) * STAGE;
        if (kt + 1 < nk) store(next);
        if (kt + 2 < nk) load(kt + 2);
        v4f ca[2] = {fa[0], fa[1]}, cb[2] = {fb[0], fb[1]};
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int q = 0; q < 2; ++q) acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(ca[q][c], cb[q][c], acc[q], 0, 0, 0);
        __syncthreads();  // tile kt read by everyone (fragments are in registers), tile kt + 1 written
        if (kt + 1 < nk) read(next);
#pragma unroll
        for (int c = 2; c < 4; ++c)
#pragma unroll
            for (int q = 0; q < 2; ++q) acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(ca[q][c], cb[q][c], acc[q], 0, 0, 0);
    }
    float *mine = smem + wave * RED;  // behind the last barrier nobody reads a stage
#pragma unroll
    for (int v = 0; v < 16; ++v) mine[(8 * (v >> 2) + 4 * h + (v & 3)) * LD + r] = acc[0][v] + acc[1][v];
    __syncthreads();
    float *__restrict__ C = static_cast<float *>(a.C);
    with_activation(a.act, [&](auto act_c) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int row = 8 * wave + 2 * p + h;
            const float *s = smem + row * LD + r;
            const float x = (s[0] + s[RED]) + (s[2 * RED] + s[3 * RED]);
            if (m0 + row < a.M && n0 + r < a.N)
                C[(size_t)(m0 + row) * a.ldc + n0 + r] = finish<GEMM_FWD, decltype(act_c)::value>(x, bias, 0.f);
        }
    });
}

int env_int(const char *name, int dflt)
{
    const char *s = getenv(name);
    return (s && *s) ? atoi(s) : dflt;
}

// ---- plan of the split-plane kernels (gemm_split.hip).
struct Shape {
    int bm, bn;
};
constexpr Shape SHAPES[] = {{64, 64}, {128, 64}, {128, 128}, {64, 64}, {64, 32}};  // by the number launch_gemm_split takes
constexpr int SHARED = 3;  // 64 x 64, the contraction shared by two groups of wavefronts ...
constexpr int SHARED_K = 256;  // ... of at least this length (32-deep: 4.6 us alone, 4.8 shared)
constexpr int HALF = 4;        // 64 x 32, the contraction shared by four groups (forward products only, long_fwd())
constexpr int CUS = 256;
constexpr int K_CHUNK_ALIGN = 32;  // slices of a split contraction are multiples of the k-tile

long long tiles_of(int sh, int M, int N)
{
    return (long long)((M + SHAPES[sh].bm - 1) / SHAPES[sh].bm) * ((N + SHAPES[sh].bn - 1) / SHAPES[sh].bn);
}

// Clocks per k-tile of a workgroup, in hundreds, from time stamps around the main loop (MI355X,
// K = 512; taken, as the times below and plan_pair's, before the operands were scaled, which adds 2 to 4 % to all shapes): 64 x 64 9 alone on its compute unit (6 with two groups of wavefronts, which fill its LDS)
// and 15 for two that share one, 128 x 64 12.5,
// 128 x 128 20 (one per compute unit).  The shape with the shortest sequence of rounds wins:
// 4096 x 512 outputs 14.6 us as 128 x 64 (256 workgroups), 16.8 as 64 x 64, 20 as 128 x 128;
// 8192 x 512 27 / 31 / 25.8; 2048 x 512 12.0 / 11.2 / 19, with two groups 10.6 (12.7 without, in a step).
double rounds_cost(int sh, long long blocks)
{
    const long long r = (blocks + CUS - 1) / CUS;
    if (sh == 2) return 20.0 * r;
    if (sh == 1) return 12.5 * r;
    if (sh == SHARED) return r <= 1 ? 6.0 : 7.5 * r;  // 4096 x 512 (two rounds): 18.6 us against 16.4 as 128 x 64
    return blocks <= CUS ? 9.0 : 15.0 * ((r + 1) / 2);
}
int pick_shape(int M, int N, int K)
{
    int best = 0;
    for (int sh = 1; sh < (K >= SHARED_K ? 4 : 3); ++sh)
        if (rounds_cost(sh, tiles_of(sh, M, N)) <= rounds_cost(best, tiles_of(best, M, N))) best = sh;
    return best;
}

struct SplitPlan {
    int splits, chunk;
};
SplitPlan slices(int K, int s)
{
    const int chunk = ((K + s - 1) / s + K_CHUNK_ALIGN - 1) / K_CHUNK_ALIGN * K_CHUNK_ALIGN;
    return {(K + chunk - 1) / chunk, chunk};
}
// Slices of a weight gradient (its contraction runs over the batch) of `tiles` output tiles for
// `wgs` workgroups in all, each slice at least 128 long.
SplitPlan plan_splits(long long tiles, int K, int max_splits, long long wgs)
{
    long long s = (wgs + tiles - 1) / tiles;
    const int by_k = (K + 4 * K_CHUNK_ALIGN - 1) / (4 * K_CHUNK_ALIGN);
    if (s > by_k) s = by_k;
    if (s > max_splits) s = max_splits;
    if (s < 1) s = 1;
    return slices(K, (int)s);
}

// Shape and batch slices of a paired backward launch: the pair with the shortest estimated time, from
// the workgroups' lengths (clocks per k-tile as above, plus 60 hundred for prologue and epilogue)
// dealt out as the hardware does, weight-gradient workgroups first, and the slices' partial sums
// written and read again at 3 TB/s.  Against one workgroup of the weight gradient per workgroup of
// the backward-data product in the largest shape that fills the device: 3001 x 1024 x 1024 84.4 ->
// 74.2 us, 3001 x 512 x 512 31.1 -> 24.5, 1500 x 512 x 512 20.3 -> 16.0, 4096 x 512 x 512 26.8 -> 26.2 (the
// same plan; a contiguous eighth of the pieces per XCD).
struct PairPlan {
    int shape;
    SplitPlan split;
};
// end of n1 pieces of length a followed by n2 of length b on `slots` servers, each piece on the first free one
double makespan(long long n1, double a, long long n2, double b, long long slots)
{
    const long long q = n1 / slots, rem = n1 % slots;
    double t0 = q * a, t1 = t0 + a;           // slots - rem servers are free at t0, rem at t1
    long long c0 = slots - rem, c1 = rem;
    const long long rounds = n2 / slots;      // whole rounds shift both groups alike
    if (rounds > 0) {
        t0 += rounds * b;
        t1 += rounds * b;
        n2 -= rounds * slots;
    }
    double end = rem ? t1 : t0;
    while (n2 > 0) {
        if (c1 > 0 && t1 < t0) {
            const double t = t0;
            const long long c = c0;
            t0 = t1; c0 = c1; t1 = t; c1 = c;
        }
        const long long k = n2 < c0 ? n2 : c0;
        if (t0 + b > end) end = t0 + b;
        t0 += b;
        n2 -= k;
    }
    return end;
}
PairPlan plan_pair(const GemmArgs &da, const GemmArgs &dw, int max_splits)
{
    // with the whole chip busy (its clock is lower then); the weight gradient's M-major tiles cost more
    constexpr double DA_K[4] = {15.0, 13.0, 20.0, 7.5}, DW_K[4] = {16.0, 15.0, 21.0, 8.0};
    constexpr int SLOTS[4] = {2 * CUS, CUS, CUS, CUS};
    const int by_k = (dw.K + 4 * K_CHUNK_ALIGN - 1) / (4 * K_CHUNK_ALIGN);  // slices of at least 128
    int most = max_splits < by_k ? max_splits : by_k;
    if (most > 16) most = 16;
    if (most < 1) most = 1;
    PairPlan best = {0, slices(dw.K, 1)};
    double best_t = -1.0;
    for (int sh = 0; sh < 4; ++sh) {
        if (sh == SHARED && da.K < SHARED_K && dw.K < SHARED_K) continue;
        const long long n = tiles_of(sh, da.M, da.N), t = tiles_of(sh, dw.M, dw.N);
        const double len_da = 60.0 + DA_K[sh] * ((da.K + 31) / 32);
        for (int s = 1; s <= most; ++s) {
            const SplitPlan sp = slices(dw.K, s);
            if (sp.splits != s) continue;
            const double len_dw = 60.0 + DW_K[sh] * (sp.chunk / 32);
            const double sums = s * (double)dw.M * dw.N * 8.0 / 3.0e12 * 22.0e6;
            const double e = makespan(t * s, len_dw, n, len_da, SLOTS[sh]) + sums;
            if (best_t < 0.0 || e < best_t) {
                best_t = e;
                best = {sh, sp};
            }
        }
    }
    return best;
}

// Products with fewer 64 x 64 output tiles than small_tiles_max() (forward / backward-data; plan_f32_pair has a line of its
// own), or a contraction shorter than small_k_max() (weight gradient, whose contraction is the batch), go to the kernels
// of small products.  Small / split planes, us, forward products 512 wide: contraction of 128 4.4 / 5.0 with 64 tiles, 5.1 / 5.4
// with 128, 5.9 / 5.6 with 152; of 256 4.7 / 6.4, 7.0 / 6.9, 8.2 / 7.0; of 512 7.5 / 9.2 with 64, 9.9 / 9.3 with 80, 9.8 / 9.4 with
// 128, 11.7 / 9.4 with 152; of 1024 11.3 / 14.6, 15.8 / 14.7, 15.8 / 14.5, 19.8 / 14.8.  So the line of 160 tiles is that of
// contractions up to 256; longer ones: long_fwd().
// Contractions below 64 stay with split planes, although the small kernels are quicker there (512 x 54 forward, 16 rows 5.3 us,
// small 4.2; pair of 512 x 40, 48 rows 6.8, 4.2): over 300 drawn networks with inputs below 64 and 4 .. 63 rows their gradients
// would be 1.035 times as far from 64 bits.
// HB_GEMM_SMALL_TILES / HB_GEMM_SMALL_K: tuning aids (0: no small kernel for outputs / for weight gradients; either
// one for the paired launch).
int small_tiles_max()
{
    static const int v = env_int("HB_GEMM_SMALL_TILES", 160);  // B = 1280 for 512-wide layers
    return v;
}
int small_k_max()
{
    static const int v = env_int("HB_GEMM_SMALL_K", 2048);
    return v;
}
bool small_out(int M, int N, int K)
{
    return K >= 64 && (long long)((M + 63) / 64) * ((N + 63) / 64) < small_tiles_max();
}
// Forward products of 80 to 159 tiles over 768 and more, and of 80 to 127 over 512 to 767, go to the split planes, in tiles
// of 64 x 32 while each has a compute unit of its own (else 64 x 64): four groups of two wavefronts share the contraction, a
// quarter of the k-tiles in a row each, where 64 x 64 tiles leave half of the device idle and fp32 MFMAs are a longer chain
// than the conversions.  Networks of w-w-w-w-w-w-4 (2048 and more: w-w-w-4), forward and loss, us, small kernels / 64 x 64 /
// 64 x 32: w = 512 640 rows 55.5 / 54.0 / 47.1, 1021 rows 56.3 / 60.9 / 54.6; 768 430 rows 72.7 / 76.7 / 64.1, 600 rows 74.3
// / 71.6 / 61.9, 800 rows (312 tiles of 64 x 32) 90.0 / 77.3; 1024 320 rows 90.0 / 82.6 / 66.9, 510 rows 93.4 / 89.8 / 80.8;
// 2048 130 rows 69.0 / 61.6 / 51.2, 250 rows 71.4 / 65.3 / 56.5; 4096 100 rows 130.7 / 116.6 / 97.8.  Shorter contractions
// stay: 320 1021 rows 41.5 / 49.7 / 45.5; 256 2047 rows 38.9 / 45.3 / 43.0; fewer tiles too: 512 330 rows 43.9 / - / 47.5,
// 768 300 rows 58.2 / - / 63.1.  Narrower outputs than the ones measured, and up to 64 rows (4096 wide 88.6 / 88.3 / -), stay
// too.  So do 128 tiles and more over less than 768: 3 % (512 1021 rows) is little to give up the sums that all small forms
// share for, by which a row comes out the same, bit for bit, in batches of any size up to there.
bool long_fwd(int M, int N, int K)
{
    const long long tiles = (long long)((M + 63) / 64) * ((N + 63) / 64);
    return K >= 512 && N >= 512 && M > 64 && tiles >= 80 && (K >= 768 || tiles < 128) && small_out(M, N, K);
}
// A weight gradient launched on its own (not paired with a backward-data product) whose output
// is only a few tiles -- the first layer of a narrow input, 512 x 54 -- stays with the small
// kernel up to four times that contraction length: with so few tiles the 64-wide kernel needs
// tens of K-slices to fill the chip, and every slice is a partial the update has to read
// (512 x 54, small / split planes: 1000 rows 4.8 / 6.9 us, 4096 rows 5.3 / 8.0, 8000 rows 7.8 / 8.3, 8192 rows 8.1 / 8.6,
// 12000 rows 11.6 / 9.8; 100 x 100: 6000 rows 5.6 / 6.3, 8000 rows 6.7 / 6.6).  For other outputs: 1024 x 300, 80 tiles,
// 1000 rows 11.3 / 12.0, 2000 rows 16.5 / 19.6 (a longer update with it), 2500 rows 21.2 / 15.5; 2048 x 600, 320 tiles,
// 500 rows 18.2 / 18.8, 1000 rows 28.1 / 27.3, 2000 rows 52 / 44; of 1024 x 1024, 256 tiles, split planes would be ahead
// at every batch (500 rows 14.3 / 11.4 and 1.7 us more in the update, 1000 rows 25 / 17, 2000 rows 46 / 27).
long long small_dw_alone_kmax(int M, int N)  // contractions below this go to the small kernel
{
    const bool few_tiles = (long long)((M + 63) / 64) * ((N + 63) / 64) <= 16;
    return few_tiles ? 4 * (long long)small_k_max() : (long long)small_k_max();
}
bool small_dw_alone(int M, int N, int K)
{
    return K >= 64 && K < small_dw_alone_kmax(M, N);
}
// Output tile of the small kernel.  16 x 16 has a quarter of the MFMA chain of 32 x 32 and reads twice as much per
// result: it pays while a compute unit gets at most two of them (forward products 512 wide: 16 rows 6.1 us with 32 x 32,
// 4.5 with 16 x 16; 128 rows 6.2 / 4.2; 256 rows 6.2 / 5.6; 400 rows 6.3 / 9.2), beside a weight gradient at most one
// (pairs 512 wide: 128 rows 7.2 / 5.3, 200 rows 7.6 / 7.9).
int small_tile(int M, int N, bool pair)
{
    return (long long)((M + 15) / 16) * ((N + 15) / 16) <= (pair ? CUS : 2 * CUS) ? 16 : 32;
}
// Forward products of more 32 x 32 blocks than compute units pass through LDS (see gemm_f32_staged_kernel).
bool small_staged(int M, int N)
{
    return (long long)((M + 31) / 32) * ((N + 31) / 32) > CUS;
}
// Weight gradient: a wavefront per block for up to 32 rows, where a block takes one wavefront no longer than eight need to
// meet, and where the blocks alone occupy the device for as long as one of them walks the batch (pairs with a workgroup per block / so: 1024 blocks, 64 rows 11.5 / 10.8 us, 128 rows 14.1 / 10.6, 220 rows 18.0 / 19.5;
// 484 blocks, 64 rows 8.7 / 6.5, 150 rows 9.4 / 10.5; 256 blocks, 16 rows 5.1 / 4.5, 64 rows 5.4 / 5.8; 4096 blocks, 32 rows
// 27.4 / 18.4).  Above 128 rows its registers would spill.
int small_dw_wave(int M, int N, int K)  // 0, or the rows in units of 64
{
    const long long blocks = (long long)((M + 31) / 32) * ((N + 31) / 32);
    if (K > 32 && (K > 128 || 6 * K > blocks)) return 0;
    return K <= 64 ? 1 : 2;
}
// K-slices of the small weight-gradient kernel: at most 512 long (multiples of its k-tile)
SplitPlan plan_small_splits(int K, int max_splits)
{
    int s = (K + 511) / 512;
    if (s > max_splits) s = max_splits;
    if (s < 1) s = 1;
    const int chunk = ((K + s - 1) / s + SMALL_CHUNK - 1) / SMALL_CHUNK * SMALL_CHUNK;
    return {(K + chunk - 1) / chunk, chunk};
}

}  // namespace

int gemm_f32_dw_splits(int M, int N, int K, int max_splits)
{
    int big = 1;
    for (int sh = 0; sh < 3; ++sh) {
        const int n = plan_splits(tiles_of(sh, M, N), K, max_splits, CUS).splits;
        if (n > big) big = n;
    }
    // longest contraction the small kernel can be given for any batch up to K
    const long long kmax = small_dw_alone_kmax(M, N);
    const int ks = K < kmax ? K : (int)(kmax - 1);
    const int small = (ks >= 64) ? plan_small_splits(ks, max_splits).splits : 1;
    return big > small ? big : small;
}

namespace {

// shape < 0: the kernels of small products (blocks of 16 x 16 or 32 x 32), else the one launch_gemm_split takes
struct F32Plan {
    int shape;
    SplitPlan split;
};
F32Plan plan_f32(GemmKind kind, int M, int N, int K, int max_splits)
{
    if (kind == GEMM_DW ? small_dw_alone(M, N, K) : small_out(M, N, K) && !(kind == GEMM_FWD && long_fwd(M, N, K))) {
        if (kind == GEMM_DW) return {-1, plan_small_splits(K, max_splits)};
        return {-1, {1, (K + SMALL_CHUNK - 1) / SMALL_CHUNK * SMALL_CHUNK}};
    }
    if (kind == GEMM_FWD && long_fwd(M, N, K) && tiles_of(HALF, M, N) <= CUS)
        return {HALF, {1, (K + K_CHUNK_ALIGN - 1) / K_CHUNK_ALIGN * K_CHUNK_ALIGN}};
    if (kind != GEMM_DW)
        return {pick_shape(M, N, K), {1, (K + K_CHUNK_ALIGN - 1) / K_CHUNK_ALIGN * K_CHUNK_ALIGN}};
    int sh = (M >= 128) ? (N >= 128 ? 2 : 1) : 0;
    const SplitPlan sp = plan_splits(tiles_of(sh, M, N), K, max_splits, CUS);
    if (sh == 0 && sp.chunk >= SHARED_K && tiles_of(sh, M, N) * sp.splits <= CUS) sh = SHARED;
    return {sh, sp};
}
// da M x N over K and dw M x N over K of one layer.  Small tiles / split-plane tiles, 512-wide layers: B = 640 (80 tiles
// of 64 x 64) 12.4 / 10.3 us, B = 768 13.4 / 10.5, B = 1024 16.4 / 10.9; 256 wide, B = 2000 12.0 / 8.8; 1024 wide, B = 512
// 29.8 / 25.0.  At just 64 tiles the small ones are ahead (512 wide, B = 512 9.1 / 10.1; 256 wide, B = 1024 6.9 / 7.7), but
// their sums on fp32 MFMAs are further from 64 bits than the split-plane ones, so the line stays below 64.  A contraction
// of 1024 and more goes to the small ones while each block of 32 x 32 has a compute unit of its own: 1024 wide, B = 128
// (128 blocks) 10.7 / 21.2 us, B = 256 (256) 18.6 / 22.2, B = 320 (320) 21.0 / 23.1, B = 512 (512) 29.6 / 25.5; 2048 wide, B = 128 (256)
// 33.3 / 44.7, B = 192 (384) 48.9 / 48.7, B = 256 (512) 58.6 / 50.9; 1536 wide, B = 170 (288) 30.3 / 36.7, B = 256 (384) 35.6 /
// 33.6; 4096 wide, B = 64 (256) 69 / 97, B = 128 (512) 118 / 118.
F32Plan plan_f32_pair(const GemmArgs &da, const GemmArgs &dw, int max_splits)
{
    const int most = small_tiles_max() < 64 ? small_tiles_max() : 64;
    const bool one_each = da.K >= 1024 && (long long)((da.M + 31) / 32) * ((da.N + 31) / 32) <= CUS;
    if (da.K >= 64 && (tiles_of(0, da.M, da.N) < most || (one_each && most > 0)) && dw.K < small_k_max())
        return {-1, plan_small_splits(dw.K, max_splits)};
    const PairPlan pp = plan_pair(da, dw, max_splits);
    return {pp.shape, pp.split};
}

}  // namespace

int gemm_f32_plan(int product, int B, int d_out, int d_in, int max_splits, int *splits)
{
    F32Plan p;
    if (product == 0) {
        p = plan_f32(GEMM_FWD, B, d_out, d_in, 1);
    } else if (product == 1 && !gemm_f32_pair_ok(B, d_out, d_in)) {
        p = plan_f32(GEMM_DA, B, d_in, d_out, 1);
        p.split.splits = plan_f32(GEMM_DW, d_out, d_in, B, max_splits).split.splits;
    } else if (product == 1) {
        GemmArgs da = {}, dw = {};
        da.M = B, da.N = d_in, da.K = d_out;
        dw.M = d_out, dw.N = d_in, dw.K = B;
        p = plan_f32_pair(da, dw, max_splits);
    } else {
        p = plan_f32(GEMM_DW, d_out, d_in, B, max_splits);
    }
    *splits = p.split.splits;
    return p.shape;
}

int gemm_f32_small_form(int product, int B, int d_out, int d_in, int max_splits)
{
    int splits = 1;
    if (gemm_f32_plan(product, B, d_out, d_in, max_splits, &splits) >= 0) return 0;
    if (product == 0) {
        const int block = small_tile(B, d_out, false);
        return block + (block == 32 && small_staged(B, d_out) ? 64 : 0);
    }
    const int wave = small_dw_wave(d_out, d_in, std::min(B, plan_small_splits(B, max_splits).chunk));
    if (product == 2) return 32 + 128 * wave;
    const bool pair = gemm_f32_pair_ok(B, d_out, d_in);
    return small_tile(B, d_in, pair) + (pair ? 128 * wave : 0);
}

hipError_t launch_gemm_f32(GemmKind kind, GemmArgs a, int max_splits, int *splits_out,
                           hipStream_t stream, const LaunchEvents &ev)
{
    if (a.M <= 0 || a.N <= 0 || a.K <= 0) return hipErrorInvalidValue;
    const F32Plan p = plan_f32(kind, a.M, a.N, a.K, max_splits);
    const int small = kind == GEMM_DW ? 32 : small_tile(a.M, a.N, false);
    const int bm = p.shape < 0 ? small : SHAPES[p.shape].bm, bn = p.shape < 0 ? small : SHAPES[p.shape].bn;
    a.tiles_m = (a.M + bm - 1) / bm;
    a.tiles_n = (a.N + bn - 1) / bn;
    const long long tiles = (long long)a.tiles_m * a.tiles_n;
    if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    a.splits = p.split.splits;
    a.k_chunk = p.split.chunk;
    if (splits_out) *splits_out = p.split.splits;
    dim3 grid((unsigned)tiles, (unsigned)p.split.splits, 1);
    if (p.shape >= 0) return launch_gemm_split(kind, a, p.shape, grid, stream, ev);
    switch (kind) {
    case GEMM_FWD:
        if (small == 16) return launch_kernel(gemm_f32_small_kernel<16, true, true, GEMM_FWD>, grid, dim3(NT), stream, ev, a);
        if (small_staged(a.M, a.N)) return launch_kernel(gemm_f32_staged_kernel, grid, dim3(STAGED_NT), stream, ev, a);
        return launch_kernel(gemm_f32_small_kernel<32, true, true, GEMM_FWD>, grid, dim3(NT), stream, ev, a);
    case GEMM_DA:
        if (small == 16) return launch_kernel(gemm_f32_small_kernel<16, true, false, GEMM_DA>, grid, dim3(NT), stream, ev, a);
        return launch_kernel(gemm_f32_small_kernel<32, true, false, GEMM_DA>, grid, dim3(NT), stream, ev, a);
    case GEMM_DW:
        if (const int nq = small_dw_wave(a.M, a.N, std::min(a.K, a.k_chunk))) {
            grid.x = (unsigned)((tiles + WAVES - 1) / WAVES);
            return launch_kernel(nq == 1 ? gemm_f32_small_dw_wave_kernel<1> : gemm_f32_small_dw_wave_kernel<2>, grid, dim3(NT), stream, ev, a);
        }
        return launch_kernel(gemm_f32_small_kernel<32, false, false, GEMM_DW>, grid, dim3(NT), stream, ev, a);
    }
    return hipErrorInvalidValue;
}

// dA_l and dW_l of one hidden layer in one launch: both only read D_l, so they are independent, and
// sharing a launch lets the prologue / epilogue of one hide under the main loop of the other and pays
// the per-launch latencies once (B = 16, 512-wide layers: 4.7 + 5.1 us apart, 4.7 together; the step of
// 54-512x4-7 70 / 55 us).  Apart only with fewer rows than a k-tile and a weight gradient of more than 2^24 values: its
// 32 x 32 tiles then outlast the backward-data product (16 rows, 8192 wide: 158 us apart, 244 together; 4096 wide 66 / 62).
// HB_NO_PAIR = 1 (tuning aid): two launches.
bool gemm_f32_pair_ok(int B, int d_out, int d_in)
{
    static const int off = env_int("HB_NO_PAIR", 0);
    return !off && (B >= SMALL_CHUNK || (long long)d_out * d_in <= (1ll << 24));
}

hipError_t launch_gemm_f32_bwd_pair(GemmArgs da, GemmArgs dw, int max_splits, int *splits_out,
                                    hipStream_t stream, const LaunchEvents &ev)
{
    const F32Plan p = plan_f32_pair(da, dw, max_splits);
    const int da_small = small_tile(da.M, da.N, true);
    for (GemmArgs *g : {&da, &dw}) {
        const int small = g == &da ? da_small : 32;
        const int bm = p.shape < 0 ? small : SHAPES[p.shape].bm, bn = p.shape < 0 ? small : SHAPES[p.shape].bn;
        g->tiles_m = (g->M + bm - 1) / bm;
        g->tiles_n = (g->N + bn - 1) / bn;
    }
    const int align = p.shape < 0 ? SMALL_CHUNK : K_CHUNK_ALIGN;
    da.splits = 1;
    da.k_chunk = (da.K + align - 1) / align * align;
    dw.splits = p.split.splits;
    dw.k_chunk = p.split.chunk;
    if (splits_out) *splits_out = p.split.splits;
    const int wave = p.shape < 0 ? small_dw_wave(dw.M, dw.N, std::min(dw.K, dw.k_chunk)) : 0;
    const long long dw_tiles = (long long)dw.tiles_m * dw.tiles_n;
    const long long n_dw = (wave ? (dw_tiles + WAVES - 1) / WAVES : dw_tiles) * p.split.splits;
    const long long blocks = (long long)da.tiles_m * da.tiles_n + n_dw;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    if (p.shape >= 0) return launch_gemm_split_pair(da, dw, p.shape, (unsigned)blocks, (int)n_dw, stream, ev);
    const auto pick = [wave](auto da_tile) {
        constexpr int T = decltype(da_tile)::value;
        return wave == 0 ? gemm_f32_small_pair_kernel<T, 0>
                         : wave == 1 ? gemm_f32_small_pair_kernel<T, 1> : gemm_f32_small_pair_kernel<T, 2>;
    };
    const auto kernel = da_small == 16 ? pick(IntC<16>()) : pick(IntC<32>());
    return launch_kernel(kernel, dim3((unsigned)blocks), dim3(NT), stream, ev, da, dw, (int)n_dw);
}

}  // namespace hb
