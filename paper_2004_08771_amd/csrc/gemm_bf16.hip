// bf16 MFMA GEMM for the mixed-precision mode (bf16 weights / activations, fp32 master
// weights and accumulation) of the mini-batch step: the same three layer products as the
// fp32 path (Section 3 of the paper, Eq. (1) forward and Eq. (2) backward).
//
// gfx950 design: v_mfma_f32_32x32x16_bf16 wants 8 consecutive k per lane.
//   forward   Z_l     = A_{l-1} . W_l^T        A = A_{l-1} [B x d],   B = W_l   [d_l x d_{l-1}]   both K-major
//   backward  D_{l-1} = (D_l . W_l) * f'       A = D_l     [B x d_l], B = W_l^T [d_{l-1} x d_l]   both K-major
//   gradient  dW_l    = D_l^T . A_{l-1}        contraction over the batch, the ROW index of both
// The weights exist as two bf16 copies (W_l and W_l^T), rewritten by the weight-gradient
// epilogue, which also applies the SGD update (Eq. (3)) to the fp32 master weights.  The
// weight gradient reads D_l and A_{l-1} as they are, batch-major, through the transposing LDS
// read of gfx950 (LDS-direct kernel) or transposed in registers (small tiles); only where it cannot
// (rows that are not 4-byte aligned, or not 16-byte aligned in a large product) do the epilogues
// that produce a tensor also write its transposed copy, and the product runs K-major like the
// other two.
// Two kernel families: gemm_bf16_dma_kernel (256 x 256 x 64 tiles, LDS-direct loads) for the large
// products, gemm_bf16_mid_kernel (64 x 64 x 64 or 128 x 128 x 64, operands global -> registers -> LDS) for all others.
#include "gemm_device.h"

#include <stdlib.h>

#include <type_traits>

namespace hb {
namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned short bf16_t;  // storage type

constexpr int NT = 256;

// fp32 -> bf16, round to nearest even: gfx950's v_cvt_pk_bf16_f32 (checked against the bit
// formula u + 0x7fff + ((u >> 16) & 1) on all 2^32 inputs: identical for every non-NaN value,
// NaN stays NaN).  One instruction per pair instead of about seven integer operations per
// value, which the epilogues of the GEMMs run 128 times per lane and tile.
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ bf16_t f2bf(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }
__device__ __forceinline__ unsigned int pack2bf(float lo, float hi)
{
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(unsigned int, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ float bf2f(bf16_t b) { return __uint_as_float((unsigned int)b << 16); }

// Guarded loads of one operand tile, ROWS x BK bf16, K-major.
template <int ROWS, int BK, int THREADS = NT>
struct TileB {
    static constexpr int VPT = ROWS * BK / 8 / THREADS;  // 16-byte vectors per thread
    static_assert(ROWS * BK / 8 % THREADS == 0, "tile must split evenly over the workgroup");

    // guarded: anything outside [0, nrows) x [.., kend) reads as zero
    static __device__ __forceinline__ void load(uint4 (&reg)[VPT], const bf16_t *__restrict__ P, long long ld,
                                                int row0, int nrows, int k0, int kend, bool vec, int tid)
    {
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
            const int idx = tid + v * THREADS;
            const int kq = idx % (BK / 8), r = idx / (BK / 8);
            const int row = row0 + r, k = k0 + kq * 8;
            uint4 x = {0u, 0u, 0u, 0u};
            if (row < nrows && k < kend) {
                const bf16_t *p = P + (size_t)row * ld + k;
                if (vec && k + 8 <= kend) {
                    x = *reinterpret_cast<const uint4 *>(p);
                } else {
                    // all eight are requested before the first is used (past the end: the last again); under a condition
                    // each would wait for the one before it
                    unsigned int b[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) b[e] = p[min(e, kend - 1 - k)];
#pragma unroll
                    for (int e = 1; e < 8; ++e) b[e] = (k + e < kend) ? b[e] : 0u;
                    x = make_uint4(b[0] | b[1] << 16, b[2] | b[3] << 16, b[4] | b[5] << 16, b[6] | b[7] << 16);
                }
            }
            reg[v] = x;
        }
    }
};

// The activation is a template argument of the epilogues: tested at run time per value, it
// became three scalar branches in front of each of a lane's 128 outputs (about 5 us per
// 256 x 256 tile, with the MFMA pipes idle).
template <int ACT>
__device__ __forceinline__ float act_fwd(float z)
{
    if (ACT == ACT_SIGMOID) return sigmoidf_fast(z);
    if (ACT == ACT_RELU) return fmaxf(z, 0.f);
    return z;
}
// calls f(IntC<activation>, IntC<mask ? 1 : 0>) with the run-time activation as a constant
template <typename F>
__device__ __forceinline__ void with_activation(int act, bool mask, F &&f)
{
    if (act == ACT_RELU) {
        if (mask) f(IntC<ACT_RELU>(), IntC<1>());
        else f(IntC<ACT_RELU>(), IntC<0>());
    } else if (act == ACT_SIGMOID) {
        f(IntC<ACT_SIGMOID>(), IntC<0>());
    } else {
        f(IntC<ACT_NONE>(), IntC<0>());
    }
}

// ReLU decision bits of one 32 x 32 block (see GemmBf16Args::mask_out): position of the value
// (q, e) = row 8 q + 4 h + e in the lane's 16-bit word, the word from the lane's 16 packed
// bf16 values (pk[q] = rows e = 0..3 of group q), and the use of a bit on a backward value.
// "Positive" is: sign clear and magnitude not zero (true for a NaN as well, where `> 0` is not).
__device__ __forceinline__ constexpr int relu_bit_pos(int q, int e) { return 8 * (e & 1) + 2 * q + (e >> 1); }
__device__ __forceinline__ unsigned relu_bits(const uint2 (&pk)[4])
{
    unsigned acc = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {  // dword k holds (q, e) = (k / 2, 2 (k % 2)) below (q, e + 1)
        const unsigned x = (k & 1) ? pk[k >> 1].y : pk[k >> 1].x;
        const unsigned t = ((x & 0x7fff7fffu) + 0x7fff7fffu) & ~x;  // bits 15 / 31: the half is positive
        acc = (t & 0x80008000u) | (acc >> 1);
    }
    // the low halves of dwords 0..7 now sit at bits 8..15, the high halves at bits 24..31
    return ((acc >> 8) & 0xffu) | ((acc >> 16) & 0xff00u);
}
__device__ __forceinline__ float relu_keep(float val, unsigned word, int q, int e)
{
    const int m = (int)(word << (31 - relu_bit_pos(q, e))) >> 31;  // 0 or -1 (one v_bfe_i32)
    return __uint_as_float(__float_as_uint(val) & (unsigned)m);
}

// Epilogue shared by both kernels.  acc[i][j][v] = C(row, col) of the wavefront's block (i, j):
// row = 8 (v / 4) + 4 h + (v % 4), col = r.  (mw, nw) is the wavefront's first row / column and
// must be wavefront-uniform: every address below is a scalar base (row, column block) plus a
// per-lane byte offset that does not change during the epilogue, so the 128 outputs of a lane
// cost no address registers.
// FULL: the wavefront's tile lies inside the matrix and the 8-byte accesses are aligned; no
// guards, and what a column block needs from memory (bias, the activations of the
// backward-data derivative, the fp32 master weights of the fused update) is requested before
// its first use, so that those loads are in flight together instead of one round trip each.
// ACT: the activation (forward, backward-data).  MASK: the ReLU decision bits are written
// (forward: mask_out) / read instead of the activations (backward-data: mask_in).
template <int KIND, int TM, int TN, bool FULL, int ACT, bool MASK>
__device__ __forceinline__ void epilogue_bf16_impl(const GemmBf16Args &a, v16f (&acc)[TM][TN], int mw, int nw, int r,
                                                   int h)
{
    const bool has_cf = a.C_f32 != nullptr, has_cb = a.C_bf16 != nullptr;
    const bool has_ct = a.Ct_bf16 != nullptr && !(KIND == GEMM_DW && a.write_grad);
    const bool use_t = (KIND == GEMM_DA) && a.aux_t != nullptr && (a.ldauxt & 3) == 0;
    constexpr bool use_mask = (KIND == GEMM_DA) && MASK;
    const bool ct_vec = (a.ldct & 3) == 0;
    // per-lane byte offsets (row part 4 h, column part r)
    const unsigned lo_cf = (unsigned)(4 * h * (int)a.ldc + r) * 4u;
    const unsigned lo_cb = (unsigned)(4 * h * (int)a.ldcb + r) * 2u;
    const unsigned lo_ct = (unsigned)(r * (int)a.ldct + 4 * h) * 2u;
    const unsigned lo_at = (unsigned)(r * (int)a.ldauxt + 4 * h) * 2u;
    const unsigned lo_ax = (unsigned)(4 * h * (int)a.ldaux + r) * 2u;
    unsigned char *const cf0 = static_cast<unsigned char *>(a.C_f32);
    unsigned char *const cb0 = static_cast<unsigned char *>(a.C_bf16);
    unsigned char *const ct0 = static_cast<unsigned char *>(a.Ct_bf16);
    const unsigned char *const at0 = static_cast<const unsigned char *>(a.aux_t);
    const unsigned char *const ax0 = static_cast<const unsigned char *>(a.aux);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int nb = nw + j * 32;  // uniform
        const int n = nb + r;
        const bool n_ok = FULL || n < a.N;
        float bias = 0.f;
        if (KIND == GEMM_FWD && a.bias != nullptr && n_ok) bias = a.bias[n];
        uint2 ot[TM][4];
        if (KIND == GEMM_DA && FULL && !use_mask) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    ot[i][q] = *reinterpret_cast<const uint2 *>(
                        at0 + ((size_t)nb * a.ldauxt + (mw + i * 32 + 8 * q)) * 2 + lo_at);
            __builtin_amdgcn_sched_barrier(0);
        }
        // ReLU decision bits: a block is addressed only when it holds a valid element (the
        // array covers ceil(M / 32) x ceil(N / 32) blocks)
        unsigned mword[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            mword[i] = 0u;
            if (KIND == GEMM_DA && use_mask && (FULL || (mw + i * 32 < a.M && nb < a.N)))
                mword[i] = a.mask_in[((size_t)((mw + i * 32) >> 5) * a.mask_nb + (nb >> 5)) * 64 + 32 * h + r];
        }
        float csum = 0.f;  // backward-data: sum of the lane's stored results of this column
        // The current row of the results, moved on by additions.  A wavefront runs through this code once, so what counts is
        // its length, and 64-bit products for the addresses were a third of it: 8192 x 1000 x 784, whose last tiles come here,
        // 48.4 us, so 45.5; 128 x 128 tiles of 8192 x 600 x 1000 31.2, so 30.0.
        unsigned char *cf = cf0 + ((size_t)mw * a.ldc + nb) * 4, *cb = cb0 + ((size_t)mw * a.ldcb + nb) * 2;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            unsigned mbits = 0u;
            float w[16];
            if (KIND == GEMM_DW && FULL && !a.write_grad) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    w[v] = *reinterpret_cast<const float *>(
                        cf0 + ((size_t)(mw + i * 32 + 8 * (v >> 2) + (v & 3)) * a.ldc + nb) * 4 + lo_cf);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {  // groups of 4 consecutive rows
                const int mb = mw + i * 32 + 8 * q;  // uniform; this lane's rows are mb + 4 h + e
                const int mq = mb + 4 * h;
                uint2 o4 = {0u, 0u};
                if (KIND == GEMM_DA && !use_mask) {
                    if (FULL) o4 = ot[i][q];
                    else if (use_t && n_ok && mq < a.M)  // rows of the copy are padded to 4: in bounds
                        o4 = *reinterpret_cast<const uint2 *>(at0 + ((size_t)nb * a.ldauxt + mb) * 2 + lo_at);
                }
                float x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float val = acc[i][j][4 * q + e];
                    if (FULL || (mq + e < a.M && n_ok)) {
                        if (KIND == GEMM_FWD) {
                            val = act_fwd<ACT>(val + bias);
                            if (has_cf) *reinterpret_cast<float *>(cf + lo_cf) = val;
                            if (MASK) {
                                const bf16_t b = f2bf(val);
                                if ((b & 0x7fffu) != 0 && (b & 0x8000u) == 0) mbits |= 1u << relu_bit_pos(q, e);
                            }
                        } else if (KIND == GEMM_DA && use_mask) {
                            val = relu_keep(val, mword[i], q, e);
                        } else if (KIND == GEMM_DA) {
                            float o;
                            if (FULL || use_t) {
                                const unsigned int pw = (e < 2) ? o4.x : o4.y;
                                o = __uint_as_float((e & 1) ? (pw & 0xffff0000u) : (pw << 16));
                            } else {
                                o = bf2f(*reinterpret_cast<const bf16_t *>(ax0 + ((size_t)(mb + e) * a.ldaux + nb) * 2 +
                                                                            lo_ax));
                            }
                            if (ACT == ACT_SIGMOID) val *= o * (1.f - o);
                            else if (ACT == ACT_RELU) val = (o > 0.f) ? val : 0.f;
                        } else {  // GEMM_DW
                            float *p = reinterpret_cast<float *>(cf + lo_cf);
                            if (!a.write_grad) val = (FULL ? w[4 * q + e] : *p) - a.lr * val;  // Eq. (3), fp32 master
                            *p = val;
                        }
                        if (has_cb) *reinterpret_cast<bf16_t *>(cb + lo_cb) = f2bf(val);
                        if (KIND == GEMM_DA && a.colsum_partial != nullptr) csum += bf2f(f2bf(val));
                    }
                    x[e] = val;
                    cf += a.ldc * (e < 3 ? 4 : 20);  // the group's last row: past the four of the other half-wavefront
                    cb += a.ldcb * (e < 3 ? 2 : 10);
                }
                if (has_ct && n_ok) {
                    unsigned char *ct = ct0 + ((size_t)nb * a.ldct + mb) * 2 + lo_ct;
                    if (FULL || (mq + 4 <= a.M && ct_vec)) {
                        uint2 pk;
                        pk.x = pack2bf(x[0], x[1]);
                        pk.y = pack2bf(x[2], x[3]);
                        *reinterpret_cast<uint2 *>(ct) = pk;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (mq + e < a.M) reinterpret_cast<bf16_t *>(ct)[e] = f2bf(x[e]);
                    }
                }
                // keep the scheduler from pulling later groups' conversions up: with 128
                // accumulators live it runs out of registers
                __builtin_amdgcn_sched_barrier(0);
            }
            if (KIND == GEMM_FWD && MASK && (FULL || (mw + i * 32 < a.M && nb < a.N)))
                a.mask_out[((size_t)((mw + i * 32) >> 5) * a.mask_nb + (nb >> 5)) * 64 + 32 * h + r] =
                    (unsigned short)mbits;
        }
        // column sums over the wavefront's 128 rows (LDS-direct kernel only: mw is a multiple of
        // 128): the two half-wavefronts hold alternate groups of four rows
        if (KIND == GEMM_DA && a.colsum_partial != nullptr) {
            csum += __shfl_xor(csum, 32, 64);
            if (h == 0 && n_ok) a.colsum_partial[(size_t)(mw >> 7) * a.N + n] = csum;
        }
    }
}

template <int KIND, int TM, int TN>
__device__ __forceinline__ void epilogue_bf16(const GemmBf16Args &a, v16f (&acc)[TM][TN], int mw, int nw, int r,
                                              int h)
{
    const bool mask = KIND == GEMM_FWD  ? (a.mask_out != nullptr && a.act == ACT_RELU)
                      : KIND == GEMM_DA ? (a.mask_in != nullptr && a.act == ACT_RELU)
                                        : false;
    const bool full = (mw + 32 * TM <= a.M) && (nw + 32 * TN <= a.N) &&
                      (a.Ct_bf16 == nullptr || (a.ldct & 3) == 0) &&
                      (KIND != GEMM_DA || mask || (a.aux_t != nullptr && (a.ldauxt & 3) == 0));
    with_activation(KIND == GEMM_DW ? (int)ACT_NONE : a.act, mask, [&](auto act_c, auto mask_c) {
        constexpr int ACT = decltype(act_c)::value;
        constexpr bool MASK = decltype(mask_c)::value != 0;
        if (full) epilogue_bf16_impl<KIND, TM, TN, true, ACT, MASK>(a, acc, mw, nw, r, h);
        else epilogue_bf16_impl<KIND, TM, TN, false, ACT, MASK>(a, acc, mw, nw, r, h);
    });
}

// One slice of a split weight gradient: the sums as they are, to a.C_f32.  By way of the general epilogue, whose code a
// wavefront runs through once and mostly waits for, the slices of 512 x 512 over 8192 rows (32 workgroups) took 32.8 us, so
// 28.8; of 1000 x 784 and the like 34.9, so 31.0.
template <int TM, int TN>
__device__ __forceinline__ void store_slice(const GemmBf16Args &a, const v16f (&acc)[TM][TN], int mw, int nw, int r, int h)
{
    const bool full = mw + 32 * TM <= a.M && nw + 32 * TN <= a.N;
    const unsigned lo = (unsigned)(4 * h * (int)a.ldc + r);
    float *row = static_cast<float *>(a.C_f32) + (size_t)mw * a.ldc + nw;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q, row += 4 * a.ldc)
#pragma unroll
            for (int e = 0; e < 4; ++e, row += a.ldc)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    if (full || (mw + 32 * i + 8 * q + 4 * h + e < a.M && nw + 32 * j + r < a.N))
                        row[lo + 32 * j] = acc[i][j][4 * q + e];
}

// The 256 x 256 kernel multiplies in 16 x 16 blocks (v_mfma_f32_16x16x32_bf16): a block has rows 4 g + e and column c in lane
// 16 g + c, register e.  Two wavefronts of a SIMD that issue v_mfma_f32_32x32x16_bf16 in turn reach only two thirds of what
// the 16 x 16 form gives (registers only, normal values: 1290-1340 against 2030 TFLOP/s, zeros 1604 against 2468; one
// wavefront alone 1807 against 2041); here, where both also read and load, four steps of 2048-4096x3-1000 over 16384 rows
// went from 18.53 to 18.06 ms with it.  The epilogues want 32 x 32 blocks (rows 8 q + 4 h + e, column r in lane 32 h + r,
// register 4 q + e): of a pair of blocks side by side, lane bit 4 (which of two groups of four rows) becomes a register and
// the column block lane bit 4, one lane exchange for two registers.  For that row c of an A fragment is row a_row(c) of the
// tile, groups 1 and 2 of four rows in each other's place; with the rows in order a second exchange was needed (8192 x 1024,
// K = 784, backward-data over 1024 and 10: 22.5 us, so 21.9).
typedef float v4f __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int a_row(int c) { return (c & 3) | (c & 4) << 1 | (c & 8) >> 1; }
template <int TM, int TN>
__device__ __forceinline__ void blocks_of_32(v16f (&out)[TM][TN], const v4f (&in)[2 * TM][2 * TN])
{
#pragma unroll
    for (int i = 0; i < 2 * TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const auto y = __builtin_amdgcn_permlane16_swap(__float_as_uint(in[i][2 * j][e]),
                                                                __float_as_uint(in[i][2 * j + 1][e]), false, false);
                out[i / 2][j][8 * (i & 1) + e] = __uint_as_float(y[0]);
                out[i / 2][j][8 * (i & 1) + 4 + e] = __uint_as_float(y[1]);
            }
}

// ---- products with too few 256 x 256 tiles: 64 x 64 or 128 x 128 tiles -----------------------
// What bounds a product of this size is latency: a k-tile of 64 is only four MFMAs per block and
// wavefront, and an L2 round trip under load takes about 550 cycles.  So four register sets keep
// four k-tiles in flight per workgroup, and the 64 x 64 tiles (32 KB of LDS, 64 with two groups of
// wavefronts; 144 to 168 registers) let several workgroups share a compute unit.  (2047 x 1024 x 1024 forward 33.7 us with
// 128 x 128 x 64 tiles and two k-tiles in flight, 12.1 now; its weight gradient, with the passes that
// transposed both operands and added the bias gradient up, 48 + 14 -> 14.7 us.)  A round of the loop still takes some 1300
// clocks: LDS write, barrier, LDS read and the chain of four MFMAs follow each other.
// LDS rows are 128 bytes, their eight 16-byte chunks exchanged by the row pair, which keeps the
// writes (8 lanes per row) and the fragment reads (32 rows at one chunk) free of bank conflicts.
// A long contraction has four k-tiles in flight; what bounds one of one or two k-tiles with many outputs is its
// epilogue (16384 x 4096 x 54 forward: 110 us with one workgroup per compute unit, 85 with two; x 33 102 -> 83).
// 16-byte buffer loads need rows that are 4-byte aligned.  SHIFT: the rows of A are not (the caller's X with
// an odd d_0, or at an odd address): a lane reads the five dwords that hold its eight values and shifts them
// down as it writes them to LDS.  (Element loads instead: 5999 x 2050 x 301 forward 141 us, with this
// 57; 1021 x 512 x 1001 41 -> 12; 16384 x 4096 x 301 558 -> 198.)  A partial k-tile is taken first, through the guarded loads of TileB; with
// SHIFT and with batch-major operands every contraction ends in one, so that no wide load reads past the end of the last row.
typedef unsigned v4u __attribute__((ext_vector_type(4)));
constexpr int MID_BK = 64;

// byte offset of chunk c of an LDS row
__device__ __forceinline__ int mid_slot(int row, int c)
{
    return row * 128 + ((c ^ (((row >> 1) ^ ((row >> 5) << 2)) & 7)) << 4);
}

template <int ROWS, int THREADS, int SETS, bool SHIFT = false>
struct MidOp {
    using T = TileB<ROWS, MID_BK, THREADS>;  // thread tid holds chunk tid % 8 of rows tid / 8 + R1 v
    static constexpr int R1 = THREADS / 8;
    static constexpr int VPT = T::VPT;
    uint4 x[SETS][VPT];
    unsigned off[VPT];
    // SHIFT: the fifth dword (its own offset: of a row that is aligned after all, the fourth again) and the bytes to shift by
    unsigned x4[SHIFT ? SETS : 1][VPT], off4[VPT], sh[VPT];

    static __device__ __forceinline__ int frag(int row, int c) { return mid_slot(row, c); }
    // tile: the first value of the tile's first row
    __device__ __forceinline__ void init(const bf16_t *tile, long long ld, int last_row, int tid)
    {
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
            unsigned row = (unsigned)(min((tid >> 3) + R1 * v, last_row) - min(R1 * v, last_row)) * (unsigned)ld * 2u;
            if (SHIFT) {
                row += (unsigned)(reinterpret_cast<size_t>(tile + (size_t)min(R1 * v, last_row) * ld) & 3);
                sh[v] = row & 2u;
                row &= ~3u;
            }
            off[v] = row + (tid & 7) * 16u;
            if (SHIFT) off4[v] = off[v] + (sh[v] ? 16u : 12u);
        }
    }
    __device__ __forceinline__ void load(int set, const bf16_t *__restrict__ tile, long long ld, int last_row)
    {
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
            size_t base = reinterpret_cast<size_t>(tile + (size_t)min(R1 * v, last_row) * ld);
            if (SHIFT) base &= ~(size_t)3;
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(base), (short)0, -1, 0x00027000);
            const v4u t = __builtin_amdgcn_raw_buffer_load_b128(rs, off[v], 0, 0);
            x[set][v] = make_uint4(t[0], t[1], t[2], t[3]);
            if (SHIFT) x4[set][v] = __builtin_amdgcn_raw_buffer_load_b32(rs, off4[v], 0, 0);
        }
    }
    // SHIFT: drops the half dword below each of the eight values that were read
    __device__ __forceinline__ void align(int set)
    {
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
            const uint4 t = x[set][v];
            x[set][v] = make_uint4(
                __builtin_amdgcn_alignbyte(t.y, t.x, sh[v]), __builtin_amdgcn_alignbyte(t.z, t.y, sh[v]),
                __builtin_amdgcn_alignbyte(t.w, t.z, sh[v]), __builtin_amdgcn_alignbyte(x4[set][v], t.w, sh[v]));
        }
    }
    // a partial k-tile (aligned at once): wide loads where another value follows in the row
    __device__ __forceinline__ void load_tail(int set, const bf16_t *__restrict__ P, long long ld, int row0, int nrows,
                                              int k0, int kend, bool vec, int tid)
    {
        if (SHIFT && k0 + 8 * (tid & 7) + 8 < kend) {
            load(set, P + (size_t)row0 * ld + k0, ld, nrows - 1 - row0);
            align(set);
        } else {
            T::load(x[set], P, ld, row0, nrows, k0, kend, vec, tid);
        }
    }
    __device__ __forceinline__ void store(int set, unsigned char *S, int tid) const
    {
#pragma unroll
        for (int v = 0; v < VPT; ++v) *reinterpret_cast<uint4 *>(S + mid_slot((tid >> 3) + R1 * v, tid & 7)) = x[set][v];
    }
};

// The same for an operand whose rows are the contraction (weight gradient: D_l and A_{l-1} as the
// other products leave them, batch-major).  A k-row of the tile is 128 bytes and goes to LDS as it comes, 16 bytes per
// load; the transposing LDS read of gfx950 makes the fragments.  (Each load instruction keeps the compute unit's address unit
// busy for about 16 clocks whatever its width: with four bytes per load and a transposition in registers 1024 x 1024 over
// 2047 rows took 18.6 us, so 16.7.)  The two 64-byte halves of a k-row change places with bit 1 of its number, so that the four rows
// that a read touches together cover all banks.
typedef short v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s *lds_v4s;
template <int SETS>
struct MidOpT {
    uint4 x[SETS][2];  // k-rows tid / 8 + 32 v, columns 8 (tid % 8) ..
    unsigned off, off2[4];
    bool wide;

    // wide: 16 bytes from every valid chunk's first column on lie inside its row.  Else (rows of X without padding, at the
    // right edge) they run on into the next row, and the last row is read in pairs of columns: rows have an even pitch.
    // Chunks past the last column read as the last.
    __device__ __forceinline__ void init(long long ld, int last_row, int tid)
    {
        wide = (ld & 7) == 0 || last_row >= 63;
        const unsigned row = (unsigned)(tid >> 3) * (unsigned)ld * 2u;
        off = row + 2u * (unsigned)min(8 * (tid & 7), last_row & ~7);
#pragma unroll
        for (int e = 0; e < 4; ++e) off2[e] = row + 2u * (unsigned)min(8 * (tid & 7) + 2 * e, last_row & ~1);
    }
    template <bool WIDE>
    __device__ __forceinline__ void load_rows(int set, int v, const bf16_t *__restrict__ rows)
    {
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(rows), (short)0, -1, 0x00027000);
        if (WIDE) {
            const v4u t = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
            x[set][v] = make_uint4(t[0], t[1], t[2], t[3]);
        } else {
            x[set][v] = make_uint4(__builtin_amdgcn_raw_buffer_load_b32(rs, off2[0], 0, 0), __builtin_amdgcn_raw_buffer_load_b32(rs, off2[1], 0, 0),
                                   __builtin_amdgcn_raw_buffer_load_b32(rs, off2[2], 0, 0), __builtin_amdgcn_raw_buffer_load_b32(rs, off2[3], 0, 0));
        }
    }
    // a whole k-tile, behind which another batch row follows
    __device__ __forceinline__ void load(int set, const bf16_t *__restrict__ tile, long long ld)
    {
#pragma unroll
        for (int v = 0; v < 2; ++v) load_rows<true>(set, v, tile + (size_t)(32 * v) * ld);
    }
    // a partial k-tile: k rows from k0, zero from kend on
    __device__ __forceinline__ void load_tail(int set, const bf16_t *__restrict__ P, long long ld, int row0, int k0, int kend,
                                              int tid)
    {
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            x[set][v] = make_uint4(0u, 0u, 0u, 0u);
            if (k0 + (tid >> 3) + 32 * v < kend) {
                if (wide) load_rows<true>(set, v, P + (size_t)(k0 + 32 * v) * ld + row0);
                else load_rows<false>(set, v, P + (size_t)(k0 + 32 * v) * ld + row0);
            }
        }
    }
    __device__ __forceinline__ void store(int set, unsigned char *S, int tid) const
    {
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int k = (tid >> 3) + 32 * v, c = tid & 7;
            *reinterpret_cast<uint4 *>(S + k * 128 + (((c >> 2) ^ ((k >> 1) & 1)) << 6) + ((c & 3) << 4)) = x[set][v];
        }
    }
    // fragment of columns 32 blk + lane % 32 for k-step `step`: lane 16 g + 4 j + q addresses k-row 16 step + 8 (g / 2) + j
    // (second read: + 4), bytes 32 (g % 2) + 8 q of the block
    static __device__ __forceinline__ v8bf frag(const unsigned char *S, int blk, int step, int lane)
    {
        const int g = lane >> 4, j = (lane >> 2) & 3;
        const unsigned char *p = S + (16 * step + 8 * (g >> 1) + j) * 128 + ((blk ^ (j >> 1)) << 6) + ((g & 1) << 5) + ((lane & 3) << 3);
        const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(v4s *)p);
        const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(v4s *)(p + 512));
        return __builtin_bit_cast(v8bf, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
};

// KG: groups of four wavefronts that share the contraction of one tile (group g takes the k-tiles
// g, g + KG, ..); their sums meet in LDS, in group order, and group 0 runs the epilogue.
// BMAJ: weight gradient with both operands batch-major; the workgroups of the first tile column also
// add up the columns of D_l, the bias gradient.
// TILE: 64 (four wavefronts of 32 x 32) or 128 (one group of eight wavefronts of 64 x 32).
// SETS: k-tiles in flight.  Two for contractions of up to two k-tiles, which fit 128 registers: two workgroups of 128 x 128
// tiles share a compute unit, and the epilogue of one runs beside the loads of the other.
// The weight gradient that follows the loss kernel also finishes the mean loss, in a workgroup of its own (a launch less).
template <int TILE, int KG>
constexpr int mid_lds_bytes()
{
    return KG * 2 * 128 * 2 * TILE;
}
template <int TILE, int KG, int KIND, bool SHIFT, bool BMAJ, int SETS>
__device__ __forceinline__ void mid_tile(const GemmBf16Args &a, int id, unsigned char *smem)
{
    constexpr int BM = TILE, BN = TILE, GT = (TILE == 64) ? NT : 2 * NT, TM = TILE / 64;  // GT: threads of a group
    static_assert(!BMAJ || (!SHIFT && KIND == GEMM_DW && TILE == 64), "batch-major operands");
    static_assert(TILE == 64 || KG == 1, "a group of eight wavefronts does not share");
    static_assert(SETS % 2 == 0, "a register set's parity is its LDS stage's");
    using OA = std::conditional_t<BMAJ, MidOpT<SETS>, MidOp<BM, GT, SETS, SHIFT>>;
    using OB = std::conditional_t<BMAJ, MidOpT<SETS>, MidOp<BN, GT, SETS>>;
    constexpr int A_BYTES = 128 * BM, STAGE = 128 * (BM + BN);
    static_assert(KG * 2 * STAGE == mid_lds_bytes<TILE, KG>(), "LDS of a workgroup");
    const int lane = threadIdx.x & 63, wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tid = threadIdx.x & (GT - 1), g = wave_all / (GT / 64), wave = wave_all % (GT / 64);
    const int r = lane & 31, h = lane >> 5;
    const int wm = wave & 1, wn = wave >> 1;
    unsigned char *const stages = smem + g * 2 * STAGE;

    if constexpr (BMAJ) {
        if (id == a.tiles_m * a.tiles_n) {
            loss_finalize(a.fin, reinterpret_cast<double *>(smem));
            return;
        }
    }
    // XCD-aware tile order: each XCD gets a block of the tiles (a.xcd_m such blocks along m)
    int tile_m, tile_n;
    if (a.xcd_m > 0) {
        const int x = id & 7, j = id >> 3, rm = a.tiles_m / a.xcd_m, rn = a.tiles_n * a.xcd_m >> 3;
        tile_m = j / rn;
        tile_n = (x / a.xcd_m) * rn + j - tile_m * rn;
        tile_m += (x & (a.xcd_m - 1)) * rm;
    } else {
        id = xcd_tile_order(id, a.tiles_m * a.tiles_n);
        tile_m = id / a.tiles_n;
        tile_n = id - tile_m * a.tiles_n;
    }
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int nk_full = (SHIFT || BMAJ ? a.K - 1 : a.K) / MID_BK, tail = (nk_full * MID_BK < a.K) ? 1 : 0, nk = nk_full + tail;
    const int rounds = (nk + KG - 1) / KG;               // k-tiles of group 0
    const int mine = (nk - g + KG - 1) / KG;             // k-tiles of this group: rounds or one less
    const int a_last = a.M - 1 - m0, b_last = a.N - 1 - n0;

    const bf16_t *__restrict__ A = static_cast<const bf16_t *>(a.A);
    const bf16_t *__restrict__ Bm = static_cast<const bf16_t *>(a.B);

    v16f acc[TM][1];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][0][v] = 0.f;

    OA oa;
    OB ob;
    if constexpr (BMAJ) {
        oa.init(a.lda, a_last, tid);
        ob.init(a.ldb, b_last, tid);
    } else {
        oa.init(A + (size_t)m0 * a.lda, a.lda, a_last, tid);
        ob.init(Bm + (size_t)n0 * a.ldb, a.ldb, b_last, tid);
    }
    auto load_guarded = [&](int set, int k0) {
        if constexpr (BMAJ) {
            oa.load_tail(set, A, a.lda, m0, k0, a.K, tid);
            ob.load_tail(set, Bm, a.ldb, n0, k0, a.K, tid);
        } else {
            oa.load_tail(set, A, a.lda, m0, a.M, k0, a.K, a.a_vec != 0, tid);
            ob.load_tail(set, Bm, a.ldb, n0, a.N, k0, a.K, a.b_vec != 0, tid);
        }
    };
    // the group's i-th k-tile; k-tile 0 is the partial one if there is one; past the end: the last
    // one again (not used)
    auto load_tile = [&](int set, int i) {
        const int f = max(g + min(i, mine - 1) * KG - tail, 0);
        if constexpr (BMAJ) {
            oa.load(set, A + (size_t)f * MID_BK * a.lda + m0, a.lda);
            ob.load(set, Bm + (size_t)f * MID_BK * a.ldb + n0, a.ldb);
        } else {
            oa.load(set, A + (size_t)m0 * a.lda + f * MID_BK, a.lda, a_last);
            ob.load(set, Bm + (size_t)n0 * a.ldb + f * MID_BK, a.ldb, b_last);
        }
    };
    const bool do_bias = BMAJ && a.bias_out != nullptr && tile_n == 0;
    float csum[8];  // columns 8 (tid % 8) ..
#pragma unroll
    for (int e = 0; e < 8; ++e) csum[e] = 0.f;
    auto store_tile = [&](int set, unsigned char *S, bool aligned) {
        if constexpr (BMAJ) {
            if (do_bias) {
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    const unsigned w[4] = {oa.x[set][v].x, oa.x[set][v].y, oa.x[set][v].z, oa.x[set][v].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        csum[2 * e] += __uint_as_float(w[e] << 16);
                        csum[2 * e + 1] += __uint_as_float(w[e] & 0xffff0000u);
                    }
                }
            }
        }
        if constexpr (SHIFT)
            if (!aligned) oa.align(set);
        oa.store(set, S, tid);
        ob.store(set, S + A_BYTES, tid);
    };
    v8bf fa[4][TM], fb[4];
    auto read_frags = [&](const unsigned char *S, int step) {
        if constexpr (BMAJ) {
            fa[step][0] = OA::frag(S, wm, step, lane);
            fb[step] = OB::frag(S + A_BYTES, wn, step, lane);
        } else {
#pragma unroll
            for (int i = 0; i < TM; ++i)
                fa[step][i] = *reinterpret_cast<const v8bf *>(S + OA::frag(wm * (TILE / 2) + i * 32 + r, 2 * step + h));
            fb[step] = *reinterpret_cast<const v8bf *>(S + A_BYTES + OB::frag(wn * 32 + r, 2 * step + h));
        }
    };

    if (mine > 0) {
        if (tail && g == 0) load_guarded(0, nk_full * MID_BK);
        else load_tile(0, 0);
    }
    // Nothing in the loop, and nothing between its first loads and its head, is conditional: where a load may not have been
    // issued, the compiler waits for all of them in front of the write to LDS, and a round takes a round trip to memory
    // (us then / now: forward 1000 x 4096 x 4096 46.9 / 39.5, 2047 x 1024 x 1024 13.3 / 12.0; weight gradient 1024 x 1024 over 5000 rows
    // 30.4 / 24.9, 256 x 256 over 3000 20.5 / 16.3).
    auto multiply = [&]() {
#pragma unroll
        for (int step = 0; step < 4; ++step)
#pragma unroll
            for (int t = 0; t < TM; ++t)
                acc[t][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[step][t], fb[step], acc[t][0], 0, 0, 0);
    };
    int i = 0;
    if (mine > 1) {  // then the group has a whole k-tile
#pragma unroll
        for (int t = 1; t < SETS; ++t) {
            load_tile(t, t);
            __builtin_amdgcn_sched_barrier(0);  // in this order: the loop's first wait is for the first
        }
        store_tile(0, stages, tail && g == 0);
        load_tile(0, SETS);
        __syncthreads();
        auto round = [&](int c, bool more) {
            const unsigned char *S = stages + (c & 1) * STAGE;
#pragma unroll
            for (int step = 0; step < 4; ++step) read_frags(S, step);
            store_tile((c + 1) % SETS, stages + ((c + 1) & 1) * STAGE, false);
            if (more) load_tile((c + 1) % SETS, i + 1 + SETS);
            multiply();
            __syncthreads();  // tile i read and tile i + 1 written by everyone
            ++i;
        };
        while (i + SETS < mine) {  // whole turns of the register sets: a way out in between would reach the head as well
#pragma unroll
            for (int c = 0; c < SETS; ++c) round(c, true);
        }
#pragma unroll
        for (int c = 0; c < SETS - 1; ++c)  // everything has been asked for
            if (i + 1 < mine) round(c, false);
    } else {
        if (mine > 0) store_tile(0, stages, tail && g == 0);
        __syncthreads();
    }
    if (mine > 0) {
#pragma unroll
        for (int step = 0; step < 4; ++step) read_frags(stages + (i & 1) * STAGE, step);
        multiply();
        if (KG > 1 && mine < rounds) __syncthreads();  // a group with one k-tile less has passed one barrier less
    }
    if (BMAJ && do_bias) {  // uniform per workgroup: 32 KG sums of each column, added in order
        float *red = reinterpret_cast<float *>(smem);
        __syncthreads();  // the stages have been read
#pragma unroll
        for (int e = 0; e < 8; ++e) red[(32 * g + (tid >> 3)) * BM + 8 * (tid & 7) + e] = csum[e];
        __syncthreads();
        if (g == 0 && tid < BM && m0 + tid < a.M) {
            float t = red[tid];
#pragma unroll 8
            for (int q = 1; q < 32 * KG; ++q) t += red[q * BM + tid];
            if (a.write_grad) a.bias_out[m0 + tid] = t;
            else a.bias_out[m0 + tid] -= a.lr * t;
        }
    }
    if (KG > 1) {
        float *red = reinterpret_cast<float *>(smem);
        __syncthreads();  // the stages (the column sums) have been read
        if (g > 0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) red[(((g - 1) * 4 + wave) * 16 + v) * 64 + lane] = acc[0][0][v];
        }
        __syncthreads();
        if (g > 0) return;
#pragma unroll
        for (int q = 0; q < KG - 1; ++q)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[0][0][v] += red[((q * 4 + wave) * 16 + v) * 64 + lane];
    }
    epilogue_bf16<KIND, TM, 1>(a, acc, m0 + wm * (TILE / 2), n0 + wn * 32, r, h);
}

template <int TILE, int KG, int KIND, bool SHIFT, bool BMAJ, int SETS>
__global__ __launch_bounds__((TILE == 64 ? NT : 2 * NT) * KG, TILE == 64 ? (KG == 1 ? 3 : 2) : SETS == 2 ? 4 : 1)
void gemm_bf16_mid_kernel(GemmBf16Args a)
{
    __shared__ __attribute__((aligned(16))) unsigned char smem[mid_lds_bytes<TILE, KG>()];
    mid_tile<TILE, KG, KIND, SHIFT, BMAJ, SETS>(a, blockIdx.x, smem);
}

// A weight gradient and the next product of the backward pass in one launch (pair_shares() below: KG).  What bounds either alone
// is latency -- of the launch, of its first loads and of the round trip to memory that a k-tile is -- so both together
// take little longer than one: 1024 x 1024 over 2047 rows 12.8 us + 2047 x 1024 x 1024 11.9 us apart, 21.3 in one launch, and
// the narrow products of the output layer or of a 300-wide input vanish behind their neighbour (300-1024x3-2, 2047 rows: 133.5 ->
// 113.1 us per step).  With two groups the register sets are two (105 registers), so that two workgroups fit a compute
// unit; with one they are four and three workgroups do.
template <int KG, int KIND>
__global__ __launch_bounds__(NT *KG, KG == 1 ? 3 : 4) void gemm_bf16_mid_pair_kernel(GemmBf16Args dw, GemmBf16Args next, int n_dw)
{
    constexpr int SETS = KG == 1 ? 4 : 2;
    __shared__ __attribute__((aligned(16))) unsigned char smem[mid_lds_bytes<64, KG>()];
    const int b = blockIdx.x;
    if (b < n_dw) mid_tile<64, KG, GEMM_DW, false, true, SETS>(dw, b, smem);
    else mid_tile<64, KG, KIND, false, KIND == GEMM_DW, SETS>(next, b - n_dw, smem);
}

// ---- 256 x 256 x 64 kernel with LDS-direct loads ------------------------------------------
// Used when both operands allow 16-byte loads and the product is large enough for 256 x 256
// tiles.  512 threads: eight wavefronts as 2 x 4, each 128 x 64 (8 x 4 MFMA blocks), two per
// SIMD.  Differences from the kernel above:
//   * operand tiles go global -> LDS directly (global_load_lds_dwordx4: lane i of a wavefront
//     writes its 16 bytes at LDS base + 16 i), no staging registers and no ds_write;
//   * a k-tile row is 128 bytes, one whole cache line: with 64-byte rows every line was
//     fetched twice from L2 (the 32 KB L1 does not keep it for an iteration), and the
//     L2 -> L1 path (64 B/clk/CU) became the limit; the square tile needs 32 B/clk/CU at
//     full MFMA rate;
//   * rows are not padded; the eight 16-byte chunks of tile row R are stored at slot
//     c ^ swz(R), which keeps both the direct loads (a wavefront fills 1 KB contiguously) and
//     the MFMA fragment reads free of bank conflicts;
//   * out-of-range rows of an edge tile are clamped to the last valid row when loading (their
//     results are never stored), so the main loop has no guards; a K tail shorter than a tile
//     is multiplied after the loop from a masked, register-staged copy.
// LDS holds two stages of the A tile and three of the B tile (32 KB each: all 160 KB).  Per
// iteration every wavefront issues eight loads, two under each of the four MFMA groups (all
// at once they fill the address queue of the vector memory unit and the MFMA pipes idle while
// it drains): A of tile kt+1 under the last group of kt-1 and the first of kt, B of tile kt+2
// under groups two and three of kt, so that every load has at least two MFMA groups (B: more
// than an iteration) to land; an L2 round trip measured here takes ~550 cycles on average.
// Waits and barriers inside the main loop are written out by hand: at a workgroup barrier the
// compiler would also wait for the direct loads that were only just issued.
typedef __attribute__((address_space(1))) const void *gptr_t;
typedef __attribute__((address_space(3))) void *lptr_t;
typedef int v2i __attribute__((ext_vector_type(2)));
template <int K>
struct KStep {
    static constexpr int value = K;
};

// gfx950's transposing LDS read of 8 bytes per lane at LDS byte address addr + OFF.  Written as
// an instruction, not through the compiler's builtin: for the builtin the compiler cannot
// tell that the read does not touch what the LDS-direct loads in flight are writing, and puts
// a wait for ALL of them (vmcnt(0)) in front of every read (the weight gradient
// 4096 x 4096 x 16384 took 530 us that way).  The compiler does not wait for the result
// either: every use below sits behind an explicit lgkmcnt(0) and a scheduling barrier.
template <int OFF>
__device__ __forceinline__ v2i lds_read_tr16_b64(unsigned addr)
{
    static_assert(OFF >= 0 && OFF < 65536, "16-bit offset field");
    v2i v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}

// slot permutation of tile row R: the sixteen rows that a fragment read touches at one chunk, and any of its sets of rows 0-3,
// 12-15 at one chunk and 4-11 at the next, lie on different banks
__device__ __forceinline__ int swz(int R) { return (R >> 1) & 7; }
// the same for k-row k of a batch-major tile (512 bytes): the four rows of a transposing read on different 64-byte segments, the
// rows eight on, which the next sixteen lanes read, on the other 32 bytes of each
__device__ __forceinline__ int swz_k(int k) { return ((k & 3) << 2) ^ (((k >> 3) & 1) << 1); }

constexpr int DMA_NT = 512;
constexpr int DMA_BM = 256, DMA_BN = 256, DMA_BK = 64;
constexpr int DMA_ROW_BYTES = DMA_BK * 2;  // 128
constexpr int DMA_A_BYTES = DMA_BM * DMA_ROW_BYTES, DMA_B_BYTES = DMA_BN * DMA_ROW_BYTES;
constexpr int DMA_A_STAGES = 2, DMA_B_STAGES = 3;
constexpr int DMA_B_BASE = DMA_A_STAGES * DMA_A_BYTES;
constexpr size_t DMA_LDS_BYTES = (size_t)DMA_B_BASE + (size_t)DMA_B_STAGES * DMA_B_BYTES;  // 163,840: all of a CU's LDS

// Epilogue of the LDS-direct kernel when the whole workgroup tile lies inside the matrix (for
// the weight gradient: the form with the fused update, whose fp32 master weights are read
// and written directly): both bf16 outputs (row-major and transposed) leave
// through LDS, so that every global store is 16 bytes per lane and covers whole cache lines
// (128 bytes per row-major row, 256 per transposed row).  Straight from the MFMA layout a
// lane owns four consecutive rows of one column: 128 two-byte stores plus 32 eight-byte
// ones per lane, and the forward product took 86 us longer with them than with plain fp32
// output of the same size.  Each wavefront has 20 KB of LDS to itself (the operand stages
// are dead by now), used twice: 128 rows x 144 bytes for the row-major tile, then 64 rows x
// 272 bytes for the transposed one.
constexpr int EPI_REGION = 20480;
constexpr int EPI_SC = 144;  // row stride of the 128 x 64 row-major tile (128 bytes + 16)
constexpr int EPI_ST = 272;  // row stride of the 64 x 128 transposed tile (256 bytes + 16)
static_assert(128 * EPI_SC <= EPI_REGION && 64 * EPI_ST <= EPI_REGION && 8 * EPI_REGION <= (int)DMA_LDS_BYTES, "LDS");

// mword: backward-data product with ReLU decision bits (use_mask): the lane's words of its eight
// blocks, requested by the caller before the main loop.
template <int KIND, int ACT, bool MASK>
__device__ __forceinline__ void epilogue_bf16_lds(const GemmBf16Args &a, v16f (&acc)[4][2], unsigned char *region,
                                                  int mw, int nw, int lane, const unsigned (&mword)[4][2])
{
    constexpr bool use_mask = (KIND == GEMM_DA) && MASK;
    constexpr int TM = 4, TN = 2;
    const int r = lane & 31, h = lane >> 5;
    // ---- values -> bf16, four consecutive rows packed per (i, j, q)
    uint2 pk[TM][TN][4];
    const unsigned lo_at = (unsigned)(r * (int)a.ldauxt + 4 * h) * 2u;
    const unsigned char *const at0 = static_cast<const unsigned char *>(a.aux_t);
    const unsigned lo_cf = (unsigned)(4 * h * (int)a.ldc + r) * 4u;
    unsigned char *const cf0 = static_cast<unsigned char *>(a.C_f32);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int nb = nw + j * 32;
        float bias = 0.f;
        if (KIND == GEMM_FWD && a.bias != nullptr) bias = a.bias[nb + r];
        uint2 ot[TM][4];
        if (KIND == GEMM_DA && !use_mask) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    ot[i][q] = *reinterpret_cast<const uint2 *>(
                        at0 + ((size_t)nb * a.ldauxt + (mw + i * 32 + 8 * q)) * 2 + lo_at);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            // weight gradient: the 16 fp32 master weights of this 32 x 32 block that the lane
            // updates are requested together.  Fetched four at a time between the stores of
            // the previous four (which the compiler must assume to alias), every group of four
            // was a round trip to memory of its own: 64 per lane and tile.
            float wm[4][4];
            if (KIND == GEMM_DW) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        wm[q][e] = *reinterpret_cast<const float *>(
                            cf0 + ((size_t)(mw + i * 32 + 8 * q + e) * a.ldc + nb) * 4 + lo_cf);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float (&w)[4] = wm[q];
                float x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float val = acc[i][j][4 * q + e];
                    if (KIND == GEMM_FWD) {
                        val = act_fwd<ACT>(val + bias);
                    } else if (KIND == GEMM_DA) {
                        if (use_mask) {
                            val = relu_keep(val, mword[i][j], q, e);
                        } else {
                            const unsigned int pw = (e < 2) ? ot[i][q].x : ot[i][q].y;
                            const float o = __uint_as_float((e & 1) ? (pw & 0xffff0000u) : (pw << 16));
                            if (ACT == ACT_SIGMOID) val *= o * (1.f - o);
                            else if (ACT == ACT_RELU) val = (o > 0.f) ? val : 0.f;
                        }
                    } else {  // Eq. (3) on the fp32 master weight, stored back directly
                        val = w[e] - a.lr * val;
                        *reinterpret_cast<float *>(cf0 + ((size_t)(mw + i * 32 + 8 * q + e) * a.ldc + nb) * 4 + lo_cf) = val;
                    }
                    x[e] = val;
                }
                pk[i][j][q].x = pack2bf(x[0], x[1]);
                pk[i][j][q].y = pack2bf(x[2], x[3]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // ---- backward-data: column sums of the stored values over the wavefront's 128 rows (the
    // bias gradient of the layer below), in a fixed order; the two half-wavefronts hold
    // alternate groups of four rows
    if (KIND == GEMM_DA && a.colsum_partial != nullptr) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint2 v = pk[i][j][q];
                    s += (__uint_as_float(v.x << 16) + __uint_as_float(v.x & 0xffff0000u)) +
                         (__uint_as_float(v.y << 16) + __uint_as_float(v.y & 0xffff0000u));
                }
            s += __shfl_xor(s, 32, 64);
            if (h == 0) a.colsum_partial[(size_t)(mw >> 7) * a.N + nw + j * 32 + r] = s;
        }
    }
    // ---- row-major copy: T[m][n], lane writes its four rows of column j*32 + r
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                unsigned char *p = region + (i * 32 + 8 * q + 4 * h) * EPI_SC + (j * 32 + r) * 2;
                *reinterpret_cast<bf16_t *>(p) = (bf16_t)(pk[i][j][q].x & 0xffffu);
                *reinterpret_cast<bf16_t *>(p + EPI_SC) = (bf16_t)(pk[i][j][q].x >> 16);
                *reinterpret_cast<bf16_t *>(p + 2 * EPI_SC) = (bf16_t)(pk[i][j][q].y & 0xffffu);
                *reinterpret_cast<bf16_t *>(p + 3 * EPI_SC) = (bf16_t)(pk[i][j][q].y >> 16);
            }
    {
        unsigned char *const cb = static_cast<unsigned char *>(a.C_bf16) + ((size_t)mw * a.ldcb + nw) * 2;
#pragma unroll
        for (int it = 0; it < 16; ++it) {  // 128 rows x 8 chunks of 16 bytes
            const int c = it * 64 + lane, row = c >> 3, ch = c & 7;
            const uint4 v = *reinterpret_cast<const uint4 *>(region + row * EPI_SC + ch * 16);
            *reinterpret_cast<uint4 *>(cb + (size_t)row * a.ldcb * 2 + ch * 16) = v;
        }
    }
    // ---- forward product of a ReLU layer: the decision bits of the lane's eight blocks, worked
    // out while the stores above drain
    if (KIND == GEMM_FWD && MASK) {
        unsigned short *const mo = a.mask_out + ((size_t)(mw >> 5) * a.mask_nb + (nw >> 5)) * 64 + lane;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) mo[((size_t)i * a.mask_nb + j) * 64] = (unsigned short)relu_bits(pk[i][j]);
    }
    if (a.Ct_bf16 == nullptr) return;  // uniform
    // ---- transposed copy: T[n][m], lane writes 8 bytes (its four rows) into row j*32 + r.  The
    // region is reused: LDS operations of a wavefront execute in order
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<uint2 *>(region + (j * 32 + r) * EPI_ST + (i * 32 + 8 * q + 4 * h) * 2) = pk[i][j][q];
    {
        unsigned char *const ct = static_cast<unsigned char *>(a.Ct_bf16) + ((size_t)nw * a.ldct + mw) * 2;
#pragma unroll
        for (int it = 0; it < 16; ++it) {  // 64 rows x 16 chunks of 16 bytes
            const int c = it * 64 + lane, row = c >> 4, ch = c & 15;
            const uint4 v = *reinterpret_cast<const uint4 *>(region + row * EPI_ST + ch * 16);
            *reinterpret_cast<uint4 *>(ct + (size_t)row * a.ldct * 2 + ch * 16) = v;
        }
    }
}

// BMAJ (weight gradient only): both operands are batch-major, A[k * lda + m] and B[k * ldb + n],
// i.e. the row-major deltas and activations themselves, so that no transposed copy of either
// has to exist.  An operand tile is then 64 k-rows of 512 bytes; the MFMA still wants 8
// consecutive k per lane, which gfx950's transposing LDS read delivers: ds_read_b64_tr_b16
// works in groups of 16 lanes, lane 4 j + q of a group supplies the address of an 8-byte word
// (k-row j, columns 4 q .. 4 q + 3 of a 16-column strip) and lane l receives column l at
// k-rows 0..3 (layout checked with an in-bounds probe).  Two such reads make one operand
// fragment.  The four k-rows a group reads together are 512 bytes apart, i.e. on the same
// banks: the 64-byte segments of k-row k are therefore stored at segment index s ^ (k & 3)
// (the direct loads fetch the permuted segment, their LDS side stays contiguous; the 32-byte halves: swz_k).
template <int KIND, bool BMAJ>
__device__ __forceinline__ void gemm_bf16_dma_tile(const GemmBf16Args &a, unsigned char *smem_raw, int id, int T,
                                                   int tid)
{
    static_assert(!BMAJ || KIND == GEMM_DW, "batch-major operands: weight gradient only");
    constexpr int BM = DMA_BM, BN = DMA_BN, BK = DMA_BK;
    constexpr int TM = 4, TN = 2;  // 32 x 32 blocks per wavefront: 128 x 64

    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: LDS bases of the direct loads are scalars
    const int r = lane & 31, h = lane >> 5;
    const int wm = wave & 1, wn = wave >> 1;

    // XCD-aware tile order.  Workgroup ids go round-robin over the 8 XCDs and an XCD runs 32
    // workgroups at a time (one per CU), so the j-th group of 32 ids of XCD x gets a block of
    // 4 x 8 (or 8 x 4) tiles: per k-tile its L2 then fetches 12 operand panels for 32 tiles,
    // against 18 for two rows of 16 (1.26 instead of 1.07 PFLOP/s on the weight gradient).
    int tile_m, tile_n;
    int bm = 0, bn = 0;
    if ((T & 255) == 0) {
        if ((a.tiles_m & 3) == 0 && (a.tiles_n & 7) == 0) { bm = 4; bn = 8; }
        else if ((a.tiles_m & 7) == 0 && (a.tiles_n & 3) == 0) { bm = 8; bn = 4; }
    }
    if (bm != 0) {
        const int L = id >> 3;
        const int sb = (id & 7) * (T >> 8) + (L >> 5), pos = L & 31;
        const int sbn = a.tiles_n / bn;
        tile_m = (sb / sbn) * bm + pos / bn;
        tile_n = (sb % sbn) * bn + pos % bn;
    } else {
        if ((T & 7) == 0) id = (id & 7) * (T >> 3) + (id >> 3);  // a contiguous run of tiles per XCD
        tile_m = id / a.tiles_n;
        tile_n = id - tile_m * a.tiles_n;
    }
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    // slice of the contraction handled by this workgroup (blockIdx.y; the whole of it unless split)
    const int kbeg = (a.k_chunk > 0) ? (int)blockIdx.y * a.k_chunk : 0;
    const int klen = (a.k_chunk > 0) ? min(a.K - kbeg, a.k_chunk) : a.K;
    const int nkf = klen / BK;  // full k-tiles

    // operand base at the first k of the slice, and the step from one k-tile to the next
    const size_t a_tile_step = BMAJ ? (size_t)BK * (size_t)a.lda * 2 : (size_t)DMA_ROW_BYTES;
    const size_t b_tile_step = BMAJ ? (size_t)BK * (size_t)a.ldb * 2 : (size_t)DMA_ROW_BYTES;
    const unsigned char *__restrict__ Ab =
        static_cast<const unsigned char *>(a.A) + (BMAJ ? (size_t)kbeg * (size_t)a.lda * 2 : (size_t)kbeg * 2);
    const unsigned char *__restrict__ Bb =
        static_cast<const unsigned char *>(a.B) + (BMAJ ? (size_t)kbeg * (size_t)a.ldb * 2 : (size_t)kbeg * 2);

    // ---- global side of the direct loads.  One wavefront load fills 1 KB of LDS, lane i its
    // bytes 16 i ..: 8 tile rows of 128 bytes (lane -> row lane / 8, slot lane % 8), or, BMAJ,
    // 2 k-rows of 512 bytes (lane -> k-row lane / 32, slot lane % 32).  The wavefront takes
    // the 1 KB blocks wave, wave + 8, ..  BMAJ: columns past the end of a row (edge tiles; their
    // results are never stored) are clamped to the row's last 16 bytes.
    const int blk_row = lane >> 3;
    unsigned offA[4], offB[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (BMAJ) {
            const int k = (wave + 8 * v) * 2 + (lane >> 5);
            const int chunk = (lane & 31) ^ swz_k(k);  // the chunk whose slot is lane % 32
            offA[v] = (unsigned)((size_t)k * (size_t)a.lda * 2 +
                                 (size_t)min((long long)m0 * 2 + chunk * 16, a.lda * 2 - 16));
            offB[v] = (unsigned)((size_t)k * (size_t)a.ldb * 2 +
                                 (size_t)min((long long)n0 * 2 + chunk * 16, a.ldb * 2 - 16));
        } else {
            const int R = (wave + 8 * v) * 8 + blk_row;
            const int chunk = (lane & 7) ^ swz(R);  // the chunk whose slot is lane % 8
            offA[v] = (unsigned)((size_t)min(m0 + R, a.M - 1) * (size_t)a.lda * 2 + chunk * 16);
            offB[v] = (unsigned)((size_t)min(n0 + R, a.N - 1) * (size_t)a.ldb * 2 + chunk * 16);
        }
    }
    // load v of the wavefront's four of an A / B tile (tile t -> given stage)
    auto issue_a = [&](int t, int stage, int v) {
        __builtin_amdgcn_global_load_lds((gptr_t)(Ab + (size_t)t * a_tile_step + offA[v]),
                                         (lptr_t)(smem_raw + stage * DMA_A_BYTES + (wave + 8 * v) * 1024), 16, 0, 0);
    };
    auto issue_b = [&](int t, int stage, int v) {
        __builtin_amdgcn_global_load_lds((gptr_t)(Bb + (size_t)t * b_tile_step + offB[v]),
                                         (lptr_t)(smem_raw + DMA_B_BASE + stage * DMA_B_BYTES + (wave + 8 * v) * 1024), 16, 0, 0);
    };

    // ---- LDS side of the fragment reads: lane 16 g + c reads chunk 4 kk + g of row c (A: a_row(c)) of its block (k-step kk:
    // 32 deep).  The block offsets i * 16 rows leave (R >> 1) & 7 unchanged, so the swizzle depends on c only.
    // BMAJ: lane 16 g + 4 j + q addresses k-row 32 kk + 8 g + 4 t + j (t = 0, 1: the two reads of a fragment), bytes 8 q ..
    // (A: 2 a_row(4 q) ..) of the block's 32, which are the (block % 2)-th half of segment block / 2; both
    // indices are exchanged as swz_k says, and the block index enters as one more XOR.
    const int c16 = lane & 15, g4 = lane >> 4;
    const int tj = c16 >> 2;
    const int arow = a_row(c16);
    const int a_off = BMAJ ? (8 * g4 + tj) * 512 + (((wm * 4) ^ tj) << 6) + 32 * (g4 & 1) + 2 * a_row(4 * (lane & 3))
                         : (wm * 128 + arow) * DMA_ROW_BYTES + ((g4 ^ swz(arow)) << 4);  // k-step kk: a_off ^ (kk << 6)
    const int b_off = DMA_B_BASE + (BMAJ ? (8 * g4 + tj) * 512 + (((wn * 2) ^ tj) << 6) + 32 * (g4 & 1) + 8 * (lane & 3)
                                       : (wn * 64 + c16) * DMA_ROW_BYTES + ((g4 ^ swz(c16)) << 4));
    v8bf fa[2][TM], fb[2][2 * TN];  // half of the wavefront's rows (64) / all of its columns at one k-step
    const unsigned lds0 = (unsigned)(size_t)(lptr_t)smem_raw;  // LDS byte address of the stages
    // one operand fragment (block q of the A or B tile at p, k-step kk; kk is a KStep<> so
    // that the batch-major form can put it into the instruction's offset field)
    auto frag = [&](const unsigned char *p, int off, int q, auto kkc) -> v8bf {
        constexpr int kk = decltype(kkc)::value;
        if (BMAJ) {
            const unsigned addr = lds0 + (unsigned)(p - smem_raw) + (unsigned)(off ^ (q << 5));
            const v2i lo = lds_read_tr16_b64<kk * 32 * 512>(addr);
            const v2i hi = lds_read_tr16_b64<kk * 32 * 512 + 4 * 512>(addr);
            return __builtin_bit_cast(v8bf, __builtin_shufflevector(lo, hi, 0, 1, 2, 3));
        } else {
            return *reinterpret_cast<const v8bf *>(p + ((off ^ (kk << 6)) + q * 16 * DMA_ROW_BYTES));
        }
    };
    // the compiler does not know when the batch-major form's fragments have arrived
    auto frags_landed = [&]() {
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
    };

    v4f acc16[2 * TM][2 * TN];
#pragma unroll
    for (int i = 0; i < 2 * TM; ++i)
#pragma unroll
        for (int j = 0; j < 2 * TN; ++j) acc16[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    // Epilogue through LDS (uniform for the workgroup): bf16 output wanted, row-major or in both
    // layouts (and, except for the fused update, nothing else), workgroup tile inside the
    // matrix, 16-byte alignment of every row
    const bool use_mask = (KIND == GEMM_DA) && a.mask_in != nullptr && a.act == ACT_RELU;
    const bool via_lds = !(KIND == GEMM_DW && a.k_chunk > 0) && a.C_bf16 != nullptr &&
                         (KIND == GEMM_DW ? (a.Ct_bf16 != nullptr && a.C_f32 != nullptr && !a.write_grad)
                                          : a.C_f32 == nullptr) &&
                         (m0 + BM <= a.M) && (n0 + BN <= a.N) && (a.ldcb & 7) == 0 &&
                         (a.Ct_bf16 == nullptr || (a.ldct & 7) == 0) &&
                         ((reinterpret_cast<size_t>(a.C_bf16) | reinterpret_cast<size_t>(a.Ct_bf16)) & 15) == 0 &&
                         (KIND != GEMM_DA || use_mask || (a.aux_t != nullptr && (a.ldauxt & 3) == 0));
    // backward-data product: the ReLU decision bits of the lane's eight blocks are requested
    // now and have arrived long before the epilogue (they are older than every operand load,
    // so the waits of the main loop cover them)
    unsigned mword[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) mword[i][j] = 0u;
    if (KIND == GEMM_DA && use_mask && via_lds) {
        const unsigned short *mi =
            a.mask_in + ((size_t)((m0 + wm * 128) >> 5) * a.mask_nb + ((n0 + wn * 64) >> 5)) * 64 + lane;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) mword[i][j] = mi[((size_t)i * a.mask_nb + j) * 64];
    }

    // One MFMA group: the sixteen MFMAs of one half of the wavefront's rows at one k-step (A fragments in fa[half], B
    // fragments in fb[bs]), and in their shadow (a wavefront can issue other instructions while its MFMA executes) the
    // requests for the next group's fragments -- the other half of the rows, or (second half) the first one of the next
    // k-step and that step's B --, one after each of the first MFMAs, and two direct loads after the sixth and eleventh
    // (eleventh and fifteenth).  Clumped, these requests are issued by both wavefronts of a SIMD at the same time (the
    // barrier keeps them in step) and the MFMA pipe idles meanwhile: with two fragments to an MFMA and the two loads together
    // four steps of 2048-4096x3-1000 over 16384 rows, their readback included, take 18.06 ms, so 17.53.  Only the requests
    // are conditional, so that there is one MFMA stream.
    auto group = [&](auto half_c, int bs, bool rd, int sa, int sb, auto kk, bool ld, bool is_a, int t, int stage, int first) {
        constexpr int half = decltype(half_c)::value;
        const unsigned char *pa = smem_raw + sa * DMA_A_BYTES;
        const unsigned char *pb = smem_raw + sb * DMA_B_BYTES;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < 2 * TN; ++j) {
                acc16[TM * half + i][j] =
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[half][i], fb[bs][j], acc16[TM * half + i][j], 0, 0, 0);
                const int b = i * 2 * TN + j;
                __builtin_amdgcn_sched_barrier(0);
                if (rd) {
                    if (b < TM) fa[half ^ 1][b] = frag(pa, a_off, b + (half ? 0 : TM), kk);
                    else if (half && b < TM + 2 * TN) fb[bs ^ 1][b - TM] = frag(pb, b_off, b - TM, kk);
                }
                if (ld && (b == (half ? 10 : 5) || b == (half ? 14 : 10))) {
                    const int v = first + (b == (half ? 14 : 10) ? 1 : 0);
                    if (is_a) issue_a(t, stage, v);
                    else issue_b(t, stage, v);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    constexpr KStep<0> LO = {}, S0 = {};
    constexpr KStep<1> HI = {}, S1 = {};
    auto read_first = [&]() {  // the first group's fragments of the tile in stages 0
#pragma unroll
        for (int q = 0; q < TM; ++q) fa[0][q] = frag(smem_raw, a_off, q, S0);
#pragma unroll
        for (int q = 0; q < 2 * TN; ++q) fb[0][q] = frag(smem_raw, b_off, q, S0);
    };

    if (nkf > 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) issue_a(0, 0, v);
#pragma unroll
        for (int v = 0; v < 4; ++v) issue_b(0, 0, v);
        if (nkf > 1) {
#pragma unroll
            for (int v = 0; v < 4; ++v) issue_b(1, 1, v);
            issue_a(1, 1, 0);
            issue_a(1, 1, 1);
            asm volatile("s_waitcnt vmcnt(6)\n\ts_barrier" ::: "memory");  // tile 0 landed
        } else {
            asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        }
        read_first();
        static_assert(BK == 64, "the load schedule below is written for two k-steps per tile");
        int b_cur = 0, b_nxt = 1, b_ld = 2;  // B stages of tiles kt, kt+1, kt+2
        for (int kt = 0; kt < nkf; ++kt) {
            const int a_cur = kt & 1;
            const bool next = (kt + 1 < nkf), next2 = (kt + 2 < nkf);
            // The explicit lgkmcnt(0) at the head of a group tells the compiler that the
            // fragments requested during the previous group have arrived (they have: five
            // MFMAs lie in between); it cannot track them across the small branches.
            // (batch-major form: the compiler does not see the reads at all, and a scheduling
            // barrier keeps the MFMAs behind the wait)
            __builtin_amdgcn_s_waitcnt(0xc07f);
            if (BMAJ) __builtin_amdgcn_sched_barrier(0);
            group(LO, 0, true, a_cur, b_cur, S0, next, true, kt + 1, a_cur ^ 1, 2);   // + second half of A(kt+1)
            __builtin_amdgcn_s_waitcnt(0xc07f);
            if (BMAJ) __builtin_amdgcn_sched_barrier(0);
            group(HI, 0, true, a_cur, b_cur, S1, next2, false, kt + 2, b_ld, 0);      // + B(kt+2): its stage held B(kt-1)
            __builtin_amdgcn_s_waitcnt(0xc07f);
            if (BMAJ) __builtin_amdgcn_sched_barrier(0);
            group(LO, 1, true, a_cur, b_cur, S1, next2, false, kt + 2, b_ld, 2);
            // Tile kt+1 must have landed (this wavefront's share; the barrier covers the others');
            // the four loads of B(kt+2) just issued may stay in flight.  This wavefront's reads of
            // tile kt must be done before anyone overwrites its stages.
            if (next2) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0) again, this time visible to the compiler
            if (BMAJ) __builtin_amdgcn_sched_barrier(0);
            // last group of tile kt; the first fragments of tile kt+1 are requested from the stages that have
            // just been completed, and the first half of A(kt+2) goes into the stage just released
            group(HI, 1, next, a_cur ^ 1, b_nxt, S0, next2, true, kt + 2, a_cur, 0);
            const int t = b_cur;
            b_cur = b_nxt;
            b_nxt = b_ld;
            b_ld = t;
        }
    }

    // ---- K tail (fewer than BK columns left): masked copy through registers into stage 0
    const int ktail = klen - nkf * BK;
    if (ktail > 0) {
        __syncthreads();  // everybody is done with the main loop's stages
        const int kbase = nkf * BK;  // relative to the slice
#pragma unroll
        for (int v = 0; v < (BM + BN) * 8 / DMA_NT; ++v) {  // 16-byte chunks of both tiles over the workgroup
            const int idx = tid + v * DMA_NT;
            const bool isA = idx < BM * 8;
            const int q = isA ? idx : idx - BM * 8;
            if (BMAJ) {  // k-row q / 32, slot q % 32; k-rows past the end of the slice are zero
                const int k = q >> 5, slot = q & 31;
                const int chunk = slot ^ swz_k(k);
                uint4 x = {0u, 0u, 0u, 0u};
                if (kbase + k < klen) {
                    const long long ld = isA ? a.lda : a.ldb;
                    const long long col = min((long long)(isA ? m0 : n0) * 2 + chunk * 16, ld * 2 - 16);
                    x = *reinterpret_cast<const uint4 *>((isA ? Ab : Bb) + (size_t)(kbase + k) * (size_t)ld * 2 + col);
                }
                *reinterpret_cast<uint4 *>(smem_raw + (isA ? 0 : DMA_B_BASE) + k * 512 + slot * 16) = x;
                continue;
            }
            const int R = q >> 3, c = q & 7;
            const int k = kbase + c * 8;
            uint4 x = {0u, 0u, 0u, 0u};
            if (k < klen) {  // rows are padded to 8 elements, so the 16 bytes are in bounds
                const int grow = isA ? min(m0 + R, a.M - 1) : min(n0 + R, a.N - 1);
                const unsigned char *p = isA ? Ab + ((size_t)grow * (size_t)a.lda + k) * 2
                                             : Bb + ((size_t)grow * (size_t)a.ldb + k) * 2;
                x = *reinterpret_cast<const uint4 *>(p);
                const int valid = klen - k;  // elements of this chunk that belong to the slice
                if (valid < 8) {
                    unsigned int w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (2 * e >= valid) w[e] = 0u;
                        else if (2 * e + 1 >= valid) w[e] &= 0xffffu;
                    }
                    x = make_uint4(w[0], w[1], w[2], w[3]);
                }
            }
            *reinterpret_cast<uint4 *>(smem_raw + (isA ? 0 : DMA_B_BASE) + R * DMA_ROW_BYTES +
                                       ((c ^ swz(R)) << 4)) = x;
        }
        __syncthreads();
        read_first();
        frags_landed();
        group(LO, 0, true, 0, 0, S0, false, false, 0, 0, 0);
        frags_landed();
        group(HI, 0, true, 0, 0, S1, false, false, 0, 0, 0);
        frags_landed();
        group(LO, 1, true, 0, 0, S1, false, false, 0, 0, 0);
        frags_landed();
        group(HI, 1, false, 0, 0, S0, false, false, 0, 0, 0);
    }
    v16f acc[TM][TN];
    blocks_of_32<TM, TN>(acc, acc16);

    if (KIND == GEMM_DW && a.k_chunk > 0) {
        GemmBf16Args as = a;  // this slice's partial product
        as.C_f32 = static_cast<float *>(a.C_f32) + (size_t)blockIdx.y * (size_t)a.c_split_stride;
        store_slice<TM, TN>(as, acc, m0 + wm * 128, n0 + wn * 64, r, h);
    } else {
        if (via_lds) {
            // Every wavefront must be done with the operand stages.  After the main loop it is:
            // the last fragments were read before the loop's last barrier.  A K tail, or no
            // whole k-tile at all, ends with reads of stage 0.
            if (ktail > 0 || nkf == 0) __syncthreads();
            const bool mask = (KIND == GEMM_FWD) ? (a.mask_out != nullptr && a.act == ACT_RELU) : use_mask;
            with_activation(KIND == GEMM_DW ? (int)ACT_NONE : a.act, mask, [&](auto act_c, auto mask_c) {
                epilogue_bf16_lds<KIND, decltype(act_c)::value, decltype(mask_c)::value != 0>(
                    a, acc, smem_raw + wave * EPI_REGION, m0 + wm * 128, n0 + wn * 64, lane, mword);
            });
        } else {
            epilogue_bf16<KIND, TM, TN>(a, acc, m0 + wm * 128, n0 + wn * 64, r, h);
        }
    }
}

// Workgroup b computes tiles b, b + gridDim.x, ..: with more tiles than compute units the
// launcher starts one workgroup per compute unit, which saves the dispatch of a new
// workgroup at every tile boundary (16384 x 4096 x 4096: 428 -> 425 us); otherwise one
// workgroup per tile.  The thread number goes through an empty asm in every round: everything
// the tile derives from it would otherwise be computed once in front of the loop and sit in
// registers through the main loop, which has none to spare.  Between two tiles every
// wavefront must be done with the LDS staging of its results before the next tile's operand
// loads may land on it.
template <int KIND, bool BMAJ = false>
__global__ __launch_bounds__(DMA_NT, 1) void gemm_bf16_dma_kernel(GemmBf16Args a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int T = a.tiles_m * a.tiles_n;
    for (int id = blockIdx.x; id < T; id += (int)gridDim.x) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        gemm_bf16_dma_tile<KIND, BMAJ>(a, smem_raw, id, T, tid);
        if (id + (int)gridDim.x < T) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
}

// out[c][r] = in[r][c] for bf16 matrices (R x C, leading dimensions ldi / ldo), 64 x 64 tiles.
// Interior tiles of 16-byte aligned matrices move 16 bytes per lane on both sides (two-byte
// accesses reach 2.3 TB/s, a third of what the memory gives): rows come in as eight 16-byte
// pieces each, go to LDS as dwords with a row stride of 33 dwords, and a lane gathers the
// eight values of its output piece from eight LDS rows (stride 33: the eight row groups of a
// wavefront fall on banks 8 apart, conflict-free).
__global__ __launch_bounds__(256) void transpose_bf16_kernel(const bf16_t *__restrict__ in, long long ldi,
                                                             bf16_t *__restrict__ out, long long ldo, int R, int C,
                                                             int vec_ok)
{
    __shared__ bf16_t t[64][66];
    const int c0 = blockIdx.x * 64, r0 = blockIdx.y * 64;
    if (vec_ok && r0 + 64 <= R && c0 + 64 <= C) {
        uint32_t *tw = reinterpret_cast<uint32_t *>(&t[0][0]);  // [64][33] dwords
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int s = threadIdx.x + 256 * p, row = s >> 3, sc = s & 7;
            const uint4 v = *reinterpret_cast<const uint4 *>(in + (size_t)(r0 + row) * ldi + c0 + sc * 8);
            uint32_t *d = tw + row * 33 + sc * 4;
            d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
        }
        __syncthreads();
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int s = threadIdx.x + 256 * p, c = s >> 3, sr = s & 7;
            uint32_t w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t lo = t[sr * 8 + 2 * j][c], hi = t[sr * 8 + 2 * j + 1][c];
                w[j] = lo | (hi << 16);
            }
            *reinterpret_cast<uint4 *>(out + (size_t)(c0 + c) * ldo + r0 + sr * 8) = make_uint4(w[0], w[1], w[2], w[3]);
        }
        return;
    }
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;  // 64 x 4
    for (int k = ty; k < 64; k += 4)
        if (r0 + k < R && c0 + tx < C) t[k][tx] = in[(size_t)(r0 + k) * ldi + c0 + tx];
    __syncthreads();
    for (int k = ty; k < 64; k += 4)
        if (c0 + k < C && r0 + tx < R) out[(size_t)(c0 + k) * ldo + r0 + tx] = t[tx][k];
}

// bf16 copies of an fp32 weight matrix W [R x C]: shadow [R x lds_] and shadow_t [C x ldt]
__global__ __launch_bounds__(256) void shadow_kernel(const float *__restrict__ W, int R, int C,
                                                     bf16_t *__restrict__ shadow, long long lds_,
                                                     bf16_t *__restrict__ shadow_t, long long ldt)
{
    __shared__ bf16_t t[64][66];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int c0 = blockIdx.x * 64, r0 = blockIdx.y * 64;
    for (int k = ty; k < 64; k += 4)
        if (r0 + k < R && c0 + tx < C) {
            const bf16_t b = f2bf(W[(size_t)(r0 + k) * C + c0 + tx]);
            t[k][tx] = b;
            shadow[(size_t)(r0 + k) * lds_ + c0 + tx] = b;
        }
    __syncthreads();
    for (int k = ty; k < 64; k += 4)
        if (c0 + k < C && r0 + tx < R) shadow_t[(size_t)(c0 + k) * ldt + r0 + tx] = t[tx][k];
}

// Sum of the slices of a split weight gradient, then Eq. (3) on the fp32 master weights or a
// plain store of the gradient.  Slices are added in index order (deterministic).
__global__ __launch_bounds__(256) void dw_reduce_kernel(const float *__restrict__ partial, int splits,
                                                        long long stride, long long count,
                                                        float *__restrict__ master, float *__restrict__ grad,
                                                        float lr)
{
    const bool vec = ((stride & 3) == 0) && ((count & 3) == 0) && ((reinterpret_cast<size_t>(partial) & 15) == 0) &&
                     ((reinterpret_cast<size_t>(grad ? grad : master) & 15) == 0);
    const long long step = (long long)gridDim.x * 256;
    if (vec) {
        for (long long q = (long long)blockIdx.x * 256 + threadIdx.x; q < (count >> 2); q += step) {
            float4 s = {0.f, 0.f, 0.f, 0.f};
            for (int k = 0; k < splits; ++k) {
                const float4 p = *reinterpret_cast<const float4 *>(partial + (size_t)k * stride + 4 * q);
                s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
            }
            if (grad) {
                *reinterpret_cast<float4 *>(grad + 4 * q) = s;
            } else {
                float4 w = *reinterpret_cast<float4 *>(master + 4 * q);
                w.x -= lr * s.x; w.y -= lr * s.y; w.z -= lr * s.z; w.w -= lr * s.w;
                *reinterpret_cast<float4 *>(master + 4 * q) = w;
            }
        }
    } else {
        for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < count; i += step) {
            float s = 0.f;
            for (int k = 0; k < splits; ++k) s += partial[(size_t)k * stride + i];
            if (grad) grad[i] = s;
            else master[i] -= lr * s;
        }
    }
}

// Bias gradient from the transposed delta (one wavefront per output unit j):
//   g = sum_b Dt[j][b];  b_l[j] -= lr g   or   grad[j] = g
__global__ __launch_bounds__(256) void rowsum_bias_kernel(const bf16_t *__restrict__ Dt, long long ld, int d,
                                                          long long B, float *__restrict__ bias,
                                                          float *__restrict__ grad, float lr)
{
    const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (j >= d) return;
    const bf16_t *row = Dt + (size_t)j * ld;
    float s = 0.f;
    long long b0 = 0;
    if ((ld & 7) == 0 && (reinterpret_cast<size_t>(Dt) & 15) == 0) {
        // 16 bytes (8 values) per lane and load, four loads in flight
        const long long nvec = B >> 3;
        const uint4 *rv = reinterpret_cast<const uint4 *>(row);
        for (long long v0 = 0; v0 < nvec; v0 += 256) {
            uint4 x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const long long v = v0 + u * 64 + lane;
                x[u] = (v < nvec) ? rv[v] : make_uint4(0u, 0u, 0u, 0u);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const unsigned int w[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) s += __uint_as_float(w[e] << 16) + __uint_as_float(w[e] & 0xffff0000u);
            }
        }
        b0 = nvec << 3;
    }
    for (long long b = b0 + lane; b < B; b += 64) s += bf2f(row[b]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) {
        if (grad) grad[j] = s;
        else bias[j] -= lr * s;
    }
}

// Bias gradient from the row-major delta D [B x ld] (16-byte aligned rows): column sums over
// the batch in two steps, both in a fixed order.  Step 1, block (x, s): columns 512 x .. + 511 of
// the rows of slice s; a thread owns 8 columns (one 16-byte load per row) and every fourth row,
// four loads in flight; the four row lanes meet in LDS.  Step 2 adds the slices in index order
// and applies Eq. (3) to the bias (or stores the gradient).
constexpr int CSB_COLS = 512, CSB_MAX_SLICES = 128;
__global__ __launch_bounds__(256) void colsum_bf16_kernel(const bf16_t *__restrict__ D, long long ld, int d,
                                                          long long B, int rows_per_slice,
                                                          float *__restrict__ partial)
{
    __shared__ float red[4][CSB_COLS + 8];
    const int cl = threadIdx.x & 63, rl = threadIdx.x >> 6;
    const long long c0 = (long long)blockIdx.x * CSB_COLS + cl * 8;
    const long long r0 = (long long)blockIdx.y * rows_per_slice, r1 = min(B, r0 + (long long)rows_per_slice);
    float s[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] = 0.f;
    auto add = [&](const uint4 &x) {
        const unsigned int w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[2 * e] += __uint_as_float(w[e] << 16);
            s[2 * e + 1] += __uint_as_float(w[e] & 0xffff0000u);
        }
    };
    if (c0 < ld) {  // ld is a multiple of 8: the whole 16-byte piece lies inside the row
        const bf16_t *p = D + c0;
        long long i = r0 + rl;
        for (; i + 12 < r1; i += 16) {
            uint4 x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = *reinterpret_cast<const uint4 *>(p + (size_t)(i + 4 * u) * ld);
#pragma unroll
            for (int u = 0; u < 4; ++u) add(x[u]);
        }
        for (; i < r1; i += 4) add(*reinterpret_cast<const uint4 *>(p + (size_t)i * ld));
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) red[rl][cl * 8 + e] = s[e];
    __syncthreads();
    for (int c = threadIdx.x; c < CSB_COLS; c += 256) {
        const long long col = (long long)blockIdx.x * CSB_COLS + c;
        if (col < d) partial[(size_t)blockIdx.y * d + col] = (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
    }
}

__global__ __launch_bounds__(256) void colsum_bias_finalize_kernel(const float *__restrict__ partial, int slices,
                                                                   int d, float *__restrict__ bias,
                                                                   float *__restrict__ grad, float lr)
{
    // 64 columns per block, four lanes per column: lane q adds slices q, q + 4, .. (eight loads
    // in flight), the four meet in LDS in lane order
    __shared__ float red[4][64];
    const int c = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int j = blockIdx.x * 64 + c;
    float s = 0.f;
    if (j < d) {
        int k = q;
        for (; k + 28 < slices; k += 32) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = partial[(size_t)(k + 4 * u) * d + j];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; k < slices; k += 4) s += partial[(size_t)k * d + j];
    }
    red[q][c] = s;
    __syncthreads();
    if (q == 0 && j < d) {
        const float t = (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
        if (grad) grad[j] = t;
        else bias[j] -= lr * t;
    }
}

int env_int_bf16(const char *name, int dflt)
{
    const char *v = getenv(name);
    return (v && *v) ? atoi(v) : dflt;
}

// Tiles of a product and the blocks of them that the 8 XCDs take: those with the fewest operand rows (4096 x 4096 x 1000:
// forward 46.9 -> 42.5 us, backward-data 47.3 -> 41.7; 1024 x 1024 x 2047 the same either way).
long long mid_tiles(GemmBf16Args &a, int tile)
{
    a.tiles_m = (a.M + tile - 1) / tile;
    a.tiles_n = (a.N + tile - 1) / tile;
    a.xcd_m = 0;
    for (int m = 1, best = 0; m <= 8; m *= 2) {
        if (a.tiles_m % m != 0 || a.tiles_n % (8 / m) != 0) continue;
        const int rows = a.tiles_m / m + a.tiles_n / (8 / m);
        if (a.xcd_m == 0 || rows < best) {
            a.xcd_m = m;
            best = rows;
        }
    }
    return (long long)a.tiles_m * a.tiles_n;
}

template <int TILE, int KG, bool SHIFT, int SETS = 4>
hipError_t launch_mid_bf16(GemmKind kind, GemmBf16Args a, hipStream_t stream, const LaunchEvents &ev)
{
    const long long tiles = mid_tiles(a, TILE);
    if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles), block((TILE == 64 ? NT : 2 * NT) * KG);
    if constexpr (TILE == 64 && !SHIFT)
        if (a.bmaj)
            return launch_kernel(gemm_bf16_mid_kernel<TILE, KG, GEMM_DW, false, true, SETS>,
                                 dim3((unsigned)tiles + (a.fin.n > 0 ? 1 : 0)), block, stream, ev, a);
    if (kind == GEMM_FWD)
        return launch_kernel(gemm_bf16_mid_kernel<TILE, KG, GEMM_FWD, SHIFT, false, SETS>, grid, block, stream, ev, a);
    if constexpr (!SHIFT) {
        if (kind == GEMM_DA)
            return launch_kernel(gemm_bf16_mid_kernel<TILE, KG, GEMM_DA, false, false, SETS>, grid, block, stream, ev, a);
        if constexpr (SETS == 4)
            return launch_kernel(gemm_bf16_mid_kernel<TILE, KG, GEMM_DW, false, false, SETS>, grid, block, stream, ev, a);
    }
    return hipErrorInvalidValue;
}

// 128 x 128 tiles where they (nearly) fill the compute units: half the operand bytes per flop
// (against 64 x 64, both in turn: 1600 x 2050 x 2050, 221 tiles: 59.1 -> 32.8 us; 3300 x 1024 x 1024, 208: 21.6 -> 18.6;
// 7001 x 1024 x 1024, 440: 34.2 -> 31.5; one and a half rounds lose a little, 3001 x 2048 x 1024, 384: 31.4 -> 32.6).  Two of them
// on a compute unit for contractions of one k-tile with more than 256 tiles, and of two with more than 512
// (4096 x 2048 x 54, 512 tiles: 17.5 -> 15.2 us; 16384 x 4096 x 100: 134 -> 123; but 8192 x 512 x 128, 256 tiles:
// 9.4 -> 13.4, and 8192 x 1000 x 100, 512 tiles: 23.2 -> 25.3).
// Else 64 x 64, with two groups of wavefronts per tile while there are no more tiles than compute units and there are
// k-tiles to share (1023 x 1024 x 1024: 12.6 -> 10.1 us, 1024 x 1024 x 2047 as a weight gradient 20.2 ->
// 17.7 us); with more tiles the compute units are shared by workgroups anyway (7001 x 1024 x 1024 in such tiles: two
// groups take a fifth longer than one).
int mid_kernel_of(GemmKind kind, const GemmBf16Args &a)
{
    const long long tiles = (long long)((a.M + 63) / 64) * ((a.N + 63) / 64);
    const long long big = (long long)((a.M + 127) / 128) * ((a.N + 127) / 128);
    if (!a.bmaj && big >= 200) {
        const bool epilogue_bound = kind != GEMM_DW && (a.K <= MID_BK ? big > 256 : a.K <= 2 * MID_BK && big > 512);
        return epilogue_bound ? BF16_K_128_SHORT : BF16_K_128;
    }
    return (tiles <= 256 && a.K >= 8 * MID_BK) ? BF16_K_64_SHARED : BF16_K_64;
}
template <bool SHIFT>
hipError_t launch_mid(GemmKind kind, const GemmBf16Args &a, hipStream_t stream, const LaunchEvents &ev)
{
    switch (mid_kernel_of(kind, a)) {
    case BF16_K_128_SHORT: return launch_mid_bf16<128, 1, SHIFT, 2>(kind, a, stream, ev);
    case BF16_K_128: return launch_mid_bf16<128, 1, SHIFT>(kind, a, stream, ev);
    case BF16_K_64_SHARED: return launch_mid_bf16<64, 2, SHIFT>(kind, a, stream, ev);
    default: return launch_mid_bf16<64, 1, SHIFT>(kind, a, stream, ev);
    }
}

hipError_t launch_dma_bf16(GemmKind kind, GemmBf16Args a, hipStream_t stream, const LaunchEvents &ev)
{
    void (*k)(GemmBf16Args) = kind == GEMM_FWD  ? gemm_bf16_dma_kernel<GEMM_FWD>
                              : kind == GEMM_DA ? gemm_bf16_dma_kernel<GEMM_DA>
                              : a.bmaj          ? gemm_bf16_dma_kernel<GEMM_DW, true>
                                                : gemm_bf16_dma_kernel<GEMM_DW>;
    const int slot = (kind == GEMM_DW && a.bmaj) ? 3 : (int)kind;
    static LdsGrant granted[4];
    const hipError_t e = grant_lds(granted[slot], DMA_LDS_BYTES, k);
    if (e != hipSuccess) return e;
    a.tiles_m = (a.M + DMA_BM - 1) / DMA_BM;
    a.tiles_n = (a.N + DMA_BN - 1) / DMA_BN;
    const long long tiles = (long long)a.tiles_m * a.tiles_n;
    if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    const int splits = (kind == GEMM_DW && a.k_chunk > 0) ? (a.K + a.k_chunk - 1) / a.k_chunk : 1;
    // one workgroup per compute unit (256 on this part) when there are more tiles than that
    // (HB_BF16_PERSIST=0, tuning aid: one workgroup per tile)
    static const int persist = env_int_bf16("HB_BF16_PERSIST", 1);
    const long long wgs = (persist && tiles > 256) ? 256 : tiles;
    const dim3 grid((unsigned)wgs, (unsigned)splits), block(DMA_NT);
    if (ev.start)
        hipExtLaunchKernelGGL(k, grid, block, (unsigned)DMA_LDS_BYTES, stream, ev.start, ev.stop, 0, a);
    else
        hipLaunchKernelGGL(k, grid, block, DMA_LDS_BYTES, stream, a);
    return hipGetLastError();
}

}  // namespace

namespace {
bool aligned4(const void *p, long long ld) { return (ld & 1) == 0 && (reinterpret_cast<size_t>(p) & 3) == 0; }
}  // namespace

int gemm_bf16_kernel(GemmKind kind, const GemmBf16Args &a)
{
    if (a.M <= 0 || a.N <= 0 || a.K <= 0) return 0;
    // The 256 x 256 LDS-direct kernel when both operands allow it and its tiles cover at least
    // half of the CUs, else the smaller tiles.  HB_BF16_TILE = 1 forces the LDS-direct kernel (tuning aid).
    static const int forced = env_int_bf16("HB_BF16_TILE", 0);
    const long long dma_tiles = (long long)((a.M + DMA_BM - 1) / DMA_BM) * ((a.N + DMA_BN - 1) / DMA_BN);
    // the LDS-direct kernel addresses each operand with 32-bit byte offsets from its base
    // (batch-major operands: rows are batch rows, and only the first k-tile is addressed that way)
    const bool dma_ok = a.a_vec && a.b_vec &&
                        (a.bmaj ? ((unsigned long long)DMA_BK * (unsigned long long)a.lda * 2 < (1ull << 32) &&
                                   (unsigned long long)DMA_BK * (unsigned long long)a.ldb * 2 < (1ull << 32) &&
                                   a.lda >= a.M && a.ldb >= a.N)
                                : ((unsigned long long)a.M * (unsigned long long)a.lda * 2 < (1ull << 32) &&
                                   (unsigned long long)a.N * (unsigned long long)a.ldb * 2 < (1ull << 32)));
    if (a.bmaj && kind != GEMM_DW) return 0;
    if (a.bmaj == BF16_DW_BMAJ_MID) return (a.k_chunk > 0) ? 0 : mid_kernel_of(kind, a);
    if (a.bmaj || a.k_chunk > 0) {  // batch-major operands, or split over the batch: the LDS-direct kernel only
        const bool slices_ok = a.k_chunk == 0 || (a.write_grad && !a.C_bf16 && !a.Ct_bf16 && (a.k_chunk % DMA_BK) == 0);
        return (kind == GEMM_DW && dma_ok && slices_ok) ? BF16_K_DMA : 0;
    }
    if (dma_ok && (forced == 1 || (forced == 0 && dma_tiles >= 128))) return BF16_K_DMA;
    // 32-bit byte offsets over 64 rows.  Rows of the weight copies, activations and deltas have a pitch of 8; only the
    // caller's X can be off.
    if (a.lda >= (1ll << 25) || a.ldb >= (1ll << 25) || !aligned4(a.B, a.ldb)) return 0;
    return (aligned4(a.A, a.lda) || kind == GEMM_FWD) ? mid_kernel_of(kind, a) : 0;
}

hipError_t launch_gemm_bf16(GemmKind kind, GemmBf16Args a, hipStream_t stream, const LaunchEvents &ev,
                            int *colsum_slices_out)
{
    if (colsum_slices_out) *colsum_slices_out = 0;
    const int kernel = gemm_bf16_kernel(kind, a);
    if (kernel == 0) return hipErrorInvalidValue;
    if (kernel == BF16_K_DMA) {
        // column sums of a backward-data result: two slices per tile row, if the caller has room
        const int slices = 2 * ((a.M + DMA_BM - 1) / DMA_BM);
        if (kind != GEMM_DA || a.colsum_partial == nullptr || slices > a.colsum_cap) a.colsum_partial = nullptr;
        else if (colsum_slices_out) *colsum_slices_out = slices;
        return launch_dma_bf16(kind, a, stream, ev);
    }
    a.colsum_partial = nullptr;  // the other kernels do not produce them
    return (a.bmaj || aligned4(a.A, a.lda)) ? launch_mid<false>(kind, a, stream, ev) : launch_mid<true>(kind, a, stream, ev);
}

// Two groups of wavefronts per tile for a pair of `tiles` 64 x 64 tiles whose weight gradient runs over K rows?  They halve the
// longest chain, the weight gradient's k-tiles, and hold half as many loads each: better where there are chains to halve and
// the workgroups have a compute unit for themselves or nearly, and for long batches always.  One group / two, us per step:
// 300-1024x3-2 64 rows 65.3 / 66.4, 500 78.0 / 78.0, 2047 (768 tiles) 113.1 / 115.6, 4000 172.6 / 170.4, 7001 287 / 281;
// 64-256x3-10 64 rows 43.0 / 45.3, 500 54.3 / 53.6, 2047 80.1 / 71.8, 7001 167 / 131; 1024-2048-2048-10 64 rows 68.5 / 73.0, 1000
// (1536 tiles) 103.9 / 107.8, 2047 157.2 / 159.3, 4000 309 / 309, 7001 400 / 392.
static bool pair_shares(long long tiles, int K) { return K >= 8 * MID_BK && (tiles <= 512 || K >= 48 * MID_BK); }

// Products that the kernels of 64 x 64 tiles take (apart / in one launch, us per step: 64-128-7 64 rows 25.7 / 21.5, 7001
// 80.1 / 50.4; 512x4-100 500 rows 83.7 / 62.9; 2048-700x3-1000 2047 rows 172 / 137, 7001 rows, which has hardly any such
// product, 395 / 394; 1024-2048-2048-10 4000 rows 309 / 309).  HB_BF16_NO_PAIR=1 (tuning and test aid; read per step): apart.
bool gemm_bf16_pairs_on() { return env_int_bf16("HB_BF16_NO_PAIR", 0) == 0; }
int gemm_bf16_pair_groups(const GemmBf16Args &dw, GemmKind kind, const GemmBf16Args &next)
{
    if (dw.bmaj != BF16_DW_BMAJ_MID || kind == GEMM_FWD || (kind == GEMM_DW && next.bmaj != BF16_DW_BMAJ_MID)) return 0;
    long long blocks = 0;
    for (const GemmBf16Args *a : {&dw, &next}) {
        const int k = gemm_bf16_kernel(a == &dw ? GEMM_DW : kind, *a);
        if (k != BF16_K_64 && k != BF16_K_64_SHARED) return 0;
        blocks += (long long)((a->M + 63) / 64) * ((a->N + 63) / 64) + (a->bmaj && a->fin.n > 0 ? 1 : 0);
    }
    if (!next.bmaj && !aligned4(next.A, next.lda)) return 0;
    return pair_shares(blocks, dw.K) ? 2 : 1;
}

hipError_t launch_gemm_bf16_pair(GemmBf16Args dw, GemmKind kind, GemmBf16Args next, hipStream_t stream, const LaunchEvents &ev)
{
    const int groups = gemm_bf16_pair_groups(dw, kind, next);
    if (groups == 0) return hipErrorInvalidValue;
    next.colsum_partial = nullptr;
    const long long n_dw = mid_tiles(dw, 64) + (dw.fin.n > 0 ? 1 : 0);
    const long long blocks = n_dw + mid_tiles(next, 64) + (kind == GEMM_DW && next.fin.n > 0 ? 1 : 0);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const bool two = groups == 2;
    const auto kernel = kind == GEMM_DA ? (two ? gemm_bf16_mid_pair_kernel<2, GEMM_DA> : gemm_bf16_mid_pair_kernel<1, GEMM_DA>)
                                        : (two ? gemm_bf16_mid_pair_kernel<2, GEMM_DW> : gemm_bf16_mid_pair_kernel<1, GEMM_DW>);
    return launch_kernel(kernel, dim3((unsigned)blocks), dim3(two ? 2 * NT : NT), stream, ev, dw, next, (int)n_dw);
}

int gemm_bf16_dw_form(int M, int N, int K, long long lda, long long ldb, const void *A, const void *B)
{
    const size_t base = reinterpret_cast<size_t>(A) | reinterpret_cast<size_t>(B);
    // 32-bit byte offsets over the k-rows of a tile (64 rows of up to 2^24 values, the widest layer there is), and whole
    // column pairs in every row
    if (((lda | ldb) & 1) || (base & 3) || lda < M + (M & 1) || ldb < N + (N & 1) || lda > (1ll << 24) ||
        ldb > (1ll << 24))
        return BF16_DW_KMAJ;
    // the LDS-direct kernel: 16-byte rows, and a product it is chosen for (split over the batch,
    // or at least 128 tiles)
    const long long tiles = (long long)((M + DMA_BM - 1) / DMA_BM) * ((N + DMA_BN - 1) / DMA_BN);
    static const int forced = env_int_bf16("HB_BF16_TILE", 0);
    if (tiles >= 128 || forced == 1 || gemm_bf16_dw_splits_cap(M, N, K) > 1)
        return ((lda | ldb) & 7) || (base & 15) || (forced == 1 && tiles < 128 && gemm_bf16_dw_splits_cap(M, N, K) < 2)
                   ? BF16_DW_KMAJ
                   : BF16_DW_BMAJ;
    return BF16_DW_BMAJ_MID;
}

int gemm_bf16_dw_splits_cap(int M, int N, int K)
{
    const long long tiles = (long long)((M + DMA_BM - 1) / DMA_BM) * ((N + DMA_BN - 1) / DMA_BN);
    if (tiles > 128 || K < 2048) return 1;
    long long s = 256 / tiles;  // fill the chip once
    if (s > 8) s = 8;
    if (s > K / 1024) s = K / 1024;  // at least 16 k-tiles per slice
    // With fewer workgroups than half of the compute units, the kernel of small tiles is faster on the whole
    // contraction: its time grows with the contraction, that of the slices hardly does, but these are
    // followed by the passes over their sums and the bias.  The lines are where the two met while every product had a launch
    // of its own; now that a weight gradient of small tiles shares its launch with the next product, they meet beyond.
    // Steps, small tiles / slices, us: 64-w-w-10, w = 256 93 / 184 at 7001 rows, 100 / 184 at 8001, 292 / 370 at 30000; 768
    // 144 / 227 at 7501; 1024 174 / 249 at 7001, 181 / 247 at 7501; 64-1280x4-10 335 / 453 at 4096 rows, 382 / 492 at 5121,
    // 419 / 530 at 5999, 730 / 742 at 12001; 54-512x4-7 233 / 336 at 8192.
    const long long small = (long long)((M + 63) / 64) * ((N + 63) / 64);
    return (s < 2 || (tiles * s < 128 && K < (small <= 256 ? 7500 : 5120))) ? 1 : (int)s;
}

int gemm_bf16_dw_splits(int M, int N, int K, long long lda, long long ldb)
{
    // the LDS-direct kernel (the only one that splits) addresses each operand with 32-bit byte
    // offsets: an operand beyond 4 GiB is not split.  This makes the count non-monotonic in K
    // (lda and ldb grow with the batch), which is why buffers are sized with ..._cap.
    if ((unsigned long long)M * (unsigned long long)lda * 2 >= (1ull << 32) ||
        (unsigned long long)N * (unsigned long long)ldb * 2 >= (1ull << 32) || (lda & 7) || (ldb & 7))
        return 1;
    return gemm_bf16_dw_splits_cap(M, N, K);
}

hipError_t launch_dw_reduce(const float *partial, int splits, long long stride, long long count, float *master,
                            float *grad, float lr, hipStream_t stream, const LaunchEvents &ev)
{
    if (count <= 0) return hipSuccess;
    const long long n4 = (count + 3) / 4;
    long long blocks = (n4 + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    return launch_kernel(dw_reduce_kernel, dim3((unsigned)blocks), dim3(256), stream, ev, partial, splits, stride,
                         count, master, grad, lr);
}

hipError_t launch_transpose_bf16(const void *in, long long ldi, void *out, long long ldo, int R, int C,
                                 hipStream_t stream, const LaunchEvents &ev)
{
    const int vec_ok = (ldi % 8 == 0) && (ldo % 8 == 0) && ((reinterpret_cast<size_t>(in) & 15) == 0) &&
                       ((reinterpret_cast<size_t>(out) & 15) == 0);
    return launch_kernel(transpose_bf16_kernel, dim3((unsigned)((C + 63) / 64), (unsigned)((R + 63) / 64)),
                         dim3(256), stream, ev, static_cast<const bf16_t *>(in), ldi, static_cast<bf16_t *>(out),
                         ldo, R, C, vec_ok);
}

hipError_t launch_shadow(const float *W, int R, int C, void *shadow, long long lds_, void *shadow_t,
                         long long ldt, hipStream_t stream)
{
    return launch_kernel(shadow_kernel, dim3((unsigned)((C + 63) / 64), (unsigned)((R + 63) / 64)), dim3(256),
                         stream, LaunchEvents(), W, R, C, static_cast<bf16_t *>(shadow), lds_,
                         static_cast<bf16_t *>(shadow_t), ldt);
}

int colsum_bias_slices(long long B)
{
    long long s = (B + 63) / 64;  // at least 64 rows per slice
    if (s > CSB_MAX_SLICES) s = CSB_MAX_SLICES;
    return s < 1 ? 1 : (int)s;
}

hipError_t launch_colsum_bias_finalize(const float *partial, int slices, int d, float *bias, float *grad, float lr,
                                       hipStream_t stream, const LaunchEvents &ev)
{
    return launch_kernel(colsum_bias_finalize_kernel, dim3((unsigned)((d + 63) / 64)), dim3(256), stream, ev,
                         partial, slices, d, bias, grad, lr);
}

hipError_t launch_colsum_bias(const void *D, long long ld, int d, long long B, float *partial, float *bias,
                              float *grad, float lr, hipStream_t stream, const LaunchEvents &ev)
{
    if ((ld & 7) != 0 || (reinterpret_cast<size_t>(D) & 15) != 0 || B <= 0) return hipErrorInvalidValue;
    const int slices = colsum_bias_slices(B);
    const int rows_per_slice = (int)((B + slices - 1) / slices);
    hipError_t e = launch_kernel(colsum_bf16_kernel, dim3((unsigned)((ld + CSB_COLS - 1) / CSB_COLS), (unsigned)slices),
                                 dim3(256), stream, ev, static_cast<const bf16_t *>(D), ld, d, B, rows_per_slice,
                                 partial);
    if (e != hipSuccess) return e;
    return launch_kernel(colsum_bias_finalize_kernel, dim3((unsigned)((d + 63) / 64)), dim3(256), stream,
                         LaunchEvents(), static_cast<const float *>(partial), slices, d, bias, grad, lr);
}

hipError_t launch_rowsum_bias(const void *Dt, long long ld, int d, long long B, float *bias, float *grad,
                              float lr, hipStream_t stream, const LaunchEvents &ev)
{
    return launch_kernel(rowsum_bias_kernel, dim3((unsigned)((d + 3) / 4)), dim3(256), stream, ev,
                         static_cast<const bf16_t *>(Dt), ld, d, B, bias, grad, lr);
}

}  // namespace hb
