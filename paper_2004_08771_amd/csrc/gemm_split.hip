// The dense fp32 products on the bf16 matrix cores, for products large enough to fill the device
// (smaller ones: gemm_f32.hip).
//
// Every fp32 operand value is split, on its way from registers to LDS, into three bf16 values
// x = x0 + x1 + x2 (leading part rounded to nearest, then the leading part of the exact remainder,
// then the rest, which fits: 3 x 8 significand bits), and the product becomes six bf16 MFMAs
//     x0 y0  +  (x0 y1 + x1 y0 + x1 y1 + x0 y2 + x2 y0)
// whose two groups have accumulators of their own and meet after the loop.  The terms left out,
// x1 y2 + x2 y1, reach 2^-24 of |x y| (significands just above 1: |x1| up to 2^-8, |x2| up to 2^-17) and are
// 2^-28 in the mean square.  The bf16 MFMA does 16 times the flop of the fp32 one per clock, so six of
// them are 2.7 times as fast, and their sums are more exact: bf16 products are exact in fp32, 16 of
// them are added per rounding, and the group of the small terms does not round at the size of
// the large one.  Against 64 bits (relative 2-norm of contractions of normal values, 8 / 54 / 512 / 4096
// deep): fp32 MFMA 5.4e-8 / 9.9e-8 / 2.9e-7 / 8.1e-7, this 2.9e-8 / 4.7e-8 / 1.3e-7 / 4.0e-7, all six in one
// accumulator 3.4e-7 at 512, three terms only 4.4e-6.  Where a sum is a single product the roundings
// that this saves do not exist and the left out terms show (largest error 1.0e-7 against 6.0e-8, rms 2.60e-8
// against 2.53e-8): a contraction of one k-tile gets them too (8 MFMAs, 6.0e-8; its launch is bound by
// latency).  In all contractions they would cost 4096 x 512 steps 171 -> 190 us.  bf16 has fp32's exponent range but only 8 significand bits, so the last part of
// a value below 2^-110 would fall under its smallest denormal: every value is multiplied by 2^24
// first, which makes the split exact for all fp32 values down to the denormals (operands of 2^-118:
// error 8.8e-6 -> 4.9e-8; one instruction per value, 4096 x 512 forward + backward steps 167 -> 171 us), and the sum
// by 2^-48 at the end.  A value without a finite x0 -- infinite, NaN, or of 2^104 and more -- makes the
// planes NaN: a wavefront that finds a non-finite result (also a sum of 2^80 and more) computes its tile
// again with fp32 MFMAs from the operands in memory, unless a NaN among the first values of its
// operands' rows explains it.  (54-512x4-7, B = 4096: step with all weights NaN 162 us, as with finite ones,
// and 869 when every block was computed again behind loads that nothing covered; gradient with all of W_2
// infinite 257 us, 421 before, 262 on fp32 MFMAs alone.)
//
// What bounds it: power, then the instruction stream.  With nothing but the MFMAs of
// 4096 x 1024 x 1024 in the loop the launch takes 33 us (clock 2.05 GHz); the whole kernel takes 47 us (45 without the scale) at
// 1.7 GHz and 2000 clocks per k-tile of a 128 x 128 tile, against 1536 of MFMA (fp32 MFMA kernel: 73 us).
// Hence: the largest tile that still gives every compute unit a workgroup (fewer operand bytes
// loaded, converted and read back per flop), eight wavefronts (one wavefront on a SIMD issues
// about five instructions in the shadow of an MFMA, and the conversion needs more: the same tile with
// four wavefronts of 64 x 64 takes 49 us), fp32 in memory (planes written by the producer would be
// 6 bytes per value through an L1 path of 64 B/clk that is already a third busy), no dot2 for the
// remainders (one instruction instead of two, but it does not run beside an MFMA).
#include "gemm_device.h"

#include <stdlib.h>

#include <type_traits>

namespace hb {
namespace {

typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));

constexpr int BK = 32;   // contraction per tile
constexpr int SETS = 2;  // register sets of loaded tiles
constexpr float SCALE = 16777216.f;  // on every operand value: 2^-149, the last bit of any, becomes a bf16 value

__device__ __forceinline__ unsigned cvt_pk_bf16(float a, float b)
{
    // through the compiler, not as asm: it has to see the wait states that a dot product's result needs
    const v2f x = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(x, v2bf));
}

// x - (low / high half of the bf16 pair u), exact.  (A dot product with {-1, 0} would be one
// instruction instead of two, but it does not run beside the matrix instructions.)
__device__ __forceinline__ float minus_lo(unsigned u, float x) { return x - __uint_as_float(u << 16); }
__device__ __forceinline__ float minus_hi(unsigned u, float x) { return x - __uint_as_float(u & 0xffff0000u); }

typedef unsigned v2u __attribute__((ext_vector_type(2)));
// N floats at (wavefront-uniform base) + (byte offset of the lane), any 4-byte alignment
template <int N>
__device__ __forceinline__ void load_lane(float *x, const float *base, unsigned off)
{
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), (short)0, -1, 0x00027000);
    if (N == 4) {
        const v4u t = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = __uint_as_float(t[c]);
    } else if (N == 2) {
        const v2u t = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
#pragma unroll
        for (int c = 0; c < 2; ++c) x[c] = __uint_as_float(t[c]);
    } else {
        x[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
    }
}

// One operand tile of ROWS rows x BK: global -> registers (fp32) -> three bf16 planes in LDS.  A
// plane has 64-byte rows of 32 k, the 16-byte slots of a row exchanged (swz) so that the 16 rows that a
// fragment read or a K-major write touches together lie on different banks.  An M-major operand is
// transposed on the way: a thread holds four k of MV neighbouring rows, packs each row's four k
// and writes row m to LDS row m / MV + R1 (m % MV), so that the lanes write consecutive LDS rows.
template <int NT, int ROWS, bool KMAJ>
struct Op {
    static constexpr int MV = ROWS * 8 / NT;  // quads of four k per thread
    static constexpr int R1 = NT / 8;         // rows (groups of MV rows) that the threads cover at once
    static constexpr int PLANE = ROWS * 64;   // bytes of one plane: 64-byte rows of 32 bf16
    static constexpr int BYTES = 3 * PLANE;

    // row of the tile -> row in LDS
    static __device__ __forceinline__ int phys(int m) { return KMAJ ? m : m / MV + R1 * (m % MV); }
    static __device__ __forceinline__ int swz(int p)
    {
        if (KMAJ || MV == 1) return (p >> 2) & 3;
        return (MV == 4) ? ((p >> 2) ^ (p / R1)) & 3 : ((p >> 2) ^ ((p / R1) << 1)) & 3;
    }

    // How a whole k-tile is loaded: 16-byte (8-byte) loads at any 4-byte alignment, or, where an M-major
    // tile is cut by the end of the matrix, single values with the row clamped to the last one.
    float x[SETS][4 * MV];  // KMAJ: [4 v + c] = (row r + 32 v, k = 4 kq + c);  else [MV q + e] = (row MV i + e, k = 4 j + q)
    unsigned off[MV];       // byte offsets of the lane (every one below 2^32 for rows of up to 2^24 floats)

    template <bool VEC>
    __device__ __forceinline__ void init(int ld, int last_row, int tid)
    {
        if (KMAJ) {
            const int kq = tid & 7, r = tid >> 3;
#pragma unroll
            for (int v = 0; v < MV; ++v)
                off[v] = (unsigned)(min(r + R1 * v, last_row) - min(R1 * v, last_row)) * (unsigned)ld * 4u + kq * 16u;
        } else {
            const int i = tid % R1, j = tid / R1;
#pragma unroll
            for (int e = 0; e < MV; ++e)
                off[e] = (unsigned)(4 * j) * (unsigned)ld * 4u + 4u * (unsigned)(VEC ? MV * i : min(MV * i + e, last_row));
        }
    }
    // piece v of LOADS of a tile that is whole along k; tile: its first element
    static constexpr int LOADS = KMAJ ? MV : 4;
    template <bool VEC>
    __device__ __forceinline__ void load(int set, int v, const float *__restrict__ tile, int ld, int last_row)
    {
        if (KMAJ) {
            load_lane<4>(&x[set][4 * v], tile + (size_t)min(R1 * v, last_row) * ld, off[v]);
        } else if (VEC) {
            load_lane<MV>(&x[set][MV * v], tile + (size_t)v * ld, off[0]);
        } else {
#pragma unroll
            for (int e = 0; e < MV; ++e) load_lane<1>(&x[set][MV * v + e], tile + (size_t)v * ld, off[e]);
        }
    }
    // a partial k-tile: everything outside [0, nrows) x [.., kend) reads as zero
    __device__ __forceinline__ void load_tail(int set, const float *__restrict__ P, int ld, int row0, int nrows, int k0,
                                              int kend, int tid)
    {
        if (KMAJ) {
            const int kq = tid & 7, r = tid >> 3;
#pragma unroll
            for (int v = 0; v < MV; ++v) {
                const int row = row0 + r + R1 * v, k = k0 + 4 * kq;
                const float *p = P + (size_t)row * ld + k;
#pragma unroll
                for (int c = 0; c < 4; ++c) x[set][4 * v + c] = (row < nrows && k + c < kend) ? p[c] : 0.f;
            }
        } else {
            const int i = tid % R1, j = tid / R1;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int k = k0 + 4 * j + q, row = row0 + MV * i;
                const float *p = P + (size_t)k * ld + row;
#pragma unroll
                for (int e = 0; e < MV; ++e) x[set][MV * q + e] = (k < kend && row + e < nrows) ? p[e] : 0.f;
            }
        }
    }
    // plane pl of quad u: the leading bf16 part goes to LDS, the remainder stays in the registers
    __device__ __forceinline__ void split_store(int set, char *S, int u, int pl, int tid)
    {
        auto &x0 = x[set][KMAJ ? 4 * u : u], &x1 = x[set][KMAJ ? 4 * u + 1 : MV + u],
             &x2 = x[set][KMAJ ? 4 * u + 2 : 2 * MV + u], &x3 = x[set][KMAJ ? 4 * u + 3 : 3 * MV + u];
        const int kq = KMAJ ? tid & 7 : tid / R1, p = (KMAJ ? tid >> 3 : tid % R1) + R1 * u;
        if (pl == 0) {
            x0 *= SCALE;
            x1 *= SCALE;
            x2 *= SCALE;
            x3 *= SCALE;
        }
        uint2 w;
        w.x = cvt_pk_bf16(x0, x1);
        w.y = cvt_pk_bf16(x2, x3);
        if (pl < 2) {
            x0 = minus_lo(w.x, x0);
            x1 = minus_hi(w.x, x1);
            x2 = minus_lo(w.y, x2);
            x3 = minus_hi(w.y, x3);
        }
        *reinterpret_cast<uint2 *>(S + p * 64 + (((kq >> 1) ^ swz(p)) << 4) + ((kq & 1) << 3) + pl * PLANE) = w;
    }
    // byte offset of the 8 k (8 h .. 8 h + 7) of tile row m in the first 16-deep step; the second: ^ 32
    static __device__ __forceinline__ int frag_off(int m, int h)
    {
        const int p = phys(m);
        return p * 64 + ((h ^ swz(p)) << 4);
    }
};

// One 32 x 32 block on fp32 MFMAs from the operands in memory, for one wavefront, the k-tile ahead while the MFMAs of
// the present one run.  Rare: sums that are infinite or beyond 2^80.
template <typename RA, typename RB>
__device__ __forceinline__ v16f fp32_block(const RA &ra, const RB &rb, int kbeg, int kend)
{
    v16f acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    float xa[2][BK / 2], xb[2][BK / 2];
    auto load = [&](int set, int k0) {
#pragma unroll
        for (int q = 0; q < BK / 8; ++q) {
            ra.template load<true>(xa[set], q, k0, kend);
            rb.template load<true>(xb[set], q, k0, kend);
        }
    };
    auto mfma = [&](int set) {
#pragma unroll
        for (int q = 0; q < BK / 2; ++q)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[set][q], xb[set][q], acc, 0, 0, 0);
    };
    const int whole = (kend - kbeg) / BK;  // k-tiles
    if (whole > 0) load(0, kbeg);
#pragma unroll 1
    for (int t = 0; t < whole; t += 2) {
        if (t + 1 < whole) load(1, kbeg + (t + 1) * BK);
        mfma(0);
        if (t + 1 < whole) {
            if (t + 2 < whole) load(0, kbeg + (t + 2) * BK);
            mfma(1);
        }
    }
    if (kbeg + whole * BK < kend) {
#pragma unroll
        for (int q = 0; q < BK / 8; ++q) {
            ra.template load<false>(xa[0], q, kbeg + whole * BK, kend);
            rb.template load<false>(xb[0], q, kbeg + whole * BK, kend);
        }
        mfma(0);
    }
    return acc;
}
// bit m: one of the first eight values of row m of a block is NaN (row: the lane's, m = lane % 32)
template <bool KMAJ>
__device__ __forceinline__ unsigned nan_rows(const float *__restrict__ P, int ld, int row, int kbeg, int kend, int h)
{
    bool nan = false;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int k = min(kbeg + 4 * h + c, kend - 1);
        const float x = KMAJ ? P[(size_t)row * ld + k] : P[(size_t)k * ld + row];
        nan |= x != x;
    }
    const unsigned long long w = __ballot(nan);
    return (unsigned)(w | (w >> 32));
}

template <int BM, int BN>
constexpr int lds_bytes()
{
    return 2 * 3 * 64 * (BM + BN);
}

// One output tile (index id in n-fastest order) of one K-slice (split) of C = A . B^T.
// KG: groups of NT threads that share the contraction (group g takes the k-tiles g, g + KG, .. from LDS
// stages of its own); their sums meet in LDS, in group order, and group 0 finishes the tile.
template <int NT, int KG, int BM, int BN, int WAVES_M, bool A_KMAJ, bool B_KMAJ, int KIND>
__device__ __forceinline__ void split_tile(const GemmArgs &a, char *smem, int id, int split)
{
    constexpr int WAVES_N = NT / 64 / WAVES_M;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int TM = WM / 32, TN = WN / 32;
    using OA = Op<NT, BM, A_KMAJ>;
    using OB = Op<NT, BN, B_KMAJ>;
    constexpr int STAGE = OA::BYTES + OB::BYTES;

    const int tid = threadIdx.x % NT;
    const int lane = tid & 63, wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = wave_all / (NT / 64), wave = wave_all % (NT / 64);
    const int r = lane & 31, h = lane >> 5;
    const int wm = wave % WAVES_M, wn = wave / WAVES_M;
    char *const smem_all = smem;
    smem += g * 2 * STAGE;

    const int tile_m = id / a.tiles_n, tile_n = id - tile_m * a.tiles_n;
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int kbeg = split * a.k_chunk;
    const int kend = min(a.K, kbeg + a.k_chunk);
    const int nk_all = (kend - kbeg + BK - 1) / BK;

    const float *__restrict__ A = static_cast<const float *>(a.A);
    const float *__restrict__ Bm = static_cast<const float *>(a.B);

    // hi: the products of the leading parts; lo: the five cross products
    v16f hi[TM][TN], lo[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) hi[i][j][v] = lo[i][j][v] = 0.f;

    const bool a_in = (m0 + BM <= a.M), b_in = (n0 + BN <= a.N);

    // forward: the lane's bias values are requested now, not after the main loop
    float bias_pre[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = n0 + wn * WN + j * 32 + r;
        bias_pre[j] = (KIND == GEMM_FWD && a.bias != nullptr && n < a.N) ? a.bias[n] : 0.f;
    }

    // DW only: column sums of the A tile (the bias gradient) by the blocks of the first tile column,
    // from the fp32 values in the staging registers
    const bool do_colsum = (KIND == GEMM_DW) && a.colsum != nullptr && tile_n == 0;
    float csum[OA::MV];
#pragma unroll
    for (int e = 0; e < OA::MV; ++e) csum[e] = 0.f;

    int fa_off[TM], fb_off[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) fa_off[i] = OA::frag_off(wm * WM + i * 32 + r, h);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb_off[j] = OA::BYTES + OB::frag_off(wn * WN + j * 32 + r, h);

    OA oa;  // two register sets: tile kt + 1 is split and written while tile kt + 2 is in flight
    OB ob;
    v8bf fa[2][TM][3], fb[2][TN][3];
    constexpr int READS = 3 * (TM + TN), MF = TM * TN, NM = 6 * MF;  // fragment reads and MFMAs of one 16-deep step
    auto read_frag = [&](int slot, const char *S, int step, int i) {
        const int pl = i / (TM + TN), b = i % (TM + TN);
        if (b < TM)
            fa[slot][b][pl] = *reinterpret_cast<const v8bf *>(S + (fa_off[b] ^ (step << 5)) + pl * OA::PLANE);
        else
            fb[slot][b - TM][pl] = *reinterpret_cast<const v8bf *>(S + (fb_off[b - TM] ^ (step << 5)) + pl * OB::PLANE);
    };
    auto read_frags = [&](int slot, const char *S, int step) {
#pragma unroll
        for (int i = 0; i < READS; ++i) read_frag(slot, S, step, i);
    };
    auto mfma = [&](int slot, int i) {
        constexpr int PA[8] = {0, 0, 1, 1, 0, 2, 1, 2}, PB[8] = {0, 1, 0, 1, 2, 0, 2, 1};
        const int q = i / MF, bi = (i % MF) / TN, bj = (i % MF) % TN;
        v16f &acc = (q == 0) ? hi[bi][bj] : lo[bi][bj];
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[slot][bi][PA[q]], fb[slot][bj][PB[q]], acc, 0, 0, 0);
    };
    constexpr int QA = OA::MV, QB = OB::MV, PIECES = 3 * (QA + QB);
    auto split_piece = [&](int set, char *S, int c, bool counts) {
        const int u = c / 3, pl = c % 3;
        if (u < QA) {
            if (KIND == GEMM_DW && pl == 0 && do_colsum && counts) {
#pragma unroll
                for (int q = 0; q < 4; ++q) csum[u] += oa.x[set][QA * q + u];
            }
            oa.split_store(set, S, u, pl, tid);
        } else {
            ob.split_store(set, S + OA::BYTES, u - QA, pl, tid);
        }
    };
    // A partial last k-tile goes first (tile 0 of the loop below); all others are whole.
    const int nk_full = (kend - kbeg) / BK, tail = nk_all - nk_full;
    const int rounds = (nk_all + KG - 1) / KG, nk = (nk_all - g + KG - 1) / KG;  // k-tiles of group 0, of this group
    auto main_loop = [&](auto a_vec, auto b_vec) {
        constexpr bool AV = decltype(a_vec)::value != 0, BV = decltype(b_vec)::value != 0;
        const int a_last = a.M - 1 - m0, b_last = a.N - 1 - n0;
        oa.template init<AV>(a.lda, a_last, tid);
        ob.template init<BV>(a.ldb, b_last, tid);
        const float *At = A_KMAJ ? A + (size_t)m0 * a.lda + kbeg : A + (size_t)kbeg * a.lda + m0;
        const float *Bt = B_KMAJ ? Bm + (size_t)n0 * a.ldb + kbeg : Bm + (size_t)kbeg * a.ldb + n0;
        const size_t a_step = A_KMAJ ? (size_t)BK : (size_t)BK * a.lda, b_step = B_KMAJ ? (size_t)BK : (size_t)BK * a.ldb;
        constexpr int LOADS = OA::LOADS + OB::LOADS;
        auto load_piece = [&](int set, int t, int v) {  // past the end: the last tile again (not used)
            const int f = max(g + min(t, nk - 1) * KG - tail, 0);
            if (v < OA::LOADS) oa.template load<AV>(set, v, At + f * a_step, a.lda, a_last);
            else ob.template load<BV>(set, v - OA::LOADS, Bt + f * b_step, a.ldb, b_last);
        };
        auto load_whole = [&](int set, int t) {
#pragma unroll
            for (int v = 0; v < LOADS; ++v) load_piece(set, t, v);
        };
        if (tail && g == 0) {
            oa.load_tail(0, A, a.lda, m0, a.M, kbeg + nk_full * BK, kend, tid);
            ob.load_tail(0, Bm, a.ldb, n0, a.N, kbeg + nk_full * BK, kend, tid);
        } else {
            load_whole(0, 0);
        }
        // nk > 1 also means that there is a whole tile to read (a lone partial one must not be read as whole)
        if (nk > 1) {
#pragma unroll
            for (int t = 1; t < SETS; ++t) load_whole(t, t);
        }
#pragma unroll
        for (int p = 0; p < PIECES; ++p) split_piece(0, smem, p, true);
        if (nk > 1) {
            load_whole(0, SETS);
#pragma unroll
            for (int p = 0; p < PIECES / 2; ++p) split_piece(1, smem + STAGE, p, true);
        }
        __syncthreads();
        read_frags(0, smem, 0);
        int kt = 0;
        auto round = [&](int c, bool more) {  // more: a tile kt + 2 is prepared (past the end: the last one again, not used)
            // Tile kt is in stage c % 2.  First half: the second half of tile kt + 1 goes to the other
            // stage.  Second half, behind the barrier, when the fragments of tile kt have all been
            // read: the first half of tile kt + 2 goes to stage c.  Every memory operation and
            // every piece of the conversion has its place behind an MFMA.
            const int s1 = (c + 1) % SETS, s2 = (c + 2) % SETS;  // register sets of tiles kt + 1, kt + 2
            char *S = smem + (c & 1) * STAGE, *N = smem + ((c + 1) & 1) * STAGE;
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                mfma(0, i);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int f = 0; f < READS; ++f)
                    if (f * (2 * NM / 3) / READS == i) read_frag(1, S, 1, f);
#pragma unroll
                for (int p = PIECES / 2; p < PIECES; ++p)
                    if ((p - PIECES / 2) * NM / (PIECES - PIECES / 2) == i) split_piece(s1, N, p, true);
#pragma unroll
                for (int v = 0; v < OA::LOADS; ++v)
                    if (more && NM / 3 + v * (2 * NM / 3) / OA::LOADS == i) load_piece(s1, kt + 1 + SETS, v);
                __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();
            const bool two = kt + 2 < nk;
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                mfma(1, i);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int f = 0; f < READS; ++f)
                    if (f * (2 * NM / 3) / READS == i) read_frag(0, N, 0, f);
#pragma unroll
                for (int p = 0; p < PIECES / 2; ++p)
                    if (more && p * NM / (PIECES / 2) == i) split_piece(s2, S, p, two);
#pragma unroll
                for (int v = 0; v < OB::LOADS; ++v)
                    if (more && v * NM / OB::LOADS == i) load_piece(s1, kt + 1 + SETS, OA::LOADS + v);
                __builtin_amdgcn_sched_barrier(0);
            }
            ++kt;
        };
        // Whole turns of the register sets: where a way out in between reaches the head of the loop as well, the compiler
        // cannot tell how many loads are in flight there and waits for all of them in every second k-tile (3001 x 1024 x 1024
        // forward 40.8 -> 37.9 us, backward 78.0 -> 75.7; 3000 x 700 x 700 31.3 -> 28.7, 46.7 -> 45.9).
        while (kt + 2 < nk) {
            round(0, true);
            round(1, true);
        }
        if (kt + 1 < nk) round(0, false);
        const bool lone = nk_all == 1, half = lone && kend - kbeg <= BK / 2;  // half: the second 16-deep step is zero
        // (8192 x 8192 weight gradient over 16 rows: 78 -> 70 us)
        if (!half) read_frags(1, smem + (kt & 1) * STAGE, 1);
#pragma unroll
        for (int i = 0; i < NM; ++i) mfma(0, i);
        if (lone) {  // the terms left out
#pragma unroll
            for (int i = NM; i < NM + 2 * MF; ++i) mfma(0, i);
        }
        if (!half) {
#pragma unroll
            for (int i = 0; i < NM; ++i) mfma(1, i);
            if (lone) {
#pragma unroll
                for (int i = NM; i < NM + 2 * MF; ++i) mfma(1, i);
            }
        }
    };
    if (nk > 0) {
        if ((A_KMAJ || a_in) && (B_KMAJ || b_in)) main_loop(IntC<1>(), IntC<1>());
        else main_loop(IntC<A_KMAJ>(), IntC<B_KMAJ>());
    }
    // a group with one k-tile less has passed one barrier less
    if (KG > 1 && nk < rounds) __syncthreads();

    if (KIND == GEMM_DW) {
        if (do_colsum) {  // uniform per workgroup
            __syncthreads();  // the last tile's fragments have been read
            float *red = reinterpret_cast<float *>(smem_all);
#pragma unroll
            for (int e = 0; e < OA::MV; ++e) red[(8 * g + tid / OA::R1) * BM + (tid % OA::R1) * OA::MV + e] = csum[e];
            __syncthreads();
            if (g == 0 && tid < BM && m0 + tid < a.M) {
                float s = red[tid];
#pragma unroll
                for (int q = 1; q < 8 * KG; ++q) s += red[q * BM + tid];
                a.colsum[(size_t)split * a.M + m0 + tid] = s;
            }
        }
    }

#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) hi[i][j][v] = (hi[i][j][v] + lo[i][j][v]) * (1.f / SCALE / SCALE);
    if constexpr (KG > 1) {
        static_assert(TM == 1 && TN == 1, "one block per wavefront");
        float *red = reinterpret_cast<float *>(smem_all);
        __syncthreads();  // the stages (the column sums) have been read
        if (g > 0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) red[(((g - 1) * (NT / 64) + wave) * 16 + v) * 64 + lane] = hi[0][0][v];
        }
        __syncthreads();
        if (g > 0) return;
#pragma unroll
        for (int q = 0; q < KG - 1; ++q)
#pragma unroll
            for (int v = 0; v < 16; ++v) hi[0][0][v] += red[((q * (NT / 64) + wave) * 16 + v) * 64 + lane];
    }
    float bad = 0.f;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) bad = fmaf(hi[i][j][v], 0.f, bad);
    if (__any(bad != 0.f) && kbeg < kend) {  // NaN: some result of this wavefront is not finite
        // A row whose first values hold a NaN (all of them, once the weights of a run are NaN) has a NaN in
        // every result in either arithmetic: only the other results that are not finite ask for the second one.
        auto row_a = [&](int i) { return min(m0 + wm * WM + i * 32 + r, a.M - 1); };
        auto row_b = [&](int j) { return min(n0 + wn * WN + j * 32 + r, a.N - 1); };
        unsigned nan_a[TM], nan_b[TN], again = 0;
#pragma unroll
        for (int i = 0; i < TM; ++i) nan_a[i] = nan_rows<A_KMAJ>(A, a.lda, row_a(i), kbeg, kend, h);
#pragma unroll
        for (int j = 0; j < TN; ++j) nan_b[j] = nan_rows<B_KMAJ>(Bm, a.ldb, row_b(j), kbeg, kend, h);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                unsigned open = 0;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = 8 * (v >> 2) + 4 * h + (v & 3);
                    open |= (hi[i][j][v] * 0.f != 0.f) ? ~(nan_a[i] >> row) & 1u : 0u;
                }
                if (__any(open & ~(nan_b[j] >> r) & 1u)) again |= 1u << (i * TN + j);
            }
#pragma unroll 1
        for (int b = 0; b < TM * TN; ++b) {
            if (!((again >> b) & 1u)) continue;  // uniform per wavefront
            const Fp32Rows<A_KMAJ> ra(A, a.lda, m0 + wm * WM + (b / TN) * 32, a.M - 1, r, h);
            const Fp32Rows<B_KMAJ> rb(Bm, a.ldb, n0 + wn * WN + (b % TN) * 32, a.N - 1, r, h);
            const v16f acc = fp32_block(ra, rb, kbeg, kend);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    if (i * TN + j == b) hi[i][j] = acc;
        }
    }

    // ---- epilogue.  hi[i][j][v] is C(row, col) with row = 8 (v / 4) + 4 h + (v % 4), col = r inside
    // its 32 x 32 block.
    float *__restrict__ C = static_cast<float *>(a.C) + (size_t)split * a.c_split_stride;
    const float *__restrict__ aux = static_cast<const float *>(a.aux);
    auto epilogue = [&](auto act_c) {
        constexpr int ACT = decltype(act_c)::value;
        auto finish = [&](float x, float bias, float o) {
            if (KIND == GEMM_FWD) {
                x += bias;
                if (ACT == ACT_SIGMOID) x = sigmoidf_fast(x);
                else if (ACT == ACT_RELU) x = fmaxf(x, 0.f);
            } else if (KIND == GEMM_DA) {
                if (ACT == ACT_SIGMOID) x *= o * (1.f - o);
                else if (ACT == ACT_RELU) x = (o > 0.f) ? x : 0.f;
            }
            return x;
        };
        if (a_in && b_in) {
            const unsigned lo_c = (unsigned)(4 * h * a.ldc + r), lo_x = (unsigned)(4 * h * a.ldaux + r);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int nb = n0 + wn * WN + j * 32;  // uniform
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const int mbu = m0 + wm * WM + i * 32;
                    float o[16];
                    if (KIND == GEMM_DA) {
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            o[v] = (aux + ((size_t)(mbu + 8 * (v >> 2) + (v & 3)) * a.ldaux + nb))[lo_x];
                    }
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        (C + ((size_t)(mbu + 8 * (v >> 2) + (v & 3)) * a.ldc + nb))[lo_c] =
                            finish(hi[i][j][v], bias_pre[j], KIND == GEMM_DA ? o[v] : 0.f);
                }
            }
            return;
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + wn * WN + j * 32 + r;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int m = m0 + wm * WM + i * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
                    if (m < a.M && n < a.N)
                        C[(size_t)m * a.ldc + n] =
                            finish(hi[i][j][v], bias_pre[j], KIND == GEMM_DA ? aux[(size_t)m * a.ldaux + n] : 0.f);
                }
        }
    };
    with_activation(KIND == GEMM_DW ? (int)ACT_NONE : a.act, epilogue);
}

template <int NT, int KG, int BM, int BN, int WM, int WGS, bool A_KMAJ, bool B_KMAJ, int KIND>
__global__ __launch_bounds__(NT *KG, WGS) void gemm_split_kernel(GemmArgs a)
{
    __shared__ __attribute__((aligned(16))) char smem[KG * lds_bytes<BM, BN>()];
    split_tile<NT, KG, BM, BN, WM, A_KMAJ, B_KMAJ, KIND>(a, smem, xcd_tile_order(blockIdx.x, gridDim.x), blockIdx.y);
}

// Backward of one hidden layer in one launch (see launch_gemm_f32_bwd_pair).
template <int NT, int KG, int BM, int BN, int WM, int WGS>
__global__ __launch_bounds__(NT *KG, WGS) void gemm_split_pair_kernel(GemmArgs da, GemmArgs dw, int n_dw)
{
    __shared__ __attribute__((aligned(16))) char smem[KG * lds_bytes<BM, BN>()];
    const int b = blockIdx.x;
    if (b < n_dw) {
        // Workgroup ids go round-robin over the 8 XCDs, each with an L2 of its own: an XCD gets a contiguous
        // eighth of the (slice, tile) pairs, so that it reads only its slices' rows of D_l and A_{l-1}, once;
        // the backward-data blocks below give it (nearly) the same rows.
        const int tiles = dw.tiles_m * dw.tiles_n, w = xcd_tile_order(b, n_dw);
        split_tile<NT, KG, BM, BN, WM, false, false, GEMM_DW>(dw, smem, w % tiles, w / tiles);
    } else {
        split_tile<NT, KG, BM, BN, WM, true, false, GEMM_DA>(da, smem, xcd_tile_order(b - n_dw, (int)gridDim.x - n_dw), 0);
    }
}

template <int NT, int KG, int BM, int BN, int WM, int WGS>
hipError_t launch_kind(GemmKind kind, const GemmArgs &a, dim3 grid, hipStream_t stream, const LaunchEvents &ev)
{
    switch (kind) {
    case GEMM_FWD:
        return launch_kernel(gemm_split_kernel<NT, KG, BM, BN, WM, WGS, true, true, GEMM_FWD>, grid, dim3(NT *KG), stream, ev, a);
    case GEMM_DA:
        return launch_kernel(gemm_split_kernel<NT, KG, BM, BN, WM, WGS, true, false, GEMM_DA>, grid, dim3(NT *KG), stream, ev, a);
    case GEMM_DW:
        return launch_kernel(gemm_split_kernel<NT, KG, BM, BN, WM, WGS, false, false, GEMM_DW>, grid, dim3(NT *KG), stream, ev, a);
    }
    return hipErrorInvalidValue;
}

}  // namespace

// shape: 0 64 x 64, 1 128 x 64, 2 128 x 128, 3 64 x 64 with two groups, 4 64 x 32 with four
hipError_t launch_gemm_split(GemmKind kind, const GemmArgs &a, int shape, dim3 grid, hipStream_t stream,
                             const LaunchEvents &ev)
{
    switch (shape) {
    case 0: return launch_kind<256, 1, 64, 64, 2, 2>(kind, a, grid, stream, ev);
    case 1: return launch_kind<512, 1, 128, 64, 4, 1>(kind, a, grid, stream, ev);
    case 2: return launch_kind<512, 1, 128, 128, 2, 1>(kind, a, grid, stream, ev);
    case 4:  // the forward product only
        if (kind != GEMM_FWD) return hipErrorInvalidValue;
        return launch_kernel(gemm_split_kernel<128, 4, 64, 32, 2, 1, true, true, GEMM_FWD>, grid, dim3(512), stream, ev, a);
    default: return launch_kind<256, 2, 64, 64, 2, 1>(kind, a, grid, stream, ev);
    }
}

hipError_t launch_gemm_split_pair(const GemmArgs &da, const GemmArgs &dw, int shape, unsigned blocks, int n_dw,
                                  hipStream_t stream, const LaunchEvents &ev)
{
    switch (shape) {
    case 0: return launch_kernel(gemm_split_pair_kernel<256, 1, 64, 64, 2, 2>, dim3(blocks), dim3(256), stream, ev, da, dw, n_dw);
    case 1: return launch_kernel(gemm_split_pair_kernel<512, 1, 128, 64, 4, 1>, dim3(blocks), dim3(512), stream, ev, da, dw, n_dw);
    case 3: return launch_kernel(gemm_split_pair_kernel<256, 2, 64, 64, 2, 1>, dim3(blocks), dim3(512), stream, ev, da, dw, n_dw);
    default: return launch_kernel(gemm_split_pair_kernel<512, 1, 128, 128, 2, 1>, dim3(blocks), dim3(512), stream, ev, da, dw, n_dw);
    }
}

}  // namespace hb
