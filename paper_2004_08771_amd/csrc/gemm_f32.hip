// fp32 MFMA GEMM for the three dense layer products of the mini-batch step
// (Section 3 of the paper: forward Eq. (1), backward Eq. (2); on a batch the
// matrix-vector products become matrix-matrix products, the dominant cost).
//
// This file: the plan (which kernel, tile shape and split a product gets) and the kernels for
// products with few output tiles (small batches), on fp32 MFMAs: 32 x 32 tiles, 256-thread
// workgroups (4 wavefronts of 64), the contraction split over the four wavefronts,
// v_mfma_f32_32x32x2_f32 blocks, operands staged global -> registers -> LDS with a double-buffered
// LDS tile.  K-major operands are read from LDS as 16-byte vectors along k (the k index is permuted
// identically for both operands, which leaves the contraction unchanged); M-major operands are
// read one float per lane with the 32 rows of a block on consecutive addresses.  Epilogues fuse
// bias + activation (forward), the activation derivative (backward-data) and the bias-gradient
// column sums (weight gradient).  The large products are in gemm_split.hip.
#include "gemm_device.h"

#include <stdlib.h>

#include <type_traits>

namespace hb {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int NT = 256;  // threads per workgroup

template <int ROWS, int BK, bool KMAJ>
struct Tile {
    static_assert(ROWS % 32 == 0 && BK % 8 == 0, "tile shape");
    static constexpr int LD = KMAJ ? (BK + 4) : (ROWS + 8);
    static constexpr int FLOATS = KMAJ ? ROWS * LD : BK * LD;
    static constexpr int VECS = ROWS * BK / 4;
    static constexpr int VPT = (VECS + NT - 1) / NT;

    // global -> registers; everything outside [0,nrows) x [.., kend) reads as zero
    static __device__ __forceinline__ void load(v4f (&reg)[VPT], const float *__restrict__ P,
                                                int ld, int row0, int nrows, int k0, int kend,
                                                bool vec, int tid)
    {
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
            const int idx = tid + v * NT;
            v4f x = {0.f, 0.f, 0.f, 0.f};
            if (VECS % NT == 0 || idx < VECS) {
                if (KMAJ) {
                    const int kq = idx % (BK / 4), r = idx / (BK / 4);
                    const int row = row0 + r, k = k0 + kq * 4;
                    if (row < nrows && k < kend) {
                        const float *p = P + (size_t)row * ld + k;
                        if (vec && k + 4 <= kend) {
                            x = *reinterpret_cast<const v4f *>(p);
                        } else {
                            x.x = p[0];
                            if (k + 1 < kend) x.y = p[1];
                            if (k + 2 < kend) x.z = p[2];
                            if (k + 3 < kend) x.w = p[3];
                        }
                    }
                } else {
                    const int mq = idx % (ROWS / 4), kk = idx / (ROWS / 4);
                    const int row = row0 + mq * 4, k = k0 + kk;
                    if (k < kend && row < nrows) {
                        const float *p = P + (size_t)k * ld + row;
                        if (vec && row + 4 <= nrows) {
                            x = *reinterpret_cast<const v4f *>(p);
                        } else {
                            x.x = p[0];
                            if (row + 1 < nrows) x.y = p[1];
                            if (row + 2 < nrows) x.z = p[2];
                            if (row + 3 < nrows) x.w = p[3];
                        }
                    }
                }
            }
            reg[v] = x;
        }
    }

    // The same tile without any guard: legal when the tile lies inside the matrix in both
    // directions.  vec: 16-byte loads, else four 4-byte loads (rows that are not 16-byte
    // aligned, e.g. the caller's X with d_0 = 54).
    static __device__ __forceinline__ void load_fast(v4f (&reg)[VPT], const float *__restrict__ P,
                                                     int ld, int row0, int k0, bool vec, int tid)
    {
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
            const int idx = tid + v * NT;
            if (VECS % NT == 0 || idx < VECS) {
                const float *p;
                if (KMAJ) {
                    const int kq = idx % (BK / 4), r = idx / (BK / 4);
                    p = P + (size_t)(row0 + r) * ld + k0 + kq * 4;
                } else {
                    const int mq = idx % (ROWS / 4), kk = idx / (ROWS / 4);
                    p = P + (size_t)(k0 + kk) * ld + row0 + mq * 4;
                }
                if (vec) {
                    reg[v] = *reinterpret_cast<const v4f *>(p);
                } else {
                    v4f x;
                    x.x = p[0];
                    x.y = p[1];
                    x.z = p[2];
                    x.w = p[3];
                    reg[v] = x;
                }
            }
        }
    }

    // registers -> LDS (same element <-> thread mapping as load)
    static __device__ __forceinline__ void store(float *S, const v4f (&reg)[VPT], int tid)
    {
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
            const int idx = tid + v * NT;
            if (VECS % NT == 0 || idx < VECS) {
                if (KMAJ) {
                    const int kq = idx % (BK / 4), r = idx / (BK / 4);
                    *reinterpret_cast<v4f *>(&S[r * LD + kq * 4]) = reg[v];
                } else {
                    const int mq = idx % (ROWS / 4), kk = idx / (ROWS / 4);
                    *reinterpret_cast<v4f *>(&S[kk * LD + mq * 4]) = reg[v];
                }
            }
        }
    }

    // The four operand values of tile row `row` for the MFMA steps of k-group g:
    // f[j] = element(row, k = 8 g + 4 h + j), h = lane / 32.
    static __device__ __forceinline__ v4f frag(const float *S, int row, int g, int h)
    {
        if (KMAJ) {
            return *reinterpret_cast<const v4f *>(&S[row * LD + g * 8 + h * 4]);
        } else {
            const float *p = &S[(g * 8 + h * 4) * LD + row];
            v4f f;
            f.x = p[0];
            f.y = p[LD];
            f.z = p[2 * LD];
            f.w = p[3 * LD];
            return f;
        }
    }
};

// LDS floats one workgroup of this shape needs (two stages of an A and a B tile)
template <int BM, int BN, int BK, bool A_KMAJ, bool B_KMAJ>
constexpr int lds_floats()
{
    return 2 * (Tile<BM, BK, A_KMAJ>::FLOATS + Tile<BN, BK, B_KMAJ>::FLOATS);
}

// ---- small products: one 32 x 32 output block per workgroup, the contraction split over
// the four wavefronts.
//
// With few output tiles (a small batch) a 64 x 64 tile leaves most compute units idle
// while each wavefront walks the whole contraction alone: K / 2 dependent-issue MFMAs of 64
// cycles each are the run time, whatever the batch.  Here every workgroup owns one 32 x 32
// block and its wavefront w takes the k-groups {w, w + 4, ...} of every k-tile, so the MFMA
// chain per wavefront is a quarter as long and four times as many workgroups exist.  The four
// partial blocks meet in LDS (the tile stages are free by then) and every wavefront finishes
// eight rows of the block with the fused epilogue.
template <int BK, bool A_KMAJ, bool B_KMAJ, int KIND>
__device__ __forceinline__ void gemm_f32_small_tile(const GemmArgs &a, float *smem, int id, int split)
{
    using TA = Tile<32, BK, A_KMAJ>;
    using TB = Tile<32, BK, B_KMAJ>;
    constexpr int STAGE = TA::FLOATS + TB::FLOATS;
    constexpr int G = BK / 8;  // k-groups of 8 per tile
    static_assert(G % 4 == 0, "k-groups are dealt to four wavefronts");
    constexpr int Q = G / 4;   // k-groups per wavefront and tile
    constexpr int RED_LD = 40, RED = 32 * RED_LD;  // 4 rows apart = 32 banks apart
    static_assert(2 * STAGE >= 4 * RED, "partial blocks reuse the tile stages");

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int r = lane & 31, h = lane >> 5;

    const int tile_m = id / a.tiles_n, tile_n = id - tile_m * a.tiles_n;
    const int m0 = tile_m * 32, n0 = tile_n * 32;
    const int kbeg = split * a.k_chunk;
    const int kend = min(a.K, kbeg + a.k_chunk);
    const int nk = (kend - kbeg + BK - 1) / BK;

    const float *__restrict__ A = static_cast<const float *>(a.A);
    const float *__restrict__ Bm = static_cast<const float *>(a.B);

    v16f acc[2];  // two independent MFMA chains
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[c][v] = 0.f;

    const bool a_in = (m0 + 32 <= a.M), b_in = (n0 + 32 <= a.N);
    float colsum = 0.f;
    const bool do_colsum = (KIND == GEMM_DW) && a.colsum != nullptr && tile_n == 0;
    // forward: the lane's bias is requested now, not after the reduction
    const float bias_pre = (KIND == GEMM_FWD && a.bias != nullptr && n0 + r < a.N) ? a.bias[n0 + r] : 0.f;

    v4f ra[TA::VPT], rb[TB::VPT];
    auto load_tile = [&](int t) {
        const int k0 = kbeg + t * BK;
        const bool kfull = (k0 + BK <= kend);
        if (a_in && kfull) TA::load_fast(ra, A, a.lda, m0, k0, a.a_vec != 0, tid);
        else TA::load(ra, A, a.lda, m0, a.M, k0, kend, a.a_vec != 0, tid);
        if (b_in && kfull) TB::load_fast(rb, Bm, a.ldb, n0, k0, a.b_vec != 0, tid);
        else TB::load(rb, Bm, a.ldb, n0, a.N, k0, kend, a.b_vec != 0, tid);
    };
    v4f fa[Q], fb[Q];
    auto read_frags = [&](const float *As, const float *Bs) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            fa[q] = TA::frag(As, r, wave + 4 * q, h);
            fb[q] = TB::frag(Bs, r, wave + 4 * q, h);
        }
    };

    // global loads run two k-tiles ahead, the LDS write one tile ahead, the fragments of tile
    // kt+1 are read right after the barrier of tile kt, under its last MFMAs
    load_tile(0);
    TA::store(smem, ra, tid);
    TB::store(smem + TA::FLOATS, rb, tid);
    if (nk > 1) load_tile(1);
    __syncthreads();
    read_frags(smem, smem + TA::FLOATS);
    for (int kt = 0; kt < nk; ++kt) {
        const float *As = smem + (kt & 1) * STAGE;
        float *An = smem + ((kt + 1) & 1) * STAGE;
        const bool next = (kt + 1 < nk);
        if (next) {
            TA::store(An, ra, tid);
            TB::store(An + TA::FLOATS, rb, tid);
        }
        if (kt + 2 < nk) load_tile(kt + 2);
        if (KIND == GEMM_DW && !A_KMAJ) {
            if (do_colsum && tid < 32) {
#pragma unroll
                for (int k = 0; k < BK; ++k) colsum += As[k * TA::LD + tid];
            }
        }
        v4f ca[Q], cb[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            ca[q] = fa[q];
            cb[q] = fb[q];
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int q = 0; q < Q; ++q)
                acc[q & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(ca[q][s], cb[q][s], acc[q & 1], 0, 0, 0);
        __syncthreads();  // tile kt read by everyone (fragments are in registers), tile kt+1 written
        if (next) read_frags(An, An + TA::FLOATS);
#pragma unroll
        for (int s = 2; s < 4; ++s)
#pragma unroll
            for (int q = 0; q < Q; ++q)
                acc[q & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(ca[q][s], cb[q][s], acc[q & 1], 0, 0, 0);
    }

    // ---- the four partial blocks meet in LDS.  acc[.][v] is C(row, col) with
    //      row = 8 (v / 4) + 4 h + (v % 4), col = r.  After the loop's last barrier nobody
    //      reads a tile stage any more (the DW column sums read theirs before it).
    float *mine = smem + wave * RED;
#pragma unroll
    for (int v = 0; v < 16; ++v)
        mine[(8 * (v >> 2) + 4 * h + (v & 3)) * RED_LD + r] = acc[0][v] + acc[1][v];
    __syncthreads();

    float *__restrict__ C = static_cast<float *>(a.C) + (size_t)split * a.c_split_stride;
    const int n = n0 + r;
    const bool n_ok = n < a.N;
    const float bias = bias_pre;
    float o4[4] = {0.f, 0.f, 0.f, 0.f};
    if (KIND == GEMM_DA && a_in && b_in) {  // the four activation values of the lane, requested together
#pragma unroll
        for (int p = 0; p < 4; ++p)
            o4[p] = static_cast<const float *>(a.aux)[(size_t)(m0 + 8 * wave + 2 * p + h) * a.ldaux + n];
    }
    with_activation(KIND == GEMM_DW ? (int)ACT_NONE : a.act, [&](auto act_c) {
        constexpr int ACT = decltype(act_c)::value;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int row = 8 * wave + 2 * p + h;
            const int m = m0 + row;
            float x = smem[row * RED_LD + r] + smem[RED + row * RED_LD + r] +
                      (smem[2 * RED + row * RED_LD + r] + smem[3 * RED + row * RED_LD + r]);
            if (m < a.M && n_ok) {
                if (KIND == GEMM_FWD) {
                    x += bias;
                    if (ACT == ACT_SIGMOID) x = sigmoidf_fast(x);
                    else if (ACT == ACT_RELU) x = fmaxf(x, 0.f);
                } else if (KIND == GEMM_DA) {
                    const float o = (a_in && b_in) ? o4[p] : static_cast<const float *>(a.aux)[(size_t)m * a.ldaux + n];
                    if (ACT == ACT_SIGMOID) x *= o * (1.f - o);
                    else if (ACT == ACT_RELU) x = (o > 0.f) ? x : 0.f;
                }
                C[(size_t)m * a.ldc + n] = x;
            }
        }
    });
    if (KIND == GEMM_DW) {
        if (do_colsum && tid < 32 && m0 + tid < a.M)
            a.colsum[(size_t)split * a.M + m0 + tid] = colsum;
    }
}

constexpr int SMALL_BK = 64;

template <bool A_KMAJ, bool B_KMAJ, int KIND>
__global__ __launch_bounds__(NT) void gemm_f32_small_kernel(GemmArgs a)
{
    __shared__ __attribute__((aligned(16))) float smem[lds_floats<32, 32, SMALL_BK, A_KMAJ, B_KMAJ>()];
    gemm_f32_small_tile<SMALL_BK, A_KMAJ, B_KMAJ, KIND>(a, smem, xcd_tile_order(blockIdx.x, gridDim.x),
                                                       blockIdx.y);
}

// The backward pair of one hidden layer (see launch_gemm_f32_bwd_pair) for small batches.  The product whose
// workgroups walk the longer contraction goes first: of a wide layer the backward-data product, whose few workgroups
// take most of the launch, while the many short ones of the weight gradient fill the other compute units (16 rows,
// 2048 wide: 35.2 us with the weight gradient first, 27 so; 4096 wide 99 -> 60).
__global__ __launch_bounds__(NT) void gemm_f32_small_pair_kernel(GemmArgs da, GemmArgs dw, int n_dw)
{
    constexpr int LDS_DA = lds_floats<32, 32, SMALL_BK, true, false>();
    constexpr int LDS_DW = lds_floats<32, 32, SMALL_BK, false, false>();
    __shared__ __attribute__((aligned(16))) float smem[LDS_DA > LDS_DW ? LDS_DA : LDS_DW];
    const int n_da = (int)gridDim.x - n_dw, dw_from = (da.K > dw.k_chunk) ? n_da : 0;
    const int b = (int)blockIdx.x - dw_from;  // of the weight gradient if in [0, n_dw)
    if (b >= 0 && b < n_dw) {
        const int tiles = dw.tiles_m * dw.tiles_n;
        gemm_f32_small_tile<SMALL_BK, false, false, GEMM_DW>(dw, smem, xcd_tile_order(b % tiles, tiles), b / tiles);
    } else {
        gemm_f32_small_tile<SMALL_BK, true, false, GEMM_DA>(da, smem, xcd_tile_order(dw_from ? (int)blockIdx.x : b - n_dw, n_da), 0);
    }
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
constexpr Shape SHAPES[] = {{64, 64}, {128, 64}, {128, 128}, {64, 64}};  // by the number launch_gemm_split takes
constexpr int SHARED = 3;  // 64 x 64, the contraction shared by two groups of wavefronts ...
constexpr int SHARED_K = 256;  // ... of at least this length (32-deep: 4.6 us alone, 4.8 shared)
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

// Products with fewer 64 x 64 output tiles than this (forward / backward-data; plan_f32_pair has a line of its own),
// or a contraction shorter than small_k_max() (weight gradient, whose contraction is the batch),
// go to the 32 x 32 split-wavefront kernel.  Both lines were measured against 64 x 64 tiles on fp32 MFMAs.
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
// A weight gradient launched on its own (not paired with a backward-data product) whose output
// is only a few tiles -- the first layer of a narrow input, 512 x 54 -- stays with the small
// kernel up to four times that contraction length: with so few tiles the 64-wide kernel needs
// tens of K-slices to fill the chip, and every slice is a partial the update has to read
// (B = 4096, 512 x 54: 12.4 -> 11.0 us, and the update 7.7 -> 7.2 us, against fp32 MFMA tiles).
long long small_dw_alone_kmax(int M, int N)  // contractions below this go to the small kernel
{
    const bool few_tiles = (long long)((M + 63) / 64) * ((N + 63) / 64) <= 16;
    return few_tiles ? 4 * (long long)small_k_max() : (long long)small_k_max();
}
bool small_dw_alone(int M, int N, int K)
{
    return K >= 64 && K < small_dw_alone_kmax(M, N);
}
// K-slices of the small weight-gradient kernel: at most 512 long (multiples of its k-tile)
SplitPlan plan_small_splits(int K, int max_splits)
{
    int s = (K + 511) / 512;
    if (s > max_splits) s = max_splits;
    if (s < 1) s = 1;
    const int chunk = ((K + s - 1) / s + SMALL_BK - 1) / SMALL_BK * SMALL_BK;
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

// shape < 0: the kernel of small products (tiles of 32 x 32), else the one launch_gemm_split takes
struct F32Plan {
    int shape;
    SplitPlan split;
};
F32Plan plan_f32(GemmKind kind, int M, int N, int K, int max_splits)
{
    if (kind == GEMM_DW ? small_dw_alone(M, N, K) : small_out(M, N, K)) {
        if (kind == GEMM_DW) return {-1, plan_small_splits(K, max_splits)};
        return {-1, {1, (K + SMALL_BK - 1) / SMALL_BK * SMALL_BK}};
    }
    if (kind != GEMM_DW)
        return {pick_shape(M, N, K), {1, (K + K_CHUNK_ALIGN - 1) / K_CHUNK_ALIGN * K_CHUNK_ALIGN}};
    int sh = (M >= 128) ? (N >= 128 ? 2 : 1) : 0;
    const SplitPlan sp = plan_splits(tiles_of(sh, M, N), K, max_splits, CUS);
    if (sh == 0 && sp.chunk >= SHARED_K && tiles_of(sh, M, N) * sp.splits <= CUS) sh = SHARED;
    return {sh, sp};
}
// da M x N over K and dw M x N over K of one layer.  Small tiles / split-plane tiles, 512-wide layers: B = 512 (64 tiles
// of 64 x 64) 14.2 / 12.8 us, B = 640 16.3 / 12.3, B = 1024 18.3 / 13.2.  A long contraction favours the small ones
// while each has a compute unit of its own: B = 256, 1024 wide (256 of 32 x 32) 22.7 / 24.2 us, B = 128, 2048 wide
// 44.4 / 48.0; but B = 384, 1536 wide (576) 55 / 42.
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

hipError_t launch_gemm_f32(GemmKind kind, GemmArgs a, int max_splits, int *splits_out,
                           hipStream_t stream, const LaunchEvents &ev)
{
    if (a.M <= 0 || a.N <= 0 || a.K <= 0) return hipErrorInvalidValue;
    const F32Plan p = plan_f32(kind, a.M, a.N, a.K, max_splits);
    const int bm = p.shape < 0 ? 32 : SHAPES[p.shape].bm, bn = p.shape < 0 ? 32 : SHAPES[p.shape].bn;
    a.tiles_m = (a.M + bm - 1) / bm;
    a.tiles_n = (a.N + bn - 1) / bn;
    const long long tiles = (long long)a.tiles_m * a.tiles_n;
    if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    a.splits = p.split.splits;
    a.k_chunk = p.split.chunk;
    if (splits_out) *splits_out = p.split.splits;
    const dim3 grid((unsigned)tiles, (unsigned)p.split.splits, 1);
    if (p.shape >= 0) return launch_gemm_split(kind, a, p.shape, grid, stream, ev);
    switch (kind) {
    case GEMM_FWD:
        return launch_kernel(gemm_f32_small_kernel<true, true, GEMM_FWD>, grid, dim3(NT), stream, ev, a);
    case GEMM_DA:
        return launch_kernel(gemm_f32_small_kernel<true, false, GEMM_DA>, grid, dim3(NT), stream, ev, a);
    case GEMM_DW:
        return launch_kernel(gemm_f32_small_kernel<false, false, GEMM_DW>, grid, dim3(NT), stream, ev, a);
    }
    return hipErrorInvalidValue;
}

// dA_l and dW_l of one hidden layer in one launch: both only read D_l, so they are independent, and
// sharing a launch lets the prologue / epilogue of one hide under the main loop of the other and pays
// the per-launch latencies once (B = 16, 512-wide layers: 9.7 + 7.8 -> 8.7 us; B = 128, 32-wide:
// 4.8 + 4.5 -> 7.4).  Apart only with fewer rows than a k-tile and a weight gradient of more than 2^24 values: its
// 32 x 32 tiles then outlast the backward-data product (16 rows, 8192 wide: 158 us apart, 244 together; 4096 wide 66 / 62).
// HB_NO_PAIR = 1 (tuning aid): two launches.
bool gemm_f32_pair_ok(int B, int d_out, int d_in)
{
    static const int off = env_int("HB_NO_PAIR", 0);
    return !off && (B >= SMALL_BK || (long long)d_out * d_in <= (1ll << 24));
}

hipError_t launch_gemm_f32_bwd_pair(GemmArgs da, GemmArgs dw, int max_splits, int *splits_out,
                                    hipStream_t stream, const LaunchEvents &ev)
{
    const F32Plan p = plan_f32_pair(da, dw, max_splits);
    const int bm = p.shape < 0 ? 32 : SHAPES[p.shape].bm, bn = p.shape < 0 ? 32 : SHAPES[p.shape].bn;
    for (GemmArgs *g : {&da, &dw}) {
        g->tiles_m = (g->M + bm - 1) / bm;
        g->tiles_n = (g->N + bn - 1) / bn;
    }
    const int align = p.shape < 0 ? SMALL_BK : K_CHUNK_ALIGN;
    da.splits = 1;
    da.k_chunk = (da.K + align - 1) / align * align;
    dw.splits = p.split.splits;
    dw.k_chunk = p.split.chunk;
    if (splits_out) *splits_out = p.split.splits;
    const long long n_dw = (long long)dw.tiles_m * dw.tiles_n * p.split.splits;
    const long long blocks = (long long)da.tiles_m * da.tiles_n + n_dw;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    if (p.shape >= 0) return launch_gemm_split_pair(da, dw, p.shape, (unsigned)blocks, (int)n_dw, stream, ev);
    return launch_kernel(gemm_f32_small_pair_kernel, dim3((unsigned)blocks), dim3(NT), stream, ev, da, dw, (int)n_dw);
}

}  // namespace hb
