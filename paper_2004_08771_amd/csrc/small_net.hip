// The whole gradient of a small network in one launch: a workgroup takes a block of the batch's rows through the forward
// pass (Section 3, Eq. (1)), the loss, and the backward pass (Eq. (2)) with every weight and everything it computes in LDS.
// A batch of one block is also updated (Eq. (3)) by the same launch; more blocks leave partial sums for update_kernel.
//
// As separate launches a step of such a network is a chain of 2 L of them, each 4 to 6 us of latency around next to no
// work (54-32-7, 64 rows: 20 us for four).  Here the parameters and rows are read from memory once, all at the same
// time, and a layer is an LDS pass of 16 x 16 blocks (v_mfma_f32_16x16x4_f32, fp32 throughout) dealt to sixteen wavefronts.
// Time stamps at 54-32-7, 64 rows: 1.6 us until the loads are issued, 1.0 until they are in LDS, 1.9 and 1.0 for the forward
// products, 1.0 for the loss, 2.0 and 1.8 backward.  What bounds it: latencies of LDS and of the descriptions of the
// layers, not the matrix cores.  (With the pieces of the parameters found by a search in the arguments of the launch, which
// lie in host memory, the step took 17 us.)
#include "gemm_device.h"

namespace hb {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int SN_NT = 1024, SN_WAVES = SN_NT / 64;
constexpr int SN_BATCH = 8;               // values that a thread has in flight
constexpr int SN_LDS_FLOATS = 156 * 256;  // of 160 KB

__host__ __device__ inline int up16(int x) { return (x + 15) & ~15; }
// Pitch of a tensor's rows in LDS: rows of a 16-byte read per lane, and the four rows that a column-wise read touches
// together, lie on different banks.
__host__ __device__ inline int pitch(int d) { return up16(d) + 4; }

// a 16 x 16 block of P . Q^T over K (a multiple of 16); each operand with k along its rows or across them.  sum: the lane's
// values of P (its row r, a quarter of the k).  The matrix unit rounds after every term, so the sum is cut short: four side by
// side over every 64 k, which then add up.  Positive terms, rms relative error and us per step of 54-32-7, 64 rows: one running
// sum 2.9e-7 over 480 terms, 1.1e-7 over 54, 10.9 us; so 5.0e-8, 4.7e-8, 10.9; eight sums 5.3e-8, 4.3e-8, 11.4; sums in 64 bits
// 12.8 us.  The kernels of single layers: 5.8e-8 over 480 terms, 4.8e-8 over 54 (there products of bf16 planes).
template <bool P_KMAJ, bool Q_KMAJ>
__device__ __forceinline__ v4f block_product(const float *P, int ldp, const float *Q, int ldq, int K, int r, int h, float &sum)
{
    v4f acc[4], t = {0.f, 0.f, 0.f, 0.f};
    const float *p = P_KMAJ ? P + r * ldp + 4 * h : P + 4 * h * ldp + r;
    const float *q = Q_KMAJ ? Q + r * ldq + 4 * h : Q + 4 * h * ldq + r;
    auto read = [](const float *s, int ld, bool kmaj) {
        if (kmaj) return *reinterpret_cast<const v4f *>(s);
        return v4f{s[0], s[ld], s[2 * ld], s[3 * ld]};
    };
    v4f x = read(p, ldp, P_KMAJ), y = read(q, ldq, Q_KMAJ);
    sum = 0.f;
    for (int k = 0;;) {
        const int end = min(k + 64, K);
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = v4f{0.f, 0.f, 0.f, 0.f};
        for (k += 16; k < end; k += 16) {
            p += P_KMAJ ? 16 : 16 * ldp;
            q += Q_KMAJ ? 16 : 16 * ldq;
            const v4f xn = read(p, ldp, P_KMAJ), yn = read(q, ldq, Q_KMAJ);
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[c], y[c], acc[c], 0, 0, 0);
            sum += (x[0] + x[1]) + (x[2] + x[3]);
            x = xn;
            y = yn;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[c], y[c], acc[c], 0, 0, 0);
        sum += (x[0] + x[1]) + (x[2] + x[3]);
        if (k < K) {
            p += P_KMAJ ? 16 : 16 * ldp;
            q += Q_KMAJ ? 16 : 16 * ldq;
            x = read(p, ldp, P_KMAJ);
            y = read(q, ldq, Q_KMAJ);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) t[v] += (acc[0][v] + acc[1][v]) + (acc[2][v] + acc[3][v]);
        if (k >= K) return t;  // t[v]: row 4 h + v, column r
    }
}

template <int ACT>
__device__ __forceinline__ float hidden(float z)
{
    return (ACT == ACT_SIGMOID) ? sigmoidf_fast(z) : fmaxf(z, 0.f);
}
template <int ACT>
__device__ __forceinline__ float derivative(float x, float o)
{
    return (ACT == ACT_SIGMOID) ? x * (o * (1.f - o)) : (o > 0.f) ? x : 0.f;
}

template <int ACT>
__global__ __launch_bounds__(SN_NT) void small_net_kernel(SmallNetArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float sm[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, h = lane >> 4;
    const SmallNetLayer *__restrict__ net = a.net;  // [0 .. L]
    const int L = a.L, R = a.R;
    const long long r0 = (long long)blockIdx.x * R;
    const int rows = (int)((a.B - r0 < R) ? a.B - r0 : R);
    const int d0 = net[0].d, x_floats = rows * d0;
    const float *__restrict__ X = a.X + (size_t)r0 * d0;

    // the row of the batch that this thread's group of T = 16, 32 or 64 lanes takes through the loss
    const int lt = 31 - __builtin_clz(SN_NT) - (31 - __builtin_clz(R)), T = 1 << lt, lrow = tid >> lt, lc = tid & (T - 1);
    const int yi = (lrow < rows) ? a.y[r0 + lrow] : 0;

    // ---- everything from memory: the flat parameters with the place in LDS of each, and the block's rows of X
    float *const act0 = sm + a.lds_act;
    const float inv_d0 = 1.0f / (float)d0;
    const int ld0 = pitch(d0), n_all = a.P + x_floats;
    for (int base = 0; base < n_all; base += SN_BATCH * SN_NT) {  // (the same rounds for every thread: there is a barrier)
        const int e0 = base + tid;
        float v[SN_BATCH];
        int to[SN_BATCH];
#pragma unroll
        for (int j = 0; j < SN_BATCH; ++j) {
            const int e = e0 + j * SN_NT;
            to[j] = -1;
            v[j] = 0.f;
            if (e < a.P) {
                v[j] = a.params[e];
                to[j] = a.place[e];
            } else if (e < n_all) {
                v[j] = X[e - a.P];
                to[j] = -2;
            }
        }
        if (base == 0) {  // the padding: under the first loads
            for (int i = 4 * tid; i < a.lds_floats; i += 4 * SN_NT) *reinterpret_cast<v4f *>(sm + i) = v4f{0.f, 0.f, 0.f, 0.f};
            __syncthreads();
        }
#pragma unroll
        for (int j = 0; j < SN_BATCH; ++j) {
            if (to[j] >= 0) sm[to[j]] = v[j];
            if (to[j] == -2) {
                const int e = e0 + j * SN_NT - a.P, row = (int)(((float)e + 0.5f) * inv_d0);  // exact: e < 2^17
                act0[row * ld0 + e - row * d0] = v[j];
            }
        }
    }
    __syncthreads();

    const int rt = R >> 4;  // row blocks
    // ---- forward.  A layer's description is read a layer ahead.
    SmallNetLayer in = net[0], o = net[1];
    for (int l = 1; l <= L; ++l) {
        const SmallNetLayer next = net[min(l + 1, L)];
        const int ldi = in.ld, ldo = o.ld;
        const float *src = act0 + R * in.cum, *W = sm + o.lds_w, *b = sm + o.lds_b;
        float *out = act0 + R * o.cum;
        float *__restrict__ const keep = (l < L) ? o.act : nullptr;
        for (int i = wave; i < rt * o.nt; i += SN_WAVES) {
            const int mi = (i * o.inv_nt) >> 16, m0 = mi * 16 + 4 * h, nb = (i - mi * o.nt) * 16, n = nb + r;
            const float bias = b[n];
            float unused;
            const v4f acc = block_product<true, true>(src + mi * 16 * ldi, ldi, W + nb * ldi, ldi, 16 * in.nt, r, h, unused);
            if (n < o.d) {  // all padding stays zero
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float x = acc[e] + bias;
                    if (keep) x = hidden<ACT>(x);
                    if (m0 + e < rows) {
                        out[(m0 + e) * ldo + n] = x;
                        if (keep) keep[(size_t)(r0 + m0 + e) * o.act_ld + n] = x;
                    }
                }
            }
        }
        __syncthreads();
        if (l < L) {
            in = o;
            o = next;
        }
    }

    // ---- loss and D_L (zero rows past the end of the batch)
    float *const red = sm + a.lds_red;
    {
        const int K = o.d, ldz = o.ld;
        const float *z = act0 + R * o.cum + lrow * ldz;
        float *D = sm + a.lds_delta[L & 1] + lrow * ldz;
        const float invB = 1.0f / (float)a.B;
        float row_loss = 0.f;
        if (a.loss == 1 && K == 1) {
            if (lc == 0 && lrow < rows) {
                const float yf = (float)yi, mg = yf * z[0];
                const float e = __expf(-fabsf(mg));
                row_loss = fmaxf(-mg, 0.f) + log1pf(e);
                D[0] = -yf * ((mg >= 0.f) ? e / (1.f + e) : 1.f / (1.f + e)) * invB;
            }
        } else {
            const int cls = (a.loss == 1) ? (yi + 1) / 2 : yi;
            const float z0 = (lc < K) ? z[lc] : -INFINITY;  // an output to a lane: K <= 16 <= T
            const float zc = (cls >= 0 && cls < K) ? z[cls] : 0.f;
            float mx = z0;
            for (int q = 8; q > 0; q >>= 1) mx = fmaxf(mx, __shfl_xor(mx, q, 64));
            float se = (lc < K) ? __expf(z0 - mx) : 0.f;
            for (int q = 8; q > 0; q >>= 1) se += __shfl_xor(se, q, 64);
            const float lse = mx + __logf(se);
            if (lrow < rows) {
                if (lc < K) D[lc] = (__expf(z0 - lse) - (lc == cls ? 1.f : 0.f)) * invB;
                row_loss = lse - zc;
            }
        }
        if (lc == 0) red[lrow] = row_loss;
        __syncthreads();
    }

    // ---- backward: D_{l-1} and dW_l of a layer side by side
    const bool one = gridDim.x == 1;  // the gradient is whole
    const bool update = one && a.update;
    for (int l = a.backward ? L : 0; l >= 1; --l) {
        const SmallNetLayer next = net[max(l - 2, 0)];
        const int d = o.d, di = in.d, ldd = o.ld, lda = in.ld, nt = in.nt;
        const float *D = sm + a.lds_delta[l & 1], *A = act0 + R * in.cum, *W = sm + o.lds_w;
        float *Dn = sm + a.lds_delta[(l - 1) & 1];
        float *const gw = one ? a.grad + o.w_off : o.partial_w + (size_t)blockIdx.x * d * di;
        float *const gb = one ? a.grad + o.b_off : o.partial_b + (size_t)blockIdx.x * d;
        const int n_da = (l > 1) ? rt * nt : 0;
        for (int i = wave; i < n_da + o.nt * nt; i += SN_WAVES) {
            const int j = (i < n_da) ? i : i - n_da, mi = (j * in.inv_nt) >> 16, m0 = mi * 16, n0 = (j - mi * nt) * 16, n = n0 + r;
            float sum;
            if (i < n_da) {
                const v4f acc = block_product<true, false>(D + m0 * ldd, ldd, W + n0, lda, 16 * o.nt, r, h, sum);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = m0 + 4 * h + e;
                    const float x = derivative<ACT>(acc[e], A[row * lda + n]);
                    Dn[row * lda + n] = (row < rows && n < di) ? x : 0.f;
                }
            } else {
                const v4f acc = block_product<false, false>(D + m0, ldd, A + n0, lda, R, r, h, sum);
                if (n < di) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int m = m0 + 4 * h + e;
                        if (m < d) gw[m * di + n] = update ? W[m * lda + n] - a.lr * acc[e] : acc[e];
                    }
                }
                if (n0 == 0) {  // the bias: the columns of D
                    sum += __shfl_xor(sum, 16, 64);
                    sum += __shfl_xor(sum, 32, 64);
                    if (h == 0 && m0 + r < d) gb[m0 + r] = update ? sm[o.lds_b + m0 + r] - a.lr * sum : sum;
                }
            }
        }
        __syncthreads();
        o = in;
        in = next;
    }

    if (wave == 0) {
        float s = (lane < R) ? red[lane] : 0.f;
#pragma unroll
        for (int q = 32; q > 0; q >>= 1) s += __shfl_xor(s, q, 64);
        if (lane == 0) {
            if (!one) {
                a.block_partials[blockIdx.x] = s;
            } else {
                const float mean = (float)((double)s / (double)a.B);
                a.loss_out[0] = mean;
                if (a.loss_out2) a.loss_out2[0] = mean;
            }
        }
    }
}

__global__ __launch_bounds__(256) void small_net_plan_kernel(SmallNetPlan p)
{
    if (blockIdx.x == 0 && (int)threadIdx.x <= p.L) p.net[threadIdx.x] = p.layer[threadIdx.x];
    for (int e = blockIdx.x * 256 + threadIdx.x; e < p.P; e += gridDim.x * 256) {
        int l = 1;
        while (l < p.L && e >= p.layer[l + 1].w_off) ++l;
        const SmallNetLayer &o = p.layer[l];
        const int i = e - o.w_off, di = p.layer[l - 1].d, row = i / di;
        p.place[e] = (e >= o.b_off) ? o.lds_b + e - o.b_off : o.lds_w + row * p.layer[l - 1].ld + i - row * di;
    }
}

// LDS of a block of R rows in floats; the offsets of `a` and the layers' places (either may be null)
int lds_floats(const int *dims, int L, int R, SmallNetArgs *a, SmallNetLayer *net)
{
    long long n = 0;
    int cum = 0, widest = 0;
    for (int l = 0; l <= L; ++l) {
        if (dims[l] > 4096) return 1 << 28;
        if (net) net[l].cum = cum;
        cum += pitch(dims[l]);
        if (l == 0) continue;
        if (net) net[l].lds_w = (int)n;
        n += (long long)up16(dims[l]) * pitch(dims[l - 1]);
        if (net) net[l].lds_b = (int)n;
        n += up16(dims[l]);
        if (pitch(dims[l]) > widest) widest = pitch(dims[l]);
        if (n > 1 << 20) return 1 << 28;
    }
    if (a) a->lds_act = (int)n;
    n += (long long)R * cum;
    for (int i = 0; i < 2; ++i) {
        if (a) a->lds_delta[i] = (int)n;
        n += (long long)R * widest;
    }
    if (a) a->lds_red = (int)n;
    n += 64;
    return (int)n;
}

}  // namespace

// A narrow output, and everything in LDS.  Up to 64 rows in one workgroup if so large a block fits; above, blocks of 16 rows
// (32, 64) for up to 128 workgroups, whose partial sums a second launch adds.  Launches of the single layers / so, us per step:
// 54-32-7 64 rows 21.1 / 11.1, 2048 rows 24.0 / 13.9; 32x8-2 64 rows 86 / 31, 5000 rows 110 / 36; 64x4-5 32 rows 36.7 / 21.3, 2000 rows
// 45.7 / 25.7; 200-60-60-10 1000 rows 38.8 / 25.3.  A chain of few layers with many parameters is as fast in launches of their own,
// each on more compute units (100-100-100-3 100 rows 27.3 / 26.5, 3000 rows 40 / 42; 100-100-7 64 rows 18.8 / 18.5; 105-108-4
// 13.9 / 17.8; 500-32-2 100 rows 19.2 / 21.1): hence the limit on the parameters.  Where a block of all rows does not fit, 17 .. 64
// rows go in blocks of 16: 64x4-5 40 rows 35.5 / 21.7, 64 rows 31.6 / 21.8; 200-60-60-10 64 rows 33.9 / 22.8; 400-20-20-3 28.4 /
// 21.1; 100-64x5-4 32 rows 46.0 / 31.9; but two layers are faster apart (80-100-4 15.5 / 17.3; 500-16-2 15.7 / 18.3; 1000-8-2 16.1 /
// 24.9).  More than 128 blocks cost as much to add up as the layers' launches: with blocks of 16 54-32-7 8193 rows 28.2 / 30.4,
// 16000 rows 31.6 / 44.4; 64x4-5 4097 rows 45.2 / 44.6; 200-60-60-10 4097 rows 45.2 / 49.5; 80-100-4 24.0 / 34.6; only a chain
// of many narrow layers would gain (32x8-2 8193 rows 128 / 75).
int small_net_rows(const int *dims, int L, long long B)
{
    if (L < 2 || L > SMALL_NET_LAYERS || dims[L] > 16) return 0;
    long long P = 0;
    for (int l = 1; l <= L; ++l) P += (long long)dims[l] * (dims[l - 1] + 1);
    if (P > 9000ll * (L - 1)) return 0;
    bool fits = false;
    for (int R = 16; R <= 64; R *= 2) {
        if (lds_floats(dims, L, R, nullptr, nullptr) > SN_LDS_FLOATS) break;
        fits = true;
        if (B <= R || (B > 64 && B <= (long long)R * SMALL_NET_BLOCKS)) return R;
    }
    return (fits && B <= 64 && L > 2) ? 16 : 0;  // too many rows for one block
}

void small_net_layers(const int *dims, int L, SmallNetPlan &plan)
{
    SmallNetLayer *net = plan.layer;
    lds_floats(dims, L, 16, nullptr, net);
    int at = 0;
    for (int l = 0; l <= L; ++l) {
        SmallNetLayer &o = net[l];
        o.d = dims[l];
        o.ld = pitch(dims[l]);
        o.nt = up16(dims[l]) / 16;
        o.inv_nt = (65536 + o.nt - 1) / o.nt;  // (i inv_nt) >> 16 = i / nt for i < 4096
        if (l == 0) continue;
        o.w_off = at;
        o.b_off = at + dims[l] * dims[l - 1];
        at = o.b_off + dims[l];
    }
    plan.L = L;
    plan.P = at;
}

hipError_t launch_small_net_plan(const SmallNetPlan &plan, hipStream_t stream)
{
    return launch_kernel(small_net_plan_kernel, dim3((unsigned)((plan.P + 255) / 256)), dim3(256), stream, LaunchEvents(), plan);
}

hipError_t launch_small_net(const int *dims, SmallNetArgs a, hipStream_t stream, const LaunchEvents &ev)
{
    a.lds_floats = lds_floats(dims, a.L, a.R, &a, nullptr);
    const size_t lds = 4 * (size_t)a.lds_floats;
    if (lds > 4 * (size_t)SN_LDS_FLOATS) return hipErrorInvalidValue;
    static LdsGrant granted;
    const hipError_t e = grant_lds(granted, lds, small_net_kernel<ACT_SIGMOID>, small_net_kernel<ACT_RELU>);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)((a.B + a.R - 1) / a.R)), block(SN_NT);
    const auto kernel = a.act == ACT_SIGMOID ? small_net_kernel<ACT_SIGMOID> : small_net_kernel<ACT_RELU>;
    if (ev.start) hipExtLaunchKernelGGL(kernel, grid, block, (unsigned)lds, stream, ev.start, ev.stop, 0, a);
    else hipLaunchKernelGGL(kernel, grid, block, lds, stream, a);
    return hipGetLastError();
}

}  // namespace hb
