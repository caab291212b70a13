// The rate-distortion loss of the differentiable layer and its gradient, and the padding of that
// layer's outputs.
//   dist = sum (ahat - aref)^2 / (Nv C),  rate = lambda sum log2(1 + |yhat| / step),  loss = dist + rate
//   d/dahat = 2 g_dist (ahat - aref) / (Nv C),  d/dyhat = g_rate lambda sgn(yhat) / (ln 2 (step + |yhat|))
//
// HBM traffic bounds both directions: the forward reads three [rows][C] matrices and writes the
// difference its backward needs, the backward reads two and writes two, each once, in one launch or in
// one for each gradient (a caller may want the terms' gradients apart; the two launches cost 5 us of
// a 500K x 56 training step of 785 more). As single
// framework operators (difference, square, two sums, absolute value, quotient, logarithm and their
// adjoints) the same step read and wrote some twenty matrices: 500K x 56 rows (112 MB a matrix).
// Terms are FP32; the sums are FP64, per block in a fixed order, then over the blocks by one
// workgroup, so results repeat bit for bit.
#include <initializer_list>

#include "gsc_device.h"

namespace gsc {

constexpr int RD_THREADS = 256;
constexpr uint32_t RD_GRID = 2048;  // workgroups (eight per CU)

struct RdArgs {
    const float *yhat, *ahat, *aref, *step;
    uint64_t units;  // rows C, or that / 4 (VEC)
    uint32_t C, cu;  // channels; units per row
    double lam, rows;
    const int64_t *nv;  // (forward) rows that count, or null (all)
    const float *count_in;  // (gradient) the forward's count
    float *diff;        // ahat - aref, or null
    double *part;       // [grid][2]
    float *loss, *dist, *rate, *count;  // results
    // gradient
    const float *g_loss, *g_dist, *g_rate;  // scalars or null
    float *g_yhat, *g_ahat;  // (one may be null)
};

// The unit's channel group steps by the grid's stride modulo a row's units.
struct RdWalk {
    uint64_t i, stride;
    uint32_t c, cs, cu;
    __device__ explicit RdWalk(uint32_t cu_) : cu(cu_)
    {
        i = (uint64_t)blockIdx.x * RD_THREADS + threadIdx.x;
        stride = (uint64_t)gridDim.x * RD_THREADS;
        c = (uint32_t)(i % cu);
        cs = (uint32_t)(stride % cu);
    }
    __device__ void next()
    {
        i += stride;
        c += cs;
        c -= c >= cu ? cu : 0u;
    }
};

// Unit i of a matrix: four values (VEC) or one, the others zero.
template <bool VEC>
__device__ inline float4 rd_load(const float *p, uint64_t i)
{
    return VEC ? gload4(gp(p) + 4 * i) : make_float4(gp(p)[i], 0.f, 0.f, 0.f);
}
template <bool VEC>
__device__ inline void rd_store(float *p, uint64_t i, const float4 &v)
{
    if (VEC) gstore4(gp(p) + 4 * i, v);
    else gp(p)[i] = v.x;
}

template <bool VEC>
__global__ __launch_bounds__(RD_THREADS) void k_rd_sums(RdArgs a)
{
    constexpr int W = VEC ? 4 : 1;
    __shared__ float s_step[GSC_MAX_CHANNELS];
    __shared__ double s_p[2][RD_THREADS / WAVE];
    if (threadIdx.x < a.C) s_step[threadIdx.x] = a.step[threadIdx.x];
    __syncthreads();
    double dist = 0.0, rate = 0.0;
    for (RdWalk w(a.cu); w.i < a.units; w.next()) {
        const float4 y = rd_load<VEC>(a.yhat, w.i), h = rd_load<VEC>(a.ahat, w.i), r = rd_load<VEC>(a.aref, w.i);
        const float4 d = make_float4(h.x - r.x, h.y - r.y, h.z - r.z, h.w - r.w);
        if (a.diff) rd_store<VEC>(a.diff, w.i, d);
        const float yy[4] = {y.x, y.y, y.z, y.w}, dd[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
        for (int e = 0; e < W; ++e) {
            dist += (double)(dd[e] * dd[e]);
            rate += (double)log2f(1.0f + fabsf(yy[e]) / s_step[W * w.c + e]);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        dist += __shfl_xor(dist, o, WAVE);
        rate += __shfl_xor(rate, o, WAVE);
    }
    if (lane_id() == 0) {
        s_p[0][threadIdx.x / WAVE] = dist;
        s_p[1][threadIdx.x / WAVE] = rate;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < RD_THREADS / WAVE; ++q) s += s_p[threadIdx.x][q];
        a.part[2 * (size_t)blockIdx.x + threadIdx.x] = s;
    }
}

// One workgroup: the blocks' partials in a fixed order, and the three results.
__global__ __launch_bounds__(RD_THREADS) void k_rd_total(RdArgs a, uint32_t blocks)
{
    __shared__ double s_p[2][RD_THREADS];
    double s[2] = {0.0, 0.0};
    for (uint32_t b = threadIdx.x; b < blocks; b += RD_THREADS)
#pragma unroll
        for (int q = 0; q < 2; ++q) s[q] += a.part[2 * (size_t)b + q];
#pragma unroll
    for (int q = 0; q < 2; ++q) s_p[q][threadIdx.x] = s[q];
    __syncthreads();
    for (uint32_t n = RD_THREADS / 2; n > 0; n >>= 1) {
        if (threadIdx.x < n)
#pragma unroll
            for (int q = 0; q < 2; ++q) s_p[q][threadIdx.x] += s_p[q][threadIdx.x + n];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double n = a.nv ? (double)a.nv[0] : a.rows;
        const float dist = (float)(s_p[0][0] / (n * a.C)), rate = (float)(a.lam * s_p[1][0]);
        *a.loss = dist + rate;
        *a.dist = dist;
        *a.rate = rate;
        *a.count = (float)n;
    }
}

template <bool VEC>
__global__ __launch_bounds__(RD_THREADS) void k_rd_grad(RdArgs a)
{
    constexpr int W = VEC ? 4 : 1;
    __shared__ float s_step[GSC_MAX_CHANNELS];
    if (a.g_yhat && threadIdx.x < a.C) s_step[threadIdx.x] = a.step[threadIdx.x];
    __syncthreads();
    const float gl = a.g_loss ? *a.g_loss : 0.0f;
    const float gd = gl + (a.g_dist ? *a.g_dist : 0.0f), gr = gl + (a.g_rate ? *a.g_rate : 0.0f);
    const float fd = a.g_ahat ? (float)(2.0 * (double)gd / ((double)*a.count_in * a.C)) : 0.0f;
    const float fr = (float)((double)gr * a.lam / 0.693147180559945309417);  // (1 / ln 2)
    for (RdWalk w(a.cu); w.i < a.units; w.next()) {
        if (a.g_ahat) {
            const float4 d = rd_load<VEC>(a.diff, w.i);
            rd_store<VEC>(a.g_ahat, w.i, make_float4(fd * d.x, fd * d.y, fd * d.z, fd * d.w));
        }
        if (!a.g_yhat) continue;
        const float4 y = rd_load<VEC>(a.yhat, w.i);
        const float yy[4] = {y.x, y.y, y.z, y.w};
        float g[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < W; ++e) {
            const float v = fr / (s_step[W * w.c + e] + fabsf(yy[e]));
            g[e] = yy[e] > 0.f ? v : yy[e] < 0.f ? -v : yy[e] == 0.f ? 0.f * v : v;  // (a NaN stays one)
        }
        rd_store<VEC>(a.g_yhat, w.i, make_float4(g[0], g[1], g[2], g[3]));
    }
}

// Rows past Nv of the layer's three outputs cleared (all rows after a device-detected error), and
// Nv as a 64-bit word. The rows below Nv were written by the forward launches.
constexpr int PAD_THREADS = 256;
template <bool VEC>
__global__ __launch_bounds__(PAD_THREADS) void k_ste_pad(const int32_t *info, uint64_t units, uint32_t cu, float *m0, float *m1,
                                                         float *m2, int64_t *nv_out)
{
    const uint32_t nv = info[0] == 0 ? (uint32_t)info[1] : 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) *nv_out = (int64_t)nv;
    const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    for (uint64_t i = (uint64_t)nv * cu + (uint64_t)blockIdx.x * PAD_THREADS + threadIdx.x; i < units;
         i += (uint64_t)gridDim.x * PAD_THREADS) {
        rd_store<VEC>(m0, i, z);
        rd_store<VEC>(m1, i, z);
        rd_store<VEC>(m2, i, z);
    }
}

// --------------------------------------------------------------------------- launches
// 16-byte accesses: whole units of four channels and aligned matrices.
static bool rd_vec(uint32_t C, std::initializer_list<const void *> ps)
{
    for (const void *p : ps)
        if (((uintptr_t)p & 15u) != 0) return false;
    return C % 4 == 0;
}
static uint32_t rd_grid(uint64_t units)
{
    const uint64_t b = (units + RD_THREADS - 1) / RD_THREADS;
    return b < RD_GRID ? (uint32_t)(b ? b : 1) : RD_GRID;
}
size_t rd_loss_workspace_bytes() { return (size_t)RD_GRID * 2 * sizeof(double); }

static RdArgs rd_args(const float *yhat, const float *step, uint64_t rows, uint32_t C, double lam, bool vec)
{
    RdArgs a = {};
    a.yhat = yhat;
    a.step = step;
    a.units = vec ? rows * C / 4 : rows * C;
    a.C = C;
    a.cu = vec ? C / 4 : C;
    a.lam = lam;
    a.rows = (double)rows;
    return a;
}

hipError_t launch_rd_loss_forward(const float *yhat, const float *ahat, const float *aref, const float *step, uint64_t rows,
                                  uint32_t C, double lam, const int64_t *nv, float *diff, float *const out[4], double *ws,
                                  hipStream_t s)
{
    const bool vec = rd_vec(C, {yhat, ahat, aref, diff});
    RdArgs a = rd_args(yhat, step, rows, C, lam, vec);
    a.nv = nv;
    a.ahat = ahat;
    a.aref = aref;
    a.diff = diff;
    a.part = ws;
    a.loss = out[0];
    a.dist = out[1];
    a.rate = out[2];
    a.count = out[3];
    const uint32_t g = rd_grid(a.units);
    if (vec) hipLaunchKernelGGL(k_rd_sums<true>, dim3(g), dim3(RD_THREADS), 0, s, a);
    else hipLaunchKernelGGL(k_rd_sums<false>, dim3(g), dim3(RD_THREADS), 0, s, a);
    hipLaunchKernelGGL(k_rd_total, dim3(1), dim3(RD_THREADS), 0, s, a, g);
    return hipGetLastError();
}

hipError_t launch_rd_loss_backward(const float *yhat, const float *diff, const float *step, uint64_t rows, uint32_t C,
                                   double lam, const float *count, const float *g_loss, const float *g_dist,
                                   const float *g_rate, float *g_yhat, float *g_ahat, hipStream_t s)
{
    const bool vec = rd_vec(C, {yhat, diff, g_yhat, g_ahat});
    RdArgs a = rd_args(yhat, step, rows, C, lam, vec);
    a.count_in = count;
    a.diff = const_cast<float *>(diff);
    a.g_loss = g_loss;
    a.g_dist = g_dist;
    a.g_rate = g_rate;
    a.g_yhat = g_yhat;
    a.g_ahat = g_ahat;
    const uint32_t g = rd_grid(a.units);
    if (vec) hipLaunchKernelGGL(k_rd_grad<true>, dim3(g), dim3(RD_THREADS), 0, s, a);
    else hipLaunchKernelGGL(k_rd_grad<false>, dim3(g), dim3(RD_THREADS), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_ste_pad(const int32_t *info, uint64_t rows, uint32_t C, float *m0, float *m1, float *m2, int64_t *nv,
                          hipStream_t s)
{
    const bool vec = rd_vec(C, {m0, m1, m2});
    const uint64_t units = vec ? rows * C / 4 : rows * C;
    const uint32_t cu = vec ? C / 4 : C;
    const uint64_t b = (units + PAD_THREADS - 1) / PAD_THREADS;
    const dim3 g((uint32_t)(b < 256 ? (b ? b : 1) : 256)), t(PAD_THREADS);  // (few rows are past Nv in a usual frame)
    if (vec) hipLaunchKernelGGL(k_ste_pad<true>, g, t, 0, s, info, units, cu, m0, m1, m2, nv);
    else hipLaunchKernelGGL(k_ste_pad<false>, g, t, 0, s, info, units, cu, m0, m1, m2, nv);
    return hipGetLastError();
}

}  // namespace gsc
