// Vector kernels of the CGLS loop (conjugate gradients on min ||b - A x||_2),
// the first-order use of the two products that the paper's closing section
// describes: each iteration is one product with A, one with A^T, and a few
// passes of vector updates and inner products, which this file fuses.
//
// The product with A is taken of s = A^T r, and q = A p is formed from it by
// linearity (p = s + beta p, so q = A s + beta q).  This leaves the update of
// the two long vectors (p, then x) free to run right before the A^T r product,
// whose scattered gathers leave memory bandwidth to spare for writing them
// back, instead of right before the A p product, whose streaming they slowed.
//
// Every inner product is formed in a fixed order, so a solve is bit-identical
// from run to run: dot_parts(len) workgroups each sum a fixed contiguous range
// (thread t adds elements t, t + BLOCK, ... of the range in order, then a
// fixed butterfly inside each wave and the waves in ascending order), and whoever needs
// the product adds those partial sums the same way.  The step sizes stay on the
// device, so the loop never waits for the host.
//
// On small and ordinary matrices the loop is bound by its chain of short kernels, so
// the partial sums are finished by the kernel that uses them, not by a launch of one
// workgroup in between: every workgroup of a short-vector pass adds the partial sums
// itself (they are few for a short vector), and its first one writes the history entry
// and the step size down for the passes over the long vectors.  Four vector launches an
// iteration instead of seven, and the residual is written in the order the next
// product reads it: ten iterations on 10,007 x 500,000 with 5e6 nonzeros 790 -> 684 us.
//
// Scalars (binary64): [0] alpha, [1] beta of the iteration.  gamma_k = ||A^T r_k||^2 and
// ||r_k||^2 live in the histories.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "spw_internal.h"

namespace spw {
namespace {

constexpr int SV_BLOCK = 256;
constexpr int SV_WAVE = 64;
constexpr int DOT_PARTS = 1024;          // partial sums per inner product, at most (one per workgroup)
constexpr int S_ALPHA = 0, S_BETA = 1;

// Partial sums of an inner product over len elements: one per 2,048, so that a short
// vector has few of them to add up.
__host__ __device__ inline int dot_parts(int64_t len)
{
    const int64_t p = (len + 2047) / 2048;
    return (int)(p < 1 ? 1 : p > DOT_PARTS ? DOT_PARTS : p);
}

// Sum of one value per thread over a workgroup of SV_BLOCK threads, in a fixed
// order: butterfly inside each wave, then the waves in ascending order.  Every
// thread gets it.
__device__ __forceinline__ double block_sum(double v, double *lds)
{
    for (int off = SV_WAVE / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, SV_WAVE);
    const int wave = threadIdx.x / SV_WAVE, lane = threadIdx.x % SV_WAVE;
    __syncthreads();                     // an earlier sum has been read
    if (lane == 0) lds[wave] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < SV_BLOCK / SV_WAVE; ++w) s += lds[w];
    return s;
}

// The inner product whose partial sums these are.
__device__ __forceinline__ double finish_dot(const double *__restrict__ partial, int parts, double *lds)
{
    double acc = 0.0;
    for (int i = threadIdx.x; i < parts; i += SV_BLOCK) acc += partial[i];
    return block_sum(acc, lds);
}

// Range of workgroup g out of parts over len elements.
__device__ __forceinline__ void part_range(int64_t len, int64_t &a, int64_t &e)
{
    a = len * (int64_t)blockIdx.x / (int64_t)gridDim.x;
    e = len * ((int64_t)blockIdx.x + 1) / (int64_t)gridDim.x;
}

// partial[g] = sum over workgroup g's range of a_i * a_i.  Eight loads are
// issued before their squares are added (in the same order as one at a time),
// so that more bytes are in flight.
__global__ __launch_bounds__(SV_BLOCK) void sq_part(const double *__restrict__ a, int64_t len,
                                                    double *__restrict__ partial)
{
    __shared__ double lds[SV_BLOCK / SV_WAVE];
    int64_t s, e;
    part_range(len, s, e);
    double acc = 0.0;
    int64_t i = s + threadIdx.x;
    for (; i + 7 * SV_BLOCK < e; i += 8 * SV_BLOCK) {
        double t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = a[i + u * SV_BLOCK];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += t[u] * t[u];
    }
    for (; i < e; i += SV_BLOCK) acc += a[i] * a[i];
    const double t = block_sum(acc, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// gamma_k from the partial sums of s; beta_k = gamma_k / gamma_{k-1} (0 for k = 0 and when
// gamma_{k-1} is 0).  The first workgroup writes both down.
__device__ __forceinline__ double finish_gamma(const double *__restrict__ spart, int sparts, int64_t k,
                                               double *__restrict__ hist_gamma, double *__restrict__ scal, double *lds)
{
    const double gamma = finish_dot(spart, sparts, lds);
    const double before = k > 0 ? hist_gamma[k - 1] : 0.0;
    const double beta = before > 0.0 ? gamma / before : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        hist_gamma[k] = gamma;
        scal[S_BETA] = beta;
    }
    return beta;
}

// One workgroup: gamma_k and beta_k, where no short-vector pass follows that finishes them.
__global__ __launch_bounds__(SV_BLOCK) void gamma_step(const double *__restrict__ spart, int sparts, int64_t k,
                                                       double *__restrict__ hist_gamma, double *__restrict__ scal)
{
    __shared__ double lds[SV_BLOCK / SV_WAVE];
    finish_gamma(spart, sparts, k, hist_gamma, scal, lds);
}

// One workgroup: out[0] = the inner product.
__global__ __launch_bounds__(SV_BLOCK) void dot_step(const double *__restrict__ partial, int parts,
                                                     double *__restrict__ out)
{
    __shared__ double lds[SV_BLOCK / SV_WAVE];
    const double sum = finish_dot(partial, parts, lds);
    if (threadIdx.x == 0) out[0] = sum;
}

// DIRECT: q = t.  Otherwise q = t + beta_k q.  Either way partial[g] = sum of
// q_i * q_i of the new q over workgroup g's range.  GAMMA: gamma_k (and beta_k) are
// finished here, else they have been (gamma_step).
template <bool DIRECT, bool GAMMA>
__global__ __launch_bounds__(SV_BLOCK) void q_step(double *__restrict__ q, const double *__restrict__ t, int64_t len,
                                                   const double *__restrict__ spart, int sparts, int64_t k,
                                                   double *__restrict__ hist_gamma, double *__restrict__ scal,
                                                   double *__restrict__ partial)
{
    __shared__ double lds[SV_BLOCK / SV_WAVE];
    double beta = 0.0;
    if (GAMMA) beta = finish_gamma(spart, sparts, k, hist_gamma, scal, lds);
    int64_t s, e;
    part_range(len, s, e);
    double acc = 0.0;
    for (int64_t i = s + threadIdx.x; i < e; i += SV_BLOCK) {
        const double qi = DIRECT ? t[i] : t[i] + beta * q[i];
        q[i] = qi;
        acc += qi * qi;
    }
    const double sum = block_sum(acc, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = sum;
}

// r = b - q, partial[g] = sum of r_i * r_i of the new r over workgroup g's range.
__global__ __launch_bounds__(SV_BLOCK) void r_init(double *__restrict__ r, const double *__restrict__ b,
                                                   const double *__restrict__ q, int64_t len,
                                                   double *__restrict__ partial)
{
    __shared__ double lds[SV_BLOCK / SV_WAVE];
    int64_t s, e;
    part_range(len, s, e);
    double acc = 0.0;
    for (int64_t i = s + threadIdx.x; i < e; i += SV_BLOCK) {
        const double ri = b[i] - q[i];
        r[i] = ri;
        acc += ri * ri;
    }
    const double t = block_sum(acc, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// alpha = gamma_k / ||q||^2 (0 when either is 0), r = r - alpha q, partial[g] = sum of
// r_i * r_i of the new r over workgroup g's range.  rank (may be NULL): r is also written to
// perm in the matrix's own row order, which the next product reads.
__global__ __launch_bounds__(SV_BLOCK) void r_step(double *__restrict__ r, const double *__restrict__ q, int64_t len,
                                                   const double *__restrict__ qpart, int qparts, int64_t k,
                                                   const double *__restrict__ hist_gamma, double *__restrict__ scal,
                                                   const int32_t *__restrict__ rank, double *__restrict__ perm,
                                                   double *__restrict__ partial)
{
    __shared__ double lds[SV_BLOCK / SV_WAVE];
    const double delta = finish_dot(qpart, qparts, lds);
    const double gamma = hist_gamma[k];
    const double alpha = (gamma > 0.0 && delta > 0.0) ? gamma / delta : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) scal[S_ALPHA] = alpha;
    int64_t s, e;
    part_range(len, s, e);
    double acc = 0.0;
    for (int64_t i = s + threadIdx.x; i < e; i += SV_BLOCK) {
        const double ri = r[i] - alpha * q[i];
        r[i] = ri;
        if (rank) perm[rank[i]] = ri;
        acc += ri * ri;
    }
    const double t = block_sum(acc, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// ||r||^2 of the iteration, by the first workgroup of a pass over the long vectors.
__device__ __forceinline__ void finish_rho(const double *__restrict__ rpart, int rparts, double *__restrict__ rho)
{
    __shared__ double lds[SV_BLOCK / SV_WAVE];
    if (blockIdx.x != 0) return;
    const double sum = finish_dot(rpart, rparts, lds);
    if (threadIdx.x == 0) *rho = sum;
}

// p = s + beta p (FIRST: p = s), then x = x + alpha p with the new p: one
// pass over the three long vectors.
template <bool FIRST>
__global__ __launch_bounds__(SV_BLOCK) void px_step(double *__restrict__ x, double *__restrict__ p,
                                                    const double *__restrict__ s, int64_t len,
                                                    const double *__restrict__ scal, const double *__restrict__ rpart,
                                                    int rparts, double *__restrict__ rho)
{
    const double alpha = scal[S_ALPHA], beta = FIRST ? 0.0 : scal[S_BETA];
    finish_rho(rpart, rparts, rho);
    const int64_t stride = (int64_t)gridDim.x * SV_BLOCK;
    for (int64_t i = blockIdx.x * (int64_t)SV_BLOCK + threadIdx.x; i < len; i += stride) {
        const double pi = FIRST ? s[i] : s[i] + beta * p[i];
        p[i] = pi;
        x[i] = x[i] + alpha * pi;
    }
}

// The two halves of px_step for an iteration that forms q = A p directly:
// p = s + beta p before the product, x = x + alpha p after alpha is known.
__global__ __launch_bounds__(SV_BLOCK) void p_step(double *__restrict__ p, const double *__restrict__ s, int64_t len,
                                                   const double *__restrict__ scal)
{
    const double beta = scal[S_BETA];
    const int64_t stride = (int64_t)gridDim.x * SV_BLOCK;
    for (int64_t i = blockIdx.x * (int64_t)SV_BLOCK + threadIdx.x; i < len; i += stride) p[i] = s[i] + beta * p[i];
}

__global__ __launch_bounds__(SV_BLOCK) void x_step(double *__restrict__ x, const double *__restrict__ p, int64_t len,
                                                   const double *__restrict__ scal, const double *__restrict__ rpart,
                                                   int rparts, double *__restrict__ rho)
{
    const double alpha = scal[S_ALPHA];
    finish_rho(rpart, rparts, rho);
    const int64_t stride = (int64_t)gridDim.x * SV_BLOCK;
    for (int64_t i = blockIdx.x * (int64_t)SV_BLOCK + threadIdx.x; i < len; i += stride) x[i] = x[i] + alpha * p[i];
}

unsigned stream_grid(int64_t len)
{
    const int64_t g = (len + SV_BLOCK - 1) / SV_BLOCK;
    return (unsigned)(g < 1 ? 1 : (g > 16384 ? 16384 : g));
}

}  // namespace

// Partial sums of the three inner products of an iteration (q, r, s).
int64_t cgls_partials() { return 3 * DOT_PARTS; }

int launch_cgls_vec(CglsVecOp op, const CglsWork &w, int64_t k, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    double *qpart = w.partial, *rpart = w.partial + DOT_PARTS, *spart = w.partial + 2 * DOT_PARTS;
    const int mp = dot_parts(w.m), np = dot_parts(w.n);
    const dim3 block(SV_BLOCK);
    switch (op) {
    case CglsVecOp::R_INIT:     // r = b - q, rho_0
        hipLaunchKernelGGL(r_init, dim3(mp), block, 0, st, w.r, w.b, w.q, w.m, rpart);
        hipLaunchKernelGGL(dot_step, dim3(1), block, 0, st, rpart, mp, w.hist_rho);
        break;
    case CglsVecOp::S_NORM:     // the partial sums of ||s||^2
        hipLaunchKernelGGL(sq_part, dim3(np), block, 0, st, w.s, w.n, spart);
        break;
    case CglsVecOp::GAMMA:      // gamma_k, beta_k
        hipLaunchKernelGGL(gamma_step, dim3(1), block, 0, st, spart, np, k, w.hist_gamma, w.scal);
        break;
    case CglsVecOp::Q_FIRST:    // gamma_k, q = t
        hipLaunchKernelGGL((q_step<true, true>), dim3(mp), block, 0, st, w.q, w.t, w.m, spart, np, k, w.hist_gamma,
                           w.scal, qpart);
        break;
    case CglsVecOp::Q:          // gamma_k, beta_k, q = t + beta q
        hipLaunchKernelGGL((q_step<false, true>), dim3(mp), block, 0, st, w.q, w.t, w.m, spart, np, k, w.hist_gamma,
                           w.scal, qpart);
        break;
    case CglsVecOp::Q_DIRECT:   // q = t
        hipLaunchKernelGGL((q_step<true, false>), dim3(mp), block, 0, st, w.q, w.t, w.m, spart, np, k, w.hist_gamma,
                           w.scal, qpart);
        break;
    case CglsVecOp::R:          // alpha, r = r - alpha q
        hipLaunchKernelGGL(r_step, dim3(mp), block, 0, st, w.r, w.q, w.m, qpart, mp, k, w.hist_gamma, w.scal, w.rank,
                           w.perm, rpart);
        break;
    case CglsVecOp::PX_FIRST:   // rho_{k+1}, p = s, x = x + alpha p
        hipLaunchKernelGGL(px_step<true>, dim3(stream_grid(w.n)), block, 0, st, w.x, w.p, w.s, w.n, w.scal, rpart, mp,
                           w.hist_rho + k + 1);
        break;
    case CglsVecOp::PX:         // rho_{k+1}, p = s + beta p, x = x + alpha p
        hipLaunchKernelGGL(px_step<false>, dim3(stream_grid(w.n)), block, 0, st, w.x, w.p, w.s, w.n, w.scal, rpart, mp,
                           w.hist_rho + k + 1);
        break;
    case CglsVecOp::P:          // p = s + beta p
        hipLaunchKernelGGL(p_step, dim3(stream_grid(w.n)), block, 0, st, w.p, w.s, w.n, w.scal);
        break;
    case CglsVecOp::X:          // rho_{k+1}, x = x + alpha p
        hipLaunchKernelGGL(x_step, dim3(stream_grid(w.n)), block, 0, st, w.x, w.p, w.n, w.scal, rpart, mp,
                           w.hist_rho + k + 1);
        break;
    }
    return (int)hipGetLastError();
}

}  // namespace spw
