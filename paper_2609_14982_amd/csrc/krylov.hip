// LSQR inner loop over the paired actions (the Krylov least-squares solve of
// Algorithm 1, which calls J and J^T once per iteration at the same
// frozen state, Section 4.5).  The harness solves min ||J x - d|| column by
// column for the B right-hand sides of a batch: model-space vectors are
// [N][B] (one model block shared by all sources, FM_DS_BROADCAST), data-space
// vectors are [S][R][B] (receiver data of every source), so J maps model
// blocks to stacked receiver data and J^T sums over the sources (Section 4.4).
//
// Every per-column scalar lives on the device and every step is a kernel on
// the batch stream: no allocation, no synchronisation and no memset after
// creation, so a whole run of iterations can be captured once as a HIP graph
// and replayed.  Column norms are two-stage reductions with a fixed
// block-to-row assignment and a fixed summation order (deterministic).
//
// The recurrences are the standard LSQR ones (Paige and Saunders):
//   beta_1 u_1 = d, alpha_1 v_1 = J^T u_1, w_1 = v_1, x_0 = 0,
//   phibar_1 = beta_1, rhobar_1 = alpha_1; then per iteration
//   beta u = J v - alpha u;  alpha v = J^T u - beta v;
//   rho = sqrt(rhobar^2 + beta^2), c = rhobar/rho, s = beta/rho,
//   theta = s alpha, rhobar = -c alpha, phi = c phibar, phibar = s phibar,
//   x += (phi/rho) w,  w = v - (theta/rho) w.
//
// CGLS (Hestenes and Stiefel's conjugate gradients on the normal equations,
// in the least-squares form that never forms J^T J) is the inner solver of the
// Gauss-Newton step through the autograd wrapper; per column b:
//   x_0 = 0, r_0 = d, s_0 = J^T r_0, p_0 = s_0, gamma_0 = ||s_0||^2; then
//   q = J p, alpha = gamma / ||q||^2, x += alpha p, r -= alpha q,
//   s = J^T r, gamma' = ||s||^2, beta = gamma' / gamma, p = s + beta p.
// Same device-resident scalars, same capture rules as LSQR.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "batch.h"

namespace fm {

constexpr int kRedBlocks = 512;     // partial sums per column norm
constexpr int kRedThreads = 256;

// per-column scalars, [kScalars][B] doubles on the device
enum : int { sAlpha = 0, sBeta, sRhobar, sPhibar, sRho, sPhi, sTheta, sInvNorm, kScalars };
// CGLS per-column scalars, [kCgScalars][B]
enum : int { cGamma = 0, cQQ, cAlpha, cGnew, cBeta, cRR, kCgScalars };

// What a pass over the rows of a vector does besides adding up its squares.
enum class Row { kRead, kSub, kAxpy };

// partial[blk][b] = sum over this block's rows of y[row][b]^2, of y as it is
// (kRead), after y = x - c y (kSub) or after y -= c x (kAxpy), c = scal[slot]:
// the update and the norm of its result are one pass over memory.  A thread
// keeps its column, so no element pays a division for its index.
template <typename V, Row OP>
__global__ __launch_bounds__(kRedThreads) void k_colsq_partial(std::conditional_t<OP == Row::kRead, const V, V>* __restrict__ y,
                                                                const V* __restrict__ x, int64_t rows, int B,
                                                                const double* __restrict__ scal, int slot,
                                                                double* __restrict__ partial) {
    __shared__ double red[kRedThreads];
    const int per = kRedThreads / B;           // rows per step (B <= 256)
    const int col = threadIdx.x % B;
    const int lr = threadIdx.x / B;
    const int64_t chunk = (rows + gridDim.x - 1) / gridDim.x;
    const int64_t r0 = blockIdx.x * chunk;
    const int64_t r1 = min(rows, r0 + chunk);
    const double c = OP == Row::kRead ? 0.0 : scal[slot * B + col];
    double acc = 0.0;
    if (lr < per)
        for (int64_t r = r0 + lr; r < r1; r += per) {
            const int64_t t = r * B + col;
            V v = y[t];
            if constexpr (OP == Row::kSub) v = (V)((double)x[t] - c * (double)v);
            if constexpr (OP == Row::kAxpy) v = (V)((double)v - c * (double)x[t]);
            if constexpr (OP != Row::kRead) y[t] = v;
            acc += (double)v * (double)v;
        }
    red[threadIdx.x] = (lr < per) ? acc : 0.0;
    __syncthreads();
    if (threadIdx.x < B) {
        double s = 0.0;
        for (int q = 0; q < per; ++q) s += red[q * B + threadIdx.x];
        partial[(int64_t)blockIdx.x * B + threadIdx.x] = s;
    }
}

// The partial sums of a column added up, then the per-column scalars that
// follow from the sum, in one launch of one workgroup.
//   kBeta        LSQR: beta and its inverse
//   kAlphaStart  LSQR: alpha and its inverse, phibar = beta, rhobar = alpha
//   kAlphaRotate LSQR: alpha and its inverse, the plane rotation
//   cStart       CGLS: gamma; the second sums are ||r||^2
//   cStep        CGLS: ||q||^2, alpha (a zero denominator, a converged column,
//                gives a zero step, so the column stays where it is)
//   cDirection   CGLS: ||s||^2, beta, gamma; the second sums are ||r||^2
// A latency chain: with one thread per column adding 512 loads in turn it took
// 122 us (32 columns) and 39 us (one); in parallel 7 us.
enum class Fin { kBeta, kAlphaStart, kAlphaRotate, cStart, cStep, cDirection };

constexpr int kFinThreads = 1024;

template <Fin OP>
__global__ __launch_bounds__(kFinThreads) void k_colsum_finalize(const double* __restrict__ partial, int nblk, int B,
                                                                 double* __restrict__ scal, double* __restrict__ hist,
                                                                 int row) {
    constexpr bool kTwo = OP == Fin::cStart || OP == Fin::cDirection;
    __shared__ double red[kTwo ? 2 : 1][kFinThreads];
    const int per = kFinThreads / B, col = threadIdx.x % B, lr = threadIdx.x / B;
    for (int w = 0; w < (kTwo ? 2 : 1); ++w) {
        double s = 0.0;
        if (lr < per)
            for (int q = lr; q < nblk; q += per) s += partial[((int64_t)w * nblk + q) * B + col];
        red[w][threadIdx.x] = s;
    }
    int half = 1;
    while (half < per) half *= 2;
    for (half /= 2; half > 0; half /= 2) {
        __syncthreads();
        if (lr < half && lr + half < per)
            for (int w = 0; w < (kTwo ? 2 : 1); ++w) red[w][threadIdx.x] += red[w][threadIdx.x + half * B];
    }
    const int b = threadIdx.x;
    if (b >= B) return;
    const double sum = red[0][b];
    if constexpr (OP == Fin::kBeta || OP == Fin::kAlphaStart || OP == Fin::kAlphaRotate) {
        const double n = sqrt(sum);
        scal[(OP == Fin::kBeta ? sBeta : sAlpha) * B + b] = n;
        scal[sInvNorm * B + b] = n > 0.0 ? 1.0 / n : 0.0;
        if constexpr (OP == Fin::kAlphaStart) {
            scal[sPhibar * B + b] = scal[sBeta * B + b];
            scal[sRhobar * B + b] = n;
        }
        if constexpr (OP == Fin::kAlphaRotate) {
            const double alpha = n, beta = scal[sBeta * B + b];
            const double rhobar = scal[sRhobar * B + b], phibar = scal[sPhibar * B + b];
            const double rho = sqrt(rhobar * rhobar + beta * beta);
            const double c = rho > 0.0 ? rhobar / rho : 0.0;
            const double s = rho > 0.0 ? beta / rho : 0.0;
            scal[sRho * B + b] = rho;
            scal[sTheta * B + b] = s * alpha;
            scal[sRhobar * B + b] = -c * alpha;
            scal[sPhi * B + b] = c * phibar;
            scal[sPhibar * B + b] = s * phibar;
        }
    } else if constexpr (OP == Fin::cStep) {
        scal[cQQ * B + b] = sum;
        scal[cAlpha * B + b] = sum > 0.0 ? scal[cGamma * B + b] / sum : 0.0;
    } else {
        if constexpr (OP == Fin::cDirection) {
            const double g = scal[cGamma * B + b];
            scal[cGnew * B + b] = sum;
            scal[cBeta * B + b] = g > 0.0 ? sum / g : 0.0;
        }
        scal[cGamma * B + b] = sum;
        scal[cRR * B + b] = red[1][b];
        if (row >= 0) hist[(int64_t)row * B + b] = red[1][b];
    }
}

// f(element, column) over the elements of a [rows][B] vector
template <class F>
__device__ __forceinline__ void each(int64_t rows, int B, F f) {
    const int64_t n = rows * B, step = (int64_t)gridDim.x * blockDim.x, t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int add = (int)(step % B);
    int b = (int)(t0 % B);
    for (int64_t t = t0; t < n; t += step) {
        f(t, b);
        b += add;
        if (b >= B) b -= B;
    }
}

// x[:, b] *= scal[sInvNorm][b]
template <typename V>
__global__ void k_scale_inv(V* __restrict__ x, int64_t rows, int B, const double* __restrict__ scal) {
    each(rows, B, [&](int64_t t, int b) { x[t] = (V)((double)x[t] * scal[sInvNorm * B + b]); });
}

// v = v / alpha; w = v; x = 0
template <typename V>
__global__ void k_lsqr_first(V* __restrict__ v, V* __restrict__ x, V* __restrict__ w, int64_t rows, int B,
                             const double* __restrict__ scal) {
    each(rows, B, [&](int64_t t, int b) {
        const V vn = (V)((double)v[t] * scal[sInvNorm * B + b]);
        v[t] = vn;
        w[t] = vn;
        x[t] = (V)0;
    });
}

// v = v / alpha; x += (phi/rho) w; w = v - (theta/rho) w
template <typename V>
__global__ void k_lsqr_xw(V* __restrict__ v, V* __restrict__ x, V* __restrict__ w, int64_t rows, int B,
                          const double* __restrict__ scal) {
    each(rows, B, [&](int64_t i, int b) {
        const double rho = scal[sRho * B + b];
        const double fphi = rho > 0.0 ? scal[sPhi * B + b] / rho : 0.0;
        const double fth = rho > 0.0 ? scal[sTheta * B + b] / rho : 0.0;
        const double vn = (double)v[i] * scal[sInvNorm * B + b];
        const double wi = (double)w[i];
        v[i] = (V)vn;
        x[i] = (V)((double)x[i] + fphi * wi);
        w[i] = (V)(vn - fth * wi);
    });
}

template <typename V>
__global__ void k_copy(V* __restrict__ y, const V* __restrict__ x, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) y[i] = x[i];
}

// p = s; x = 0 (a fill without memset, safe inside captured graphs)
template <typename V>
__global__ void k_cgls_first(V* __restrict__ p, V* __restrict__ x, const V* __restrict__ s, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        p[i] = s[i];
        x[i] = (V)0;
    }
}

// x += alpha p, then p = s + beta p (x waits for the end of its iteration, so
// that p is read once)
template <typename V>
__global__ void k_cgls_xp(V* __restrict__ x, V* __restrict__ p, const V* __restrict__ s, int64_t rows, int B,
                          const double* __restrict__ scal) {
    each(rows, B, [&](int64_t i, int b) {
        const double pi = (double)p[i];
        x[i] = (V)((double)x[i] + scal[cAlpha * B + b] * pi);
        p[i] = (V)((double)s[i] + scal[cBeta * B + b] * pi);
    });
}

}  // namespace fm

struct fm_lsqr {
    fm_batch* b = nullptr;
    void* u = nullptr;       // [S][R][B]
    void* td = nullptr;      // [S][R][B] J v
    void* v = nullptr;       // [N][B]
    void* w = nullptr;       // [N][B]
    void* x = nullptr;       // [N][B]
    void* tv = nullptr;      // [N][B] J^T u
    double* scal = nullptr;  // [kScalars][B]
    double* partial = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    int32_t graph_iters = 0;
};

struct fm_cgls {
    fm_batch* b = nullptr;
    void* x = nullptr;       // [N][B]
    void* p = nullptr;       // [N][B]
    void* s = nullptr;       // [N][B] J^T r
    void* r = nullptr;       // [S][R][B]
    void* q = nullptr;       // [S][R][B] J p
    double* scal = nullptr;  // [kCgScalars][B]
    double* partial = nullptr;
    double* hist = nullptr;  // [max_iter + 1][B] ||r||^2 after start and after each iteration
    int32_t max_iter = 0;
    int32_t it = 0;          // iterations enqueued since start (a graph records its own positions)
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

namespace fm {

static int grid_for(int64_t n) { return (int)std::min<int64_t>((n + 255) / 256, 8192); }

template <typename V>
static void colsq(const fm_batch* b, double* partial, const void* y, int64_t rows) {
    hipLaunchKernelGGL((k_colsq_partial<V, Row::kRead>), dim3(kRedBlocks), dim3(kRedThreads), 0, b->stream, (const V*)y,
                       (const V*)nullptr, rows, b->B, (const double*)nullptr, 0, partial);
}

// y = x - c y or y -= c x, and the partial sums of its squares
template <typename V, Row OP>
static void update_sq(const fm_batch* b, double* partial, void* y, const void* x, int64_t rows, const double* scal, int slot) {
    hipLaunchKernelGGL((k_colsq_partial<V, OP>), dim3(kRedBlocks), dim3(kRedThreads), 0, b->stream, (V*)y, (const V*)x,
                       rows, b->B, scal, slot, partial);
}

template <Fin OP>
static void finalize(const fm_batch* b, const double* partial, double* scal, double* hist = nullptr, int row = -1) {
    hipLaunchKernelGGL(k_colsum_finalize<OP>, dim3(1), dim3(kFinThreads), 0, b->stream, partial, kRedBlocks, b->B, scal,
                       hist, row);
}

template <typename V>
static int lsqr_start(fm_lsqr* L, const void* d) {
    fm_batch* b = L->b;
    const int64_t nd = (int64_t)b->S * b->R, nm = b->N;
    hipLaunchKernelGGL(k_copy<V>, dim3(grid_for(nd * b->B)), dim3(256), 0, b->stream, (V*)L->u, (const V*)d, nd * b->B);
    colsq<V>(b, L->partial, L->u, nd);
    finalize<Fin::kBeta>(b, L->partial, L->scal);
    hipLaunchKernelGGL(k_scale_inv<V>, dim3(grid_for(nd * b->B)), dim3(256), 0, b->stream, (V*)L->u, nd, b->B,
                       (const double*)L->scal);
    int rc = apply_JT(b, L->u, FM_W_RECEIVERS, L->v, FM_JT_SUMMED);
    if (rc) return rc;
    colsq<V>(b, L->partial, L->v, nm);
    finalize<Fin::kAlphaStart>(b, L->partial, L->scal);
    hipLaunchKernelGGL(k_lsqr_first<V>, dim3(grid_for(nm * b->B)), dim3(256), 0, b->stream, (V*)L->v, (V*)L->x, (V*)L->w,
                       nm, b->B, (const double*)L->scal);
    return hipGetLastError() == hipSuccess ? FM_OK : FM_EHIP;
}

template <typename V>
static int lsqr_iterate(fm_lsqr* L, int n) {
    fm_batch* b = L->b;
    const int64_t nd = (int64_t)b->S * b->R, nm = b->N;
    for (int it = 0; it < n; ++it) {
        int rc = apply_J(b, L->v, FM_DS_BROADCAST, L->td, FM_OUT_RECEIVERS);
        if (rc) return rc;
        update_sq<V, Row::kSub>(b, L->partial, L->u, L->td, nd, L->scal, sAlpha);
        finalize<Fin::kBeta>(b, L->partial, L->scal);
        hipLaunchKernelGGL(k_scale_inv<V>, dim3(grid_for(nd * b->B)), dim3(256), 0, b->stream, (V*)L->u, nd, b->B,
                           (const double*)L->scal);
        rc = apply_JT(b, L->u, FM_W_RECEIVERS, L->tv, FM_JT_SUMMED);
        if (rc) return rc;
        update_sq<V, Row::kSub>(b, L->partial, L->v, L->tv, nm, L->scal, sBeta);
        finalize<Fin::kAlphaRotate>(b, L->partial, L->scal);
        hipLaunchKernelGGL(k_lsqr_xw<V>, dim3(grid_for(nm * b->B)), dim3(256), 0, b->stream, (V*)L->v, (V*)L->x,
                           (V*)L->w, nm, b->B, (const double*)L->scal);
        if (hipGetLastError() != hipSuccess) { set_error("LSQR kernel launch failed"); return FM_EHIP; }
    }
    return FM_OK;
}

static void lsqr_release(fm_lsqr* L) {
    if (!L) return;
    if (L->exec) (void)hipGraphExecDestroy(L->exec);
    if (L->graph) (void)hipGraphDestroy(L->graph);
    void* bufs[] = {L->u, L->td, L->v, L->w, L->x, L->tv, L->scal, L->partial};
    for (void* p : bufs)
        if (p) (void)hipFree(p);
    delete L;
}

int lsqr_create(fm_batch* b, fm_lsqr** out) {
    if (!b || !out) { set_error("null argument"); return FM_EINVAL; }
    *out = nullptr;
    if (b->R == 0) { set_error("the states have no receivers"); return FM_EINVAL; }
    if (b->B > 256) { set_error("LSQR supports at most 256 right-hand sides"); return FM_EINVAL; }
    fm_lsqr* L = new fm_lsqr();
    L->b = b;
    const size_t vb = b->prec == FM_FP64 ? 8 : 4;
    const size_t nd = (size_t)b->S * b->R * b->B * vb, nm = (size_t)b->N * b->B * vb;
    hipError_t e = hipSuccess;
    void** targets[] = {&L->u, &L->td, &L->v, &L->w, &L->x, &L->tv};
    size_t sizes[] = {nd, nd, nm, nm, nm, nm};
    for (int i = 0; i < 6 && e == hipSuccess; i++) e = hipMalloc(targets[i], sizes[i]);
    if (e == hipSuccess) e = hipMalloc((void**)&L->scal, sizeof(double) * kScalars * b->B);
    if (e == hipSuccess) e = hipMalloc((void**)&L->partial, sizeof(double) * kRedBlocks * b->B);
    if (e != hipSuccess) {
        lsqr_release(L);
        set_error("LSQR allocation failed: %s", hipGetErrorString(e));
        return e == hipErrorOutOfMemory ? FM_ENOMEM : FM_EHIP;
    }
    *out = L;
    return FM_OK;
}

int lsqr_start_any(fm_lsqr* L, const void* d) {
    if (!L || !d) { set_error("null argument"); return FM_EINVAL; }
    return L->b->prec == FM_FP64 ? lsqr_start<double>(L, d) : lsqr_start<float>(L, d);
}

int lsqr_iterate_any(fm_lsqr* L, int32_t n) {
    if (!L || n < 0) { set_error("bad arguments"); return FM_EINVAL; }
    return L->b->prec == FM_FP64 ? lsqr_iterate<double>(L, n) : lsqr_iterate<float>(L, n);
}

int lsqr_capture(fm_lsqr* L, int32_t n) {
    if (!L || n < 1) { set_error("bad arguments"); return FM_EINVAL; }
    if (L->exec) { (void)hipGraphExecDestroy(L->exec); L->exec = nullptr; }
    if (L->graph) { (void)hipGraphDestroy(L->graph); L->graph = nullptr; }
    hipStream_t s = L->b->stream;
    if (s == nullptr) { set_error("graph capture needs a non-null batch stream"); return FM_EINVAL; }
    HIP_TRY(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
    int rc = lsqr_iterate_any(L, n);
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(s, &g);
    if (rc) { if (g) (void)hipGraphDestroy(g); return rc; }
    if (e != hipSuccess) { set_error("hipStreamEndCapture failed: %s", hipGetErrorString(e)); return FM_EHIP; }
    e = hipGraphInstantiate(&L->exec, g, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        (void)hipGraphDestroy(g);
        set_error("hipGraphInstantiate failed: %s", hipGetErrorString(e));
        return FM_EHIP;
    }
    L->graph = g;
    L->graph_iters = n;
    return FM_OK;
}

int lsqr_replay(fm_lsqr* L) {
    if (!L || !L->exec) { set_error("no captured graph"); return FM_ESTATE; }
    HIP_TRY(hipGraphLaunch(L->exec, L->b->stream));
    return FM_OK;
}

int lsqr_buffers(const fm_lsqr* L, void** x, void** u, void** v, double** scal) {
    if (!L) { set_error("null argument"); return FM_EINVAL; }
    if (x) *x = L->x;
    if (u) *u = L->u;
    if (v) *v = L->v;
    if (scal) *scal = L->scal;
    return FM_OK;
}

void lsqr_free(fm_lsqr* L) { lsqr_release(L); }

// ---------------------------------------------------------------------------
// CGLS
// ---------------------------------------------------------------------------
// (the second half of the partial sums is the residual's)
template <typename V>
static int cgls_start(fm_cgls* C, const void* d) {
    fm_batch* b = C->b;
    const int64_t nd = (int64_t)b->S * b->R, nm = b->N;
    double* const partial_r = C->partial + (size_t)kRedBlocks * b->B;
    hipLaunchKernelGGL(k_copy<V>, dim3(grid_for(nd * b->B)), dim3(256), 0, b->stream, (V*)C->r, (const V*)d, nd * b->B);
    int rc = apply_JT(b, C->r, FM_W_RECEIVERS, C->s, FM_JT_SUMMED);
    if (rc) return rc;
    hipLaunchKernelGGL(k_cgls_first<V>, dim3(grid_for(nm * b->B)), dim3(256), 0, b->stream, (V*)C->p, (V*)C->x,
                       (const V*)C->s, nm * b->B);
    colsq<V>(b, C->partial, C->s, nm);
    colsq<V>(b, partial_r, C->r, nd);
    C->it = 0;
    finalize<Fin::cStart>(b, C->partial, C->scal, C->hist, 0);
    if (hipGetLastError() != hipSuccess) { set_error("CGLS kernel launch failed"); return FM_EHIP; }
    return FM_OK;
}

template <typename V>
static int cgls_iterate(fm_cgls* C, int n) {
    fm_batch* b = C->b;
    const int64_t nd = (int64_t)b->S * b->R, nm = b->N;
    double* const partial_r = C->partial + (size_t)kRedBlocks * b->B;
    for (int it = 0; it < n; ++it) {
        int rc = apply_J(b, C->p, FM_DS_BROADCAST, C->q, FM_OUT_RECEIVERS);
        if (rc) return rc;
        colsq<V>(b, C->partial, C->q, nd);
        finalize<Fin::cStep>(b, C->partial, C->scal);
        update_sq<V, Row::kAxpy>(b, partial_r, C->r, C->q, nd, C->scal, cAlpha);
        rc = apply_JT(b, C->r, FM_W_RECEIVERS, C->s, FM_JT_SUMMED);
        if (rc) return rc;
        colsq<V>(b, C->partial, C->s, nm);
        ++C->it;
        finalize<Fin::cDirection>(b, C->partial, C->scal, C->hist, C->it <= C->max_iter ? C->it : -1);
        hipLaunchKernelGGL(k_cgls_xp<V>, dim3(grid_for(nm * b->B)), dim3(256), 0, b->stream, (V*)C->x, (V*)C->p,
                           (const V*)C->s, nm, b->B, (const double*)C->scal);
        if (hipGetLastError() != hipSuccess) { set_error("CGLS kernel launch failed"); return FM_EHIP; }
    }
    return FM_OK;
}

static void cgls_release(fm_cgls* C) {
    if (!C) return;
    if (C->exec) (void)hipGraphExecDestroy(C->exec);
    if (C->graph) (void)hipGraphDestroy(C->graph);
    void* bufs[] = {C->x, C->p, C->s, C->r, C->q, C->scal, C->partial, C->hist};
    for (void* p : bufs)
        if (p) (void)hipFree(p);
    delete C;
}

int cgls_create(fm_batch* b, int32_t max_iter, fm_cgls** out) {
    if (!b || !out) { set_error("null argument"); return FM_EINVAL; }
    if (max_iter < 0) { set_error("max_iter must be >= 0"); return FM_EINVAL; }
    *out = nullptr;
    if (b->R == 0) { set_error("the states have no receivers"); return FM_EINVAL; }
    if (b->B > 256) { set_error("CGLS supports at most 256 right-hand sides"); return FM_EINVAL; }
    fm_cgls* C = new fm_cgls();
    C->b = b;
    C->max_iter = max_iter;
    const size_t vb = b->prec == FM_FP64 ? 8 : 4;
    const size_t nd = (size_t)b->S * b->R * b->B * vb, nm = (size_t)b->N * b->B * vb;
    hipError_t e = hipSuccess;
    void** targets[] = {&C->x, &C->p, &C->s, &C->r, &C->q};
    size_t sizes[] = {nm, nm, nm, nd, nd};
    for (int i = 0; i < 5 && e == hipSuccess; i++) e = hipMalloc(targets[i], sizes[i]);
    if (e == hipSuccess) e = hipMalloc((void**)&C->scal, sizeof(double) * kCgScalars * b->B);
    if (e == hipSuccess) e = hipMalloc((void**)&C->partial, sizeof(double) * 2 * kRedBlocks * b->B);
    if (e == hipSuccess) e = hipMalloc((void**)&C->hist, sizeof(double) * ((size_t)max_iter + 1) * b->B);
    if (e != hipSuccess) {
        cgls_release(C);
        set_error("CGLS allocation failed: %s", hipGetErrorString(e));
        return e == hipErrorOutOfMemory ? FM_ENOMEM : FM_EHIP;
    }
    *out = C;
    return FM_OK;
}

int cgls_start_any(fm_cgls* C, const void* d) {
    if (!C || !d) { set_error("null argument"); return FM_EINVAL; }
    return C->b->prec == FM_FP64 ? cgls_start<double>(C, d) : cgls_start<float>(C, d);
}

int cgls_iterate_any(fm_cgls* C, int32_t n) {
    if (!C || n < 0) { set_error("bad arguments"); return FM_EINVAL; }
    return C->b->prec == FM_FP64 ? cgls_iterate<double>(C, n) : cgls_iterate<float>(C, n);
}

int cgls_capture(fm_cgls* C, int32_t n) {
    if (!C || n < 1) { set_error("bad arguments"); return FM_EINVAL; }
    if (C->exec) { (void)hipGraphExecDestroy(C->exec); C->exec = nullptr; }
    if (C->graph) { (void)hipGraphDestroy(C->graph); C->graph = nullptr; }
    hipStream_t s = C->b->stream;
    if (s == nullptr) { set_error("graph capture needs a non-null batch stream"); return FM_EINVAL; }
    HIP_TRY(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
    int rc = cgls_iterate_any(C, n);
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(s, &g);
    if (rc) { if (g) (void)hipGraphDestroy(g); return rc; }
    if (e != hipSuccess) { set_error("hipStreamEndCapture failed: %s", hipGetErrorString(e)); return FM_EHIP; }
    e = hipGraphInstantiate(&C->exec, g, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        (void)hipGraphDestroy(g);
        set_error("hipGraphInstantiate failed: %s", hipGetErrorString(e));
        return FM_EHIP;
    }
    C->graph = g;
    return FM_OK;
}

int cgls_replay(fm_cgls* C) {
    if (!C || !C->exec) { set_error("no captured graph"); return FM_ESTATE; }
    HIP_TRY(hipGraphLaunch(C->exec, C->b->stream));
    return FM_OK;
}

int cgls_buffers(const fm_cgls* C, void** x, void** r, double** scal, double** hist) {
    if (!C) { set_error("null argument"); return FM_EINVAL; }
    if (x) *x = C->x;
    if (r) *r = C->r;
    if (scal) *scal = C->scal;
    if (hist) *hist = C->hist;
    return FM_OK;
}

void cgls_free(fm_cgls* C) { cgls_release(C); }

}  // namespace fm
