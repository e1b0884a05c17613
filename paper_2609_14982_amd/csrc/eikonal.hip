// First-arrival traveltimes on the GPU: the state of Section 2.1, T the
// viscosity solution of |grad_x T| = s with T = 0 at the source, computed for
// S sources at once before the tangent setup (Algorithm 1, Phase I).
//
// Discretisation (the paper only cites its factored solver): a monotone
// semi-Lagrangian update on the boundary-conforming grid.  Node i's stencil
// is its face neighbours (one logical step along each axis); its simplices
// are the neighbours, the segments joining neighbours on two different axes
// and, in 3-D, the triangles with one neighbour per axis.  The update is
//   T_i = min over simplices S, min over y in S, of T_S(y) + s_i |x_i - y|,
// T_S linear over S, x the physical node positions.  The inner minimum is
// convex in the barycentric coordinates: it is the least of the vertex
// values, the stationary points inside the segments, and the stationary
// points inside the triangles, all in closed form.  The update is monotone
// in the neighbour values, so from T = +inf off the seeds every iteration
// order decreases T to the same (largest) fixed point; here it is Jacobi
// iteration, T^{n+1} = min(T^n, F(T^n)), double-buffered, until an
// iteration changes nothing.
//
// Seeds: the nodes within max-norm logical distance rho of the source's
// logical coordinates xi keep the straight-ray time
// (s_src + s_p)/2 |x_p - x_src|, s_src and x_src multilinear over xi's cell
// (a source on a node is the case of integer xi).
//
// Work per iteration: a node is recomputed only when a neighbour changed in
// the previous iteration (one bit per node and source, the word of 64 nodes the
// unit); the others keep their value, which the buffer being written already
// holds unless the node changed in the previous iteration.  The per-iteration
// amount of work of each is read by the host once per chunk of iterations.  Built with
// -ffp-contract=off: every product and sum is rounded as written.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "fmbtf.h"
#include "devmem.h"
#include "internal.h"
#include "batch.h"

struct fm_eikonal {
    int dim = 3;
    int64_t n[3] = {1, 1, 1};
    int64_t N = 0;
    int32_t S = 0;                  // capacity in sources
    fm::DevBlocks block;            // holds the device arrays below
    double* X = nullptr;            // device [N][dim]
    double* Tb = nullptr;           // device [S][N] second buffer
    int64_t W = 0;                  // words of 64 nodes per source (a multiple of kTile)
    // (not on small grids:)
    uint16_t* list = nullptr;       // device [S][W / 64][4096] nodes of a tile to recompute
    int32_t* count = nullptr;       // device [S][W / 64] their number
    uint32_t* batch = nullptr;      // device [S][W] batches of 64 of them: tile * 64 + batch
    uint64_t* chg[2] = {nullptr, nullptr};   // device [S][W] nodes changed by the last iteration
    uint64_t* seed = nullptr;       // device [S][W] seed nodes
    uint64_t* edge = nullptr;       // device [4][W] nodes with a lower / upper neighbour on axes 0 and 1
    double* xi = nullptr;           // device [S][3]
    unsigned* n_batch = nullptr;    // device [kChunk + 1] batches of each iteration of a chunk and the next
    unsigned* n_batch_h = nullptr;  // pinned host copy
    hipStream_t stream = nullptr;
    int device = -1;
    int waves = 0;                  // waves of an iteration's recomputation
};

namespace fm {

namespace {

constexpr int kChunk = 16;          // iterations between convergence checks
constexpr int kTile = 64;           // words of 64 nodes listed by one wave
constexpr int kThreads = 256;
// Words (all sources) up to which an iteration is one launch, k_eik_word.  A
// whole solve with it and with the lists: 2-D 401x201, 1, 4, 8 and 16 sources
// (1280 words each) 4.3 and 7.4 ms, 7.1 and 9.7, 9.7 and 10.4, 14.4 and 11.5; 3-D
// 41x41x25, 1, 2, 4 and 8 sources (704 words each) 1.9 and 2.7, 2.6 and 3.0, 3.4
// and 3.5, 4.8 and 4.1; 60x60x35, 1 and 2 sources (1984 each) 3.3 and 3.8, 4.9 and
// 4.6.  (One lane per node and a state byte, on the same sizes: 401x201, 1, 4 and
// 16 sources 3.9, 8.6 and 23.9 ms; 41x41x25, 1, 4 and 16 2.1, 3.8 and 8.5; 77x40, 3
// sources 1.24 against 1.07 with k_eik_word.)
constexpr int64_t kSmall2 = 8192, kSmall3 = 2048;
bool is_small(int dim, int64_t words) { return words <= (dim == 3 ? kSmall3 : kSmall2); }
constexpr uint16_t kCopy = 1u << 15;   // list entry: the value is only copied

struct EikDims {
    int dim;
    int64_t n0, n1, n2, N, W;
};

__device__ __forceinline__ void logical(const EikDims& d, int64_t p, int64_t c[3]) {
    c[0] = p % d.n0;
    const int64_t r = p / d.n0;
    c[1] = r % d.n1;
    c[2] = r / d.n1;
}

__device__ __forceinline__ double dist(const double* a, const double* b, int dim) {
    double acc = 0.0;
    for (int k = 0; k < dim; ++k) {
        const double t = a[k] - b[k];
        acc = acc + t * t;
    }
    return sqrt(acc);
}

__device__ __forceinline__ double dot(const double* a, const double* b, int dim) {
    double acc = 0.0;
    for (int k = 0; k < dim; ++k) acc = acc + a[k] * b[k];
    return acc;
}

// Stationary point inside the segment [x1, x2] of t(y) + si |xi - y| (t
// linear, t1 at x1, t2 at x2), or +inf when there is none inside.  With
// e = x2 - x1, d0 = xi - x1, a = |e|^2, b = d0.e, delta = t2 - t1: the
// distance from xi to the segment's line is rperp, and at the stationary
// point |xi - y| = rperp / sqrt(1 - delta^2 / (a si^2)) and
// lambda = b/a - (|xi - y| / si) delta / a.
__device__ __forceinline__ double seg_inner(const double* xi, double si, const double* x1, double t1,
                                           const double* x2, double t2, int dim) {
    if (!(t1 < INFINITY) || !(t2 < INFINITY)) return INFINITY;
    double e[3], d0[3];
    for (int k = 0; k < dim; ++k) { e[k] = x2[k] - x1[k]; d0[k] = xi[k] - x1[k]; }
    const double a = dot(e, e, dim), b = dot(d0, e, dim), c = dot(d0, d0, dim);
    const double delta = t2 - t1;
    if (!(a * si * si > delta * delta)) return INFINITY;
    const double rperp2 = fmax(c - b * b / a, 0.0);
    const double rn = sqrt(rperp2) / sqrt(1.0 - delta * delta / (a * si * si));
    const double lam = b / a - (rn / si) * delta / a;
    if (!(lam > 0.0 && lam < 1.0)) return INFINITY;
    return t1 + lam * delta + si * rn;
}

// Stationary point inside the triangle (x1, x2, x3), or +inf.  With
// E = [x2 - x1, x3 - x1], Gm = E^T E, mu = Gm^{-1} E^T (xi - x1) (the
// projection of xi), delta = (t2 - t1, t3 - t1), q = delta^T Gm^{-1} delta:
// |xi - y| = rperp / sqrt(1 - q / si^2), lambda = mu - (|xi - y| / si) Gm^{-1} delta.
__device__ __forceinline__ double tri_inner(const double* xi, double si, const double* x1, double t1,
                                           const double* x2, double t2, const double* x3, double t3) {
    if (!(t1 < INFINITY) || !(t2 < INFINITY) || !(t3 < INFINITY)) return INFINITY;
    double e2[3], e3[3], d0[3];
    for (int k = 0; k < 3; ++k) { e2[k] = x2[k] - x1[k]; e3[k] = x3[k] - x1[k]; d0[k] = xi[k] - x1[k]; }
    const double g22 = dot(e2, e2, 3), g23 = dot(e2, e3, 3), g33 = dot(e3, e3, 3);
    const double h2 = dot(e2, d0, 3), h3 = dot(e3, d0, 3);
    const double det = g22 * g33 - g23 * g23;
    if (!(det > 0.0)) return INFINITY;
    const double mu2 = (g33 * h2 - g23 * h3) / det;
    const double mu3 = (g22 * h3 - g23 * h2) / det;
    const double rperp2 = fmax(dot(d0, d0, 3) - (mu2 * h2 + mu3 * h3), 0.0);
    const double d2 = t2 - t1, d3 = t3 - t1;
    const double i2 = (g33 * d2 - g23 * d3) / det;
    const double i3 = (g22 * d3 - g23 * d2) / det;
    const double q = d2 * i2 + d3 * i3;
    if (!(si * si > q)) return INFINITY;
    const double rn = sqrt(rperp2) / sqrt(1.0 - q / (si * si));
    const double l2 = mu2 - (rn / si) * i2;
    const double l3 = mu3 - (rn / si) * i3;
    if (!(l2 > 0.0 && l3 > 0.0 && l2 + l3 < 1.0)) return INFINITY;
    return t1 + l2 * d2 + l3 * d3 + si * rn;
}

// Seeds and +inf in both buffers (an iteration leaves a node's value in the
// buffer it writes untouched when that buffer already holds it), and the seeds
// as the nodes changed last: one wave per word, one lane per node.  The first
// source's waves also write the nodes with a lower and an upper neighbour on
// axes 0 and 1 (the last axis needs none: its shifts leave the grid).
__global__ __launch_bounds__(kThreads) void k_eik_init(EikDims d, int32_t S, const double* __restrict__ X,
                                                       const double* __restrict__ s, const double* __restrict__ xi,
                                                       double rho, double* __restrict__ T, double* __restrict__ T2,
                                                       uint64_t* __restrict__ chg, uint64_t* __restrict__ seeds,
                                                       uint64_t* __restrict__ edge) {
    const int64_t total = (int64_t)S * d.W;
    for (int64_t i = (blockIdx.x * (int64_t)kThreads + threadIdx.x) / 64; i < total; i += (int64_t)gridDim.x * (kThreads / 64)) {
        const int64_t alpha = i / d.W, p = (i - alpha * d.W) * 64 + (threadIdx.x & 63);
        const int64_t t = alpha * d.N + p;
        const double* xs = xi + alpha * 3;
        int64_t c[3];
        logical(d, p, c);
        bool seed = p < d.N;
        for (int k = 0; k < d.dim; ++k) seed = seed && fabs((double)c[k] - xs[k]) <= rho;
        const uint64_t word = __ballot(seed);
        if ((threadIdx.x & 63) == 0) {
            chg[i] = word;
            seeds[i] = word;
        }
        if (alpha == 0) {
            const bool in = p < d.N;
            const uint64_t w[4] = {__ballot(in && c[0] > 0), __ballot(in && c[0] < d.n0 - 1), __ballot(in && c[1] > 0),
                                   __ballot(in && c[1] < d.n1 - 1)};
            if ((threadIdx.x & 63) == 0)
                for (int k = 0; k < 4; ++k) edge[k * d.W + i] = w[k];
        }
        if (p >= d.N) continue;
        if (!seed) {
            T[t] = INFINITY;
            T2[t] = INFINITY;
            continue;
        }
        // the source's cell: corners and multilinear weights
        const int64_t nn[3] = {d.n0, d.n1, d.n2};
        int64_t base[3] = {0, 0, 0};
        double fr[3] = {0.0, 0.0, 0.0};
        for (int k = 0; k < d.dim; ++k) {
            int64_t b = (int64_t)floor(xs[k]);
            b = b < 0 ? 0 : b;
            b = b > nn[k] - 2 ? (nn[k] - 2 < 0 ? 0 : nn[k] - 2) : b;
            base[k] = b;
            fr[k] = xs[k] - (double)b;
        }
        double s_src = 0.0, x_src[3] = {0.0, 0.0, 0.0};
        for (int corner = 0; corner < (1 << d.dim); ++corner) {
            double w = 1.0;
            int64_t q = 0, stride = 1;
            for (int k = 0; k < d.dim; ++k) {
                const int up = (corner >> k) & 1;
                w = w * (up ? fr[k] : 1.0 - fr[k]);
                q += (base[k] + (nn[k] > 1 ? up : 0)) * stride;
                stride *= nn[k];
            }
            s_src = s_src + w * s[q];
            for (int k = 0; k < d.dim; ++k) x_src[k] = x_src[k] + w * X[q * d.dim + k];
        }
        const double v = 0.5 * (s_src + s[p]) * dist(X + p * d.dim, x_src, d.dim);
        T[t] = v;
        T2[t] = v;
    }
}

__global__ void k_clear_counts(unsigned* f) {
    if (threadIdx.x <= kChunk) f[threadIdx.x] = 0u;
}

// Word i of the mask m [W] shifted so that bit p holds bit p - off.
__device__ __forceinline__ uint64_t shifted(const uint64_t* __restrict__ m, int64_t i, int64_t W, int64_t off) {
    const int64_t bit = i * 64 - off;              // source bit of bit 0 of the result
    const int64_t lo = bit >> 6;                   // (rounds towards minus infinity)
    const int sh = (int)(bit & 63);
    const uint64_t a = lo >= 0 && lo < W ? m[lo] : 0ull;
    if (sh == 0) return a;
    const uint64_t b = lo + 1 >= 0 && lo + 1 < W ? m[lo + 1] : 0ull;
    return a >> sh | b << (64 - sh);
}

// Word i of the nodes with a changed face neighbour.
template <int DIM>
__device__ __forceinline__ uint64_t spread(const EikDims& d, const uint64_t* __restrict__ co,
                                           const uint64_t* __restrict__ edge, int64_t i) {
    uint64_t a = (shifted(co, i, d.W, 1) & edge[i]) | (shifted(co, i, d.W, -1) & edge[d.W + i]) |
                 (shifted(co, i, d.W, d.n0) & edge[2 * d.W + i]) | (shifted(co, i, d.W, -d.n0) & edge[3 * d.W + i]);
    if (DIM == 3) a |= shifted(co, i, d.W, d.n0 * d.n1) | shifted(co, i, d.W, -d.n0 * d.n1);
    const int64_t left = d.N - i * 64;
    if (left < 64) a &= left > 0 ? (1ull << left) - 1ull : 0ull;
    return a;
}

// F(T) at a node that is no seed, or its value where that is lower.
template <int DIM>
__device__ __forceinline__ double recompute(const EikDims& d, const double* __restrict__ X, const double* __restrict__ s,
                                            const double* __restrict__ Told, uint32_t p32, double told) {
    const uint32_t n0 = (uint32_t)d.n0, n1 = (uint32_t)d.n1, n2 = (uint32_t)d.n2;
    const int64_t stride[3] = {1, d.n0, d.n0 * d.n1}, p = p32;
    const uint32_t nn[3] = {n0, n1, n2};
    const uint32_t r = p32 / n0;
    const uint32_t c[3] = {p32 - r * n0, r % n1, r / n1};
    int64_t nb[DIM][2];
    for (int k = 0; k < DIM; ++k) {
        nb[k][0] = c[k] > 0 ? p - stride[k] : -1;
        nb[k][1] = c[k] < nn[k] - 1 ? p + stride[k] : -1;
    }
    const double si = s[p];
    double xi[3], xk[DIM][2][3], tk[DIM][2];
    for (int k = 0; k < DIM; ++k) xi[k] = X[p * DIM + k];
    double best = INFINITY;
    for (int k = 0; k < DIM; ++k)
        for (int side = 0; side < 2; ++side) {
            const int64_t q = nb[k][side];
            tk[k][side] = q >= 0 ? Told[q] : INFINITY;
            for (int m = 0; m < DIM; ++m) xk[k][side][m] = q >= 0 ? X[q * DIM + m] : 0.0;
            if (q >= 0) best = fmin(best, tk[k][side] + si * dist(xi, xk[k][side], DIM));
        }
    // a simplex whose vertex values are all >= best cannot lower it:
    // its interior values exceed its least vertex value
    for (int a = 0; a < DIM; ++a)
        for (int b = a + 1; b < DIM; ++b)
            for (int sa = 0; sa < 2; ++sa)
                for (int sb = 0; sb < 2; ++sb)
                    if (nb[a][sa] >= 0 && nb[b][sb] >= 0 && fmin(tk[a][sa], tk[b][sb]) < best)
                        best = fmin(best, seg_inner(xi, si, xk[a][sa], tk[a][sa], xk[b][sb], tk[b][sb], DIM));
    if constexpr (DIM == 3) {
        for (int s0 = 0; s0 < 2; ++s0)
            for (int s1 = 0; s1 < 2; ++s1)
                for (int s2 = 0; s2 < 2; ++s2)
                    if (nb[0][s0] >= 0 && nb[1][s1] >= 0 && nb[2][s2] >= 0 &&
                        fmin(fmin(tk[0][s0], tk[1][s1]), tk[2][s2]) < best)
                        best = fmin(best, tri_inner(xi, si, xk[0][s0], tk[0][s0], xk[1][s1], tk[1][s1],
                                                    xk[2][s2], tk[2][s2]));
    }
    return fmin(told, best);
}

// One iteration in one launch, a wave per word and a lane per node: for small
// grids, where a second launch costs more than the lanes without work.
template <int DIM>
__global__ __launch_bounds__(64) void k_eik_word(EikDims d, int32_t S, const double* __restrict__ X,
                                                 const double* __restrict__ s, const double* __restrict__ Told_,
                                                 double* __restrict__ Tnew_, const uint64_t* __restrict__ cold,
                                                 uint64_t* __restrict__ cnew, const uint64_t* __restrict__ seeds,
                                                 const uint64_t* __restrict__ edge, unsigned* __restrict__ any) {
    const int lane = (int)threadIdx.x;
    for (int64_t w = blockIdx.x; w < (int64_t)S * d.W; w += gridDim.x) {
        const int64_t alpha = w / d.W, i = w - alpha * d.W;
        const uint64_t* __restrict__ co = cold + alpha * d.W;
        const uint64_t open = ~seeds[w];
        const uint64_t a = spread<DIM>(d, co, edge, i) & open, t = a | (co[i] & open);
        const double* __restrict__ Told = Told_ + alpha * d.N;
        double* __restrict__ Tnew = Tnew_ + alpha * d.N;
        bool changed = false;
        if (t >> lane & 1ull) {
            const uint32_t p = (uint32_t)(i * 64) + (uint32_t)lane;
            const double told = Told[p];
            const double v = a >> lane & 1ull ? recompute<DIM>(d, X, s, Told, p, told) : told;
            Tnew[p] = v;
            changed = v != told;
        }
        const uint64_t ch = __ballot(changed);
        if (lane == 0) {
            cnew[w] = ch;
            if (ch) *any = 1u;         // (every wave stores the same)
        }
    }
}

// On other grids an iteration is two launches.  The first spreads the changed bits to their
// face neighbours (a few words per 64 nodes) and lists the nodes to recompute,
// one wave per tile of 64 words: the tile's nodes in order, and a batch for
// every 64 of them, so that the second launch finds all its work in full waves
// wherever the front is.
// With one lane per node and a state byte each, an iteration of 8 sources on
// 101x101x51 took 212 us, front or not; now 11 us and 57 us.  With each
// workgroup listing and recomputing its own 1024 nodes it was 95 us (with 512
// nodes 120, with 256 183: the workgroups away from the front, each of which
// only reads its words, took the time).  Neither kernel updates a word that
// every wave shares: those updates queue, 10 ns each (a counter that dealt out
// the batches cost 40 us, one flag set by every wave 15 us).
template <int DIM>
__global__ __launch_bounds__(kThreads) void k_eik_list(EikDims d, int32_t S, const uint64_t* __restrict__ cold,
                                                       uint64_t* __restrict__ cnew, const uint64_t* __restrict__ seeds,
                                                       const uint64_t* __restrict__ edge, uint16_t* __restrict__ list,
                                                       int32_t* __restrict__ count, uint32_t* __restrict__ batch,
                                                       unsigned* __restrict__ n_batch) {
    __shared__ unsigned wave_n[kThreads / 64], wave_at;
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    const int64_t tiles = (int64_t)S * (d.W / kTile);
    for (int64_t t0 = blockIdx.x * (int64_t)(kThreads / 64); t0 < tiles; t0 += (int64_t)gridDim.x * (kThreads / 64)) {
        const int64_t tile = t0 + wave;
        int total = 0;
        if (tile < tiles) {
            const int64_t alpha = tile / (d.W / kTile), i = (tile - alpha * (d.W / kTile)) * kTile + lane;
            const uint64_t* __restrict__ co = cold + alpha * d.W;
            const uint64_t open = ~seeds[alpha * d.W + i];
            const uint64_t a = spread<DIM>(d, co, edge, i) & open;
            const uint64_t t = a | (co[i] & open);
            cnew[alpha * d.W + i] = 0ull;
            int n = __popcll(t);       // running sum over the lanes
            for (int o = 1; o < 64; o <<= 1) {
                const int x = __shfl_up(n, o);
                if (lane >= o) n += x;
            }
            total = __shfl(n, 63);
            uint16_t* __restrict__ out = list + tile * (kTile * 64);
            for (uint64_t m = __ballot(t != 0ull); m; m &= m - 1ull) {
                const int w = __ffsll((unsigned long long)m) - 1;
                const uint64_t tw = __shfl((unsigned long long)t, w), aw = __shfl((unsigned long long)a, w);
                const int end = __shfl(n, w);
                if (tw >> lane & 1ull)
                    out[end - __popcll(tw >> lane)] = (uint16_t)(w * 64 + lane) | (aw >> lane & 1ull ? (uint16_t)0 : kCopy);
            }
        }
        // places for the batches of the whole workgroup at once: one atomic on
        // the counter (from every wave of the card they queue, 10 ns each)
        const int nb = (total + 63) / 64;
        if (lane == 0) wave_n[wave] = (unsigned)nb;
        __syncthreads();
        unsigned before = 0u, all = 0u;
        for (int w = 0; w < kThreads / 64; ++w) {
            before += w < wave ? wave_n[w] : 0u;
            all += wave_n[w];
        }
        if (all && threadIdx.x == 0) wave_at = atomicAdd(n_batch, all);
        __syncthreads();
        if (total && lane == 0) count[tile] = total;
        if (lane < nb) batch[wave_at + before + lane] = (uint32_t)(tile * kTile + lane);
    }
}

// The listed nodes, one per lane.  Bound by the FP64 divisions and square
// roots (divergent: simplices that cannot lower the value are skipped) and
// their registers (three waves per SIMD in 3-D).
template <int DIM>
__global__ __launch_bounds__(64, 3) void k_eik_step(EikDims d, const double* __restrict__ X,
                                                 const double* __restrict__ s, const double* __restrict__ Told_,
                                                 double* __restrict__ Tnew_, unsigned long long* __restrict__ cnew,
                                                 const uint16_t* __restrict__ list, const int32_t* __restrict__ count,
                                                 const uint32_t* __restrict__ batch, const unsigned* __restrict__ n_batch) {
    __shared__ unsigned long long ch[kTile];           // changed nodes of the batch's tile
    const int lane = (int)threadIdx.x;
    const uint32_t tps = (uint32_t)(d.W / kTile);      // tiles per source
    const unsigned n_b = *n_batch;
    ch[lane] = 0ull;
    for (unsigned at = blockIdx.x; at < n_b; at += gridDim.x) {
        const uint32_t e = batch[at], tile = e / kTile;
        const int32_t k = (int32_t)(e - tile * kTile) * 64 + lane;
        const uint32_t alpha = tile / tps;
        if (k < count[tile]) {
            const uint32_t entry = list[(size_t)tile * (kTile * 64) + k];
            const uint32_t p32 = (tile - alpha * tps) * (kTile * 64) + (entry & (kCopy - 1u));
            const int64_t p = p32;
            const double* __restrict__ Told = Told_ + alpha * d.N;
            double* __restrict__ Tnew = Tnew_ + alpha * d.N;
            if (entry & kCopy) {
                // T^{n+1} = T^n; the buffer written now holds T^{n-1}, which is
                // the same value unless the node changed in the last iteration
                Tnew[p] = Told[p];
            } else {
                const double told = Told[p], v = recompute<DIM>(d, X, s, Told, p32, told);
                Tnew[p] = v;
                if (v != told) atomicOr(&ch[p32 >> 6 & (kTile - 1)], 1ull << (p32 & 63u));
            }
        }
        // one global update per changed word (a wave's own LDS order is program order)
        __syncthreads();
        const unsigned long long m = ch[lane];
        if (m) {
            atomicOr(cnew + alpha * d.W + (size_t)(tile - alpha * tps) * kTile + lane, m);
            ch[lane] = 0ull;
        }
        __syncthreads();
    }
}

}  // namespace

}  // namespace fm

extern "C" {

int fm_eikonal_create(int32_t dim, int64_t n1, int64_t n2, int64_t n3, const double* X, int32_t max_sources,
                      void* hip_stream, fm_eikonal** out) {
    using namespace fm;
    clear_error();
    if (!out) { set_error("null output pointer"); return FM_EINVAL; }
    *out = nullptr;
    if (dim != 2 && dim != 3) { set_error("dim must be 2 or 3, got %d", dim); return FM_EINVAL; }
    if (dim == 2 && n2 != 1) { set_error("2-D grids need n2 == 1"); return FM_EINVAL; }
    if (n1 < 1 || n2 < 1 || n3 < 1) { set_error("grid sizes must be >= 1"); return FM_EINVAL; }
    if (!X) { set_error("null node coordinates"); return FM_EINVAL; }
    if (max_sources < 1) { set_error("max_sources must be >= 1"); return FM_EINVAL; }
    const int64_t N = n1 * n2 * n3;
    if (N >= ((int64_t)1 << 31)) { set_error("grid too large: %lld nodes", (long long)N); return FM_EINVAL; }
    for (int64_t i = 0; i < N * dim; i++)
        if (!std::isfinite(X[i])) { set_error("node coordinate %lld is not finite", (long long)i); return FM_EINVAL; }
    fm_eikonal* e = new (std::nothrow) fm_eikonal();
    if (!e) { set_error("out of host memory"); return FM_ENOMEM; }
    e->dim = dim;
    e->n[0] = n1;
    e->n[1] = dim == 3 ? n2 : n3;
    e->n[2] = dim == 3 ? n3 : 1;
    e->N = N;
    e->S = max_sources;
    e->stream = (hipStream_t)hip_stream;
    hipError_t h = hipGetDevice(&e->device);
    e->W = (N + 64 * kTile - 1) / (64 * kTile) * kTile;
    const size_t src = (size_t)max_sources, W = (size_t)e->W, listed = is_small(dim, (int64_t)src * e->W) ? 0 : src * W;
    if (h == hipSuccess)
        h = e->block.take({{(void**)&e->X, sizeof(double) * (size_t)N * dim},
                           {(void**)&e->Tb, sizeof(double) * src * (size_t)N},
                           {(void**)&e->chg[0], sizeof(uint64_t) * src * W},
                           {(void**)&e->chg[1], sizeof(uint64_t) * src * W},
                           {(void**)&e->seed, sizeof(uint64_t) * src * W},
                           {(void**)&e->edge, sizeof(uint64_t) * 4 * W},
                           {(void**)&e->list, sizeof(uint16_t) * 64 * listed},
                           {(void**)&e->count, sizeof(int32_t) * (listed / kTile)},
                           {(void**)&e->batch, sizeof(uint32_t) * listed},
                           {(void**)&e->xi, sizeof(double) * 3 * src},
                           {(void**)&e->n_batch, sizeof(unsigned) * (kChunk + 1)}});
    int cus = 0;
    if (h == hipSuccess) h = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, e->device);
    e->waves = cus * 24;    // 12 a CU are resident; more for the batches' different lengths
    if (h == hipSuccess) h = hipHostMalloc((void**)&e->n_batch_h, sizeof(unsigned) * (kChunk + 1), hipHostMallocDefault);
    if (h == hipSuccess) h = hipMemcpy(e->X, X, sizeof(double) * (size_t)N * dim, hipMemcpyHostToDevice);
    if (h != hipSuccess) {
        set_error("first-arrival solver allocation failed: %s", hipGetErrorString(h));
        fm_eikonal_free(e);
        return h == hipErrorOutOfMemory ? FM_ENOMEM : FM_EHIP;
    }
    *out = e;
    return FM_OK;
}

int fm_eikonal_set_stream(fm_eikonal* e, void* hip_stream) {
    fm::clear_error();
    if (!e) { fm::set_error("null solver"); return FM_EINVAL; }
    e->stream = (hipStream_t)hip_stream;
    return FM_OK;
}

int fm_eikonal_solve(fm_eikonal* e, const double* s, int32_t S, const double* xi_src, double seed_radius,
                     int32_t max_iter, double* T, int32_t* iterations) {
    using namespace fm;
    clear_error();
    if (iterations) *iterations = 0;
    if (!e || !s || !xi_src || !T) { set_error("null argument"); return FM_EINVAL; }
    if (S < 1 || S > e->S) { set_error("S = %d outside 1..%d (the solver's capacity)", S, e->S); return FM_EINVAL; }
    if (!(seed_radius >= 0.0) || !std::isfinite(seed_radius)) { set_error("seed radius must be finite and >= 0"); return FM_EINVAL; }
    if (max_iter < 1) { set_error("max_iter must be >= 1"); return FM_EINVAL; }
    if (((uintptr_t)s & 7u) || ((uintptr_t)T & 7u)) { set_error("device buffers must be 8-byte aligned"); return FM_EINVAL; }
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != e->device) { set_error("solver lives on device %d (current device %d)", e->device, dev); return FM_ESTATE; }
    std::vector<double> xi((size_t)3 * S, 0.0);
    for (int32_t a = 0; a < S; a++) {
        for (int k = 0; k < e->dim; k++) {
            const double v = xi_src[(size_t)a * e->dim + k];
            if (!(v >= 0.0) || !(v <= (double)(e->n[k] - 1))) {
                set_error("source %d: coordinate %d (%g) outside [0, %lld]", a, k, v, (long long)(e->n[k] - 1));
                return FM_EINVAL;
            }
            // the seed region must hold a node along every axis
            const double lo = std::max(0.0, std::ceil(v - seed_radius));
            const double hi = std::min((double)(e->n[k] - 1), std::floor(v + seed_radius));
            if (lo > hi) {
                set_error("source %d: the seed region (radius %g) holds no node", a, seed_radius);
                return FM_EINVAL;
            }
            xi[(size_t)a * 3 + k] = v;
        }
    }
    hipStream_t st = e->stream;
    HIP_TRY(hipMemcpyAsync(e->xi, xi.data(), sizeof(double) * xi.size(), hipMemcpyHostToDevice, st));
    EikDims d{e->dim, e->n[0], e->n[1], e->n[2], e->N, e->W};
    const int64_t total = (int64_t)S * e->N;
    const int grid = (int)std::min<int64_t>(((int64_t)S * e->W + 3) / 4, 16384);
    const int tiles = (int)std::min<int64_t>(((int64_t)S * (e->W / kTile) + 3) / 4, 16384);
    double* buf[2] = {T, e->Tb};
    hipLaunchKernelGGL(k_eik_init, dim3(grid), dim3(256), 0, st, d, S, e->X, s, e->xi, seed_radius, buf[0], buf[1],
                       e->chg[0], e->seed, e->edge);
    HIP_TRY(hipGetLastError());
    const auto list_fn = e->dim == 3 ? k_eik_list<3> : k_eik_list<2>;
    const auto step_fn = e->dim == 3 ? k_eik_step<3> : k_eik_step<2>;
    const auto word_fn = e->dim == 3 ? k_eik_word<3> : k_eik_word<2>;
    const int64_t words = (int64_t)S * e->W;
    const bool small = is_small(e->dim, words);
    int cur = 0;
    int32_t done = 0;
    while (done < max_iter) {
        const int n = std::min<int32_t>(kChunk, max_iter - done);
        hipLaunchKernelGGL(k_clear_counts, dim3(1), dim3(64), 0, st, e->n_batch);
        // word j + 1 stays 0 when iteration j changed nothing: on small grids the
        // iteration writes it; otherwise it is the length of the next list, and
        // one more list follows the chunk (its iteration lists the same again)
        for (int j = 0; small && j < n; j++, cur ^= 1)
            hipLaunchKernelGGL(word_fn, dim3((unsigned)words), dim3(64), 0, st, d, S, e->X, s, buf[cur], buf[cur ^ 1],
                               e->chg[cur], e->chg[cur ^ 1], e->seed, e->edge, e->n_batch + j + 1);
        for (int j = 0; !small && j <= n; j++) {
            hipLaunchKernelGGL(list_fn, dim3(tiles), dim3(kThreads), 0, st, d, S, e->chg[cur], e->chg[cur ^ 1],
                               e->seed, e->edge, e->list, e->count, e->batch, e->n_batch + j);
            if (j == n) break;
            hipLaunchKernelGGL(step_fn, dim3(e->waves), dim3(64), 0, st, d, e->X, s, buf[cur], buf[cur ^ 1],
                               (unsigned long long*)e->chg[cur ^ 1], e->list, e->count, e->batch, e->n_batch + j);
            cur ^= 1;
        }
        HIP_TRY(hipGetLastError());
        HIP_TRY(hipMemcpyAsync(e->n_batch_h, e->n_batch, sizeof(unsigned) * (n + 1), hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
        for (int j = 0; j < n; j++) {
            if (!e->n_batch_h[j + 1]) {
                // iteration done + j + 1 changed nothing; the later ones of the
                // chunk left the same values in the buffer now current
                if (iterations) *iterations = done + j + 1;
                if (cur != 0)
                    HIP_TRY(hipMemcpyAsync(T, e->Tb, sizeof(double) * (size_t)total, hipMemcpyDeviceToDevice, st));
                HIP_TRY(hipStreamSynchronize(st));
                return FM_OK;
            }
        }
        done += n;
    }
    if (iterations) *iterations = done;
    if (cur != 0) HIP_TRY(hipMemcpyAsync(T, e->Tb, sizeof(double) * (size_t)total, hipMemcpyDeviceToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));
    set_error("no fixed point within %d iterations (T holds the last iterate)", max_iter);
    return FM_ESTATE;
}

void fm_eikonal_free(fm_eikonal* e) {
    if (!e) return;
    e->block.release();
    if (e->n_batch_h) (void)hipHostFree(e->n_batch_h);
    delete e;
}

}  // extern "C"
