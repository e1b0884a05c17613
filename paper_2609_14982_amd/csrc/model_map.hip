// Cell-velocity model map M_alpha (Section 4.4, eq. (source-jacobian)): the
// inversion unknowns are cell velocities, the transport takes nodal slowness.
// A node's slowness is the reciprocal of the mean velocity of the cells that
// share it, s_p = 1 / vbar_p with vbar_p = (1/n_p) sum_{c around p} v_c, so
// the linearised map and its transpose are
//   (M dv)_p    = a_p sum_{c around p} dv_c,      a_p = -1 / (n_p vbar_p^2),
//   (M^T g)_c   = sum_{p corner of c} a_p g_p.
// Cells are the logical hexahedra (quadrilaterals in 2-D) between nodes,
// cell id c = ci + (n1-1) (cj + (n2-1) ck); a node has 1, 2, 4 or 8 cells.
// M is the same for every source, so one application serves a whole batch
// (J M = stacked J_alpha of the broadcast model block, M^T after the source
// sum).  Both products are gathers with a fixed summation order (ascending
// cell or node id): deterministic, no atomics.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "fmbtf.h"
#include "internal.h"
#include "batch.h"

struct fm_model_map {
    int dim = 3;
    int64_t n[3] = {1, 1, 1};    // nodes per logical axis (axis 0 fastest; 2-D: n[1] = n3, n[2] = 1)
    int64_t c[3] = {1, 1, 1};    // cells per axis (1 for an axis of one node)
    int64_t N = 0, Nc = 0;
    std::vector<double> slow;    // host [N] background slowness 1 / vbar
    double* scale = nullptr;     // device [N] a_p
    hipStream_t stream = nullptr;
    int device = -1;
};

namespace fm {

struct MapDims {
    int64_t n0, n1, n2, c0, c1, c2;
};

__device__ __forceinline__ void cell_range(int64_t i, int64_t n, int64_t& lo, int64_t& hi) {
    if (n == 1) { lo = 0; hi = 0; return; }
    lo = i > 0 ? i - 1 : 0;
    hi = i < n - 1 ? i : n - 2;
}

// VW right-hand sides of one row: 16 bytes where rows and pointers allow it.
template <typename V, int VW>
struct alignas(sizeof(V) * VW) Row {
    V v[VW];
};

// Both products are bound by the rows they move (each input row read from
// memory once, each output row written once) as long as the indices cost
// little: a thread takes VW right-hand sides of a column of kc planes of the
// last axis, so that it splits its index once for the column and reads a plane
// once for the two outputs that share it.  The sums stay in ascending order:
// the plane's own sum, needed first by the next output, is formed beside the
// output that continues the previous plane's.  201x201x101, 16 right-hand
// sides, FP64: 680 us (M) and 691 us (M^T) with one thread per output value,
// eight loads and five 64-bit divisions each.
template <typename V, int VW>
__global__ __launch_bounds__(256) void k_model_map(MapDims d, const double* __restrict__ a, const V* __restrict__ dv,
                                                   V* __restrict__ ds, int B, int kc) {
    typedef Row<V, VW> R;
    const int64_t L = B / VW, total = d.n0 * d.n1 * L;
    const R* __restrict__ in = (const R*)dv;
    R* __restrict__ out = (R*)ds;
    for (int64_t t = blockIdx.x * (int64_t)256 + threadIdx.x; t < total; t += (int64_t)gridDim.x * 256) {
        const int64_t r = t / L, col = t - r * L, j = r / d.n0, i = r - j * d.n0;
        int64_t i0, i1, j0, j1;
        cell_range(i, d.n0, i0, i1);
        cell_range(j, d.n1, j0, j1);
        const bool two_i = i1 > i0, two_j = j1 > j0;
        const int64_t plane = d.c0 * d.c1 * L, di = L, dj = d.c0 * L;
        const R* __restrict__ base = in + (i0 + d.c0 * j0) * L + col;
        auto add = [](R& x, const R& y) {
#pragma unroll
            for (int v = 0; v < VW; ++v) x.v[v] += y.v[v];
        };
        // acc continues with plane ck, own starts with it
        auto cells = [&](int64_t ck, R& acc, R& own) {
            const R* __restrict__ x = base + ck * plane;
            R y[4];
            y[0] = x[0];
            if (two_i) y[1] = x[di];
            if (two_j) {
                y[2] = x[dj];
                if (two_i) y[3] = x[dj + di];
            }
            own = R{};
            add(acc, y[0]);
            add(own, y[0]);
            if (two_i) { add(acc, y[1]); add(own, y[1]); }
            if (two_j) {
                add(acc, y[2]);
                add(own, y[2]);
                if (two_i) { add(acc, y[3]); add(own, y[3]); }
            }
        };
        for (int64_t k0 = (int64_t)blockIdx.y * kc; k0 < d.n2; k0 += (int64_t)gridDim.y * kc) {
            const int64_t k1 = k0 + kc < d.n2 ? k0 + kc : d.n2;
            R acc{}, own{};
            if (k0 > 0) cells(k0 - 1, acc, own);
            for (int64_t k = k0; k < k1; ++k) {
                acc = own;
                if (k < d.c2) cells(k, acc, own);
                const int64_t p = i + d.n0 * (j + d.n1 * k);
                const V c = (V)a[p];
                R o;
#pragma unroll
                for (int v = 0; v < VW; ++v) o.v[v] = c * acc.v[v];
                out[p * L + col] = o;
            }
        }
    }
}

template <typename V, int VW>
__global__ __launch_bounds__(256) void k_model_map_t(MapDims d, const double* __restrict__ a, const V* __restrict__ g,
                                                     V* __restrict__ out_, int B, int kc) {
    typedef Row<V, VW> R;
    const int64_t L = B / VW, total = d.c0 * d.c1 * L;
    const R* __restrict__ in = (const R*)g;
    R* __restrict__ out = (R*)out_;
    for (int64_t t = blockIdx.x * (int64_t)256 + threadIdx.x; t < total; t += (int64_t)gridDim.x * 256) {
        const int64_t r = t / L, col = t - r * L, j = r / d.c0, i = r - j * d.c0;
        const bool two_i = d.n0 > 1, two_j = d.n1 > 1;
        const int64_t row = i + d.n0 * j;
        auto add = [](R& x, V c, const R& y) {
#pragma unroll
            for (int v = 0; v < VW; ++v) x.v[v] += c * y.v[v];
        };
        auto nodes = [&](int64_t k, R& acc, R& own) {
            const int64_t p = row + d.n0 * d.n1 * k;
            const R* __restrict__ x = in + p * L + col;
            R y[4];
            V c[4];
            y[0] = x[0];
            c[0] = (V)a[p];
            if (two_i) { y[1] = x[L]; c[1] = (V)a[p + 1]; }
            if (two_j) {
                y[2] = x[d.n0 * L];
                c[2] = (V)a[p + d.n0];
                if (two_i) { y[3] = x[(d.n0 + 1) * L]; c[3] = (V)a[p + d.n0 + 1]; }
            }
            own = R{};
            add(acc, c[0], y[0]);
            add(own, c[0], y[0]);
            if (two_i) { add(acc, c[1], y[1]); add(own, c[1], y[1]); }
            if (two_j) {
                add(acc, c[2], y[2]);
                add(own, c[2], y[2]);
                if (two_i) { add(acc, c[3], y[3]); add(own, c[3], y[3]); }
            }
        };
        for (int64_t k0 = (int64_t)blockIdx.y * kc; k0 < d.c2; k0 += (int64_t)gridDim.y * kc) {
            const int64_t k1 = k0 + kc < d.c2 ? k0 + kc : d.c2;
            R acc{}, own{};
            nodes(k0, acc, own);
            for (int64_t k = k0; k < k1; ++k) {
                acc = own;
                if (d.n2 > 1) nodes(k + 1, acc, own);
                out[(i + d.c0 * (j + d.c1 * k)) * L + col] = acc;
            }
        }
    }
}

// (2-D: the second axis is the one walked, over rows of one node)
static MapDims dims_of(const fm_model_map* m) {
    if (m->dim == 2) return MapDims{m->n[0], 1, m->n[1], m->c[0], 1, m->c[1]};
    return MapDims{m->n[0], m->n[1], m->n[2], m->c[0], m->c[1], m->c[2]};
}

static int check_map(const fm_model_map* m, int32_t B, int32_t precision, const void* x, const void* y) {
    if (!m) { set_error("null model map"); return FM_EINVAL; }
    if (B < 1) { set_error("B must be >= 1"); return FM_EINVAL; }
    if (precision != FM_FP64 && precision != FM_FP32) { set_error("precision must be FM_FP64 or FM_FP32"); return FM_EINVAL; }
    if (!x || !y) { set_error("null vector"); return FM_EINVAL; }
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != m->device) { set_error("model map lives on device %d (current device %d)", m->device, dev); return FM_ESTATE; }
    return FM_OK;
}

// One launch of either product over `rows` rows of `planes` planes.  Columns of
// 16 planes read one in 17 twice; shorter ones where that leaves fewer than
// eight workgroups a CU.
template <typename V>
static void launch_map(void (*fn)(MapDims, const double*, const V*, V*, int, int), const fm_model_map* m, int64_t rows,
                       int64_t planes, int B, int vw, const void* x, void* y) {
    const int64_t bx = std::min<int64_t>((rows * (B / vw) + 255) / 256, 1 << 20);
    int64_t kc = 16;
    while (kc > 1 && bx * ((planes + kc - 1) / kc) < 2048) kc /= 2;
    const int64_t by = std::min<int64_t>((planes + kc - 1) / kc, 65535);
    hipLaunchKernelGGL(fn, dim3((unsigned)bx, (unsigned)by), dim3(256), 0, m->stream, dims_of(m), m->scale, (const V*)x, (V*)y, B,
                       (int)kc);
}

// rows of whole 16-byte parts, on such addresses
template <typename V>
static bool wide(int B, const void* x, const void* y) {
    return B % (16 / sizeof(V)) == 0 && (((uintptr_t)x | (uintptr_t)y) & 15u) == 0;
}

template <typename V>
static void map_apply(const fm_model_map* m, int B, const void* dv, void* ds) {
    const MapDims d = dims_of(m);
    constexpr int vw = 16 / sizeof(V);
    if (wide<V>(B, dv, ds)) launch_map<V>(k_model_map<V, vw>, m, d.n0 * d.n1, d.n2, B, vw, dv, ds);
    else launch_map<V>(k_model_map<V, 1>, m, d.n0 * d.n1, d.n2, B, 1, dv, ds);
}

template <typename V>
static void map_apply_t(const fm_model_map* m, int B, const void* g, void* out) {
    const MapDims d = dims_of(m);
    constexpr int vw = 16 / sizeof(V);
    if (wide<V>(B, g, out)) launch_map<V>(k_model_map_t<V, vw>, m, d.c0 * d.c1, d.c2, B, vw, g, out);
    else launch_map<V>(k_model_map_t<V, 1>, m, d.c0 * d.c1, d.c2, B, 1, g, out);
}

}  // namespace fm

extern "C" {

int fm_model_map_create(int32_t dim, int64_t n1, int64_t n2, int64_t n3, const double* v_cell, void* hip_stream,
                        fm_model_map** out) {
    using namespace fm;
    clear_error();
    if (!out) { set_error("null output pointer"); return FM_EINVAL; }
    *out = nullptr;
    if (dim != 2 && dim != 3) { set_error("dim must be 2 or 3, got %d", dim); return FM_EINVAL; }
    if (dim == 2 && n2 != 1) { set_error("2-D grids need n2 == 1"); return FM_EINVAL; }
    if (n1 < 2 || n3 < 2 || (dim == 3 && n2 < 2)) { set_error("every axis of the grid needs at least 2 nodes"); return FM_EINVAL; }
    if (!v_cell) { set_error("null cell velocities"); return FM_EINVAL; }
    fm_model_map* m = new (std::nothrow) fm_model_map();
    if (!m) { set_error("out of host memory"); return FM_ENOMEM; }
    m->dim = dim;
    m->n[0] = n1;
    m->n[1] = dim == 3 ? n2 : n3;
    m->n[2] = dim == 3 ? n3 : 1;
    for (int d = 0; d < 3; d++) m->c[d] = m->n[d] > 1 ? m->n[d] - 1 : 1;
    m->N = m->n[0] * m->n[1] * m->n[2];
    m->Nc = m->c[0] * m->c[1] * m->c[2];
    for (int64_t c = 0; c < m->Nc; c++)
        if (!(v_cell[c] > 0.0) || !std::isfinite(v_cell[c])) {
            set_error("cell velocity %lld must be finite and > 0", (long long)c);
            delete m;
            return FM_EINVAL;
        }
    std::vector<double> a;
    try {
        m->slow.resize(m->N);
        a.resize(m->N);
    } catch (const std::bad_alloc&) {
        delete m;
        set_error("out of host memory");
        return FM_ENOMEM;
    }
    auto range = [&](int64_t i, int d, int64_t& lo, int64_t& hi) {
        if (m->n[d] == 1) { lo = hi = 0; return; }
        lo = i > 0 ? i - 1 : 0;
        hi = i < m->n[d] - 1 ? i : m->n[d] - 2;
    };
    for (int64_t p = 0; p < m->N; p++) {
        const int64_t i = p % m->n[0], r = p / m->n[0], j = r % m->n[1], k = r / m->n[1];
        int64_t i0, i1, j0, j1, k0, k1;
        range(i, 0, i0, i1);
        range(j, 1, j0, j1);
        range(k, 2, k0, k1);
        double sum = 0.0;
        int cnt = 0;
        for (int64_t ck = k0; ck <= k1; ++ck)
            for (int64_t cj = j0; cj <= j1; ++cj)
                for (int64_t ci = i0; ci <= i1; ++ci) {
                    sum += v_cell[ci + m->c[0] * (cj + m->c[1] * ck)];
                    cnt++;
                }
        const double vbar = sum / cnt;
        m->slow[p] = 1.0 / vbar;
        a[p] = -1.0 / ((double)cnt * vbar * vbar);
    }
    hipError_t e = hipGetDevice(&m->device);
    if (e == hipSuccess) e = hipMalloc((void**)&m->scale, sizeof(double) * (size_t)m->N);
    if (e == hipSuccess) e = hipMemcpy(m->scale, a.data(), sizeof(double) * (size_t)m->N, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        if (m->scale) (void)hipFree(m->scale);
        set_error("model map upload failed: %s", hipGetErrorString(e));
        const bool oom = e == hipErrorOutOfMemory;
        delete m;
        return oom ? FM_ENOMEM : FM_EHIP;
    }
    m->stream = (hipStream_t)hip_stream;
    *out = m;
    return FM_OK;
}

int fm_model_map_sizes(const fm_model_map* m, int64_t* n_nodes, int64_t* n_cells) {
    fm::clear_error();
    if (!m) { fm::set_error("null model map"); return FM_EINVAL; }
    if (n_nodes) *n_nodes = m->N;
    if (n_cells) *n_cells = m->Nc;
    return FM_OK;
}

int fm_model_map_slowness(const fm_model_map* m, double* s_out) {
    fm::clear_error();
    if (!m || !s_out) { fm::set_error("null argument"); return FM_EINVAL; }
    std::copy(m->slow.begin(), m->slow.end(), s_out);
    return FM_OK;
}

int fm_model_map_set_stream(fm_model_map* m, void* hip_stream) {
    fm::clear_error();
    if (!m) { fm::set_error("null model map"); return FM_EINVAL; }
    m->stream = (hipStream_t)hip_stream;
    return FM_OK;
}

int fm_model_map_apply(fm_model_map* m, int32_t B, int32_t precision, const void* dv, void* ds) {
    using namespace fm;
    clear_error();
    int rc = check_map(m, B, precision, dv, ds);
    if (rc) return rc;
    if (precision == FM_FP64) map_apply<double>(m, B, dv, ds);
    else map_apply<float>(m, B, dv, ds);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("model map launch failed: %s", hipGetErrorString(e)); return FM_EHIP; }
    return FM_OK;
}

int fm_model_map_apply_T(fm_model_map* m, int32_t B, int32_t precision, const void* g, void* dv_out) {
    using namespace fm;
    clear_error();
    int rc = check_map(m, B, precision, g, dv_out);
    if (rc) return rc;
    if (precision == FM_FP64) map_apply_t<double>(m, B, g, dv_out);
    else map_apply_t<float>(m, B, g, dv_out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("model map transpose launch failed: %s", hipGetErrorString(e)); return FM_EHIP; }
    return FM_OK;
}

void fm_model_map_free(fm_model_map* m) {
    if (!m) return;
    if (m->scale) (void)hipFree(m->scale);
    delete m;
}

}  // extern "C"
