// Fractional-step time integration on the GPU (Section 3.2 and Algorithm 1).
//
// Algorithm 1 assembles the Laplacian matrix once before the time loop, then
// per time step runs three Runge-Kutta stages (element assembly, momentum
// update) and one pressure solve by Jacobi-preconditioned conjugate gradients.
// The paper names a third-order Runge-Kutta scheme without its coefficients;
// the tableau here is Heun's third-order method, c = (0, 1/3, 2/3),
// a21 = 1/3, a32 = 2/3, b = (1/4, 0, 3/4).  Projection (incremental):
//   u*     = u^n + dt (k1/4 + 3 k3/4),  k_s = M_L^-1 rhs(u_s, p^n)
//   K dp   = -(1/dt) D u*   (right-hand side projected to zero mean; dp zero mean)
//   u^n+1  = u* - dt M_L^-1 G dp,   p^n+1 = p^n + dp
// with K = int grad N_a . grad N_b, (D u)_a = int N_a div u, (G p)_a = int N_a grad p.
// Everything is FP64.  The Laplacian's values, and divergence and gradient on
// meshes without chunks, are added with device atomics; on chunked meshes these
// two sum a chunk's nodes in LDS first.
#include <algorithm>
#include <cmath>

#include "element.hpp"

namespace lesasm {

// ---- element operators -----------------------------------------------------

template <int T>
__device__ __forceinline__ void load_geometry(const CatView &c, int e, const double *__restrict__ xyz,
                                              double (&x)[Ref<T>::nn][3], int (&fid)[Ref<T>::nn]) {
    constexpr int nn = Ref<T>::nn;
#pragma unroll
    for (int a = 0; a < nn; ++a) {
        const int g = c.cg[(size_t)a * c.ld + e];
        fid[a] = c.cf[(size_t)a * c.ld + e];
#pragma unroll
        for (int k = 0; k < 3; ++k) x[a][k] = xyz[3 * (size_t)g + k];
    }
#pragma unroll
    for (int a = nn - 1; a >= 0; --a)
#pragma unroll
        for (int k = 0; k < 3; ++k) x[a][k] -= x[0][k];
}

// Jacobian at Gauss point g, its inverse (K[k][i] = dxi_k/dx_i) and det.
template <int T>
__device__ __forceinline__ double jac_inverse(const double (&x)[Ref<T>::nn][3], int g, double (&Ki)[3][3]) {
    constexpr int nn = Ref<T>::nn;
    double J[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
#pragma unroll
    for (int a = 1; a < nn; ++a)
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k) J[i][k] += x[a][i] * Ref<T>::tab.dN[g][a][k];
    double adj[3][3];
    adj[0][0] = J[1][1] * J[2][2] - J[1][2] * J[2][1];
    adj[0][1] = J[0][2] * J[2][1] - J[0][1] * J[2][2];
    adj[0][2] = J[0][1] * J[1][2] - J[0][2] * J[1][1];
    adj[1][0] = J[1][2] * J[2][0] - J[1][0] * J[2][2];
    adj[1][1] = J[0][0] * J[2][2] - J[0][2] * J[2][0];
    adj[1][2] = J[0][2] * J[1][0] - J[0][0] * J[1][2];
    adj[2][0] = J[1][0] * J[2][1] - J[1][1] * J[2][0];
    adj[2][1] = J[0][1] * J[2][0] - J[0][0] * J[2][1];
    adj[2][2] = J[0][0] * J[1][1] - J[0][1] * J[1][0];
    const double det = J[0][0] * adj[0][0] + J[0][1] * adj[1][0] + J[0][2] * adj[2][0];
    const double r = 1.0 / det;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) Ki[i][k] = adj[i][k] * r;
    return det;
}

// (D u)_a += sum_g w det N_a div u
template <int T>
__global__ __launch_bounds__(256) void k_divergence(CatView c, const double *__restrict__ xyz,
                                                    const double *__restrict__ u, double *__restrict__ out) {
    using E = Ref<T>;
    constexpr int nn = E::nn;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= c.n) return;
    double x[nn][3], uu[nn][3], m[nn];
    int fid[nn];
    load_geometry<T>(c, e, xyz, x, fid);
#pragma unroll
    for (int a = 0; a < nn; ++a) {
        m[a] = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) uu[a][k] = u[3 * (size_t)fid[a] + k];
    }
#pragma unroll
    for (int g = 0; g < E::ng; ++g) {
        double Ki[3][3];
        const double det = jac_inverse<T>(x, g, Ki);
        double div = 0.0;
#pragma unroll
        for (int a = 0; a < nn; ++a)
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const double dnx = Ki[0][i] * E::tab.dN[g][a][0] + Ki[1][i] * E::tab.dN[g][a][1] +
                                   Ki[2][i] * E::tab.dN[g][a][2];
                div += uu[a][i] * dnx;
            }
        const double wd = E::tab.w[g] * det * div;
#pragma unroll
        for (int a = 0; a < nn; ++a) m[a] += wd * E::tab.N[g][a];
    }
#pragma unroll
    for (int a = 0; a < nn; ++a) unsafeAtomicAdd(out + fid[a], m[a]);
}

// (G p)_a += sum_g w det N_a grad p
template <int T>
__global__ __launch_bounds__(256) void k_gradient(CatView c, const double *__restrict__ xyz,
                                                  const double *__restrict__ p, double *__restrict__ out) {
    using E = Ref<T>;
    constexpr int nn = E::nn;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= c.n) return;
    double x[nn][3], pp[nn], m[nn][3];
    int fid[nn];
    load_geometry<T>(c, e, xyz, x, fid);
#pragma unroll
    for (int a = 0; a < nn; ++a) {
        pp[a] = p[fid[a]];
        m[a][0] = m[a][1] = m[a][2] = 0.0;
    }
#pragma unroll
    for (int g = 0; g < E::ng; ++g) {
        double Ki[3][3];
        const double det = jac_inverse<T>(x, g, Ki);
        double gp[3] = {0, 0, 0};
#pragma unroll
        for (int a = 0; a < nn; ++a)
#pragma unroll
            for (int i = 0; i < 3; ++i)
                gp[i] += pp[a] * (Ki[0][i] * E::tab.dN[g][a][0] + Ki[1][i] * E::tab.dN[g][a][1] +
                                  Ki[2][i] * E::tab.dN[g][a][2]);
        const double wd = E::tab.w[g] * det;
#pragma unroll
        for (int a = 0; a < nn; ++a)
#pragma unroll
            for (int i = 0; i < 3; ++i) m[a][i] += wd * E::tab.N[g][a] * gp[i];
    }
#pragma unroll
    for (int a = 0; a < nn; ++a)
#pragma unroll
        for (int i = 0; i < 3; ++i) unsafeAtomicAdd(out + 3 * (size_t)fid[a] + i, m[a][i]);
}

// ---- the same operators on chunked meshes ---------------------------------------
//
// The kernels above add every element's nodes with device atomics (28 G/s:
// 1.2 ms for the gradient of a 2.0 M-element box, whose bytes take 0.02 ms).
// Meshes with chunks use these instead: one launch over the chunks of all four
// types, a chunk's nodes staged in LDS and its contributions summed there
// (LDS atomics), nodes owned by the chunk stored and only shared ones added
// with device atomics into the zeroed output.  They keep nothing between the
// calls (in particular not the mesh's staging rows), so calls on several
// streams stay independent.  With adj = det J^-1 the quadrature sums
//   (D u)_a = sum_g w N_a tr(Gx adj),   (G p)_a = sum_g w N_a px adj
// need no division; nodes enter (relative to the element's node 0, as above)
// and leave through the modal coefficients.
// 2.0 M hybrid box: gradient 79 us against 1200 (four kernels), divergence 60
// against 307.  One thread per output entry in the write-back, not per node, so
// that a wavefront's atomics fill cache lines: gradient 87 against 139 us; then
// 79 (divergence 66 -> 60) with the nodes of a chunk loaded as in chunk_body and
// their tags kept in LDS.
template <int T, bool GRAD, class XA, class VA>
__device__ __forceinline__ void element_project(XA xa, VA va, double (&r)[GRAD ? 3 : 1][Ref<T>::nn]) {
    constexpr int nn = Ref<T>::nn, NI = GRAD ? 1 : 3, NO = GRAD ? 3 : 1;
    auto adjugate = [](const double (&J)[3][3], double (&adj)[3][3]) {
        adj[0][0] = J[1][1] * J[2][2] - J[1][2] * J[2][1];
        adj[0][1] = J[0][2] * J[2][1] - J[0][1] * J[2][2];
        adj[0][2] = J[0][1] * J[1][2] - J[0][2] * J[1][1];
        adj[1][0] = J[1][2] * J[2][0] - J[1][0] * J[2][2];
        adj[1][1] = J[0][0] * J[2][2] - J[0][2] * J[2][0];
        adj[1][2] = J[0][2] * J[1][0] - J[0][0] * J[1][2];
        adj[2][0] = J[1][0] * J[2][1] - J[1][1] * J[2][0];
        adj[2][1] = J[0][1] * J[2][0] - J[0][0] * J[2][1];
        adj[2][2] = J[0][0] * J[1][1] - J[0][1] * J[1][0];
    };
    // weight times the operator's value at a point, from the reference gradients of the input
    auto point = [](const double (&g)[NI][3], const double (&adj)[3][3], double w, double (&f)[NO]) {
        if constexpr (GRAD) {
#pragma unroll
            for (int i = 0; i < 3; ++i) f[i] = w * (g[0][0] * adj[0][i] + g[0][1] * adj[1][i] + g[0][2] * adj[2][i]);
        } else {
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) s += g[i][j] * adj[j][i];
            f[0] = w * s;
        }
    };
    if constexpr (T == LESASM_TET04) {  // constant gradients: sum_g w_g N_a(g) = 1/24
        double J[3][3], g[NI][3], adj[3][3], f[NO];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
#pragma unroll
            for (int i = 0; i < 3; ++i) J[i][k] = xa(k + 1, i) - xa(0, i);
#pragma unroll
            for (int i = 0; i < NI; ++i) g[i][k] = va(k + 1, i) - va(0, i);
        }
        adjugate(J, adj);
        point(g, adj, 1.0 / 24.0, f);
#pragma unroll
        for (int o = 0; o < NO; ++o)
#pragma unroll
            for (int a = 0; a < 4; ++a) r[o][a] = f[o];
    } else {
        using M = Modal<T>;
        constexpr int nm = M::nm;
        double X[3][nm], C[NI][nm], F[NO][nm], v[nn];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
#pragma unroll
            for (int a = 0; a < nn; ++a) v[a] = xa(a, i) - xa(0, i);
            M::to_modal(v, X[i]);
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
#pragma unroll
            for (int a = 0; a < nn; ++a) v[a] = va(a, i) - va(0, i);
            M::to_modal(v, C[i]);
        }
#pragma unroll
        for (int o = 0; o < NO; ++o)
#pragma unroll
            for (int m = 0; m < nm; ++m) F[o][m] = 0.0;
        const auto &pt = M::pts();
#pragma unroll 1
        for (int gp = 0; gp < M::ng; ++gp) {
            const double *q = pt.q[gp];
            double J[3][3], g[NI][3], adj[3][3], f[NO];
#pragma unroll
            for (int i = 0; i < 3; ++i) M::grad(X[i], q, J[i]);
#pragma unroll
            for (int i = 0; i < NI; ++i) M::grad(C[i], q, g[i]);
            adjugate(J, adj);
            point(g, adj, -pt.w[gp], f);  // (the weights carry the residual's sign)
#pragma unroll
            for (int o = 0; o < NO; ++o) M::test_value(F[o], q, f[o]);
        }
#pragma unroll
        for (int o = 0; o < NO; ++o) M::to_nodal(F[o], r[o]);
    }
}

template <int T, bool GRAD, bool PERIODIC>
__device__ __forceinline__ void project_chunk(const ChunkView &c, int j, double *lds, const double *__restrict__ xyz,
                                              const double *__restrict__ in, double *__restrict__ out) {
    constexpr int nn = Ref<T>::nn, NI = GRAD ? 1 : 3, NO = GRAD ? 3 : 1;
    const int e0 = c.eoff[j], e1 = c.eoff[j + 1];
    const int g0 = c.goff[j], ng = c.goff[j + 1] - g0;
    const int f0 = PERIODIC ? c.foff[j] : g0;
    const int nf = PERIODIC ? c.foff[j + 1] - f0 : ng;
    double *sx = lds, *sv = sx + 3 * ng, *sacc = sv + NI * nf;
    uint32_t *stag = (uint32_t *)(sacc + NO * nf);  // the write-back waits for no index
    const int step = (int)blockDim.x;
    if constexpr (PERIODIC)
        for (int k = threadIdx.x; k < ng; k += step) {
            const size_t g = (size_t)c.gnodes[g0 + k];
#pragma unroll
            for (int i = 0; i < 3; ++i) sx[3 * k + i] = xyz[3 * g + i];
        }
    // kStage nodes of a thread under way together, as in chunk_body
    for (int k0 = threadIdx.x; k0 < nf; k0 += kStage * step) {
        uint32_t tag[kStage];
        double x[kStage][3], v[kStage][NI];
#pragma unroll
        for (int q = 0; q < kStage; ++q)
            if (k0 + q * step < nf) tag[q] = (uint32_t)c.fnodes[f0 + k0 + q * step];
#pragma unroll
        for (int q = 0; q < kStage; ++q)
            if (k0 + q * step < nf) {
                const size_t f = tag[q] & ~kOwnedBit;
                if constexpr (!PERIODIC) {  // the field nodes are the geometry nodes
#pragma unroll
                    for (int i = 0; i < 3; ++i) x[q][i] = xyz[3 * f + i];
                }
#pragma unroll
                for (int i = 0; i < NI; ++i) v[q][i] = in[NI * f + i];
            }
#pragma unroll
        for (int q = 0; q < kStage; ++q) {
            const int k = k0 + q * step;
            if (k >= nf) continue;
            stag[k] = tag[q];
            if constexpr (!PERIODIC) {
#pragma unroll
                for (int i = 0; i < 3; ++i) sx[3 * k + i] = x[q][i];
            }
#pragma unroll
            for (int i = 0; i < NI; ++i) sv[NI * k + i] = v[q][i];
#pragma unroll
            for (int o = 0; o < NO; ++o) sacc[NO * k + o] = 0.0;
        }
    }
    __syncthreads();
    for (int base = e0; base < e1; base += blockDim.x) {
        // neighbouring elements on different wavefronts, as in chunk_body
        const int e = base + (int)blockDim.x <= e1
                          ? base + (int)(threadIdx.x & 63) * (int)(blockDim.x >> 6) + (int)(threadIdx.x >> 6)
                          : base + (int)threadIdx.x;
        if (e >= e1) break;
        int lg[nn], lf[nn];
#pragma unroll
        for (int a = 0; a < nn; ++a) {
            lg[a] = c.lg[(size_t)a * c.ld + e];
            lf[a] = PERIODIC ? (int)c.lf[(size_t)a * c.ld + e] : lg[a];
        }
        double r[NO][nn];
        element_project<T, GRAD>([&](int a, int i) { return sx[3 * lg[a] + i]; },
                                 [&](int a, int i) { return sv[NI * lf[a] + i]; }, r);
#pragma unroll
        for (int a = 0; a < nn; ++a)
#pragma unroll
            for (int o = 0; o < NO; ++o) unsafeAtomicAdd(sacc + NO * lf[a] + o, r[o][a]);
    }
    __syncthreads();
    // one thread per entry, so that the atomics of neighbouring lanes fall into the same cache lines
    for (int t = threadIdx.x; t < NO * nf; t += blockDim.x) {
        const int k = t / NO;
        const uint32_t tag = stag[k];
        double *dst = out + NO * (size_t)(tag & ~kOwnedBit) + (t - NO * k);
        if (tag & kOwnedBit) *dst = sacc[t];
        else unsafeAtomicAdd(dst, sacc[t]);
    }
}

template <bool GRAD, bool PERIODIC>
__global__ __launch_bounds__(256) void k_project_chunks(ChunkViews pv, const double *__restrict__ xyz,
                                                        const double *__restrict__ in, double *__restrict__ out) {
    extern __shared__ __align__(16) double lds[];
    const int b = blockIdx.x;
    auto chunk = [&](int k) { return xcd_block(b - pv.first[k], pv.first[k + 1] - pv.first[k]); };
    if (b < pv.first[1]) project_chunk<LESASM_HEX08, GRAD, PERIODIC>(pv.v[0], chunk(0), lds, xyz, in, out);
    else if (b < pv.first[2]) project_chunk<LESASM_PEN06, GRAD, PERIODIC>(pv.v[1], chunk(1), lds, xyz, in, out);
    else if (b < pv.first[3]) project_chunk<LESASM_PYR05, GRAD, PERIODIC>(pv.v[2], chunk(2), lds, xyz, in, out);
    else project_chunk<LESASM_TET04, GRAD, PERIODIC>(pv.v[3], chunk(3), lds, xyz, in, out);
}

// Adds the operator's contributions into the zeroed out (chunked meshes).
template <bool GRAD>
void launch_project_chunks(const lesasm_mesh *m, const double *in, double *out, hipStream_t s) {
    const ChunkViews pv = chunk_views(m);
    int doubles = 0;
    for (const Category &c : m->cat) doubles = std::max(doubles, c.project_doubles);
    const dim3 grid(pv.first[kNumCat]), block(256);
    const size_t shm = sizeof(double) * (size_t)doubles;
    if (grid.x == 0) return;
    if (mesh_is_periodic(m)) hipLaunchKernelGGL((k_project_chunks<GRAD, true>), grid, block, shm, s, pv, m->d_xyz, in, out);
    else hipLaunchKernelGGL((k_project_chunks<GRAD, false>), grid, block, shm, s, pv, m->d_xyz, in, out);
}

__device__ __forceinline__ int find_col(const int32_t *__restrict__ col, int lo, int hi, int key) {
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (col[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// K_ab += sum_g w det grad N_a . grad N_b into the CSR matrix (rows = field nodes)
template <int T>
__global__ __launch_bounds__(256) void k_laplacian(CatView c, const double *__restrict__ xyz,
                                                   const int32_t *__restrict__ rowptr,
                                                   const int32_t *__restrict__ col, double *__restrict__ val) {
    using E = Ref<T>;
    constexpr int nn = E::nn;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= c.n) return;
    double x[nn][3], Ke[nn][nn];
    int fid[nn];
    load_geometry<T>(c, e, xyz, x, fid);
#pragma unroll
    for (int a = 0; a < nn; ++a)
#pragma unroll
        for (int b = 0; b < nn; ++b) Ke[a][b] = 0.0;
#pragma unroll
    for (int g = 0; g < E::ng; ++g) {
        double Ki[3][3], dx[nn][3];
        const double det = jac_inverse<T>(x, g, Ki);
#pragma unroll
        for (int a = 0; a < nn; ++a)
#pragma unroll
            for (int i = 0; i < 3; ++i)
                dx[a][i] = Ki[0][i] * E::tab.dN[g][a][0] + Ki[1][i] * E::tab.dN[g][a][1] +
                           Ki[2][i] * E::tab.dN[g][a][2];
        const double wd = E::tab.w[g] * det;
#pragma unroll
        for (int a = 0; a < nn; ++a)
#pragma unroll
            for (int b = 0; b < nn; ++b) Ke[a][b] += wd * (dx[a][0] * dx[b][0] + dx[a][1] * dx[b][1] + dx[a][2] * dx[b][2]);
    }
#pragma unroll
    for (int a = 0; a < nn; ++a) {
        const int r0 = rowptr[fid[a]], r1 = rowptr[fid[a] + 1];
#pragma unroll
        for (int b = 0; b < nn; ++b) unsafeAtomicAdd(val + find_col(col, r0, r1, fid[b]), Ke[a][b]);
    }
}

// ---- vector kernels ----------------------------------------------------------

// Conjugate-gradient kernels: three launches an iteration (product, residual
// update, direction), each on a grid fixed by the row count, so every reduction
// runs in a fixed order.  A kernel leaves one partial sum per workgroup; the
// workgroups of the next one each add all of them, while their first rows are on
// the way, instead of a single-workgroup reduction launch (5 us) between them.
// An iteration with 2.9 k rows takes 15 us against 24 with five launches, with
// 117 k rows 19 against 31, 0.45 M 37 against 55, 0.89 M 66 against 86, 8.8 M
// (bound by the bytes) 667 against 676.
constexpr int kSpmvBlocks = 8192;       // most workgroups (partial sums) of the product
constexpr int kVecBlocks = 1024;        // and of the vector kernels
constexpr int kVecRows = 2;             // rows a thread of the vector kernels has in flight
constexpr int kMaxCapturedCg = 100000;  // CG iterations a step graph may hold
constexpr int kLanesPerRow = 8;         // CSR product: lanes per row
constexpr int kRowUnroll = 4;           // and row entries in flight per lane

// CG iteration `it` runs only while it <= *state, where *state is the iteration
// that met the tolerance (INT32_MAX until then).
__device__ __forceinline__ bool cg_skip(const int *state, int it) { return state && it > *state; }

// Fixed-order sum of v over a workgroup of 256 threads, in every thread.
__device__ __forceinline__ double block_sum_256(double v, double *sh) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();  // sh may still be read from a previous sum
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// The same of two values at once (sh: 8 doubles).
__device__ __forceinline__ void block_sum2_256(double &v, double &w, double *sh) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        v += __shfl_xor(v, o);
        w += __shfl_xor(w, o);
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        sh[threadIdx.x >> 6] = v;
        sh[4 + (threadIdx.x >> 6)] = w;
    }
    __syncthreads();
    v = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    w = (sh[4] + sh[5]) + (sh[6] + sh[7]);
}

// Sum of partial[b], b < nb, in every thread; and of pairs partial[2b], partial[2b+1].
__device__ __forceinline__ double partial_sum_256(const double *__restrict__ partial, int nb, double *sh) {
    double v = 0.0;
#pragma unroll 4
    for (int b = threadIdx.x; b < nb; b += 256) v += partial[b];
    return block_sum_256(v, sh);
}
__device__ __forceinline__ void partial_sum2_256(const double *__restrict__ partial, int nb, double &v, double &w,
                                                 double *sh) {
    v = w = 0.0;
#pragma unroll 4
    for (int b = threadIdx.x; b < nb; b += 256) {
        v += partial[2 * b];
        w += partial[2 * b + 1];
    }
    block_sum2_256(v, w, sh);
}

// q = K p with kLanesPerRow lanes per row (coalesced reads of the row's
// entries, kRowUnroll of them in flight per lane, fixed shuffle tree), and
// partial[b] = block sums of p.q.  Each lane adds its entries in row order.
__global__ __launch_bounds__(256) void k_spmv_dot(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                                                  const double *__restrict__ val, const double *__restrict__ p,
                                                  double *__restrict__ q, int n, double *__restrict__ partial,
                                                  const int *state, int it) {
    if (cg_skip(state, it)) return;
    __shared__ double sh[4];
    const int lane = threadIdx.x % kLanesPerRow;
    const int rows_per_block = 256 / kLanesPerRow;
    double pq = 0.0;
    for (int64_t base = blockIdx.x * rows_per_block; base < n; base += gridDim.x * rows_per_block) {
        const int64_t row = base + (int)threadIdx.x / kLanesPerRow;
        double s = 0.0;
        if (row < n) {
            const int k1 = rowptr[row + 1];
            for (int64_t k = rowptr[row] + lane; k < k1; k += kRowUnroll * kLanesPerRow) {
                int c[kRowUnroll];
                double v[kRowUnroll];
#pragma unroll
                for (int j = 0; j < kRowUnroll; ++j) {
                    const int64_t kk = k + j * kLanesPerRow;
                    c[j] = kk < k1 ? col[kk] : -1;
                    v[j] = kk < k1 ? val[kk] : 0.0;
                }
#pragma unroll
                for (int j = 0; j < kRowUnroll; ++j)
                    if (c[j] >= 0) s += v[j] * p[c[j]];
            }
        }
#pragma unroll
        for (int o = kLanesPerRow / 2; o > 0; o >>= 1) s += __shfl_down(s, o, kLanesPerRow);
        if (lane == 0 && row < n) {
            q[row] = s;
            pq += s * p[row];
        }
    }
    pq = block_sum_256(pq, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = pq;
}

#ifndef LESASM_CG_SELL
#define LESASM_CG_SELL 1
#endif
constexpr int kSlice = 64;  // rows per slice of the sliced-ELLPACK copy (one wavefront)

// Entries j .. j + U - 1 of a slice's 64 rows: columns and values.  The loads go
// through a buffer descriptor of the slice's extent, so entries past its width
// cost no branch and no traffic (they read as 0 and are not added).  The whole
// position is in the lane offset, which the descriptor's extent bounds; the scalar
// offset operand is 0, because the bounds check does not cover it.
template <bool NT, int U> struct SellBatch {
    int c[U];
    double v[U];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t cols, __amdgpu_buffer_rsrc_t vals, unsigned lane, int j) {
        constexpr int aux = NT ? 2 : 0;  // nontemporal
        const unsigned at = lane + kSlice * (unsigned)j;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            c[k] = (int)__builtin_amdgcn_raw_buffer_load_b32(cols, 4 * at + 4 * kSlice * k, 0, aux);
            v[k] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(vals, 8 * at + 8 * kSlice * k, 0, aux));
        }
    }
    __device__ __forceinline__ void gather(const double *__restrict__ p, double (&g)[U]) const {
#pragma unroll
        for (int k = 0; k < U; ++k) g[k] = p[(unsigned)c[k]];
    }
    __device__ __forceinline__ double add(double s, const double (&g)[U], int j, int w) const {
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const double t = fma(v[k], g[k], s);
            s = j + k < w ? t : s;
        }
        return s;
    }
};

// q = K p on the sliced-ELLPACK copy of K: slice s holds rows 64 s .. 64 s +
// 63, padded to its longest row and stored column-major, so entry j of all 64
// rows is one coalesced load; lane l adds row 64 s + l's entries in column
// order.  Padding entries hold value 0 and a valid column.  One wavefront per
// slice, slices in a fixed grid-stride order; partial[b] = block sums of p.q.
// Bound by the matrix bytes (12 B an entry) once enough loads are in flight:
// U entries are loaded while the U before them gather p and are added.  U = 4
// with plain loads (entries of 0.45 M rows: 24.0 us; 3, 6, 8: 25.0, 25.0, 26.2;
// four at a time without the overlap 28.6), 3 with nontemporal ones (8.8 M rows:
// 527 us; 2, 4, 6, 8: 546, 535, 551, 576; without the overlap 532).
// NT: nontemporal matrix loads (see kKeepBytes).
template <bool NT>
__global__ __launch_bounds__(256) void k_spmv_sell_dot(const int32_t *__restrict__ soff,
                                                       const int32_t *__restrict__ scol,
                                                       const double *__restrict__ sval, const double *__restrict__ p,
                                                       double *__restrict__ q, int n, int nslices,
                                                       double *__restrict__ partial, const int *state, int it) {
    if (cg_skip(state, it)) return;
    __shared__ double sh[4];
    const unsigned lane = threadIdx.x % kSlice;
    const int waves = 256 / kSlice;
    constexpr int U = NT ? 3 : 4;
    double pq = 0.0;
    for (int sl = __builtin_amdgcn_readfirstlane(blockIdx.x * waves + threadIdx.x / kSlice); sl < nslices;
         sl += gridDim.x * waves) {
        const int o0 = soff[sl], w = (soff[sl + 1] - o0) / kSlice;
        const auto cols = __builtin_amdgcn_make_buffer_rsrc((void *)(scol + o0), 0, 4 * kSlice * w, 0x00020000);
        const auto vals = __builtin_amdgcn_make_buffer_rsrc((void *)(sval + o0), 0, 8 * kSlice * w, 0x00020000);
        double s = 0.0;
        SellBatch<NT, U> a, b;
        a.load(cols, vals, lane, 0);
        // loads return in order: a batch's gathers are issued before the next
        // batch's loads, so that adding them does not wait for those
        for (int j = 0; j < w; j += 2 * U) {
            double g[U];
            a.gather(p, g);
            __builtin_amdgcn_sched_barrier(0);
            b.load(cols, vals, lane, j + U);
            __builtin_amdgcn_sched_barrier(0);
            s = a.add(s, g, j, w);
            b.gather(p, g);
            __builtin_amdgcn_sched_barrier(0);
            a.load(cols, vals, lane, j + 2 * U);
            __builtin_amdgcn_sched_barrier(0);
            s = b.add(s, g, j + U, w);
        }
        const int row = sl * kSlice + (int)lane;
        if (row < n) {
            q[row] = s;
            pq += s * p[row];
        }
    }
    pq = block_sum_256(pq, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = pq;
}

// sliced-ELLPACK values from the assembled CSR values (src < 0: padding)
__global__ void k_sell_fill(const int32_t *__restrict__ src, const double *__restrict__ val, double *__restrict__ sval,
                            int64_t total) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x)
        sval[i] = src[i] >= 0 ? val[src[i]] : 0.0;
}

// pq = sum of the product's nb partial sums (kept in scal[i_pq]);
// alpha = rz / pq;  r -= alpha q;  z = r / diag  (x is advanced with the old
// direction by k_cg_direction, which reads p anyway);
// partial[2b] = block sums of r.z, partial[2b+1] = of r.r
__global__ __launch_bounds__(256) void k_cg_update(double *__restrict__ r, double *__restrict__ z,
                                                   const double *__restrict__ q, const double *__restrict__ diag,
                                                   double *scal, int i_rz, int i_pq, int n,
                                                   const double *__restrict__ pq_partial, int nb,
                                                   double *__restrict__ partial, const int *state, int it) {
    if (cg_skip(state, it)) return;
    __shared__ double sh[8];
    const int64_t stride = (int64_t)gridDim.x * 256;
    int64_t i = blockIdx.x * 256 + threadIdx.x;
    // rows i, i + stride, ... kVecRows at a time; the first ones are loaded
    // before the partial sums are waited for
    double rv[kVecRows], qv[kVecRows], dv[kVecRows];
    auto load = [&](int64_t at) {
#pragma unroll
        for (int k = 0; k < kVecRows; ++k)
            if (at + k * stride < n) {
                rv[k] = r[at + k * stride];
                qv[k] = q[at + k * stride];
                dv[k] = diag[at + k * stride];
            }
    };
    load(i);
    const double pq = partial_sum_256(pq_partial, nb, sh);
    if (blockIdx.x == 0 && threadIdx.x == 0) scal[i_pq] = pq;
    const double alpha = scal[i_rz] / pq;
    double rz = 0.0, rr = 0.0;
    while (i < n) {
#pragma unroll
        for (int k = 0; k < kVecRows; ++k)
            if (i + k * stride < n) {
                const double ri = rv[k] - alpha * qv[k];
                const double zi = ri / dv[k];
                r[i + k * stride] = ri;
                z[i + k * stride] = zi;
                rz += ri * zi;
                rr += ri * ri;
            }
        i += kVecRows * stride;
        load(i);
    }
    block_sum2_256(rz, rr, sh);
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = rz;
        partial[2 * blockIdx.x + 1] = rr;
    }
}

// rz_new, r.r = sums of the update's nb partial sums (kept in scal);
// x += (rz_old / pq) p;  p = z + (rz_new / rz_old) p.
// An iteration with |r| <= tol |b| records itself in *state, which ends the
// solve: tol is rtol where the solve tests and a level below it in between (see
// pressure_solve).  host, if given, receives {r.r, b.b, met, it} in host[0..3]
// from a test and in host[4..7] from an iteration that ended the solve between
// two tests.
__global__ __launch_bounds__(256) void k_cg_direction(double *__restrict__ x, double *__restrict__ p,
                                                      const double *__restrict__ z, double *scal, int i_new, int i_old,
                                                      int i_pq, int i_rr, int i_bb, int n,
                                                      const double *__restrict__ partial, int nb, int *state, int it,
                                                      bool test, double tol, double *host) {
    if (cg_skip(state, it)) return;
    __shared__ double sh[8];
    const int64_t stride = (int64_t)gridDim.x * 256;
    int64_t i = blockIdx.x * 256 + threadIdx.x;
    double xv[kVecRows], pv[kVecRows], zv[kVecRows];
    auto load = [&](int64_t at) {  // as in k_cg_update
#pragma unroll
        for (int k = 0; k < kVecRows; ++k)
            if (at + k * stride < n) {
                xv[k] = x[at + k * stride];
                pv[k] = p[at + k * stride];
                zv[k] = z[at + k * stride];
            }
    };
    load(i);
    double rz, rr;
    partial_sum2_256(partial, nb, rz, rr, sh);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const double bb = scal[i_bb];
        const bool met = sqrt(rr) <= tol * sqrt(bb);
        scal[i_new] = rz;
        scal[i_rr] = rr;
        if (met) *state = it;
        if (host && (test || met)) {
            double *rec = test ? host : host + 4;
            rec[0] = rr;
            rec[1] = bb;
            rec[2] = met ? 1.0 : 0.0;
            rec[3] = it;
        }
    }
    const double alpha = scal[i_old] / scal[i_pq];
    const double beta = rz / scal[i_old];
    while (i < n) {
#pragma unroll
        for (int k = 0; k < kVecRows; ++k)
            if (i + k * stride < n) {
                x[i + k * stride] = xv[k] + alpha * pv[k];
                p[i + k * stride] = zv[k] + beta * pv[k];
            }
        i += kVecRows * stride;
        load(i);
    }
}

// y = a0 x0 + a1 x1 + a2 x2 (x1, x2 may be NULL)
__global__ void k_lincomb(double *__restrict__ y, double a0, const double *__restrict__ x0, double a1,
                          const double *__restrict__ x1, double a2, const double *__restrict__ x2, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        double v = a0 * x0[i];
        if (x1) v += a1 * x1[i];
        if (x2) v += a2 * x2[i];
        y[i] = v;
    }
}

__global__ void k_diag(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                       const double *__restrict__ val, double *__restrict__ d, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double v = 0.0;
    for (int q = rowptr[i]; q < rowptr[i + 1]; ++q)
        if (col[q] == i) v = val[q];
    d[i] = v;
}

// u_new = u* - dt M^-1 (G dp)
__global__ void k_correct(double *__restrict__ u, const double *__restrict__ ustar, const double *__restrict__ gdp,
                          const double *__restrict__ mass, double dt, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const double s = dt / mass[i];
        u[3 * (size_t)i + 0] = ustar[3 * (size_t)i + 0] - s * gdp[3 * (size_t)i + 0];
        u[3 * (size_t)i + 1] = ustar[3 * (size_t)i + 1] - s * gdp[3 * (size_t)i + 1];
        u[3 * (size_t)i + 2] = ustar[3 * (size_t)i + 2] - s * gdp[3 * (size_t)i + 2];
    }
}

// Block sums of a (the first of two passes that take a mean).
__global__ __launch_bounds__(256) void k_sum_partial(const double *__restrict__ a, int n, double *__restrict__ partial) {
    __shared__ double sh[4];
    double v = 0.0;
#pragma unroll 4
    for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) v += a[i];
    v = block_sum_256(v, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = v;
}

// x -= mean(x), from the block sums of x
__global__ __launch_bounds__(256) void k_sub_mean(double *__restrict__ x, const double *__restrict__ partial, int nb, int n) {
    __shared__ double sh[4];
    const double m = partial_sum_256(partial, nb, sh) / n;
    for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) x[i] -= m;
}

// Start of a CG from the block sums of b: r = b - mean(b), x = 0, z = r / diag,
// p = z; out[2k], out[2k+1] = block sums of r.r (= b.b) and r.z.  x may be b.
__global__ __launch_bounds__(256) void k_cg_setup(const double *b, const double *__restrict__ diag,
                                                  double *x, double *__restrict__ r, double *__restrict__ z,
                                                  double *__restrict__ p, int n,
                                                  const double *__restrict__ partial, int nb, double *__restrict__ out) {
    __shared__ double sh[8];
    const double m = partial_sum_256(partial, nb, sh) / n;
    double bb = 0.0, rz = 0.0;
    for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const double ri = b[i] - m, zi = ri / diag[i];
        x[i] = 0.0;
        r[i] = ri;
        z[i] = zi;
        p[i] = zi;
        bb += ri * ri;
        rz += ri * zi;
    }
    block_sum2_256(bb, rz, sh);
    if (threadIdx.x == 0) {
        out[2 * blockIdx.x] = bb;
        out[2 * blockIdx.x + 1] = rz;
    }
}

// b.b and r.z of the start, and *state: no iteration yet met the tolerance;
// with a zero right-hand side every iteration is skipped.
__global__ __launch_bounds__(256) void k_cg_begin(const double *__restrict__ partial, int nb, double *scal, int i_bb,
                                                  int i_rz, int *state) {
    __shared__ double sh[8];
    double bb, rz;
    partial_sum2_256(partial, nb, bb, rz, sh);
    if (threadIdx.x == 0) {
        scal[i_bb] = bb;
        scal[i_rz] = rz;
        state[0] = bb > 0.0 ? INT32_MAX : 0;
    }
}

// End of a captured CG: rec = {iterations run, relative residual, converged}.
__global__ void k_cg_end(const int *state, const double *scal, int i_rr, int i_bb, int maxit, double *rec) {
    if (threadIdx.x != 0) return;
    const int conv = state[0];
    const double bb = scal[i_bb];
    rec[0] = (double)(conv < maxit ? conv : maxit);
    rec[1] = bb > 0.0 ? sqrt(scal[i_rr] / bb) : 0.0;
    rec[2] = conv <= maxit ? 1.0 : 0.0;
}

__global__ void k_zero(double *__restrict__ a, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        a[i] = 0.0;
}

// Launches KERNEL<type> over every non-empty category of mesh m on stream s.
#define LESASM_PER_CATEGORY(KERNEL, m, s, ...)                                                              \
    for (int k_ = 0; k_ < kNumCat; ++k_) {                                                                 \
        const Category &c_ = (m)->cat[k_];                                                                 \
        if (c_.n == 0) continue;                                                                           \
        CatView v_{c_.d_cg, c_.d_cf, c_.d_delta, (int32_t)c_.n, 0, (int32_t)c_.n};                         \
        const dim3 g_((unsigned)((c_.n + 255) / 256)), b_(256);                                            \
        switch (c_.type) {                                                                                 \
        case LESASM_TET04: hipLaunchKernelGGL(KERNEL<LESASM_TET04>, g_, b_, 0, (s), v_, __VA_ARGS__); break; \
        case LESASM_PYR05: hipLaunchKernelGGL(KERNEL<LESASM_PYR05>, g_, b_, 0, (s), v_, __VA_ARGS__); break; \
        case LESASM_PEN06: hipLaunchKernelGGL(KERNEL<LESASM_PEN06>, g_, b_, 0, (s), v_, __VA_ARGS__); break; \
        case LESASM_HEX08: hipLaunchKernelGGL(KERNEL<LESASM_HEX08>, g_, b_, 0, (s), v_, __VA_ARGS__); break; \
        }                                                                                                  \
    }

}  // namespace lesasm

using namespace lesasm;

struct lesasm_stepper {
    lesasm_mesh *mesh = nullptr;
    double nu = 0.0, dt = 0.0, rtol = 1e-12;
    int maxit = 1000, check_every = 16;
    int n = 0;
    int32_t *rowptr = nullptr, *col = nullptr;
    double *val = nullptr, *diag = nullptr;
    double *k1 = nullptr, *k3 = nullptr, *us = nullptr, *ustar = nullptr, *gdp = nullptr;  // [n][3]
    double *x = nullptr, *r = nullptr, *z = nullptr, *pv = nullptr, *q = nullptr;  // [n]
    double *partial = nullptr, *scal = nullptr;  // reductions
    std::vector<void *> allocs;
    int spmv_blocks = 0, vec_blocks = 0;  // grids of the CG kernels
    int last_iters = 0;
    double last_res = 0.0;
    int64_t nnz = 0;
    // sliced-ELLPACK copy of K for the CG's SpMV (empty if not built)
    int32_t *soff = nullptr, *scol = nullptr;
    double *sval = nullptr;
    int nslices = 0;
    int64_t sell_entries = 0;
    int *d_cgstate = nullptr;   // iteration that met the tolerance (see cg_skip)
    double *h_rec = nullptr;    // pinned: two records of k_cg_direction
    hipEvent_t ev_check = nullptr;  // end of the iteration that made it
};

// A whole time step captured in a HIP graph, bound to one (u, p) pair.
struct lesasm_step_graph {
    lesasm_stepper *st = nullptr;
    double *u = nullptr, *p = nullptr;
    int cg_iters = 0;
    double *d_rec = nullptr;        // {iterations, relative residual, converged} of the last replay
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipEvent_t ev_last = nullptr;   // recorded after every replay
    bool launched = false;
};

namespace {

template <class T> int salloc(lesasm_stepper *st, T **p, size_t n) {
    *p = nullptr;
    if (!n) return LESASM_OK;
    void *q = nullptr;
    int rc = device_alloc(&q, n * sizeof(T), "stepper");
    if (rc) return rc;
    st->allocs.push_back(q);
    *p = (T *)q;
    return LESASM_OK;
}

void stepper_free(lesasm_stepper *st) {
    if (!st) return;
    (void)hipDeviceSynchronize();
    for (void *p : st->allocs) device_free(p);
    if (st->h_rec) (void)hipHostFree(st->h_rec);
    if (st->ev_check) (void)hipEventDestroy(st->ev_check);
    delete st;
}

enum { S_RZ = 0, S_PQ, S_RR, S_RZN, S_BB, S_NUM };

// A matrix copy up to this size stays in the 256 MB Infinity Cache between
// products; a larger one is read past it (nontemporal), so that p and the other
// vectors keep the caches.  Per iteration, plain against nontemporal: 122 MB 41
// against 51 us, 242 MB 72 against 82, 476 MB 157 against 150.
constexpr int64_t kKeepBytes = (int64_t)320 << 20;

void launch_spmv(const lesasm_stepper *st, const double *p, double *q, const int *state, int it, hipStream_t s) {
    const dim3 g(st->spmv_blocks), b(256);
    if (!st->sval)
        hipLaunchKernelGGL(k_spmv_dot, g, b, 0, s, st->rowptr, st->col, st->val, p, q, st->n, st->partial, state, it);
    else if (12 * st->sell_entries > kKeepBytes)
        hipLaunchKernelGGL(k_spmv_sell_dot<true>, g, b, 0, s, st->soff, st->scol, st->sval, p, q, st->n, st->nslices,
                           st->partial, state, it);
    else
        hipLaunchKernelGGL(k_spmv_sell_dot<false>, g, b, 0, s, st->soff, st->scol, st->sval, p, q, st->n, st->nslices,
                           st->partial, state, it);
}

// CG iteration it (1, 2, ...) for solution x.  The old and new r.z use two slots
// alternately, so that no scalar is overwritten while a kernel may still read it.
void launch_cg_iteration(lesasm_stepper *st, double *x, int it, bool test, double tol, double *host, hipStream_t s) {
    const int i_rz = it & 1 ? S_RZ : S_RZN, i_rzn = it & 1 ? S_RZN : S_RZ;
    int *state = st->d_cgstate;
    const dim3 g(st->vec_blocks), b(256);
    double *rpart = st->partial + kSpmvBlocks;
    launch_spmv(st, st->pv, st->q, state, it, s);
    hipLaunchKernelGGL(k_cg_update, g, b, 0, s, st->r, st->z, st->q, st->diag, st->scal, i_rz, (int)S_PQ, st->n,
                       st->partial, st->spmv_blocks, rpart, (const int *)state, it);
    hipLaunchKernelGGL(k_cg_direction, g, b, 0, s, x, st->pv, st->z, st->scal, i_rzn, i_rz, (int)S_PQ, (int)S_RR,
                       (int)S_BB, st->n, rpart, st->vec_blocks, state, it, test, tol, host);
}

// Start of a solve (before iteration 1) and its end (x to zero mean).
void launch_cg_start(lesasm_stepper *st, const double *b_in, double *x, hipStream_t s) {
    const dim3 g(st->vec_blocks), b(256);
    double *rpart = st->partial + kSpmvBlocks;
    hipLaunchKernelGGL(k_sum_partial, g, b, 0, s, b_in, st->n, st->partial);
    hipLaunchKernelGGL(k_cg_setup, g, b, 0, s, b_in, st->diag, x, st->r, st->z, st->pv, st->n, st->partial,
                       st->vec_blocks, rpart);
    hipLaunchKernelGGL(k_cg_begin, dim3(1), b, 0, s, rpart, st->vec_blocks, st->scal, (int)S_BB, (int)S_RZ,
                       st->d_cgstate);
}

void launch_cg_finish(lesasm_stepper *st, double *x, hipStream_t s) {
    const dim3 g(st->vec_blocks), b(256);
    hipLaunchKernelGGL(k_sum_partial, g, b, 0, s, x, st->n, st->partial);
    hipLaunchKernelGGL(k_sub_mean, g, b, 0, s, x, st->partial, st->vec_blocks, st->n);
}

// The convergence test runs on the device every check_every iterations (and
// after the last) and tells the host through pinned memory.  The host queues
// kCgAhead iterations behind a test before it waits for it, so the GPU does not
// idle while the answer travels (0.45 M rows: 36.9 against 38.8 us an iteration
// with a copy and a wait); if the test was met they return at once.
// Between two tests a solve also ends once the residual is at rounding: K is
// singular on closed and periodic meshes, and an iteration on a residual of
// rounding errors, whose constant part K cannot reduce, throws the solution off
// (8^3 periodic cube, 17 to 32 iterations: 2 to 12 % of the solves came back with
// residuals of 1e-8 to 1e-5).  Above rounding it goes on to the test whatever the
// tolerance: on a coarse one the iterations up to it are worth digits.
constexpr int kCgAhead = 4;
constexpr double kCgRounding = 1e-14;  // of |b|

int pressure_solve(lesasm_stepper *st, const double *b_in, double *x, hipStream_t s) {
    for (int k = 0; k < 8; ++k) st->h_rec[k] = -1.0;
    launch_cg_start(st, b_in, x, s);
    const double below = std::min(st->rtol, kCgRounding);
    int queued = 0, at = 0, iters = 0;
    double res = 0.0;
    bool met = false;
    while (at < st->maxit && !met) {
        at = std::min(at + st->check_every, st->maxit);
        const int next = std::min(at + st->check_every, st->maxit);
        auto queue = [&](int upto) {
            while (queued < upto) {
                ++queued;
                launch_cg_iteration(st, x, queued, queued == at, queued == at ? st->rtol : below, st->h_rec, s);
            }
        };
        queue(at);
        LESASM_HIP_TRY(hipEventRecord(st->ev_check, s));
        queue(std::min(at + kCgAhead, next - 1));
        LESASM_HIP_TRY(hipGetLastError());
        LESASM_HIP_TRY(hipEventSynchronize(st->ev_check));
        const volatile double *rec = st->h_rec;
        if (rec[3] != at) rec += 4;  // the test was skipped: the solve ended before it
        if (rec[3] < 0.0) break;     // or had nothing to do: zero right-hand side, x = 0
        iters = (int)rec[3];
        res = std::sqrt(rec[0]) / std::sqrt(rec[1]);
        met = rec[2] > 0.0;
    }
    st->last_iters = iters;
    st->last_res = res;
    launch_cg_finish(st, x, s);
    LESASM_HIP_TRY(hipGetLastError());
    return LESASM_OK;
}

// The same solve for graph capture, without host reads.  Exactly cg_iters
// iterations are captured; once the residual meets the tolerance (tested after
// every iteration) the remaining iterations return at once.  rec receives the
// iteration count, relative residual and convergence flag.
int pressure_solve_captured(lesasm_stepper *st, const double *b_in, double *x, hipStream_t s, int cg_iters,
                            double *rec) {
    launch_cg_start(st, b_in, x, s);
    for (int it = 1; it <= cg_iters; ++it) launch_cg_iteration(st, x, it, true, st->rtol, nullptr, s);
    hipLaunchKernelGGL(k_cg_end, dim3(1), dim3(64), 0, s, (const int *)st->d_cgstate, (const double *)st->scal,
                       (int)S_RR, (int)S_BB, cg_iters, rec);
    launch_cg_finish(st, x, s);
    LESASM_HIP_TRY(hipGetLastError());
    return LESASM_OK;
}

}  // namespace

extern "C" int lesasm_divergence(lesasm_mesh *m, const double *d_u, double *d_out, void *stream) {
    if (!m || (m->n_field && (!d_u || !d_out))) return fail(LESASM_E_INVALID_ARG, "divergence: NULL argument");
    hipStream_t s = (hipStream_t)stream;
    if (!m->n_field) return LESASM_OK;
    hipLaunchKernelGGL(k_zero, dim3(grid_for(m->n_field, 256)), dim3(256), 0, s, d_out, (size_t)m->n_field);
    if (mesh_is_chunked(m)) launch_project_chunks<false>(m, d_u, d_out, s);
    else LESASM_PER_CATEGORY(k_divergence, m, s, (const double *)m->d_xyz, d_u, d_out);
    LESASM_HIP_TRY(hipGetLastError());
    return LESASM_OK;
}

extern "C" int lesasm_gradient(lesasm_mesh *m, const double *d_p, double *d_out, void *stream) {
    if (!m || (m->n_field && (!d_p || !d_out))) return fail(LESASM_E_INVALID_ARG, "gradient: NULL argument");
    hipStream_t s = (hipStream_t)stream;
    if (!m->n_field) return LESASM_OK;
    hipLaunchKernelGGL(k_zero, dim3(grid_for(3 * (size_t)m->n_field, 256)), dim3(256), 0, s, d_out,
                       3 * (size_t)m->n_field);
    if (mesh_is_chunked(m)) launch_project_chunks<true>(m, d_p, d_out, s);
    else LESASM_PER_CATEGORY(k_gradient, m, s, (const double *)m->d_xyz, d_p, d_out);
    LESASM_HIP_TRY(hipGetLastError());
    return LESASM_OK;
}

extern "C" int lesasm_stepper_create(lesasm_mesh *m, double nu, double dt, double rtol, int maxit,
                                     lesasm_stepper **out) {
    if (!out) return fail(LESASM_E_INVALID_ARG, "stepper_create: out is NULL");
    *out = nullptr;
    if (!m || !(dt > 0.0) || !(rtol > 0.0) || maxit < 1)
        return fail(LESASM_E_INVALID_ARG, "stepper_create: need a mesh, dt > 0, rtol > 0, maxit >= 1");
    int dev = -1;
    LESASM_HIP_TRY(hipGetDevice(&dev));
    if (dev != m->device) return fail(LESASM_E_STATE, "stepper_create: current device differs from the mesh's");
    auto *st = new lesasm_stepper();
    struct Guard {
        lesasm_stepper *p;
        ~Guard() { stepper_free(p); }
    } guard{st};
    st->mesh = m;
    st->nu = nu;
    st->dt = dt;
    st->rtol = rtol;
    st->maxit = maxit;
    st->n = (int)m->n_field;
    const int n = st->n;
    st->spmv_blocks = std::max(1, std::min((int)(((int64_t)n + 4 * kSlice - 1) / (4 * kSlice)), kSpmvBlocks));
    st->vec_blocks = std::max(1, std::min((int)(((int64_t)n + 255) / 256), kVecBlocks));

    // CSR pattern of K: for each field node, the field nodes of its elements
    std::vector<int32_t> ninc(n + 1, 0);
    for (int k = 0; k < kNumCat; ++k) {
        const Category &c = m->cat[k];
        const std::vector<int32_t> &cf = c.h_cf.empty() ? c.h_cg : c.h_cf;
        for (int32_t f : cf) ninc[f + 1]++;
    }
    for (int i = 0; i < n; ++i) ninc[i + 1] += ninc[i];
    std::vector<int64_t> elem_of(ninc[n]);
    std::vector<int32_t> fill(ninc.begin(), ninc.end() - 1);
    int64_t gbase = 0;
    for (int k = 0; k < kNumCat; ++k) {
        const Category &c = m->cat[k];
        const std::vector<int32_t> &cf = c.h_cf.empty() ? c.h_cg : c.h_cf;
        for (int a = 0; a < c.type; ++a)
            for (int64_t e = 0; e < c.n; ++e) elem_of[fill[cf[(size_t)a * c.n + e]]++] = gbase + e;
        gbase += c.n;
    }
    auto elem_nodes = [&](int64_t ge, std::vector<int32_t> &outv) {
        for (int k = 0; k < kNumCat; ++k) {
            const Category &c = m->cat[k];
            if (ge < c.first || ge >= c.first + c.n) continue;
            const std::vector<int32_t> &cf = c.h_cf.empty() ? c.h_cg : c.h_cf;
            for (int a = 0; a < c.type; ++a) outv.push_back(cf[(size_t)a * c.n + (ge - c.first)]);
            return;
        }
    };
    std::vector<int32_t> rowptr(n + 1, 0), col, tmp;
    for (int i = 0; i < n; ++i) {
        tmp.clear();
        tmp.push_back(i);
        for (int32_t q = ninc[i]; q < ninc[i + 1]; ++q) elem_nodes(elem_of[q], tmp);
        std::sort(tmp.begin(), tmp.end());
        tmp.erase(std::unique(tmp.begin(), tmp.end()), tmp.end());
        col.insert(col.end(), tmp.begin(), tmp.end());
        rowptr[i + 1] = (int32_t)col.size();
    }
    st->nnz = (int64_t)col.size();
    int rc;
    if ((rc = salloc(st, &st->rowptr, rowptr.size())) || (rc = salloc(st, &st->col, col.size())) ||
        (rc = salloc(st, &st->val, col.size())) || (rc = salloc(st, &st->diag, (size_t)n)) ||
        (rc = salloc(st, &st->k1, 3 * (size_t)n)) || (rc = salloc(st, &st->k3, 3 * (size_t)n)) ||
        (rc = salloc(st, &st->us, 3 * (size_t)n)) || (rc = salloc(st, &st->ustar, 3 * (size_t)n)) ||
        (rc = salloc(st, &st->gdp, 3 * (size_t)n)) || (rc = salloc(st, &st->x, (size_t)n)) || (rc = salloc(st, &st->r, (size_t)n)) ||
        (rc = salloc(st, &st->z, (size_t)n)) || (rc = salloc(st, &st->pv, (size_t)n)) ||
        (rc = salloc(st, &st->q, (size_t)n)) || (rc = salloc(st, &st->partial, kSpmvBlocks + 2 * kVecBlocks)) ||
        (rc = salloc(st, &st->scal, S_NUM)) || (rc = salloc(st, &st->d_cgstate, 4)))
        return rc;
    LESASM_HIP_TRY(hipHostMalloc((void **)&st->h_rec, 8 * sizeof(double), hipHostMallocCoherent));
    LESASM_HIP_TRY(hipEventCreateWithFlags(&st->ev_check, hipEventDisableTiming));
    if (n) {
        LESASM_HIP_TRY(hipMemcpy(st->rowptr, rowptr.data(), sizeof(int32_t) * rowptr.size(), hipMemcpyHostToDevice));
        LESASM_HIP_TRY(hipMemcpy(st->col, col.data(), sizeof(int32_t) * col.size(), hipMemcpyHostToDevice));
        LESASM_HIP_TRY(hipMemset(st->val, 0, sizeof(double) * col.size()));
        hipStream_t s0 = 0;
        LESASM_PER_CATEGORY(k_laplacian, m, s0, (const double *)m->d_xyz, (const int32_t *)st->rowptr,
                            (const int32_t *)st->col, st->val);
        hipLaunchKernelGGL(k_diag, dim3((n + 255) / 256), dim3(256), 0, 0, st->rowptr, st->col, st->val, st->diag, n);
        LESASM_HIP_TRY(hipGetLastError());
        if (LESASM_CG_SELL) {
            // slices of kSlice rows, each padded to its longest row, column-major
            const int ns = (n + kSlice - 1) / kSlice;
            std::vector<int32_t> soff(ns + 1, 0);
            int64_t total = 0;
            for (int sl = 0; sl < ns; ++sl) {
                int w = 0;
                for (int r = sl * kSlice; r < std::min(n, (sl + 1) * kSlice); ++r) w = std::max(w, rowptr[r + 1] - rowptr[r]);
                total += (int64_t)w * kSlice;
                soff[sl + 1] = (int32_t)std::min<int64_t>(total, INT32_MAX);
            }
            if (total < INT32_MAX) {  // otherwise the CSR kernel serves the CG
                std::vector<int32_t> scol((size_t)total), src((size_t)total);
                for (int sl = 0; sl < ns; ++sl) {
                    const int w = (soff[sl + 1] - soff[sl]) / kSlice;
                    for (int l = 0; l < kSlice; ++l) {
                        const int r = sl * kSlice + l;
                        const int len = r < n ? rowptr[r + 1] - rowptr[r] : 0;
                        for (int j = 0; j < w; ++j) {
                            const size_t at = (size_t)soff[sl] + (size_t)j * kSlice + l;
                            if (j < len) {
                                scol[at] = col[(size_t)rowptr[r] + j];
                                src[at] = rowptr[r] + j;
                            } else {
                                scol[at] = r < n ? r : 0;
                                src[at] = -1;
                            }
                        }
                    }
                }
                int32_t *d_src = nullptr;
                if ((rc = salloc(st, &st->soff, soff.size())) || (rc = salloc(st, &st->scol, scol.size())) ||
                    (rc = salloc(st, &st->sval, scol.size())) || (rc = salloc(st, &d_src, src.size())))
                    return rc;
                LESASM_HIP_TRY(hipMemcpy(st->soff, soff.data(), sizeof(int32_t) * soff.size(), hipMemcpyHostToDevice));
                LESASM_HIP_TRY(hipMemcpy(st->scol, scol.data(), sizeof(int32_t) * scol.size(), hipMemcpyHostToDevice));
                LESASM_HIP_TRY(hipMemcpy(d_src, src.data(), sizeof(int32_t) * src.size(), hipMemcpyHostToDevice));
                hipLaunchKernelGGL(k_sell_fill, dim3(grid_for((size_t)total, 256)), dim3(256), 0, 0, d_src, st->val,
                                   st->sval, total);
                LESASM_HIP_TRY(hipGetLastError());
                LESASM_HIP_TRY(hipDeviceSynchronize());
                st->allocs.erase(std::find(st->allocs.begin(), st->allocs.end(), (void *)d_src));
                device_free(d_src);
                st->nslices = ns;
                st->sell_entries = total;
            }
        }
        LESASM_HIP_TRY(hipDeviceSynchronize());
    }
    guard.p = nullptr;
    *out = st;
    return LESASM_OK;
}

extern "C" int lesasm_stepper_destroy(lesasm_stepper *st) {
    stepper_free(st);
    return LESASM_OK;
}

extern "C" int lesasm_stepper_laplacian(lesasm_stepper *st, int32_t *rowptr, int32_t *col, double *val, int64_t *nnz) {
    if (!st || !nnz) return fail(LESASM_E_INVALID_ARG, "stepper_laplacian: NULL argument");
    *nnz = st->nnz;
    if (rowptr) LESASM_HIP_TRY(hipMemcpy(rowptr, st->rowptr, sizeof(int32_t) * (st->n + 1), hipMemcpyDeviceToHost));
    if (col) LESASM_HIP_TRY(hipMemcpy(col, st->col, sizeof(int32_t) * st->nnz, hipMemcpyDeviceToHost));
    if (val) LESASM_HIP_TRY(hipMemcpy(val, st->val, sizeof(double) * st->nnz, hipMemcpyDeviceToHost));
    return LESASM_OK;
}

extern "C" int lesasm_stepper_spmv(lesasm_stepper *st, const double *d_p, double *d_q, void *stream) {
    if (!st || (st->n && (!d_p || !d_q))) return fail(LESASM_E_INVALID_ARG, "stepper_spmv: NULL argument");
    if (d_p == d_q) return fail(LESASM_E_INVALID_ARG, "stepper_spmv: p and q must not alias");
    if (!st->n) return LESASM_OK;
    hipStream_t s = (hipStream_t)stream;
    launch_spmv(st, d_p, d_q, nullptr, 0, s);
    LESASM_HIP_TRY(hipGetLastError());
    return LESASM_OK;
}

extern "C" int lesasm_stepper_sell_entries(const lesasm_stepper *st, int64_t *entries) {
    if (!st || !entries) return fail(LESASM_E_INVALID_ARG, "stepper_sell_entries: NULL argument");
    *entries = st->sell_entries;
    return LESASM_OK;
}

extern "C" int lesasm_pressure_solve(lesasm_stepper *st, const double *d_b, double *d_x, void *stream) {
    if (!st || (st->n && (!d_b || !d_x))) return fail(LESASM_E_INVALID_ARG, "pressure_solve: NULL argument");
    if (!st->n) return LESASM_OK;
    return pressure_solve(st, d_b, d_x, (hipStream_t)stream);
}

// Three explicit stages only: d_ustar = u^n + dt (k1/4 + 3 k3/4).
static int rk3_stages(lesasm_stepper *st, const double *u, const double *p, double *ustar, hipStream_t s) {
    lesasm_mesh *m = st->mesh;
    const size_t n3 = 3 * (size_t)st->n;
    const int g = grid_for(n3, 256);
    int rc;
    // stage 1: k1 = dt M^-1 rhs(u^n); u2 = u^n + k1/3
    if ((rc = assemble_into(m, u, p, st->nu, st->dt, st->k1, s, true))) return rc;
    hipLaunchKernelGGL(k_lincomb, dim3(g), dim3(256), 0, s, st->us, 1.0, u, 1.0 / 3.0, st->k1, 0.0, nullptr, n3);
    // stage 2: k2 = dt M^-1 rhs(u2); u3 = u^n + 2 k2/3   (k2 held in k3)
    if ((rc = assemble_into(m, st->us, p, st->nu, st->dt, st->k3, s, true))) return rc;
    hipLaunchKernelGGL(k_lincomb, dim3(g), dim3(256), 0, s, st->us, 1.0, u, 2.0 / 3.0, st->k3, 0.0, nullptr, n3);
    // stage 3: k3 = dt M^-1 rhs(u3); u* = u^n + k1/4 + 3 k3/4
    if ((rc = assemble_into(m, st->us, p, st->nu, st->dt, st->k3, s, true))) return rc;
    hipLaunchKernelGGL(k_lincomb, dim3(g), dim3(256), 0, s, ustar, 1.0, u, 0.25, st->k1, 0.75, st->k3, n3);
    LESASM_HIP_TRY(hipGetLastError());
    return LESASM_OK;
}

extern "C" int lesasm_stepper_rk3_stages(lesasm_stepper *st, const double *d_u, const double *d_p, double *d_ustar,
                                         void *stream) {
    if (!st || (st->n && (!d_u || !d_ustar))) return fail(LESASM_E_INVALID_ARG, "rk3_stages: NULL argument");
    if (!st->n) return LESASM_OK;
    return rk3_stages(st, d_u, d_p, d_ustar, (hipStream_t)stream);
}

// One time step on s: the stages, b = -(1/dt) D u*, the pressure solve (eager
// with host convergence checks, or captured with cg_iters device-terminated
// iterations when rec is given), the correction and the pressure update.
static int step_body(lesasm_stepper *st, double *d_u, double *d_p, hipStream_t s, int cg_iters, double *rec) {
    lesasm_mesh *m = st->mesh;
    const int n = st->n;
    int rc;
    if ((rc = rk3_stages(st, d_u, d_p, st->ustar, s))) return rc;
    // b = -(1/dt) D u*
    if ((rc = lesasm_divergence(m, st->ustar, st->q, s))) return rc;
    hipLaunchKernelGGL(k_lincomb, dim3(grid_for(n, 256)), dim3(256), 0, s, st->q, -1.0 / st->dt, st->q, 0.0, nullptr,
                       0.0, nullptr, (size_t)n);
    if (rec) rc = pressure_solve_captured(st, st->q, st->x, s, cg_iters, rec);
    else rc = pressure_solve(st, st->q, st->x, s);
    if (rc) return rc;
    if ((rc = lesasm_gradient(m, st->x, st->gdp, s))) return rc;
    hipLaunchKernelGGL(k_correct, dim3(grid_for(n, 256)), dim3(256), 0, s, d_u, st->ustar, st->gdp, m->d_mass,
                       st->dt, n);
    hipLaunchKernelGGL(k_lincomb, dim3(grid_for(n, 256)), dim3(256), 0, s, d_p, 1.0, d_p, 1.0, st->x, 0.0, nullptr,
                       (size_t)n);
    LESASM_HIP_TRY(hipGetLastError());
    return LESASM_OK;
}

extern "C" int lesasm_stepper_step(lesasm_stepper *st, double *d_u, double *d_p, void *stream) {
    if (!st || (st->n && (!d_u || !d_p))) return fail(LESASM_E_INVALID_ARG, "stepper_step: NULL argument");
    int dev = -1;
    LESASM_HIP_TRY(hipGetDevice(&dev));
    if (dev != st->mesh->device) return fail(LESASM_E_STATE, "stepper_step: wrong current device");
    if (!st->n) return LESASM_OK;
    return step_body(st, d_u, d_p, (hipStream_t)stream, 0, nullptr);
}

// ---- step graph ----------------------------------------------------------------

static void step_graph_free(lesasm_step_graph *g) {
    if (!g) return;
    // a replay may still be queued: wait for the last one before the
    // executable graph goes away
    if (g->launched && g->ev_last) (void)hipEventSynchronize(g->ev_last);
    if (g->exec) (void)hipGraphExecDestroy(g->exec);
    if (g->graph) (void)hipGraphDestroy(g->graph);
    if (g->ev_last) (void)hipEventDestroy(g->ev_last);
    device_free(g->d_rec);
    delete g;
}

extern "C" int lesasm_step_graph_create(lesasm_stepper *st, double *d_u, double *d_p, int cg_iters,
                                        lesasm_step_graph **out, void *stream) {
    if (!out) return fail(LESASM_E_INVALID_ARG, "step_graph_create: out is NULL");
    *out = nullptr;
    if (!st || !d_u || !d_p) return fail(LESASM_E_INVALID_ARG, "step_graph_create: NULL argument");
    if (cg_iters < 1 || cg_iters > kMaxCapturedCg)
        return fail(LESASM_E_INVALID_ARG, "step_graph_create: cg_iters must be in 1.." + std::to_string(kMaxCapturedCg));
    if (!st->n) return fail(LESASM_E_INVALID_ARG, "step_graph_create: the mesh has no field nodes");
    hipStream_t s = (hipStream_t)stream;
    if (!s) return fail(LESASM_E_INVALID_ARG, "step_graph_create: capture needs a non-default stream");
    int dev = -1;
    LESASM_HIP_TRY(hipGetDevice(&dev));
    if (dev != st->mesh->device) return fail(LESASM_E_STATE, "step_graph_create: wrong current device");
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    LESASM_HIP_TRY(hipStreamIsCapturing(s, &cs));
    if (cs != hipStreamCaptureStatusNone) return fail(LESASM_E_STATE, "step_graph_create: stream is already capturing");
    auto *g = new lesasm_step_graph();
    struct Guard {
        lesasm_step_graph *p;
        ~Guard() { step_graph_free(p); }
    } guard{g};
    g->st = st;
    g->u = d_u;
    g->p = d_p;
    g->cg_iters = cg_iters;
    {
        void *q = nullptr;
        const int rc = device_alloc(&q, 4 * sizeof(double), "step graph");
        if (rc) return rc;
        g->d_rec = (double *)q;
    }
    LESASM_HIP_TRY(hipEventCreateWithFlags(&g->ev_last, hipEventDisableTiming));
    // the mesh's previous work must not overlap the capture's first launches
    LESASM_HIP_TRY(hipStreamSynchronize(s));
    LESASM_HIP_TRY(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
    int rc = step_body(st, d_u, d_p, s, cg_iters, g->d_rec);
    hipGraph_t graph = nullptr;
    hipError_t e = hipStreamEndCapture(s, &graph);
    if (rc) {
        if (graph) (void)hipGraphDestroy(graph);
        return rc;
    }
    if (e != hipSuccess) return fail(LESASM_E_HIP, std::string("step_graph_create: capture failed: ") + hipGetErrorString(e));
    g->graph = graph;
    LESASM_HIP_TRY(hipGraphInstantiate(&g->exec, graph, nullptr, nullptr, 0));
    guard.p = nullptr;
    *out = g;
    return LESASM_OK;
}

extern "C" int lesasm_step_graph_launch(lesasm_step_graph *g, double *d_u, double *d_p, void *stream) {
    if (!g) return fail(LESASM_E_INVALID_ARG, "step_graph_launch: graph is NULL");
    if (d_u != g->u || d_p != g->p)
        return fail(LESASM_E_STATE, "step_graph_launch: u and p must be the buffers the graph was captured with");
    int dev = -1;
    LESASM_HIP_TRY(hipGetDevice(&dev));
    if (dev != g->st->mesh->device) return fail(LESASM_E_STATE, "step_graph_launch: wrong current device");
    hipStream_t s = (hipStream_t)stream;
    LESASM_HIP_TRY(hipGraphLaunch(g->exec, s));
    LESASM_HIP_TRY(hipEventRecord(g->ev_last, s));
    g->launched = true;
    return LESASM_OK;
}

extern "C" int lesasm_step_graph_stats(lesasm_step_graph *g, int *cg_iters, double *cg_rel_residual, int *converged) {
    if (!g || !cg_iters || !cg_rel_residual || !converged)
        return fail(LESASM_E_INVALID_ARG, "step_graph_stats: NULL argument");
    if (!g->launched) return fail(LESASM_E_STATE, "step_graph_stats: the graph has not been launched");
    LESASM_HIP_TRY(hipEventSynchronize(g->ev_last));
    double rec[3] = {0.0, 0.0, 0.0};
    LESASM_HIP_TRY(hipMemcpy(rec, g->d_rec, sizeof(rec), hipMemcpyDeviceToHost));
    *cg_iters = (int)rec[0];
    *cg_rel_residual = rec[1];
    *converged = rec[2] != 0.0;
    return LESASM_OK;
}

extern "C" int lesasm_step_graph_destroy(lesasm_step_graph *g) {
    step_graph_free(g);
    return LESASM_OK;
}

extern "C" int lesasm_stepper_stats(const lesasm_stepper *st, int *cg_iters, double *cg_rel_residual) {
    if (!st || !cg_iters || !cg_rel_residual) return fail(LESASM_E_INVALID_ARG, "stepper_stats: NULL argument");
    *cg_iters = st->last_iters;
    *cg_rel_residual = st->last_res;
    return LESASM_OK;
}
