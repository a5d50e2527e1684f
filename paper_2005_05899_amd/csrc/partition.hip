// Space-filling-curve mesh partitioner and correction-coefficient load
// balancing (Section "Mesh partitioning and load balancing").
//
// Partitioner, on the device, in the paper's five steps:
//   i)   bounding box of the element locations   k_bbox_partial, k_bbox_final
//   ii)  regular 2^L grid in it;
//   iii) integer bin weights (64-bit atomics)     k_bins
//   iv)  bins in Hilbert order; v) inclusive scan of their weights along the
//        curve, targets T_i = Lambda_i W / P, and the midpoint split of every
//        element's bin                            k_scan_tile_sums, k_scan_apply, k_assign
// Bins are stored and addressed row by row (x fastest), and only the scan walks
// them in Hilbert order, so the curve is computed per bin, not per element, and
// the weights and midpoints of neighbouring elements share cache lines.
// Everything after the binning is integer arithmetic (weights, prefix sums)
// or the comparison of an exact integer with a target, so the parts do not
// depend on the launch shape or the order of the atomics.
//
// Balancing (host): per splitting point a weighted linear regression of
// (Lambda_i^k, Upsilon_i^k) cut with y = i.
#include <algorithm>
#include <cmath>
#include <vector>

#include "common.hpp"

namespace lesasm {

namespace {

constexpr int kBboxBlocks = 2048;
constexpr int kScanTile = 4096;  // bins per scan block: 512 threads x 8
constexpr int kMaxLevel = 8;

// Row-by-row indices of the 8 bins at positions 8 o .. 8 o + 7 on the Hilbert
// curve of a 2^level grid (J. Skilling, "Programming the Hilbert curve", AIP Conf.
// Proc. 707, 2004, from the index to the axes): the index is read as transposed
// bits, most significant level first, x before y before z, Gray-decoded, and the
// axes are transformed back level by level from the bottom.  The 8 positions
// differ in the lowest level only, whose bits no condition reads: they are
// carried as 8-bit vectors below the other levels' bits, one bit per position.
struct HilbertOctet {
    uint32_t a[3];
    __device__ __forceinline__ HilbertOctet(uint32_t o, int level) {
        uint32_t u[3] = {0, 0, 0};
        for (int b = level - 2; b >= 0; --b)
#pragma unroll
            for (int i = 0; i < 3; ++i) u[i] |= ((o >> (3 * b + 2 - i)) & 1u) << b;
        a[0] = u[0] << 8 | 0xF0u;
        a[1] = u[1] << 8 | 0xCCu;
        a[2] = u[2] << 8 | 0xAAu;
        const uint32_t t0 = (u[2] >> 1) << 8 | (u[2] & 1u ? 0xFFu : 0u);  // a[2] one level down
        a[2] ^= a[1];
        a[1] ^= a[0];
        a[0] ^= t0;
        for (uint32_t q = 1u << 8; q < 1u << (7 + level); q <<= 1) {
            const uint32_t low = q - 1;
#pragma unroll
            for (int i = 2; i >= 0; --i) {
                if (a[i] & q) {
                    a[0] ^= low;
                } else {
                    const uint32_t t = (a[0] ^ a[i]) & low;
                    a[0] ^= t;
                    a[i] ^= t;
                }
            }
        }
    }
    __device__ __forceinline__ uint32_t bin(int v, int level) const {
        auto axis = [&](int i) { return (a[i] >> 8) << 1 | ((a[i] >> v) & 1u); };
        return axis(2) << (2 * level) | axis(1) << level | axis(0);
    }
};

// Bin of coordinate c on an axis with bounds lo, hi: floor((c - lo) / (hi -
// lo) * nb), clamped into [0, nb - 1] (0 on a flat axis or for a NaN).
__device__ __forceinline__ uint32_t bin_of(double c, double lo, double hi, int nb) {
    const double ext = hi - lo;
    if (!(ext > 0.0)) return 0;
    const double t = floor((c - lo) / ext * (double)nb);
    if (!(t >= 0.0)) return 0;
    return t >= (double)(nb - 1) ? (uint32_t)(nb - 1) : (uint32_t)t;
}

// One thread per element.  All node ids are loaded, then all coordinates, so an
// element waits for memory three times and not twice per node.  Bound by its bytes:
// 4.0 M hybrid elements 73 us (77 node by node), 20 M 427 us (460; 458 on a grid
// of 8192 workgroups), 3.7 and 3.2 TB/s of the bytes it cannot do without.
// Contiguous eighths of the elements per XCD: 129 us at 4.0 M; runs of 4 to 256
// workgroups per XCD within 1 %; three threads per element 138 us.
__global__ __launch_bounds__(256) void k_centroids(int64_t n, const int64_t *__restrict__ off,
                                                   const int32_t *__restrict__ conn, int64_t conn_len, int64_t n_nodes,
                                                   const double *__restrict__ xyz, double *__restrict__ cen,
                                                   int32_t *__restrict__ wts, int32_t *__restrict__ flag) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = off[e], k64 = off[e + 1] - b;
        const int k = (k64 >= 4 && k64 <= 8) ? (int)k64 : 0;
        const int w = k == 4 ? 4 : k == 5 ? 8 : k == 6 ? 6 : k == 8 ? 8 : 0;
        if (!w || b < 0 || b + k > conn_len) {
            atomicOr(flag, 1);
            continue;
        }
        int32_t g[8];
        bool ok = true;
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            g[a] = a < k ? conn[b + a] : 0;
            ok = ok && (a >= k || (g[a] >= 0 && g[a] < n_nodes));
        }
        if (!ok) {
            atomicOr(flag, 2);
            continue;
        }
        double s[3] = {0.0, 0.0, 0.0};
        auto add4 = [&](int a0) {
            double x[4][3];
#pragma unroll
            for (int a = 0; a < 4; ++a)
                if (a0 + a < k)
#pragma unroll
                    for (int d = 0; d < 3; ++d) x[a][d] = xyz[3 * (size_t)g[a0 + a] + d];
#pragma unroll
            for (int a = 0; a < 4; ++a)
                if (a0 + a < k)
#pragma unroll
                    for (int d = 0; d < 3; ++d) s[d] += x[a][d];
        };
        add4(0);
        if (k > 4) add4(4);
#pragma unroll
        for (int d = 0; d < 3; ++d) cen[3 * e + d] = s[d] / (double)k;
        if (wts) wts[e] = w;
    }
}

// Per block: min and max of each coordinate over a grid-stride slice; and the
// bin weights are zeroed on the way.
__global__ __launch_bounds__(256) void k_bbox_partial(int64_t n, const double *__restrict__ c,
                                                      double *__restrict__ partial,
                                                      unsigned long long *__restrict__ binw, int64_t nbins) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nbins; i += (int64_t)gridDim.x * blockDim.x)
        binw[i] = 0ull;
    __shared__ double sh[6][256];
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double v = c[3 * e + d];
            lo[d] = fmin(lo[d], v);
            hi[d] = fmax(hi[d], v);
        }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        sh[d][threadIdx.x] = lo[d];
        sh[3 + d][threadIdx.x] = hi[d];
    }
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                sh[d][threadIdx.x] = fmin(sh[d][threadIdx.x], sh[d][threadIdx.x + w]);
                sh[3 + d][threadIdx.x] = fmax(sh[3 + d][threadIdx.x], sh[3 + d][threadIdx.x + w]);
            }
        __syncthreads();
    }
    if (threadIdx.x < 6) partial[6 * blockIdx.x + threadIdx.x] = sh[threadIdx.x][0];
}

__global__ __launch_bounds__(256) void k_bbox_final(const double *__restrict__ partial, int nb,
                                                    double *__restrict__ box) {
    __shared__ double sh[6][256];
    double v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int b = threadIdx.x; b < nb; b += blockDim.x)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            v[d] = fmin(v[d], partial[6 * b + d]);
            v[3 + d] = fmax(v[3 + d], partial[6 * b + 3 + d]);
        }
#pragma unroll
    for (int d = 0; d < 6; ++d) sh[d][threadIdx.x] = v[d];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                sh[d][threadIdx.x] = fmin(sh[d][threadIdx.x], sh[d][threadIdx.x + w]);
                sh[3 + d][threadIdx.x] = fmax(sh[3 + d][threadIdx.x], sh[3 + d][threadIdx.x + w]);
            }
        __syncthreads();
    }
    if (threadIdx.x < 6) box[threadIdx.x] = sh[threadIdx.x][0];
}

// Value of v d lanes below, within rows of 16 lanes (0 from outside the row).
template <int D> __device__ __forceinline__ uint32_t row_up(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x110 + D, 0xf, 0xf, true);  // row_shr:D
}
template <int D>
__device__ __forceinline__ void merge_run(unsigned long long &v, uint32_t run, int lane) {
    const unsigned long long up = ((unsigned long long)row_up<D>((uint32_t)(v >> 32)) << 32) | row_up<D>((uint32_t)v);
    const uint32_t run_up = row_up<D>(run);
    if ((lane & 15) >= D && run_up == run) v += up;
}

// Bin of each element; bin weights summed with 64-bit atomics.  Neighbouring
// elements mostly share a bin or lie in adjacent ones, so rows of 16 lanes first
// merge runs of equal bins in lane order (segmented scan over run ids) and only
// the last lane of a run adds the run's weight; adjacent bins are adjacent in
// memory.  Integer sums: the weights are exact whatever the grouping.
// 4.0 M elements 43 us, against 86 with the Hilbert position computed per element,
// weights scattered along the curve and merging by cross-lane reads of whole
// wavefronts; the whole split 101 against 157 us, of 20 M elements 413 against 585.
__global__ __launch_bounds__(256) void k_bins(int64_t n, const double *__restrict__ c, const int32_t *__restrict__ wts,
                                              const double *__restrict__ box, int level, uint32_t *__restrict__ key,
                                              unsigned long long *__restrict__ binw) {
    const int nb = 1 << level;
    const double lo0 = box[0], lo1 = box[1], lo2 = box[2], hi0 = box[3], hi1 = box[4], hi2 = box[5];
    const int lane = threadIdx.x & 63;
    const int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x;
    uint32_t bin = 0xffffffffu;
    unsigned long long v = 0ull;
    if (e < n) {  // (every lane goes on: the merging works on whole rows)
        const uint32_t bx = bin_of(c[3 * e + 0], lo0, hi0, nb);
        const uint32_t by = bin_of(c[3 * e + 1], lo1, hi1, nb);
        const uint32_t bz = bin_of(c[3 * e + 2], lo2, hi2, nb);
        bin = (bz << (2 * level)) | (by << level) | bx;
        key[e] = bin;
        v = (unsigned long long)(long long)(wts ? wts[e] : 1);
    }
    const uint32_t prev = __shfl_up(bin, 1);
    const bool head = (lane & 15) == 0 || prev != bin;
    const unsigned long long heads = __ballot(head);
    const uint32_t run = (uint32_t)__popcll(heads & (~0ull >> (63 - lane)));  // runs started at or before this lane
    merge_run<1>(v, run, lane);
    merge_run<2>(v, run, lane);
    merge_run<4>(v, run, lane);
    merge_run<8>(v, run, lane);
    const bool tail = lane == 63 || ((heads >> (lane + 1)) & 1);
    if (tail && bin != 0xffffffffu) atomicAdd(binw + bin, v);
}

// Inclusive sums over a workgroup of 512 threads; total receives the sum of all.
__device__ __forceinline__ unsigned long long block_inclusive_512(unsigned long long v, unsigned long long *sh,
                                                                  unsigned long long &total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long up = __shfl_up(v, o);
        if (lane >= o) v += up;
    }
    __syncthreads();  // sh may still be read from a previous scan
    if (lane == 63) sh[wave] = v;
    __syncthreads();
    unsigned long long before = 0ull, all = 0ull;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        const unsigned long long x = sh[w];
        before += w < wave ? x : 0ull;
        all += x;
    }
    total = all;
    return v + before;
}

// Sums of tiles of kScanTile bins along the curve.
__global__ __launch_bounds__(512) void k_scan_tile_sums(const unsigned long long *__restrict__ binw, int64_t n, int level,
                                                        unsigned long long *__restrict__ sums) {
    __shared__ unsigned long long sh[8];
    const int64_t first = (int64_t)blockIdx.x * kScanTile + 8 * threadIdx.x;
    unsigned long long v = 0, total;
    if (first < n) {  // (the bins are a power of 8)
        const HilbertOctet o((uint32_t)(first >> 3), level);
#pragma unroll
        for (int j = 0; j < 8; ++j) v += binw[o.bin(j, level)];
    }
    (void)block_inclusive_512(v, sh, total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// Replaces each bin's weight w by twice its midpoint on the curve, 2 S + w (S
// the weight before it: the tiles before its own, added up here, and the scan
// within the tile).  The last tile leaves the total weight in *all.
__global__ __launch_bounds__(512) void k_scan_apply(unsigned long long *__restrict__ binw, int64_t n, int level,
                                                    const unsigned long long *__restrict__ sums,
                                                    unsigned long long *__restrict__ all) {
    __shared__ unsigned long long sh[8];
    const int64_t first = (int64_t)blockIdx.x * kScanTile + 8 * threadIdx.x;
    const HilbertOctet o((uint32_t)((first < n ? first : 0) >> 3), level);
    unsigned long long v[8], own = 0ull, before = 0ull, total;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        v[j] = first < n ? binw[o.bin(j, level)] : 0ull;
        own += v[j];
    }
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += 512) before += sums[t];
    (void)block_inclusive_512(before, sh, before);
    unsigned long long run = before + block_inclusive_512(own, sh, total) - own;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (first < n) binw[o.bin(j, level)] = 2 * run + v[j];
        run += v[j];
    }
    if (threadIdx.x == 0 && blockIdx.x == gridDim.x - 1) *all = before + total;
}

// Running sums of the correction coefficients, Lambda_1 .. Lambda_(P-1), passed
// by value up to kArgLambda parts.
constexpr int kArgLambda = 256;
constexpr int kLambdaPiece = 4096;  // sums of more parts are copied in pieces of this many
struct LambdaArg {
    double v[kArgLambda];
};

// part = number of targets T_i = Lambda_i W / P at or below the midpoint of the
// element's bin (both doubled).  Running sums from `lam` (device) if set, else
// from `la` if use_arg, else Lambda_i = i.
__global__ __launch_bounds__(256) void k_assign(int64_t n, const uint32_t *__restrict__ key,
                                                const unsigned long long *__restrict__ mid2,
                                                const unsigned long long *__restrict__ all,
                                                const double *__restrict__ lam, LambdaArg la, int use_arg, int P,
                                                int32_t *__restrict__ part) {
    __shared__ double t2[kArgLambda];
    const double W = (double)*all;
    auto target = [&](int i) {
        const double acc = lam ? lam[i] : use_arg ? la.v[i] : (double)(i + 1);
        return 2.0 * (acc * W / (double)P);
    };
    const bool staged = P <= kArgLambda;
    if (staged) {
        if ((int)threadIdx.x < P - 1) t2[threadIdx.x] = target(threadIdx.x);
        __syncthreads();
    }
    const int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (e >= n) return;
    const double m = (double)mid2[key[e]];
    int lo = 0, hi = P - 1;  // first index in [0, P-1) with t2 > m, else P - 1
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if ((staged ? t2[mid] : target(mid)) <= m)
            lo = mid + 1;
        else
            hi = mid;
    }
    part[e] = lo;
}

struct Workspace {
    double *partial, *box, *lam;
    unsigned long long *all, *binw, *tiles;
    uint32_t *key;
    size_t bytes;
};

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

Workspace layout(void *base, int64_t n, int P, int level) {
    const int64_t nbins = (int64_t)1 << (3 * level);
    const int64_t ntiles = (nbins + kScanTile - 1) / kScanTile;
    char *p = (char *)base;
    size_t o = 0;
    Workspace w{};
    auto take = [&](size_t b) {
        char *q = p ? p + o : nullptr;
        o += align256(b);
        return q;
    };
    w.partial = (double *)take(sizeof(double) * 6 * kBboxBlocks);
    w.box = (double *)take(sizeof(double) * 6);
    w.all = (unsigned long long *)take(sizeof(unsigned long long));
    w.lam = (double *)take(sizeof(double) * (size_t)P);
    w.binw = (unsigned long long *)take(sizeof(unsigned long long) * (size_t)nbins);
    w.tiles = (unsigned long long *)take(sizeof(unsigned long long) * (size_t)ntiles);
    w.key = (uint32_t *)take(sizeof(uint32_t) * (size_t)(n > 0 ? n : 1));
    w.bytes = o;
    return w;
}

}  // namespace

}  // namespace lesasm

using namespace lesasm;

extern "C" int lesasm_element_centroids(int64_t n_elems, const int64_t *d_off, const int32_t *d_conn, int64_t conn_len,
                                        int64_t n_nodes, const double *d_coords, double *d_cen, int32_t *d_wts,
                                        int32_t *d_status, void *stream) {
    if (n_elems < 0 || n_nodes < 0 || conn_len < 0) return fail(LESASM_E_INVALID_ARG, "element_centroids: negative size");
    if (n_elems == 0) return LESASM_OK;
    if (!d_off || !d_conn || !d_coords || !d_cen || !d_status)
        return fail(LESASM_E_INVALID_ARG, "element_centroids: NULL argument");
    hipLaunchKernelGGL(k_centroids, dim3((unsigned)std::min<int64_t>((n_elems - 1) / 256 + 1, 1 << 20)), dim3(256), 0, (hipStream_t)stream, n_elems,
                       d_off, d_conn, conn_len, n_nodes, d_coords, d_cen, d_wts, d_status);
    LESASM_HIP_TRY(hipGetLastError());
    return LESASM_OK;
}

extern "C" int lesasm_sfc_workspace_bytes(int64_t n_elems, int n_parts, int level, size_t *bytes) {
    if (!bytes || n_elems < 0 || n_parts < 1 || level < 1 || level > kMaxLevel)
        return fail(LESASM_E_INVALID_ARG, "sfc_workspace_bytes: bad argument");
    *bytes = layout(nullptr, n_elems, n_parts, level).bytes;
    return LESASM_OK;
}

extern "C" int lesasm_sfc_partition(int64_t n, const double *d_cen, const int32_t *d_wts, int P, const double *h_lambda,
                                    int level, void *d_work, size_t work_bytes, int32_t *d_part, void *stream) {
    if (n < 0 || P < 1 || level < 1 || level > kMaxLevel)
        return fail(LESASM_E_INVALID_ARG, "sfc_partition: bad size, part count or level");
    if (n > (int64_t)INT32_MAX) return fail(LESASM_E_INVALID_ARG, "sfc_partition: more than 2^31-1 elements");
    if (n == 0) return LESASM_OK;
    if (!d_cen || !d_part || !d_work) return fail(LESASM_E_INVALID_ARG, "sfc_partition: NULL argument");
    if (((uintptr_t)d_work & 255) != 0) return fail(LESASM_E_INVALID_ARG, "sfc_partition: workspace not 256-byte aligned");
    const Workspace w = layout(d_work, n, P, level);
    if (work_bytes < w.bytes) return fail(LESASM_E_INVALID_ARG, "sfc_partition: workspace too small");
    if (h_lambda)
        for (int i = 0; i < P; ++i)
            if (!std::isfinite(h_lambda[i]) || h_lambda[i] < 0.0)
                return fail(LESASM_E_INVALID_ARG, "sfc_partition: correction coefficient negative or not finite");
    hipStream_t s = (hipStream_t)stream;
    const int64_t nbins = (int64_t)1 << (3 * level);
    const int ntiles = (int)((nbins + kScanTile - 1) / kScanTile);
    // the running sums of the coefficients: up to kArgLambda travel in the kernel
    // arguments; more are copied and waited for, so h_lambda is never read after
    // the call returns
    LambdaArg la{};
    const bool by_arg = h_lambda && P <= kArgLambda;
    if (h_lambda) {
        double piece[kLambdaPiece], acc = 0.0;  // (no allocation that could throw)
        double *to = by_arg ? la.v : piece;
        for (int i = 0, k = 0; i < P; ++i) {
            to[k++] = acc = acc + h_lambda[i];
            if (by_arg || (k < kLambdaPiece && i + 1 < P)) continue;
            LESASM_HIP_TRY(hipMemcpyAsync(w.lam + (i + 1 - k), piece, sizeof(double) * k, hipMemcpyHostToDevice, s));
            LESASM_HIP_TRY(hipStreamSynchronize(s));
            k = 0;
        }
    }
    const int g = (int)((n - 1) / 256 + 1);
    const int gb = std::min(kBboxBlocks, std::max(g, grid_for((size_t)nbins, 1024)));
    hipLaunchKernelGGL(k_bbox_partial, dim3(gb), dim3(256), 0, s, n, d_cen, w.partial, w.binw, nbins);
    hipLaunchKernelGGL(k_bbox_final, dim3(1), dim3(256), 0, s, w.partial, gb, w.box);
    hipLaunchKernelGGL(k_bins, dim3(g), dim3(256), 0, s, n, d_cen, d_wts, w.box, level, w.key, w.binw);
    hipLaunchKernelGGL(k_scan_tile_sums, dim3(ntiles), dim3(512), 0, s, w.binw, nbins, level, w.tiles);
    hipLaunchKernelGGL(k_scan_apply, dim3(ntiles), dim3(512), 0, s, w.binw, nbins, level, w.tiles, w.all);
    hipLaunchKernelGGL(k_assign, dim3(g), dim3(256), 0, s, n, w.key, w.binw, w.all,
                       (h_lambda && !by_arg) ? w.lam : nullptr, la, by_arg ? 1 : 0, P, d_part);
    LESASM_HIP_TRY(hipGetLastError());
    return LESASM_OK;
}

extern "C" int lesasm_balance_update(int P, int K, const double *lam_hist, const double *t_hist, double growth,
                                     double *lam_out) {
    if (!lam_hist || !t_hist || !lam_out || P < 1 || K < 1 || !(growth > 0.0) || !std::isfinite(growth))
        return fail(LESASM_E_INVALID_ARG, "balance_update: bad argument");
    std::vector<double> X((size_t)K * P), Y((size_t)K * P), wk(K);
    for (int k = 0; k < K; ++k) {
        double lam_sum = 0.0, t_sum = 0.0;
        for (int i = 0; i < P; ++i) {
            const double l = lam_hist[(size_t)k * P + i], t = t_hist[(size_t)k * P + i];
            if (!std::isfinite(l) || l < 0.0 || !std::isfinite(t) || t < 0.0)
                return fail(LESASM_E_INVALID_ARG, "balance_update: coefficient or time negative or not finite");
            t_sum += t;
        }
        const double mean = t_sum / P;
        if (!(mean > 0.0)) return fail(LESASM_E_INVALID_ARG, "balance_update: zero mean time");
        double run = 0.0;
        for (int i = 0; i < P; ++i) {
            lam_sum += lam_hist[(size_t)k * P + i];
            run += t_hist[(size_t)k * P + i];
            X[(size_t)k * P + i] = lam_sum;  // Lambda_{i+1}^k
            Y[(size_t)k * P + i] = run / mean;  // Upsilon_{i+1}^k
        }
        wk[k] = std::pow(growth, (double)k);
    }
    std::vector<double> cut(P + 1);
    cut[0] = 0.0;
    cut[P] = (double)P;
    for (int i = 1; i < P; ++i) {
        double next = 0.0;
        bool have = false;
        if (K >= 2) {
            double sw = 0.0, sx = 0.0, sy = 0.0, xmin = INFINITY, xmax = -INFINITY;
            for (int k = 0; k < K; ++k) {
                const double xv = X[(size_t)k * P + i - 1], yv = Y[(size_t)k * P + i - 1];
                sw += wk[k];
                sx += wk[k] * xv;
                sy += wk[k] * yv;
                xmin = std::fmin(xmin, xv);
                xmax = std::fmax(xmax, xv);
            }
            const double mx = sx / sw, my = sy / sw;
            double sxx = 0.0, sxy = 0.0;
            for (int k = 0; k < K; ++k) {
                const double dx = X[(size_t)k * P + i - 1] - mx, dy = Y[(size_t)k * P + i - 1] - my;
                sxx += wk[k] * dx * dx;
                sxy += wk[k] * dx * dy;
            }
            if (xmax - xmin > 1e-12 * P && sxx > 0.0) {
                const double beta = sxy / sxx, alpha = my - beta * mx;
                if (beta > 0.0) {
                    next = ((double)i - alpha) / beta;
                    have = true;
                }
            }
        }
        if (!have) {
            const double xl = X[(size_t)(K - 1) * P + i - 1], yl = Y[(size_t)(K - 1) * P + i - 1];
            next = yl > 0.0 ? (double)i * xl / yl : xl;
        }
        cut[i] = next;
    }
    for (int i = 1; i < P; ++i) cut[i] = std::fmin(std::fmax(cut[i], cut[i - 1]), (double)P);
    for (int i = 0; i < P; ++i) lam_out[i] = cut[i + 1] - cut[i];
    return LESASM_OK;
}
