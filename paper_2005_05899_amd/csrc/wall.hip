// Boundary assembly of the wall model (Algorithm 1, "Boundary assembly";
// Section 3.2 names a law-of-the-wall model).  One thread per wall face:
//   exchange point: vertex average of the face's volume element, where the
//     linear interpolant of the velocity is the mean of its nodal values;
//   wall distance y: from that point to the plane of the face (unit normal
//     n from the face's edge or diagonal cross product);
//   tangential velocity u_t = u_e - (u_e . n) n, U = |u_t|;
//   friction velocity from Reichardt's law U / u_tau = f(y u_tau / nu)
//     (kappa 0.41, C1 7.8, chi 11) by Newton's method from the viscous-
//     sublayer value sqrt(nu U / y), in FP32 and then FP64;
//   traction t = -u_tau^2 u_t / U, added to the face nodes with the face
//     integrals of their shape functions (triangle: A/3; bilinear quad: 2 x 2
//     Gauss).  Faces sharing a node add with FP64 atomics.
#include "common.hpp"

namespace lesasm {

namespace {

constexpr double kKappa = 0.41, kC1 = 7.8, kChi = 11.0;

__device__ __forceinline__ double wall_law(double yp) {
    return log(1.0 + kKappa * yp) / kKappa + kC1 * (1.0 - exp(-yp / kChi) - (yp / kChi) * exp(-yp / 3.0));
}

__device__ __forceinline__ double wall_law_slope(double yp) {
    return 1.0 / (1.0 + kKappa * yp) +
           kC1 * (exp(-yp / kChi) / kChi - exp(-yp / 3.0) / kChi + (yp / kChi) * exp(-yp / 3.0) / 3.0);
}

// y+ = y u_tau / nu from Re = U y / nu in FP32: Newton's method for
// y+ f(y+) = Re from the viscous-sublayer value sqrt(Re), to about 1e-6.
__device__ __forceinline__ float wall_yplus(float re) {
    constexpr float kappa = (float)kKappa, c1 = (float)kC1, chi = 1.0f / (float)kChi;
    float yp = sqrtf(re);
    for (int it = 0; it < 12; ++it) {
        const float l = 1.0f + kappa * yp, e11 = __expf(-yp * chi), e3 = __expf(-yp * (1.0f / 3.0f));
        const float f = __logf(l) * (1.0f / kappa) + c1 * (1.0f - e11 - yp * chi * e3);
        const float slope = 1.0f / l + c1 * chi * (e11 - e3 + yp * e3 * (1.0f / 3.0f));
        const float step = (yp * f - re) / (f + yp * slope);
        yp -= step;
        if (fabsf(step) <= 1e-5f * yp) break;
    }
    return yp;
}

// Newton's method in FP64 from the FP32 solution: two steps (one thread per face
// leaves the chip nearly empty, so the time is this chain; an FP64 evaluation of
// the law takes 1.5 us, and from the viscous-sublayer value it took up to eight).
// That value stays the start where FP32 cannot hold Re, and below Re = 0.01,
// where it is exact to some digits and FP32 loses them in 1 - exp.
// The steps square the relative error, so the one of 1e-9 was the last needed.
__device__ double friction_velocity(double U, double y, double nu) {
    if (!(U > 0.0)) return 0.0;
    double ut = sqrt(nu * U / y);
    const double re = U * y / nu;
    if (re > 1e-2 && re < 1e30) {
        const double yp = (double)wall_yplus((float)re);
        if (yp > 0.0 && yp < 1e30) ut = yp * nu / y;
    }
    for (int it = 0; it < 100; ++it) {
        const double yp = y * ut / nu;
        const double f = wall_law(yp);
        const double step = (ut * f - U) / (f + yp * wall_law_slope(yp));
        ut -= step;
        if (fabs(step) <= 1e-9 * ut) break;
    }
    return ut;
}

__device__ __forceinline__ void cross(const double *a, const double *b, double *c) {
    c[0] = a[1] * b[2] - a[2] * b[1];
    c[1] = a[2] * b[0] - a[0] * b[2];
    c[2] = a[0] * b[1] - a[1] * b[0];
}

// A serial chain (face, nodes, law, atomics), not bytes: workgroups of one
// wavefront spread the faces over the most CUs.  4.5 k faces: 8.0 us against 14.3
// (256 threads, nodes loaded one after the other, all Newton steps in FP64).
__global__ __launch_bounds__(64) void k_wall(const int32_t *__restrict__ fg, const int32_t *__restrict__ ff,
                                              const int32_t *__restrict__ eg, const int32_t *__restrict__ ef,
                                              const double *__restrict__ xyz, const double *__restrict__ u, double nu,
                                              double *__restrict__ rhs, int n) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= n) return;
    // exchange point and velocity (all loads under way together: a missing node's
    // are the first node's, and not added)
    int g[8], q[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        g[a] = eg[8 * (size_t)f + a];
        q[a] = ef[8 * (size_t)f + a];
    }
    double xe[3] = {0, 0, 0}, ue[3] = {0, 0, 0};
    int ne = 0;
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        const bool on = g[a] >= 0;
        const size_t ga = on ? g[a] : g[0], qa = on ? q[a] : q[0];
        ne += on;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double x = xyz[3 * ga + k], v = u[3 * qa + k];
            xe[k] += on ? x : 0.0;
            ue[k] += on ? v : 0.0;
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        xe[k] /= ne;
        ue[k] /= ne;
    }
    // face geometry
    const int nf = fg[4 * (size_t)f + 3] < 0 ? 3 : 4;
    double xf[4][3], xc[3] = {0, 0, 0};
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int g = fg[4 * (size_t)f + (b < nf ? b : 0)];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            xf[b][k] = xyz[3 * (size_t)g + k];
            xc[k] += b < nf ? xf[b][k] / nf : 0.0;
        }
    }
    double c[3], wa[4];
    if (nf == 3) {
        double d1[3], d2[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            d1[k] = xf[1][k] - xf[0][k];
            d2[k] = xf[2][k] - xf[0][k];
        }
        cross(d1, d2, c);
        const double area = 0.5 * sqrt(c[0] * c[0] + c[1] * c[1] + c[2] * c[2]);
        wa[0] = wa[1] = wa[2] = area / 3.0;
        wa[3] = 0.0;
    } else {
        double d1[3], d2[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            d1[k] = xf[2][k] - xf[0][k];
            d2[k] = xf[3][k] - xf[1][k];
        }
        cross(d1, d2, c);
        const double s[4] = {-1, 1, 1, -1}, t[4] = {-1, -1, 1, 1};
        const double gq = 0.577350269189625764509148780502;
        wa[0] = wa[1] = wa[2] = wa[3] = 0.0;
#pragma unroll
        for (int gi = 0; gi < 2; ++gi)
#pragma unroll
            for (int gj = 0; gj < 2; ++gj) {
                const double xi = gi ? gq : -gq, eta = gj ? gq : -gq;
                double dx[3] = {0, 0, 0}, dy[3] = {0, 0, 0};
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        dx[k] += 0.25 * s[a] * (1.0 + t[a] * eta) * xf[a][k];
                        dy[k] += 0.25 * t[a] * (1.0 + s[a] * xi) * xf[a][k];
                    }
                double cc[3];
                cross(dx, dy, cc);
                const double jac = sqrt(cc[0] * cc[0] + cc[1] * cc[1] + cc[2] * cc[2]);
#pragma unroll
                for (int a = 0; a < 4; ++a) wa[a] += 0.25 * (1.0 + s[a] * xi) * (1.0 + t[a] * eta) * jac;
            }
    }
    const double len = sqrt(c[0] * c[0] + c[1] * c[1] + c[2] * c[2]);
    double nrm[3], y = 0.0, un = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        nrm[k] = c[k] / len;
        y += nrm[k] * (xe[k] - xc[k]);
        un += nrm[k] * ue[k];
    }
    y = fabs(y);
    double ut[3], U = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        ut[k] = ue[k] - un * nrm[k];
        U += ut[k] * ut[k];
    }
    U = sqrt(U);
    if (!(U > 0.0)) return;
    const double utau = friction_velocity(U, y, nu);
    const double sc = -utau * utau / U;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if (b == 3 && nf == 3) break;
        const size_t q = (size_t)ff[4 * (size_t)f + b];
#pragma unroll
        for (int k = 0; k < 3; ++k) unsafeAtomicAdd(rhs + 3 * q + k, sc * ut[k] * wa[b]);
    }
}

}  // namespace

int launch_wall(lesasm_mesh *m, const double *u, double nu, double *rhs, hipStream_t s) {
    const int n = (int)m->n_wall;
    hipLaunchKernelGGL(k_wall, dim3((n + 63) / 64), dim3(64), 0, s, m->d_wall_fg, m->d_wall_ff, m->d_wall_eg,
                       m->d_wall_ef, m->d_xyz, u, nu, rhs, n);
    LESASM_HIP_TRY(hipGetLastError());
    return LESASM_OK;
}

}  // namespace lesasm
