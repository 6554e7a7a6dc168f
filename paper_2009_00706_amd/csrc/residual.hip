// Residual and matrix-free Jacobian action of the VMS weak form (gfx950): one
// quadrature point per lane.
//
// Both are the same sum over points: fields interpolated at the point, the 16
// coefficients r^i[k] of the integrand (eq. (vms) with eq. (uprime) and eq.
// (pprime)) or their derivative along the direction x with tau_M, tau_C and
// taubar frozen, and the product with the basis. No matrix is formed, so there
// is nothing for the matrix cores: the work per point is about 300 operations
// (480 along a direction), and what counts is that all lanes of a wave do it
// for different points and that the interpolation uses the tensor structure.
//
//   OUT elements (k_vec_out): a wave holds 8 elements x 8 points, and its lanes
//     are the element's corners before the interpolation and its Gauss points
//     after it. The 2-point interpolation of one axis is a butterfly between
//     the two lanes that differ in that axis' bit (lane bits 0, 1 and 3: quad
//     permutes and a row rotation by 8, no LDS), and the product with the basis
//     is the same butterflies in reverse.
//   INTERCEPTED items (k_vec_sub): a wave holds one item, lane = point, in
//     rounds of 64. The element's trilinear fields are kept as coefficients of
//     1, x, y, xy, z, xz, yz, xyz in LDS (every lane reads the same address),
//     evaluated by nested products; the tests are summed in the same basis and
//     reduced over the lanes once per item.
//
// Eight lanes per point with the basis tabulated in LDS (the element-matrix
// kernel's first phases) took, on the 194k-octant sphere (1.1M and 4.0M points,
// FP64), 0.20 and 0.72 ms for the residual and 0.28 and 0.94 ms for the action;
// these kernels take 0.033 and 0.102, 0.047 and 0.160 ms. The FP32 form of the
// mixed contexts (k_vec32, residual and action together 1.12 -> 0.43 ms) has the
// same waves of points but keeps the order of every rounding.
#include "item_dev.h"
#include "vms_point.h"

namespace vmsk {

namespace {

constexpr double KA = 0.5 + 0.5 * VMS_XI, KB = 0.5 - 0.5 * VMS_XI;

// value of the lane whose bit AX (0: x, 1: y, 2: z) of the corner index differs
template <int AX>
__device__ inline double other(double v) {
    constexpr int ctrl = AX == 0 ? 0xB1 : (AX == 1 ? 0x4E : 0x128);
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

__device__ inline double weight_of(uint32_t code) {
    return code == 3u ? 1.0 : (code == 2u ? 0.5 : (code == 1u ? 0.25 : 0.0));
}

// fields of a point: u_theta, its gradient, p, grad p, the rate (u - u_prev)/dt,
// and along a direction x_u, its gradient, x_p, grad x_p
struct PointIn {
    double u[3], gu[3][3], p, gp[3], at[3];
    double du[3], dgu[3][3], dp, dgp[3];
};

struct PointPar {
    double rho, irho, mu, th, idt, gG, tau0, h2_12;
};

// residual coefficients r^i[k] (i test component, k = 0 against N, 1 + m
// against dN/dx_m), or their derivative along the direction, without the weight
template <bool JV>
__device__ inline void point_coeffs(const PointIn &I, const PointPar &P, double r[4][4]) {
    double up[3], acc[3];
    for (int c = 0; c < 3; ++c) {
        acc[c] = I.at[c] + I.u[0] * I.gu[c][0] + I.u[1] * I.gu[c][1] + I.u[2] * I.gu[c][2];
        up[c] = P.rho * acc[c] + I.gp[c];
    }
    const double s0 = P.tau0 + P.gG * (I.u[0] * I.u[0] + I.u[1] * I.u[1] + I.u[2] * I.u[2]);
    const double tauM = rsq<double>(s0);
    const double tauC = P.h2_12 * s0 * tauM;
    for (int c = 0; c < 3; ++c) up[c] *= -tauM;
    const double upg = P.gG * (up[0] * up[0] + up[1] * up[1] + up[2] * up[2]);
    const double tb = upg > 0.0 ? rsq<double>(upg) : 0.0;
    if constexpr (!JV) {
        const double div = I.gu[0][0] + I.gu[1][1] + I.gu[2][2];
        const double pt = I.p - P.rho * tauC * div;
        for (int c = 0; c < 3; ++c) {
            const double sv = up[0] * I.gu[c][0] + up[1] * I.gu[c][1] + up[2] * I.gu[c][2];
            r[c][0] = P.rho * acc[c] + sv;
            const double tu = tb * sv - up[c] * P.irho;
            for (int k = 0; k < 3; ++k)
                r[c][1 + k] = P.mu * (I.gu[c][k] + I.gu[k][c]) - I.u[k] * up[c] + up[k] * tu;
            r[c][1 + c] -= pt;
        }
        r[3][0] = div;
        for (int k = 0; k < 3; ++k) r[3][1 + k] = -up[k] * P.irho;
    } else {
        double dut[3], dup[3], dacc[3], dg[3][3];
        for (int c = 0; c < 3; ++c) {
            dut[c] = P.th * I.du[c];
            for (int m = 0; m < 3; ++m) dg[c][m] = P.th * I.dgu[c][m];
        }
        for (int c = 0; c < 3; ++c) {
            dacc[c] = I.du[c] * P.idt + dut[0] * I.gu[c][0] + dut[1] * I.gu[c][1] + dut[2] * I.gu[c][2] +
                      I.u[0] * dg[c][0] + I.u[1] * dg[c][1] + I.u[2] * dg[c][2];
            dup[c] = -tauM * (P.rho * dacc[c] + I.dgp[c]);
        }
        const double ddiv = dg[0][0] + dg[1][1] + dg[2][2];
        const double dpt = I.dp - P.rho * tauC * ddiv;
        for (int c = 0; c < 3; ++c) {
            const double sv = up[0] * I.gu[c][0] + up[1] * I.gu[c][1] + up[2] * I.gu[c][2];
            const double dsv = dup[0] * I.gu[c][0] + dup[1] * I.gu[c][1] + dup[2] * I.gu[c][2] +
                          up[0] * dg[c][0] + up[1] * dg[c][1] + up[2] * dg[c][2];
            r[c][0] = P.rho * dacc[c] + dsv;
            const double tu = tb * sv - up[c] * P.irho, dtu = tb * dsv - dup[c] * P.irho;
            for (int k = 0; k < 3; ++k)
                r[c][1 + k] = P.mu * (dg[c][k] + dg[k][c]) - dut[k] * up[c] - I.u[k] * dup[c] + dup[k] * tu +
                              up[k] * dtu;
            r[c][1 + c] -= dpt;
        }
        r[3][0] = ddiv;
        for (int k = 0; k < 3; ++k) r[3][1 + k] = -dup[k] * P.irho;
    }
}

__device__ inline PointPar point_par(const AsmArgs &a, double h, double two_over_h) {
    // G = (2/h)^2 I: tau_M^-2 = c_t/dt^2 + gG |u|^2 + c_i nu^2 G:G, tau_C = (h^2/12)/tau_M
    const double gG = two_over_h * two_over_h;
    return {a.rho, a.irho, a.mu, a.theta, a.idt, gG, (a.tau_a + a.tau_b * gG * gG),
            (h * h * (1.0 / 12.0))};
}

// ---- OUT elements ----------------------------------------------------------

// interpolation along one axis: the lane's point from its own corner and the other one
template <int AX>
__device__ inline double interp(double v) {
    return KA * v + KB * other<AX>(v);
}
// value and gradient at the lane's Gauss point of the field with corner value v
// (sg: +-1/h by the lane's bit of each axis)
__device__ inline void field_at(double v, const double sg[3], double &val, double g[3]) {
    const double ox = other<0>(v);
    const double ix = KA * v + KB * ox, dx = sg[0] * (v - ox);
    const double oy = other<1>(ix);
    const double iy = KA * ix + KB * oy, dy = sg[1] * (ix - oy);
    const double oz = other<2>(iy);
    val = KA * iy + KB * oz;
    g[2] = sg[2] * (iy - oz);
    g[1] = interp<2>(dy);
    g[0] = interp<2>(interp<1>(dx));
}
__device__ inline double value_at(double v) {
    return interp<2>(interp<1>(interp<0>(v)));
}
// the transpose: corner value of sum over the points of r0 N + r . grad N
__device__ inline double test_sum(const double r[4], const double sg[3]) {
    double t = interp<2>(r[0]) + sg[2] * (r[3] + other<2>(r[3]));
    const double ty = interp<2>(r[2]);
    const double tx = interp<1>(interp<2>(r[1]));
    t = interp<1>(t) + sg[1] * (ty + other<1>(ty));
    return interp<0>(t) + sg[0] * (tx + other<0>(tx));
}

template <bool JV>
__global__ __launch_bounds__(256) void k_vec_out(AsmArgs a, const double *x) {
    const int lane = threadIdx.x & 63;
    const int s = (lane & 3) | ((lane >> 1) & 4);               // corner / point: x bit 0, y bit 1, z bit 3
    const int el = ((lane >> 2) & 1) | ((lane >> 4) << 1);      // element of the wave
    const int64_t item = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 8 + el;
    const bool valid = item < a.n_items;
    const int e = a.items[valid ? item : a.n_items - 1];
    const int m = a.masters[8 * (int64_t)e + s];
    const bool hang = a.has_hang[e] != 0;
    const int lev = a.level[e];
    const double h = ldexp(a.root_len, -lev), two_over_h = ldexp(a.two_over_root, lev);
    const double th = a.theta, idt = a.idt;
    double f[JV ? 11 : 7];  // u_theta, p, rate, x_u, x_p at the lane's master slot, then at its corner
    for (int c = 0; c < (JV ? 11 : 7); ++c) f[c] = 0.0;
    if (m >= 0) {
        for (int c = 0; c < 3; ++c) {
            const double u = a.f[c][m], u0 = a.f[4 + c][m];
            f[c] = th * u + (1.0 - th) * u0;
            f[4 + c] = (u - u0) * idt;
        }
        f[3] = a.f[3][m];
        if constexpr (JV)
            for (int c = 0; c < 4; ++c) f[7 + c] = x[4 * (int64_t)m + c];
    }
    // constraint codes of the lane's corner (2 bits per slot)
    uint32_t code = 0;
    const int l0 = lane & ~0xb;
    const bool any_hang = __any(hang);
    if (any_hang) {
        code = a.ccode[4 * (int64_t)e + (s >> 1)] >> (16 * (s & 1));
        double g[JV ? 11 : 7];
        for (int c = 0; c < (JV ? 11 : 7); ++c) g[c] = 0.0;
#pragma unroll 1
        for (int t = 0; t < 8; ++t) {
            const double w = weight_of((code >> (2 * t)) & 3u);
            const int src = l0 | (t & 3) | ((t & 4) << 1);
            for (int c = 0; c < (JV ? 11 : 7); ++c) g[c] += w * __shfl(f[c], src, 64);
        }
        for (int c = 0; c < (JV ? 11 : 7); ++c) f[c] = g[c];
    }
    const double ih = (0.5 * two_over_h);
    const double sg[3] = {(s & 1) ? ih : -ih, (s & 2) ? ih : -ih, (s & 4) ? ih : -ih};
    PointIn I;
    for (int c = 0; c < 3; ++c) {
        field_at(f[c], sg, I.u[c], I.gu[c]);
        I.at[c] = value_at(f[4 + c]);
    }
    field_at(f[3], sg, I.p, I.gp);
    if constexpr (JV) {
        for (int c = 0; c < 3; ++c) field_at(f[7 + c], sg, I.du[c], I.dgu[c]);
        field_at(f[10], sg, I.dp, I.dgp);
    }
    const PointPar P = point_par(a, h, two_over_h);
    double r[4][4];
    point_coeffs<JV>(I, P, r);
    const double W = 0.125 * h * h * h;
    double y[4];
    for (int i = 0; i < 4; ++i) y[i] = W * (double)test_sum(r[i], sg);
    if (any_hang) {
        // C^T: slot s takes every corner's value times C[corner][s]
        double z[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
        for (int t = 0; t < 8; ++t) {
            const int src = l0 | (t & 3) | ((t & 4) << 1);
            const double w = weight_of(((uint32_t)__shfl((int)code, src, 64) >> (2 * s)) & 3u);
            for (int i = 0; i < 4; ++i) z[i] += w * __shfl(y[i], src, 64);
        }
        for (int i = 0; i < 4; ++i) y[i] = z[i];
    }
    typedef double v2 __attribute__((ext_vector_type(2)));
    if (valid) {
        v2 *dst = (v2 *)(a.rrec + (a.slot0 + item) * 32 + 4 * s);
        dst[0] = v2{y[0], y[1]};
        dst[1] = v2{y[2], y[3]};
    }
}

// ---- INTERCEPTED items -----------------------------------------------------

// value and gradient of sum_m c[m] phi_m at (x, y, z); phi: 1, x, y, xy, z, xz, yz, xyz
__device__ inline void poly_at(const double *c, const double x[3], double &val, double g[3]) {
    const double e0 = c[0] + x[2] * c[4], e1 = c[1] + x[2] * c[5], e2 = c[2] + x[2] * c[6], e3 = c[3] + x[2] * c[7];
    g[0] = e1 + x[1] * e3;
    g[1] = e2 + x[0] * e3;
    g[2] = c[4] + x[0] * c[5] + x[1] * (c[6] + x[0] * c[7]);
    val = e0 + x[0] * g[0] + x[1] * e2;
}
__device__ inline double poly_value(const double *c, const double x[3]) {
    const double e0 = c[0] + x[2] * c[4], e1 = c[1] + x[2] * c[5], e2 = c[2] + x[2] * c[6], e3 = c[3] + x[2] * c[7];
    return e0 + x[0] * e1 + x[1] * (e2 + x[0] * e3);
}

// The scheduler may not move work across FENCE: hoisting the LDS reads of all
// fields to the front took 352 VGPRs (FP64 action, one wave per SIMD, 0.27 ms on
// the 4.0M points) instead of 202.
#define FENCE __builtin_amdgcn_sched_barrier(0)

template <bool JV>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_vec_sub(AsmArgs a, const double *x) {
    constexpr int NF = JV ? 11 : 7;
    __shared__ double sN[NF][8];
    __shared__ __attribute__((aligned(16))) double sP[NF][8];
    const int lane = threadIdx.x;
    const int64_t item = blockIdx.x;
    const int e = a.items[item];
    const bool hang = a.has_hang[e] != 0;
    const int lev = a.level[e];
    const double h = ldexp(a.root_len, -lev), two_over_h = ldexp(a.two_over_root, lev);
    const double th = a.theta, idt = a.idt;
    const int npts = a.pt_cnt[item];
    const uint32_t *ent = a.entries + a.pt_off[item];
    const int s = lane & 7;
    const int m = a.masters[8 * (int64_t)e + s];
    const uint32_t code = a.ccode[4 * (int64_t)e + (s >> 1)] >> (16 * (s & 1));
    for (int idx = lane; idx < NF * 8; idx += 64) {
        const int f = idx >> 3;
        double v = 0.0;
        if (m >= 0) {
            if (f == 3) {
                v = a.f[3][m];
            } else if (f < 7) {
                const int c = f & 3;
                const double u = field_in(a, c)[m], u0 = field_in(a, 4 + c)[m];
                v = f < 3 ? th * u + (1.0 - th) * u0 : (u - u0) * idt;
            } else {
                v = x[4 * (int64_t)m + (f - 7)];
            }
        }
        sN[f][s] = v;
    }
    __syncthreads();
    // corner values, then coefficients in x = (h/2) xi (every lane of a group of
    // 8 takes part; the last group of the second pass may be idle as a whole)
    for (int idx = lane; idx < NF * 8; idx += 64) {
        const int f = idx >> 3;
        double v = sN[f][s];
        if (hang) {
            v = 0.0;
            for (int t = 0; t < 8; ++t) v += weight_of((code >> (2 * t)) & 3u) * sN[f][t];
        }
        const double ih = 0.5 * two_over_h;  // x runs over +-h/2: slope (v1 - v0) / h
        for (int b = 1; b < 8; b <<= 1) {
            const double o = __shfl_xor(v, b, 64);
            v = (s & b) ? (v - o) * ih : 0.5 * (v + o);
        }
        sP[f][s] = v;
    }
    __syncthreads();
    const PointPar P = point_par(a, h, two_over_h);
    double M[4][8];
    for (int i = 0; i < 4; ++i)
        for (int k = 0; k < 8; ++k) M[i][k] = 0.0;
    for (int base = 0; base < npts; base += 64) {
        const int pt = base + lane;
        if (pt < npts) {
            double xi[3], w;
            point_xw<true>(a, ent[pt], 0, h, xi, w);
            const double X[3] = {(0.5 * h * xi[0]), (0.5 * h * xi[1]), (0.5 * h * xi[2])};
            const double W = w;
            PointIn I;
            for (int c = 0; c < 3; ++c) {
                FENCE;
                poly_at(sP[c], X, I.u[c], I.gu[c]);
                FENCE;
                I.at[c] = poly_value(sP[4 + c], X);
            }
            FENCE;
            poly_at(sP[3], X, I.p, I.gp);
            if constexpr (JV) {
                for (int c = 0; c < 3; ++c) {
                    FENCE;
                    poly_at(sP[7 + c], X, I.du[c], I.dgu[c]);
                }
                FENCE;
                poly_at(sP[10], X, I.dp, I.dgp);
            }
            FENCE;
            double r[4][4];
            point_coeffs<JV>(I, P, r);
            const double xy = X[0] * X[1];
            for (int i = 0; i < 4; ++i) {
                FENCE;
                const double r0 = W * r[i][0], rx = W * r[i][1], ry = W * r[i][2], rz = W * r[i][3];
                const double px = r0 * X[0] + rx, py = r0 * X[1] + ry, pz = r0 * X[2] + rz;
                const double pxy = px * X[1] + ry * X[0];
                M[i][0] += r0;
                M[i][1] += px;
                M[i][2] += py;
                M[i][3] += pxy;
                M[i][4] += pz;
                M[i][5] += px * X[2] + rz * X[0];
                M[i][6] += py * X[2] + rz * X[1];
                M[i][7] += pxy * X[2] + rz * xy;
            }
        }
    }
    // sum over the lanes: each step halves the values a lane keeps; lane bits 5
    // and 4 choose the component, bits 3, 2 and 1 the coefficient
    double v[32];
    for (int t = 0; t < 32; ++t) v[t] = (double)M[t >> 3][t & 7];
#pragma unroll
    for (int n = 16; n >= 1; n >>= 1) {
        const bool up = (lane & (2 * n)) != 0;
#pragma unroll
        for (int t = 0; t < n; ++t) {
            const double keep = up ? v[t + n] : v[t], send = up ? v[t] : v[t + n];
            v[t] = keep + __shfl_xor(send, 2 * n, 64);
        }
    }
    double y = v[0] + __shfl_xor(v[0], 1, 64);
    const int q = (lane >> 1) & 7, i = lane >> 4;
    // coefficients back to corners: N = prod (1 +- x / (h/2)) / 2
    for (int b = 1; b < 8; b <<= 1) {
        const double o = __shfl_xor(y, 2 * b, 64);
        const double lo = (q & b) ? o : y, hi = ((q & b) ? y : o) * two_over_h;
        y = 0.5 * ((q & b) ? lo + hi : lo - hi);
    }
    if (hang) {
        double z = 0.0;
        for (int t = 0; t < 8; ++t) {
            const uint32_t ct = a.ccode[4 * (int64_t)e + (t >> 1)] >> (16 * (t & 1));
            z += weight_of((ct >> (2 * q)) & 3u) * __shfl(y, (lane & 0x30) | (2 * t), 64);
        }
        y = z;
    }
    if (!(lane & 1)) a.rrec[(a.slot0 + item) * 32 + 4 * q + i] = y;
}

// ---- FP32 point work (mixed contexts) --------------------------------------

// The FP32 results of the mixed forms are a fixed sequence of roundings: the
// constrained basis of the point, every field and its gradient as the sum of
// basis times slot value in slot order, the coefficients from u and u_prev
// separately, and every test function's sum over the points one after the
// other, the same as in the mixed element matrices' kernel, whose residual has
// the same bits. What is free is where it happens: here a lane holds a
// point with its 32 basis values in registers (8 OUT elements or 64 points of
// an item per wave), and only the products with the tests pass through LDS,
// where a lane then owns a (test function, component) chain. Eight lanes per
// point took 2.3 times as long.
constexpr int VB = 52;  // floats of a point in LDS: 32 basis values (slot, derivative), 16 coefficients, padding

template <bool SUB, bool JV>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_vec32(AsmArgs a, const double *x) {
    constexpr int NF = JV ? 11 : 7, NE = SUB ? 1 : 8;
    __shared__ __attribute__((aligned(16))) float sP[64 * VB];
    __shared__ __attribute__((aligned(16))) float sU[NE][NF][8];
    __shared__ float sC[NE][64];
    typedef float v4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x;
    const int el = SUB ? 0 : lane >> 3, s8 = lane & 7;
    const int64_t item = SUB ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * 8 + el;
    const bool valid = item < a.n_items;
    const int64_t it = valid ? item : a.n_items - 1;
    const int e = a.items[it];
    const bool hang = a.has_hang[e] != 0;
    const int lev = a.level[e];
    const double hd = ldexp(a.root_len, -lev), two_over_h = ldexp(a.two_over_root, lev);
    if (SUB) {
        for (int idx = lane; idx < NF * 8; idx += 64) {
            const int f = idx >> 3, m = a.masters[8 * (int64_t)e + (idx & 7)];
            double v = 0.0;
            if (m >= 0) v = f < 7 ? field_in(a, f)[m] : x[4 * (int64_t)m + (f - 7)];
            sU[0][f][idx & 7] = (float)v;
        }
    } else {
        const int m = a.masters[8 * (int64_t)e + s8];
        for (int f = 0; f < NF; ++f) {
            double v = 0.0;
            if (m >= 0) v = f < 7 ? a.f[f < 7 ? f : 0][m] : x[4 * (int64_t)m + (f - 7)];
            sU[el][f][s8] = (float)v;
        }
    }
    const bool any_hang = __any(hang);
    if (any_hang) {
        // lane (corner v = s8 of its element; of the one element: all 64 codes)
        if (SUB) {
            const int bit = 2 * lane;
            sC[0][lane] = (float)weight_of((a.ccode[4 * (int64_t)e + (bit >> 5)] >> (bit & 31)) & 3u);
        } else {
            const uint32_t row = a.ccode[4 * (int64_t)e + (s8 >> 1)] >> (16 * (s8 & 1));
            for (int t = 0; t < 8; ++t) sC[el][8 * s8 + t] = (float)weight_of((row >> (2 * t)) & 3u);
        }
    }
    const float rho = (float)a.rho, mu = (float)a.mu, th = (float)a.theta, idt = (float)a.idt, irho = (float)a.irho;
    const double gGd = two_over_h * two_over_h;
    const float gG = (float)gGd, tau0 = (float)(a.tau_a + a.tau_b * gGd * gGd), h2_12 = (float)(hd * hd * (1.0 / 12.0));
    const int npts = SUB ? a.pt_cnt[it] : 8;
    const uint32_t *ent = SUB ? a.entries + a.pt_off[it] : nullptr;
    float R[SUB ? 1 : 4];
    for (int i = 0; i < (SUB ? 1 : 4); ++i) R[i] = 0.f;
    for (int base = 0; base < npts; base += 64) {
        __syncthreads();
        const int pt = SUB ? base + lane : s8;
        if (pt < npts) {
            double xi[3], w;
            point_xw<SUB>(a, SUB ? ent[pt] : 0u, pt, hd, xi, w);
            const float xt[3] = {(float)xi[0], (float)xi[1], (float)xi[2]};
            const float hg = 0.5f * (float)two_over_h;
            float B[8][4];
            for (int v = 0; v < 8; ++v) {
                float f[3], g[3];
                for (int k = 0; k < 3; ++k) {
                    const bool up = (v >> k) & 1;
                    f[k] = 0.5f * (up ? 1.f + xt[k] : 1.f - xt[k]);
                    g[k] = up ? hg : -hg;
                }
                B[v][0] = f[0] * f[1] * f[2];
                B[v][1] = g[0] * f[1] * f[2];
                B[v][2] = f[0] * g[1] * f[2];
                B[v][3] = f[0] * f[1] * g[2];
            }
            if (any_hang) {
                // constrained slot s: the corners v with C[v][s] != 0 (weights are
                // powers of two: only the additions round)
                float c[8][4];
                for (int s = 0; s < 8; ++s)
                    for (int k = 0; k < 4; ++k) c[s][k] = 0.f;
                for (int v = 0; v < 8; ++v)
                    for (int s = 0; s < 8; ++s) {
                        const float cw = hang ? sC[el][8 * v + s] : (v == s ? 1.f : 0.f);
                        for (int k = 0; k < 4; ++k) c[s][k] += cw * B[v][k];
                    }
                for (int s = 0; s < 8; ++s)
                    for (int k = 0; k < 4; ++k) B[s][k] = c[s][k];
            }
            float *q = sP + lane * VB;
            for (int s = 0; s < 8; ++s) *(v4 *)(q + 4 * s) = v4{B[s][0], B[s][1], B[s][2], B[s][3]};
            float I[NF][4];
            for (int f = 0; f < NF; ++f) {
                FENCE;
                const v4 ua = *(const v4 *)&sU[el][f][0], ub = *(const v4 *)&sU[el][f][4];
                float v[4] = {0.f, 0.f, 0.f, 0.f};
                for (int s = 0; s < 8; ++s) {
                    const float u = s < 4 ? ua[s & 3] : ub[s & 3];
                    for (int k = 0; k < 4; ++k) v[k] += B[s][k] * u;
                }
                for (int k = 0; k < 4; ++k) I[f][k] = v[k];
            }
            FENCE;
            const float W = (float)w;
            // a zero the compiler does not see: terms that vanish keep their place
            // in the chain of multiply-adds
            float zero = 0.f;
            asm volatile("" : "+v"(zero));
            float r[16];
            float ut[3], gu[3][3], up[3], at[3], conv[3];
            for (int c = 0; c < 3; ++c) {
                ut[c] = th * I[c][0] + (1.f - th) * I[4 + c][0];
                for (int m = 0; m < 3; ++m) gu[c][m] = th * I[c][1 + m] + (1.f - th) * I[4 + c][1 + m];
            }
            for (int c = 0; c < 3; ++c) {
                at[c] = (I[c][0] - I[4 + c][0]) * idt;
                conv[c] = ut[0] * gu[c][0] + ut[1] * gu[c][1] + ut[2] * gu[c][2];
            }
            const float s0 = tau0 + gG * (ut[0] * ut[0] + ut[1] * ut[1] + ut[2] * ut[2]);
            const float tauM = rsq<float>(s0);
            const float tauC = h2_12 * s0 * tauM;
            for (int c = 0; c < 3; ++c) {
                const float rM = rho * (at[c] + conv[c]) + I[3][1 + c];
                up[c] = -tauM * rM;
            }
            const float upg = gG * (up[0] * up[0] + up[1] * up[1] + up[2] * up[2]);
            const float tb = upg > 0.f ? rsq<float>(upg) : 0.f;
            if constexpr (!JV) {
                const float div = gu[0][0] + gu[1][1] + gu[2][2];
                const float pp = -rho * tauC * div, pr = I[3][0];
                for (int c = 0; c < 3; ++c) {
                    const float svc = up[0] * gu[c][0] + up[1] * gu[c][1] + up[2] * gu[c][2];
                    r[4 * c] = W * (rho * at[c] + rho * conv[c] + svc);
                    for (int k = 0; k < 3; ++k)
                        r[4 * c + 1 + k] = W * (mu * (gu[c][k] + gu[k][c]) - (k == c ? pr + pp : zero) - ut[k] * up[c] -
                                                up[k] * up[c] * irho + tb * up[k] * svc);
                }
                r[12] = W * div;
                for (int k = 0; k < 3; ++k) r[13 + k] = -W * up[k] * irho;
            } else {
                float dut[3], dgu[3][3], dat[3], dup[3], dconv[3];
                for (int c = 0; c < 3; ++c) {
                    dut[c] = th * I[7 + c][0];
                    dat[c] = I[7 + c][0] * idt;
                    for (int m = 0; m < 3; ++m) dgu[c][m] = th * I[7 + c][1 + m];
                }
                for (int c = 0; c < 3; ++c) {
                    dconv[c] = dut[0] * gu[c][0] + dut[1] * gu[c][1] + dut[2] * gu[c][2] + ut[0] * dgu[c][0] +
                               ut[1] * dgu[c][1] + ut[2] * dgu[c][2];
                    const float dr = rho * (dat[c] + dconv[c]) + I[10][1 + c];
                    dup[c] = dr * -tauM;
                }
                const float ddiv = dgu[0][0] + dgu[1][1] + dgu[2][2];
                const float dpp = -rho * tauC * ddiv, dpr = I[10][0];
                for (int c = 0; c < 3; ++c) {
                    float sv = 0.f, dsv = 0.f;
                    for (int m = 0; m < 3; ++m) {
                        sv += up[m] * gu[c][m];
                        dsv += dup[m] * gu[c][m] + up[m] * dgu[c][m];
                    }
                    r[4 * c] = W * (rho * dat[c] + rho * dconv[c] + dsv);
                    // the products that round by themselves are fixed: (c, k) and
                    // (k, c) must not become one value
                    for (int k = 0; k < 3; ++k)
                        r[4 * c + 1 + k] = W * (mu * __builtin_fmaf(I[7 + k][1 + c], th, dgu[c][k]) -
                                                (k == c ? dpr + dpp : zero) - dut[k] * up[c] - ut[k] * dup[c] -
                                                __builtin_fmaf(dup[k], up[c], up[k] * dup[c]) * irho +
                                                tb * __builtin_fmaf(dup[k], sv, up[k] * dsv));
                }
                r[12] = W * ddiv;
                for (int k = 0; k < 3; ++k) r[13 + k] = -W * dup[k] * irho;
            }
            for (int i = 0; i < 4; ++i) *(v4 *)(q + 32 + 4 * i) = v4{r[4 * i], r[4 * i + 1], r[4 * i + 2], r[4 * i + 3]};
        }
        __syncthreads();
        // sums over the points in order: of the item, lane (a = lane % 8, i = lane / 8);
        // of the OUT elements, lane (element, a) for every i
        if (SUB) {
            if (lane < 32) {
                const int n = min(64, npts - base);
                for (int p = 0; p < n; ++p) {
                    const v4 b = *(const v4 *)(sP + p * VB + 4 * (lane & 7)), r = *(const v4 *)(sP + p * VB + 32 + 4 * (lane >> 3));
                    R[0] += b[0] * r[0] + b[1] * r[1] + b[2] * r[2] + b[3] * r[3];
                }
            }
        } else {
            for (int p = 0; p < 8; ++p) {
                const float *q = sP + (8 * el + p) * VB;
                const v4 b = *(const v4 *)(q + 4 * s8);
                for (int i = 0; i < 4; ++i) {
                    const v4 r = *(const v4 *)(q + 32 + 4 * i);
                    R[i % (SUB ? 1 : 4)] += b[0] * r[0] + b[1] * r[1] + b[2] * r[2] + b[3] * r[3];
                }
            }
        }
    }
    if (SUB) {
        if (lane < 32) a.rrec[(a.slot0 + item) * 32 + 4 * (lane & 7) + (lane >> 3)] = (double)R[0];
    } else if (valid) {
        typedef double v2 __attribute__((ext_vector_type(2)));
        v2 *dst = (v2 *)(a.rrec + (a.slot0 + item) * 32 + 4 * s8);
        dst[0] = v2{(double)R[0], (double)R[1 % (SUB ? 1 : 4)]};
        dst[1] = v2{(double)R[2 % (SUB ? 1 : 4)], (double)R[3 % (SUB ? 1 : 4)]};
    }
}

template <bool JV>
void launch64(hipStream_t s, const AsmArgs &a, bool sub, const double *x) {
    if (sub)
        hipLaunchKernelGGL((k_vec_sub<JV>), dim3((unsigned)a.n_items), dim3(64), 0, s, a, x);
    else
        hipLaunchKernelGGL((k_vec_out<JV>), dim3((unsigned)((a.n_items + 31) / 32)), dim3(256), 0, s, a, x);
}
template <bool JV>
void launch32(hipStream_t s, const AsmArgs &a, bool sub, const double *x) {
    if (sub)
        hipLaunchKernelGGL((k_vec32<true, JV>), dim3((unsigned)a.n_items), dim3(64), 0, s, a, x);
    else
        hipLaunchKernelGGL((k_vec32<false, JV>), dim3((unsigned)((a.n_items + 7) / 8)), dim3(64), 0, s, a, x);
}

}  // namespace

void launch_residual(hipStream_t s, const AsmArgs &a, bool sub, bool fp64, const double *x) {
    if (a.n_items <= 0) return;
    if (fp64) {
        if (x) launch64<true>(s, a, sub, x);
        else launch64<false>(s, a, sub, x);
    } else {
        if (x) launch32<true>(s, a, sub, x);
        else launch32<false>(s, a, sub, x);
    }
}

}  // namespace vmsk
