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
// the figures of these kernels are at their launches below.
#include "item_dev.h"
#include "vms_point.h"

namespace vmsk {

namespace {

constexpr double KA = 0.5 + 0.5 * VMS_XI, KB = 0.5 - 0.5 * VMS_XI;

// value of the lane whose bit AX (0: x, 1: y, 2: z) of the corner index differs
template <int AX>
__device__ inline float other(float v) {
    constexpr int ctrl = AX == 0 ? 0xB1 : (AX == 1 ? 0x4E : 0x128);
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), ctrl, 0xf, 0xf, true));
}
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
template <typename T>
struct PointIn {
    T u[3], gu[3][3], p, gp[3], at[3];
    T du[3], dgu[3][3], dp, dgp[3];
};

template <typename T>
struct PointPar {
    T rho, irho, mu, th, idt, gG, tau0, h2_12;
};

// residual coefficients r^i[k] (i test component, k = 0 against N, 1 + m
// against dN/dx_m), or their derivative along the direction, without the weight
template <typename T, bool JV>
__device__ inline void point_coeffs(const PointIn<T> &I, const PointPar<T> &P, T r[4][4]) {
    T up[3], acc[3];
    for (int c = 0; c < 3; ++c) {
        acc[c] = I.at[c] + I.u[0] * I.gu[c][0] + I.u[1] * I.gu[c][1] + I.u[2] * I.gu[c][2];
        up[c] = P.rho * acc[c] + I.gp[c];
    }
    const T s0 = P.tau0 + P.gG * (I.u[0] * I.u[0] + I.u[1] * I.u[1] + I.u[2] * I.u[2]);
    const T tauM = rsq<T>(s0);
    const T tauC = P.h2_12 * s0 * tauM;
    for (int c = 0; c < 3; ++c) up[c] *= -tauM;
    const T upg = P.gG * (up[0] * up[0] + up[1] * up[1] + up[2] * up[2]);
    const T tb = upg > T(0) ? rsq<T>(upg) : T(0);
    if constexpr (!JV) {
        const T div = I.gu[0][0] + I.gu[1][1] + I.gu[2][2];
        const T pt = I.p - P.rho * tauC * div;
        for (int c = 0; c < 3; ++c) {
            const T sv = up[0] * I.gu[c][0] + up[1] * I.gu[c][1] + up[2] * I.gu[c][2];
            r[c][0] = P.rho * acc[c] + sv;
            const T tu = tb * sv - up[c] * P.irho;
            for (int k = 0; k < 3; ++k)
                r[c][1 + k] = P.mu * (I.gu[c][k] + I.gu[k][c]) - I.u[k] * up[c] + up[k] * tu;
            r[c][1 + c] -= pt;
        }
        r[3][0] = div;
        for (int k = 0; k < 3; ++k) r[3][1 + k] = -up[k] * P.irho;
    } else {
        T dut[3], dup[3], dacc[3], dg[3][3];
        for (int c = 0; c < 3; ++c) {
            dut[c] = P.th * I.du[c];
            for (int m = 0; m < 3; ++m) dg[c][m] = P.th * I.dgu[c][m];
        }
        for (int c = 0; c < 3; ++c) {
            dacc[c] = I.du[c] * P.idt + dut[0] * I.gu[c][0] + dut[1] * I.gu[c][1] + dut[2] * I.gu[c][2] +
                      I.u[0] * dg[c][0] + I.u[1] * dg[c][1] + I.u[2] * dg[c][2];
            dup[c] = -tauM * (P.rho * dacc[c] + I.dgp[c]);
        }
        const T ddiv = dg[0][0] + dg[1][1] + dg[2][2];
        const T dpt = I.dp - P.rho * tauC * ddiv;
        for (int c = 0; c < 3; ++c) {
            const T sv = up[0] * I.gu[c][0] + up[1] * I.gu[c][1] + up[2] * I.gu[c][2];
            const T dsv = dup[0] * I.gu[c][0] + dup[1] * I.gu[c][1] + dup[2] * I.gu[c][2] +
                          up[0] * dg[c][0] + up[1] * dg[c][1] + up[2] * dg[c][2];
            r[c][0] = P.rho * dacc[c] + dsv;
            const T tu = tb * sv - up[c] * P.irho, dtu = tb * dsv - dup[c] * P.irho;
            for (int k = 0; k < 3; ++k)
                r[c][1 + k] = P.mu * (dg[c][k] + dg[k][c]) - dut[k] * up[c] - I.u[k] * dup[c] + dup[k] * tu +
                              up[k] * dtu;
            r[c][1 + c] -= dpt;
        }
        r[3][0] = ddiv;
        for (int k = 0; k < 3; ++k) r[3][1 + k] = -dup[k] * P.irho;
    }
}

template <typename T>
__device__ inline PointPar<T> point_par(const AsmArgs &a, double h, double two_over_h) {
    // G = (2/h)^2 I: tau_M^-2 = c_t/dt^2 + gG |u|^2 + c_i nu^2 G:G, tau_C = (h^2/12)/tau_M
    const double gG = two_over_h * two_over_h;
    return {(T)a.rho, (T)a.irho, (T)a.mu, (T)a.theta, (T)a.idt, (T)gG, (T)(a.tau_a + a.tau_b * gG * gG),
            (T)(h * h * (1.0 / 12.0))};
}

// ---- OUT elements ----------------------------------------------------------

// interpolation along one axis: the lane's point from its own corner and the other one
template <int AX, typename T>
__device__ inline T interp(T v) {
    return T(KA) * v + T(KB) * other<AX>(v);
}
// value and gradient at the lane's Gauss point of the field with corner value v
// (sg: +-1/h by the lane's bit of each axis)
template <typename T>
__device__ inline void field_at(T v, const T sg[3], T &val, T g[3]) {
    const T ox = other<0>(v);
    const T ix = T(KA) * v + T(KB) * ox, dx = sg[0] * (v - ox);
    const T oy = other<1>(ix);
    const T iy = T(KA) * ix + T(KB) * oy, dy = sg[1] * (ix - oy);
    const T oz = other<2>(iy);
    val = T(KA) * iy + T(KB) * oz;
    g[2] = sg[2] * (iy - oz);
    g[1] = interp<2>(dy);
    g[0] = interp<2>(interp<1>(dx));
}
template <typename T>
__device__ inline T value_at(T v) {
    return interp<2>(interp<1>(interp<0>(v)));
}
// the transpose: corner value of sum over the points of r0 N + r . grad N
template <typename T>
__device__ inline T test_sum(const T r[4], const T sg[3]) {
    T t = interp<2>(r[0]) + sg[2] * (r[3] + other<2>(r[3]));
    const T ty = interp<2>(r[2]);
    const T tx = interp<1>(interp<2>(r[1]));
    t = interp<1>(t) + sg[1] * (ty + other<1>(ty));
    return interp<0>(t) + sg[0] * (tx + other<0>(tx));
}

template <typename T, bool JV>
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
    const T ih = (T)(0.5 * two_over_h);
    const T sg[3] = {(s & 1) ? ih : -ih, (s & 2) ? ih : -ih, (s & 4) ? ih : -ih};
    PointIn<T> I;
    for (int c = 0; c < 3; ++c) {
        field_at<T>((T)f[c], sg, I.u[c], I.gu[c]);
        I.at[c] = value_at<T>((T)f[4 + c]);
    }
    field_at<T>((T)f[3], sg, I.p, I.gp);
    if constexpr (JV) {
        for (int c = 0; c < 3; ++c) field_at<T>((T)f[7 + c], sg, I.du[c], I.dgu[c]);
        field_at<T>((T)f[10], sg, I.dp, I.dgp);
    }
    const PointPar<T> P = point_par<T>(a, h, two_over_h);
    T r[4][4];
    point_coeffs<T, JV>(I, P, r);
    const double W = 0.125 * h * h * h;
    double y[4];
    for (int i = 0; i < 4; ++i) y[i] = W * (double)test_sum<T>(r[i], sg);
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
template <typename T>
__device__ inline void poly_at(const T *c, const T x[3], T &val, T g[3]) {
    const T e0 = c[0] + x[2] * c[4], e1 = c[1] + x[2] * c[5], e2 = c[2] + x[2] * c[6], e3 = c[3] + x[2] * c[7];
    g[0] = e1 + x[1] * e3;
    g[1] = e2 + x[0] * e3;
    g[2] = c[4] + x[0] * c[5] + x[1] * (c[6] + x[0] * c[7]);
    val = e0 + x[0] * g[0] + x[1] * e2;
}
template <typename T>
__device__ inline T poly_value(const T *c, const T x[3]) {
    const T e0 = c[0] + x[2] * c[4], e1 = c[1] + x[2] * c[5], e2 = c[2] + x[2] * c[6], e3 = c[3] + x[2] * c[7];
    return e0 + x[0] * e1 + x[1] * (e2 + x[0] * e3);
}

// The scheduler may not move work across FENCE: hoisting the LDS reads of all
// fields to the front took 352 VGPRs (FP64 action, one wave per SIMD, 0.27 ms on
// the 4.0M points) instead of 202.
#define FENCE __builtin_amdgcn_sched_barrier(0)

template <typename T, bool JV>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_vec_sub(AsmArgs a, const double *x) {
    constexpr int NF = JV ? 11 : 7;
    __shared__ double sN[NF][8];
    __shared__ __attribute__((aligned(16))) T sP[NF][8];
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
        sP[f][s] = (T)v;
    }
    __syncthreads();
    const PointPar<T> P = point_par<T>(a, h, two_over_h);
    T M[4][8];
    for (int i = 0; i < 4; ++i)
        for (int k = 0; k < 8; ++k) M[i][k] = T(0);
    for (int base = 0; base < npts; base += 64) {
        const int pt = base + lane;
        if (pt < npts) {
            double xi[3], w;
            point_xw<true>(a, ent[pt], 0, h, xi, w);
            const T X[3] = {(T)(0.5 * h * xi[0]), (T)(0.5 * h * xi[1]), (T)(0.5 * h * xi[2])};
            const T W = (T)w;
            PointIn<T> I;
            for (int c = 0; c < 3; ++c) {
                FENCE;
                poly_at<T>(sP[c], X, I.u[c], I.gu[c]);
                FENCE;
                I.at[c] = poly_value<T>(sP[4 + c], X);
            }
            FENCE;
            poly_at<T>(sP[3], X, I.p, I.gp);
            if constexpr (JV) {
                for (int c = 0; c < 3; ++c) {
                    FENCE;
                    poly_at<T>(sP[7 + c], X, I.du[c], I.dgu[c]);
                }
                FENCE;
                poly_at<T>(sP[10], X, I.dp, I.dgp);
            }
            FENCE;
            T r[4][4];
            point_coeffs<T, JV>(I, P, r);
            const T xy = X[0] * X[1];
            for (int i = 0; i < 4; ++i) {
                FENCE;
                const T r0 = W * r[i][0], rx = W * r[i][1], ry = W * r[i][2], rz = W * r[i][3];
                const T px = r0 * X[0] + rx, py = r0 * X[1] + ry, pz = r0 * X[2] + rz;
                const T pxy = px * X[1] + ry * X[0];
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

template <typename T, bool JV>
void launch(hipStream_t s, const AsmArgs &a, bool sub, const double *x) {
    if (sub)
        hipLaunchKernelGGL((k_vec_sub<T, JV>), dim3((unsigned)a.n_items), dim3(64), 0, s, a, x);
    else
        hipLaunchKernelGGL((k_vec_out<T, JV>), dim3((unsigned)((a.n_items + 31) / 32)), dim3(256), 0, s, a, x);
}

}  // namespace

void launch_residual(hipStream_t s, const AsmArgs &a, bool sub, bool fp64, const double *x) {
    if (a.n_items <= 0) return;
    if (fp64) {
        if (x) launch<double, true>(s, a, sub, x);
        else launch<double, false>(s, a, sub, x);
    } else {
        if (x) launch<float, true>(s, a, sub, x);
        else launch<float, false>(s, a, sub, x);
    }
}

}  // namespace vmsk
