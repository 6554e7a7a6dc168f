// VMS element assembly of libvms (gfx950): two-stage contraction with MFMA.
//
// Residual and Jacobian of the VMS weak form, eq. (vms), with the fine
// scales u' = -tau_M r_M (eq. uprime, f = 0, the viscous part of div sigma
// dropped for trilinear fields) and p' = -rho tau_C div u (eq. pprime),
// Crank-Nicolson in theta form (u_theta = theta u + (1-theta) u_prev), tau's
// frozen at the current state.
//
// At each quadrature point q (weight W) the element matrix gains
//   K[(a,i),(b,j)] += sum_{k,l} B[k][a] (W D^{ij}[k][l]) B[l][b],
// B = [N; dN/dx; dN/dy; dN/dz] of the constrained basis (B C, C the
// hanging-node operator M_e of Alg. 3) and D^{ij} the 4x4 coefficient block
// of the linearised integrand for test component i and trial component j:
//   D^{ij}[0][0] multiplies N_a N_b,  D^{ij}[0][1+l] N_a d_l N_b,
//   D^{ij}[1+k][0] d_k N_a N_b,       D^{ij}[1+k][1+l] d_k N_a d_l N_b.
// This is the precomputed-operator form of Alg. 6 / App. A (basis values and
// gradients tabulated at Gauss points; the element matrix is a contraction
// over points), split in two stages:
//   stage 1:  F_q[(i,k)][(b,j)] = sum_l W D^{ij}[k][l] B[l][b]
//   stage 2:  K[a][(b,j,i)]     = sum_{q,k} B_q[k][a] F_q[(i,k)][(b,j)]
// Stage 2 is a GEMM over the 8 basis rows a, the contraction over (point,
// derivative) and the 128 columns (b, j, i).
//
// Precision forms. FP64 runs both stages on v_mfma_f64_4x4x4 (asm_item64).
// MIXED_BF16 splits both stage-2 operands into three bf16 terms and
// MIXED_FP16 into two fp16 terms (with power-of-two scaling), accumulating in
// FP32 with v_mfma_f32_16x16x32 (eight points per k-step; rows a in 16-row
// tiles with the second split term in rows 8-15); stage 1 and everything
// before the contraction run in FP32 on the VALU and the result is written
// as FP32 (asm_item32).
//
// One 64-lane workgroup per element, points in chunks of 8 (FP64 sub-cell items: 16).
#include "item_dev.h"
#include "vms_point.h"

#include <type_traits>

namespace vmsk {
using namespace vmsd;


typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));


// split x into three bf16 terms with x ~= h + m + l
__device__ inline void split3(float x, __bf16 &h, __bf16 &m, __bf16 &l) {
    h = (__bf16)x;
    const float r1 = x - (float)h;
    m = (__bf16)r1;
    l = (__bf16)(r1 - (float)m);
}
__device__ inline void split2h(float x, _Float16 &h, _Float16 &l) {
    h = (_Float16)x;
    l = (_Float16)(x - (float)h);
}
// the same on pairs (one packed conversion per pair)
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
__device__ inline void split3x2(v2f x, v2bf &h, v2bf &m, v2bf &l) {
    h = __builtin_convertvector(x, v2bf);
    const v2f r1 = x - __builtin_convertvector(h, v2f);
    m = __builtin_convertvector(r1, v2bf);
    l = __builtin_convertvector(r1 - __builtin_convertvector(m, v2f), v2bf);
}
__device__ inline void split2hx2(v2f x, v2h &h, v2h &l) {
    h = __builtin_convertvector(x, v2h);
    l = __builtin_convertvector(x - __builtin_convertvector(h, v2f), v2h);
}

constexpr int LU = 9, LB = 40;  // padded strides in LDS (FP64): fields, basis rows of a point

// Per-lane element data of one OUT work item, loaded ahead of its use: the
// element, its level and hanging flag, the master of slot lane % 8, the
// constraint weight code of (corner lane / 8, slot lane % 8) and, for lanes
// < 56, nodal field lane / 8 at that master.
struct ItemPre {
    int32_t e, m, hang, level;
    uint32_t code;
    double fv;
};

// The loads of two OUT items interleaved, so that the second item's chain
// (item -> element -> masters -> fields) is in flight while the first is
// assembled.
__device__ inline void load_pre2(const AsmArgs &a, int64_t i0, int64_t i1, bool has1, ItemPre &P0,
                                 ItemPre &P1) {
    const int lane = threadIdx.x, s = lane & 7, bit = 2 * ((lane >> 3) * 8 + s);
    P0.e = a.items[i0];
    P1.e = has1 ? a.items[i1] : P0.e;
    P0.hang = a.has_hang[P0.e];
    P1.hang = a.has_hang[P1.e];
    P0.level = a.level[P0.e];
    P1.level = a.level[P1.e];
    P0.code = (a.ccode[4 * (int64_t)P0.e + (bit >> 5)] >> (bit & 31)) & 3u;
    P1.code = (a.ccode[4 * (int64_t)P1.e + (bit >> 5)] >> (bit & 31)) & 3u;
    P0.m = a.masters[8 * (int64_t)P0.e + s];
    P1.m = a.masters[8 * (int64_t)P1.e + s];
    P0.fv = (lane < 56 && P0.m >= 0) ? field_in(a, lane >> 3)[P0.m] : 0.0;
    P1.fv = (lane < 56 && P1.m >= 0) ? field_in(a, lane >> 3)[P1.m] : 0.0;
}

// ---------------------------------------------------------------------------
// FP64 element matrices
// ---------------------------------------------------------------------------
//
// Both contraction stages run on v_mfma_f64_4x4x4 (four 4x4 blocks per
// instruction, block = test component i). Stage 1 forms, per trial component
// j and half bh of the trial functions, F^{ij}[r][4 bh + n] = sum_c
// D^{ij}[r][c] B[c][4 bh + n]; its output registers have the layout of stage
// 2's second operand, and stage 2 adds B^T F into the 4x4 blocks of the 8x8
// component-pair block.
//
// The D blocks never exist as blocks: lane (c, i, r) of stage 1's first operand
// needs one entry D^{ij}[r][c] per j, and evaluates it from the point's table
// (PQ below) with lane constants in place of the case distinctions. With
// T1 = (rho, Y), T2 = (-tau rho, X), T3 = (1, taubar u') over the rows r,
// alpha = (1/dt, theta u) over the columns c, k = r - 1, l = c - 1,
// c_3 = tau_M and H = (grad u)^2, all times the weight:
//   D^{ij}[r][c] = g_ij (alpha T2 + z0 T1) + d_ij (alpha T1 + theta u'_l T3 + mu theta d_kl)
//                + d_kj (alpha c_i - z0 u'_i + mu theta d_il) + z0 (T2 H_ij + c_i g_kj)
//                + d_lj (rho tau_C theta d_ki + theta d_i3 d_r0),     j < 3,
//   D^{i3}[r][c] = (T2 g_il + d_il T1 + d_kl c_i) / rho (c > 0), -d_ki (c = 0),
// z0 = theta on c = 0 and 0 elsewhere, terms with k dropped on r = 0 and terms
// with l on c = 0. This is dblock_mv / dblock_simple of vms_point.h written per
// entry.
//
// What bounds it: issue. A probe of independent chains (four waves per SIMD)
// takes 18 cycles per v_mfma_f64_4x4x4 and 5.4 per v_fma_f64 at a nominal 2.4
// GHz, and a loop of both takes their sum: the matrix instruction does not run
// beside FP64 or FP32 VALU work, so every instruction counts. Per point 25
// MFMA, about 30 FP64 operations and 20 LDS reads for the D entries; with the
// blocks evaluated in two divergent passes, written to LDS (17.2 KB per
// workgroup, 2.25 waves per SIMD) and read back, the OUT elements of the
// 194k-octant sphere took 0.63 ms and its sub-cell items 2.2 ms; now 0.47 and 1.50 ms
// with 9.7 and 20.5 KB. The point tables (a quarter of the sub-cell items'
// VALU work) take four lanes per point: 16 points at a time fill the wave, in what
// LDS two waves per SIMD leave (8 at a time: 4% longer). An OUT element has only 8
// points, and those of two elements at once would cost a wave per SIMD; the batch
// kernel, which serves both, keeps 8 (8 trees of 30k octants: 3.59 ms, 3.85 at 16).
#define PQ_T12 0   // (T1, T2)[r], pairs
#define PQ_AUP 8   // (alpha, theta u')[c], pairs
#define PQ_CUP 16  // (c, u')[i], pairs; i = 3: (tau_M, 0)
#define PQ_T3 24   // T3[r]
#define PQ_G 28    // grad u rows i, 3 entries each; row 3 zero
#define PQ_H 40    // (grad u)^2 rows i
#define PQ_E1 49   // 0 0 rho tau_C theta 0 0: the unit row l starts at 2 - l
#define PQ_E2 54   // 0 0 theta 0 0
#define PQ_W 59
#define PQ_RC 60   // 16 residual coefficients r^i[k]
#define PQ_N 77

// Fields at the master slots are combined as they are loaded: rows 0-2
// u_theta, 3 p, 4-6 the rate (u - u_prev) / dt, of which only the value is
// interpolated.
template <int N>
struct Smem64T {
    static constexpr int NP = N;  // points tabulated at once
    double sU[7 * LU];
    double sC[64];
    double sB[NP * LB];
    double sI[NP * 19];  // per point: u_theta and gradient (4 each), p and gradient, rate (3)
    double sQ[NP * PQ_N - 1];  // the last row ends without its pad
};
// OUT elements: all 8 points
using Smem64 = Smem64T<8>;
// sub-cell items: reference coordinates and weights of 64 points
template <int N>
struct Smem64Sub : Smem64T<N> {
    double sX[64][4];
};

template <bool SUB, typename SM>  // SM: Smem64 or Smem64Sub<8 or 16>
__device__ __forceinline__ void asm_item64(const AsmArgs &a, const int64_t item, SM &sm,
                                           const ItemPre *pre) {
    constexpr int NP = SUB ? SM::NP : 8;
    const int lane = threadIdx.x;
    __syncthreads();  // the previous item of this workgroup is done with the LDS
    const int e = pre ? pre->e : a.items[item];
    const bool hang = (pre ? pre->hang : a.has_hang[e]) != 0;
    const int lev = pre ? pre->level : (int)a.level[e];
    const double h = ldexp(a.root_len, -lev);
    const double two_over_h = ldexp(a.two_over_root, lev);
    const double rho = a.rho, mu = a.mu, th = a.theta, idt = a.idt, irho = a.irho;
    {
        uint32_t code;
        double fv;
        if (pre) {
            code = pre->code;
            fv = pre->fv;
        } else {
            const int bit = 2 * lane;
            code = (a.ccode[4 * (int64_t)e + (bit >> 5)] >> (bit & 31)) & 3u;
            const int m = a.masters[8 * (int64_t)e + (lane & 7)];
            fv = (lane < 56 && m >= 0) ? field_in(a, lane >> 3)[m] : 0.0;
        }
        sm.sC[lane] = code == 3u ? 1.0 : (code == 2u ? 0.5 : (code == 1u ? 0.25 : 0.0));
        const double other = __shfl_xor(fv, 32, 64);  // fields f and f + 4
        if (lane < 24) fv = th * fv + (1.0 - th) * other;
        else if (lane >= 32) fv = (other - fv) * idt;
        if (lane < 56) sm.sU[(lane >> 3) * LU + (lane & 7)] = fv;
    }
    const int npts = SUB ? a.pt_cnt[item] : 8;
    // G = (2/h)^2 I: u.G.u = gG |u|^2; tau_M^-2 = c_t/dt^2 + gG |u|^2 + c_i nu^2 G:G;
    // tau_C = 1/(tau_M tr G) = (h^2/12)/tau_M
    const double gG = two_over_h * two_over_h;
    const double tau0 = a.tau_a + a.tau_b * gG * gG;
    const double h2_12 = h * h * (1.0 / 12.0);

    // lane constants of the D entries
    const int c4 = lane >> 4, i4 = (lane >> 2) & 3, r4 = lane & 3, kr = r4 - 1, lc = c4 - 1;
    const double z0 = c4 == 0 ? th : 0.0, n0 = c4 == 0 ? 0.0 : 1.0;
    double dk[3], di[3];
    for (int j = 0; j < 3; ++j) {
        dk[j] = kr == j ? 1.0 : 0.0;
        di[j] = i4 == j ? 1.0 : 0.0;
    }
    const double kil = (c4 > 0 && i4 == lc) ? mu * th : 0.0;
    const double kkl = (c4 > 0 && kr == lc) ? mu * th : 0.0;
    const double mc = c4 > 0 ? irho : 0.0;
    const double m1 = (c4 > 0 && i4 == lc && r4 > 0) ? irho : 0.0, m2 = (c4 > 0 && kr == lc) ? irho : 0.0;
    const double m3 = (c4 == 0 && r4 > 0 && kr == i4) ? -1.0 : 0.0;
    const int x_at = c4 == 0 ? (i4 < 3 ? PQ_H + 3 * i4 : PQ_G + 9)
                             : (r4 > 0 && kr == i4 ? PQ_E1 + 2 - lc
                                                   : (i4 == 3 && r4 == 0 ? PQ_E2 + 2 - lc : PQ_G + 9));
    const int gi_at = PQ_G + 3 * i4, gk_at = PQ_G + (r4 > 0 ? 3 * kr : 9);
    const int gl_at = gi_at + (c4 > 0 ? lc : 0);

    // K^{ij}[4 ah + m][4 bh + n] in lane (m = lane / 16, i, n = lane % 4)
    double acc[2][2][4];
    for (int t = 0; t < 16; ++t) acc[t >> 3][(t >> 2) & 1][t & 3] = 0.0;
    // the residual is one more MFMA whose blocks 0 and 1 are the two halves of
    // the rows a (columns i carry r^i[k]): lane l holds R[4 ((l / 4) % 4) + l / 16][l % 4]
    double accr = 0.0;
    const int p8 = lane >> 3, s8 = lane & 7;
    // the lane's sub-cell entry, loaded 64 points ahead
    const int64_t eoff = SUB ? a.pt_off[item] : 0;
    uint32_t en_cur = (SUB && lane < npts) ? a.entries[eoff + lane] : 0u;
    if (lane < NP) sm.sB[lane * LB + 32] = 0.0;  // the zero that idle blocks of the residual read
    const int r_at = i4 < 2 ? c4 * 8 + 4 * i4 + r4 : 32;
    __syncthreads();

    for (int base = 0; base < npts; base += NP) {
        const int np = min(NP, npts - base);
        if constexpr (SUB) {
            // decoded 64 points at a time, one per lane (8 lanes per point would
            // decode each point 8 times)
            if ((base & 63) == 0) {
                double xi[3], w;
                point_xw<true>(a, en_cur, 0, h, xi, w);
                if (base + lane >= npts) w = 0.0;  // points beyond the item's last weigh nothing
                for (int k = 0; k < 3; ++k) sm.sX[lane][k] = xi[k];
                sm.sX[lane][3] = w;
                const int pn = base + 64 + lane;
                en_cur = pn < npts ? a.entries[eoff + pn] : 0u;
                __syncthreads();
            }
        }
        // ---- phase 1: constrained basis at the chunk's points (lane = (p, s))
        double w = 0.0;
        // the chunk's points, 8 at a time. A loop also where there are only 8: without
        // it the OUT elements' kernel spills at three waves per SIMD, with it the
        // batch's loses 1% (its registers suffice either way).
        auto eights = [&](auto f) {
            if constexpr (std::is_same_v<SM, Smem64Sub<8>>) {
                f(p8);
            } else {
#pragma unroll 1
                for (int p = p8; p < NP && p - p8 < np; p += 8) f(p);
            }
        };
        eights([&](int p) {
            double xi[3], b[4];
            if constexpr (SUB) {
                const double *X = sm.sX[(base & 63) + p];
                for (int k = 0; k < 3; ++k) xi[k] = X[k];
                w = X[3];
            } else {
                point_xw<false>(a, 0u, p8, h, xi, w);
            }
            const double hg = 0.5 * two_over_h;
            if (!hang) {
                // slot s is corner s
                double f[3], g[3];
                for (int k = 0; k < 3; ++k) {
                    const bool up = (s8 >> k) & 1;
                    f[k] = 0.5 + (up ? 0.5 : -0.5) * xi[k];
                    g[k] = up ? hg : -hg;
                }
                b[0] = f[0] * f[1] * f[2];
                b[1] = g[0] * f[1] * f[2];
                b[2] = f[0] * g[1] * f[2];
                b[3] = f[0] * f[1] * g[2];
            } else {
                // every corner v with C[v][s] != 0
                for (int k = 0; k < 4; ++k) b[k] = 0.0;
#pragma unroll 1
                for (int v = 0; v < 8; ++v) {
                    const double c = sm.sC[v * 8 + s8];
                    if (c == 0.0) continue;
                    double f[3], g[3];
                    for (int k = 0; k < 3; ++k) {
                        const bool up = (v >> k) & 1;
                        f[k] = 0.5 * (up ? 1.0 + xi[k] : 1.0 - xi[k]);
                        g[k] = up ? hg : -hg;
                    }
                    b[0] += c * (f[0] * f[1] * f[2]);
                    b[1] += c * (g[0] * f[1] * f[2]);
                    b[2] += c * (f[0] * g[1] * f[2]);
                    b[3] += c * (f[0] * f[1] * g[2]);
                }
            }
            for (int k = 0; k < 4; ++k) sm.sB[p * LB + k * 8 + s8] = b[k];
        });
        __syncthreads();
        // ---- phase 2: interpolation of the nodal fields (lane = (p, field))
        if (s8 < 7)
            eights([&](int p) {
                double v[4] = {0.0, 0.0, 0.0, 0.0};
                for (int s = 0; s < 8; ++s) {
                    const double u = sm.sU[s8 * LU + s];
                    for (int k = 0; k < 4; ++k) v[k] += sm.sB[p * LB + k * 8 + s] * u;
                }
                double *I = sm.sI + p * 19;
                if (s8 < 4) {
                    for (int k = 0; k < 4; ++k) I[4 * s8 + k] = v[k];
                } else {
                    I[12 + s8] = v[0];
                }
            });
        __syncthreads();
        // ---- phase 3: the point's table. Lanes r < 3 of point p take row / component
        // r of it; with every component index rotated by r their own row is index
        // 0, so that no register array is indexed by the lane. Lane r = 3 writes
        // the scalars and the continuity row.
        const int p3 = NP == 16 ? lane >> 2 : p8, r3 = NP == 16 ? lane & 3 : s8;
        if constexpr (NP == 16) w = sm.sX[(base & 63) + p3][3];
        if (r3 < 4) {
            const double *I = sm.sI + p3 * 19;
            const int o[3] = {r3 < 3 ? r3 : 0, r3 < 3 ? (r3 + 1 < 3 ? r3 + 1 : 0) : 1,
                              r3 < 3 ? (r3 + 2 < 3 ? r3 + 2 : r3 - 1) : 2};
            double ut[3], gu[3][3], up[3], acl[3];
            for (int c = 0; c < 3; ++c) {
                ut[c] = I[4 * o[c]];
                for (int m = 0; m < 3; ++m) gu[c][m] = I[4 * o[c] + 1 + o[m]];
            }
            const double s0 = tau0 + gG * (ut[0] * ut[0] + ut[1] * ut[1] + ut[2] * ut[2]);
            const double tauM = rsq<double>(s0);
            const double tauC = h2_12 * s0 * tauM;
            for (int c = 0; c < 3; ++c) {
                acl[c] = I[16 + o[c]] + ut[0] * gu[c][0] + ut[1] * gu[c][1] + ut[2] * gu[c][2];
                up[c] = -tauM * (rho * acl[c] + I[13 + o[c]]);
            }
            const double div = gu[0][0] + gu[1][1] + gu[2][2];
            const double pp = -rho * tauC * div;
            const double upg = gG * (up[0] * up[0] + up[1] * up[1] + up[2] * up[2]);
            const double tb = upg > 0.0 ? rsq<double>(upg) : 0.0;
            double *q = sm.sQ + p3 * PQ_N;
            if (r3 < 3) {
                const int c = r3;
                const double sv = up[0] * gu[0][0] + up[1] * gu[0][1] + up[2] * gu[0][2];
                const double Wt = w * tauM, tbr = tb * rho;
                q[PQ_T12 + 2 * (c + 1)] = Wt * (rho * ut[0] + up[0]);
                q[PQ_T12 + 2 * (c + 1) + 1] = -Wt * tbr * up[0];
                q[PQ_AUP + 2 * (c + 1)] = th * ut[0];
                q[PQ_AUP + 2 * (c + 1) + 1] = th * up[0];
                q[PQ_CUP + 2 * c] = Wt * (up[0] - tbr * sv);
                q[PQ_CUP + 2 * c + 1] = w * up[0];
                q[PQ_T3 + 1 + c] = w * tb * up[0];
                for (int m = 0; m < 3; ++m) {
                    q[PQ_G + 3 * c + o[m]] = gu[0][m];
                    q[PQ_H + 3 * c + o[m]] = gu[0][0] * gu[0][m] + gu[0][1] * gu[1][m] + gu[0][2] * gu[2][m];
                    const double t = mu * (gu[0][m] + gu[m][0]) - ut[m] * up[0] - up[m] * up[0] * irho + tb * up[m] * sv;
                    q[PQ_RC + 4 * c + 1 + o[m]] = w * (m == 0 ? t - (I[12] + pp) : t);
                }
                q[PQ_RC + 4 * c] = w * (rho * acl[0] + sv);
                q[PQ_G + 9 + c] = 0.0;
            } else {
                q[PQ_T12] = w * rho;
                q[PQ_T12 + 1] = -w * tauM * rho;
                q[PQ_AUP] = idt;
                q[PQ_AUP + 1] = 0.0;
                q[PQ_CUP + 6] = w * tauM;
                q[PQ_CUP + 7] = 0.0;
                q[PQ_T3] = w;
                q[PQ_E1] = q[PQ_E1 + 1] = q[PQ_E1 + 3] = q[PQ_E1 + 4] = 0.0;
                q[PQ_E2] = q[PQ_E2 + 1] = q[PQ_E2 + 3] = q[PQ_E2 + 4] = 0.0;
                q[PQ_E1 + 2] = w * rho * tauC * th;
                q[PQ_E2 + 2] = w * th;
                q[PQ_W] = w;
                q[PQ_RC + 12] = w * div;
                for (int k = 0; k < 3; ++k) q[PQ_RC + 13 + k] = -w * up[k] * irho;
            }
        }
        __syncthreads();
        // ---- phase 4: D entries, stage 1, stage 2
        // an odd tail runs a point of weight zero (a loop to np: 6.02 -> 6.11 ms for the
        // sub-cell items of the 721k-octant sphere)
        const int n2 = SUB ? (np + 1) & ~1 : 8;
#pragma unroll 1
        for (int p = 0; p < n2; ++p) {
            const double *q = sm.sQ + p * PQ_N;
            const double *B = sm.sB + p * LB + c4 * 8 + r4;
            const double A0 = B[0], A1 = B[4];
            const double T1 = q[PQ_T12 + 2 * r4], T2 = q[PQ_T12 + 2 * r4 + 1];
            const double al = q[PQ_AUP + 2 * c4], ul = q[PQ_AUP + 2 * c4 + 1];
            const double ci = q[PQ_CUP + 2 * i4], ui = q[PQ_CUP + 2 * i4 + 1];
            const double T3 = q[PQ_T3 + r4], W = q[PQ_W], gl = q[gl_at];
            const double Ar = sm.sB[p * LB + r_at];
            accr = __builtin_amdgcn_mfma_f64_4x4x4f64(Ar, q[PQ_RC + 4 * r4 + c4], accr, 0, 0, 0);
            const double a1 = al * T2 + z0 * T1;
            const double bk = al * ci - z0 * ui + kil * W;
            const double a5 = al * T1 + ul * T3 + kkl * W;
            const double y1 = z0 * T2 + n0, y2 = z0 * ci;
            double D[4];
            for (int j = 0; j < 3; ++j)
                D[j] = a1 * q[gi_at + j] + y1 * q[x_at + j] + y2 * q[gk_at + j] + dk[j] * bk + di[j] * a5;
            D[3] = mc * T2 * gl + m1 * T1 + m2 * ci + m3 * W;
            double F[4][2];
            for (int j = 0; j < 4; ++j)
                for (int bh = 0; bh < 2; ++bh)
                    F[j][bh] = __builtin_amdgcn_mfma_f64_4x4x4f64(D[j], bh ? A1 : A0, 0.0, 0, 0, 0);
            for (int j = 0; j < 4; ++j)
                for (int bh = 0; bh < 2; ++bh) {
                    acc[0][bh][j] = __builtin_amdgcn_mfma_f64_4x4x4f64(A0, F[j][bh], acc[0][bh][j], 0, 0, 0);
                    acc[1][bh][j] = __builtin_amdgcn_mfma_f64_4x4x4f64(A1, F[j][bh], acc[1][bh][j], 0, 0, 0);
                }
        }
        __syncthreads();
    }

    if (!std::is_same_v<SM, Smem64Sub<8>> && a.vals) {  // not in batches
        // atomic scatter: no record; each entry is added into its CSR place
        // (the summation order is the hardware's)
        double *vals = (double *)a.vals;
        const int32_t *mst = a.masters + 8 * (int64_t)e;
        const uint16_t *kk = a.el_kk + 64 * (int64_t)e;
        int al = threadIdx.x;
        asm volatile("" : "+v"(al));  // lane constants formed here, not kept through the point loop
        const int c4 = al >> 4, i4 = (al >> 2) & 3, r4 = al & 3;
#pragma unroll
        for (int ah = 0; ah < 2; ++ah) {
            const int av = 4 * ah + c4, ma = mst[av];
            if (ma < 0) continue;
            const int64_t r0 = a.nrow_ptr[ma], deg = a.nrow_ptr[ma + 1] - r0;
#pragma unroll
            for (int bh = 0; bh < 2; ++bh) {
                __builtin_amdgcn_sched_barrier(0);  // one block's registers at a time
                // 16 lanes trade (row i, column b) x entries j for (b, j) x rows, so
                // that each addition's lanes take four blocks of one row, often one
                // line (64 places in as many lines otherwise: 47.6 ms for the OUT
                // elements of two boxes in 1.64 M octants)
                auto pick = [](double v0, double v1, double v2, double v3, int k) {
                    const double lo = (k & 1) ? v1 : v0, hi = (k & 1) ? v3 : v2;
                    return (k & 2) ? hi : lo;
                };
                const double v0 = acc[ah][bh][0], v1 = acc[ah][bh][1], v2 = acc[ah][bh][2], v3 = acc[ah][bh][3];
                double w[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) w[s] = __shfl_xor(pick(v0, v1, v2, v3, r4 ^ s), s, 64);
                const double u0 = pick(w[0], w[1], w[2], w[3], r4), u1 = pick(w[0], w[1], w[2], w[3], r4 ^ 1),
                             u2 = pick(w[0], w[1], w[2], w[3], r4 ^ 2), u3 = pick(w[0], w[1], w[2], w[3], r4 ^ 3);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < 4; ++s) w[s] = __shfl_xor(pick(u0, u1, u2, u3, i4 ^ s), 4 * s, 64);
                __builtin_amdgcn_sched_barrier(0);
                const int b = 4 * bh + i4;
                if (mst[b] >= 0) {
                    double *dst = vals + 16 * r0 + 4 * (int64_t)kk[8 * av + b] + r4;
#pragma unroll
                    for (int n = 0; n < 4; ++n) atomicAdd(dst + 4 * n * deg, pick(w[0], w[1], w[2], w[3], i4 ^ n));
                }
            }
        }
    } else {
        // record of the work item, block-major (block (a, b) of master slots,
        // entry 4 i + j): a lane's four entries j are 32 contiguous bytes, 16
        // lanes write 512
        double *dst = (double *)a.em + (a.slot0 + item) * 1024;
        for (int ah = 0; ah < 2; ++ah)
            for (int bh = 0; bh < 2; ++bh) {
                const double *v = acc[ah][bh];
                *(v4d *)(dst + ((4 * ah + c4) * 8 + 4 * bh + r4) * 16 + 4 * i4) = v4d{v[0], v[1], v[2], v[3]};
            }
    }
    // residual record of the work item (entry 4 a + i)
    if (i4 < 2 && a.rrec) a.rrec[(a.slot0 + item) * 32 + 4 * (4 * i4 + c4) + r4] = accr;
}

// ---------------------------------------------------------------------------
// Mixed element matrices (BF16x3, FP16x2)
// ---------------------------------------------------------------------------
//
// Everything before the contraction is FP32; its roundings (the order of every
// sum and which products are fused) are those of the residual kernels of the
// mixed contexts too, whose results it must equal bit for bit.
//
// What bounds it: latency, then VALU issue. LDS decides the occupancy, so only
// the D blocks of two test components are there at a time (4.2 KB instead of
// 8.8), all arrays are in groups of four read and written as 16 bytes, and the
// record leaves through LDS in whole lines: 8.8 KB and 126 VGPRs, four waves per
// SIMD (13 KB and three before). Steps, then: adaptive mesh of 165,656 octants BF16x3
// 0.817 -> 0.695 ms, 194k-octant sphere FP16x2 2.47 -> 2.07 ms, sphere of 721,169
// octants BF16x3 9.00 -> 7.84 ms.
#define FQ_UT 0    // u_theta, W
#define FQ_UP 4    // u', tau_M
#define FQ_Y 8     // Y, taubar
#define FQ_X 12    // X, tau_C
#define FQ_A 16    // I/dt + theta grad u by columns j, 4 apart
#define FQ_G 28    // grad u rows, 4 apart
#define FQ_GA 40   // grad u A rows, 4 apart
#define FQ_CP 52
#define FQ_YM 56
#define FQ_XM 60
#define FQ_CM 64
#define FQ_RC 68   // 16 residual coefficients
#define FQ_SV 84
#define FQ_N 92
constexpr int FB = 36;   // floats of a point's basis: (slot, derivative), padded
constexpr int FD = 132;  // floats of a point's D blocks of two test components, padded

struct SmemF {
    __attribute__((aligned(16))) float sU[7 * 8];
    float sC[64];
    __attribute__((aligned(16))) float sB[8 * FB];
    __attribute__((aligned(16))) float sQ[8 * FQ_N];
    union {
        __attribute__((aligned(16))) float sI[8 * 28];  // interpolated fields (field, derivative)
        // blocks (i % 2, j), rows k; points 2 g + pp at 4 pp + g, so that the four
        // lane groups of the contraction read different banks
        __attribute__((aligned(16))) float sD[8 * FD];
        __attribute__((aligned(16))) float sOut[1024];  // the record, on its way out
    };
    float sSc[8];  // fp16 form: per-point bound of the contraction operands
};
// sub-cell items: reference coordinates and weights of 64 points
struct SmemFSub : SmemF {
    __attribute__((aligned(16))) float sX[64][4];
};

// One 4x4 D block, weight folded in (dblock_mv and dblock_simple of vms_point.h
// on the packed table).
__device__ inline void dblock_f(const float *q, int i, int j, float rho, float mu, float th, float irho, v4f D[4]) {
    const v4f UT = *(const v4f *)(q + FQ_UT), UP = *(const v4f *)(q + FQ_UP), Yv = *(const v4f *)(q + FQ_Y),
              Xv = *(const v4f *)(q + FQ_X);
    const float W = UT[3], tauM = UP[3], tb = Yv[3], tC = Xv[3];
    if (i < 3 && j < 3) {
        const v4f Acol = *(const v4f *)(q + FQ_A + 4 * j);
        float ei[3], ej[3];
        for (int l = 0; l < 3; ++l) {
            ei[l] = l == i ? 1.f : 0.f;
            ej[l] = l == j ? 1.f : 0.f;
        }
        const float Aij = q[FQ_A + 4 * j + i], gij = q[FQ_G + 4 * i + j], GAij = q[FQ_GA + 4 * i + j];
        const float cpi = q[FQ_CP + i], upi = q[FQ_UP + i];
        const float tr = tauM * rho;
        const float dth = (i == j) ? th * W : 0.f;
        const float thw = th * W;
        D[0][0] = W * (rho * Aij - tr * GAij);
        const float a0 = dth * rho - thw * tr * gij;
        for (int l = 0; l < 3; ++l) D[0][1 + l] = a0 * UT[l] + dth * UP[l];
        const float c1 = dth * tr, c2 = dth * tauM, c3 = -thw * tb * tr * gij, c4 = dth * tb;
        const float AW = Aij * W, GW = GAij * W, cW = cpi * W;
        const float mthw = mu * thw, rtcw = rho * tC * thw;
        const float dm = (i == j) ? mthw : 0.f;
        for (int k = 0; k < 3; ++k) {
            const float kj = ej[k], ki = ei[k];
            D[1 + k][0] = AW * Yv[k] + cW * Acol[k] + GW * Xv[k] - kj * (thw * upi);
            const float al = c1 * UT[k] + (c2 + c3) * UP[k] + kj * (thw * cpi);
            const float be = c4 * UP[k];
            const float s1 = kj * mthw, s2 = ki * rtcw;
            for (int l = 0; l < 3; ++l) {
                float v = al * UT[l] + be * UP[l] + s1 * ei[l] + s2 * ej[l];
                if (k == l) v += dm;
                D[1 + k][1 + l] = v;
            }
        }
    } else {
        const bool mp = i < 3 && j == 3, cv = i == 3 && j < 3;
        const float wmp = mp ? W : 0.f, wcv = cv ? W : 0.f, wcc = (!mp && !cv) ? W : 0.f;
        const int ii = i < 3 ? i : 0, jj = j < 3 ? j : 0;
        const v4f g = *(const v4f *)(q + FQ_G + 4 * ii), Acol = *(const v4f *)(q + FQ_A + 4 * jj),
                  ym = *(const v4f *)(q + FQ_YM), xm = *(const v4f *)(q + FQ_XM);
        float ei[3], ej[3];
        for (int l = 0; l < 3; ++l) {
            ei[l] = l == i ? 1.f : 0.f;
            ej[l] = l == j ? 1.f : 0.f;
        }
        const float cmi = q[FQ_CM + ii];
        const float tw = wcv * tauM, tthw = tw * th, mtau = -wmp * tauM, thw = wcv * th;
        const float diag = wmp * cmi + wcc * tauM * irho;
        D[0][0] = 0.f;
        for (int l = 0; l < 3; ++l) D[0][1 + l] = mtau * g[l] + thw * ej[l];
        for (int k = 0; k < 3; ++k) {
            D[1 + k][0] = tw * Acol[k] - wmp * ei[k];
            const float xk = wmp * xm[k], yk = wmp * ym[k], sk = tthw * ej[k];
            for (int l = 0; l < 3; ++l) {
                float v = xk * g[l] + sk * UT[l] + yk * ei[l];
                if (k == l) v += diag;
                D[1 + k][1 + l] = v;
            }
        }
    }
}

// TIGHT: the lane's addresses and masks are formed anew for every chunk; kept
// over the loop they take the sub-cell items from 126 VGPRs to over 160
template <int MODE, bool SUB, bool TIGHT = SUB>
__device__ __forceinline__ void asm_item32(const AsmArgs &a, const int64_t item, std::conditional_t<SUB, SmemFSub, SmemF> &sm,
                                           const ItemPre *pre) {
    const int lane = threadIdx.x;
    __syncthreads();  // the previous item of this workgroup is done with the LDS
    const int e = pre ? pre->e : a.items[item];
    const bool hang = (pre ? pre->hang : a.has_hang[e]) != 0;
    const int lev = pre ? pre->level : (int)a.level[e];
    const double hd = ldexp(a.root_len, -lev);
    const double two_over_h = ldexp(a.two_over_root, lev);
    {
        uint32_t code;
        double fv;
        if (pre) {
            code = pre->code;
            fv = pre->fv;
        } else {
            const int bit = 2 * lane;
            code = (a.ccode[4 * (int64_t)e + (bit >> 5)] >> (bit & 31)) & 3u;
            const int m = a.masters[8 * (int64_t)e + (lane & 7)];
            fv = (lane < 56 && m >= 0) ? field_in(a, lane >> 3)[m] : 0.0;
        }
        sm.sC[lane] = code == 3u ? 1.f : (code == 2u ? 0.5f : (code == 1u ? 0.25f : 0.f));
        if (lane < 56) sm.sU[lane] = (float)fv;
    }
    const int npts = SUB ? a.pt_cnt[item] : 8;
    const float rho = (float)a.rho, mu = (float)a.mu, th = (float)a.theta, idt = (float)a.idt, irho = (float)a.irho;
    // G = (2/h)^2 I: u.G.u = gG |u|^2; tau_M^-2 = c_t/dt^2 + gG |u|^2 + c_i nu^2 G:G;
    // tau_C = 1/(tau_M tr G) = (h^2/12)/tau_M
    const double gGd = two_over_h * two_over_h;
    const float gG = (float)gGd, tau0 = (float)(a.tau_a + a.tau_b * gGd * gGd);
    const float h2_12 = (float)(hd * hd * (1.0 / 12.0));
    // fp16 form: gradient rows of the basis scaled by h/2 (all rows within
    // [-1, 1]); s16 = exponent of the product scale (accumulators carry 2^s16)
    const float hhalf = (float)(0.5 * hd), gh = (float)two_over_h;
    int s16 = INT_MAX;

    v4f acc[4][2];
    for (int t = 0; t < 8; ++t) acc[t >> 1][t & 1] = v4f{0, 0, 0, 0};
    float R = 0.f;  // lanes < 32: residual of (a = lane & 7, i = lane >> 3)
    // the lane's sub-cell entry, loaded 64 points ahead
    const int64_t eoff = SUB ? a.pt_off[item] : 0;
    uint32_t en_cur = (SUB && lane < npts) ? a.entries[eoff + lane] : 0u;
    __syncthreads();

    for (int base = 0; base < npts; base += 8) {
        const int np = min(8, npts - base);
        int lane = threadIdx.x;
        if (TIGHT) asm volatile("" : "+v"(lane));
        if constexpr (SUB) {
            // decoded 64 points at a time, one per lane (8 lanes per point would
            // decode each point 8 times)
            if ((base & 63) == 0) {
                double xi[3], w;
                point_xw<true>(a, en_cur, 0, hd, xi, w);
                *(v4f *)sm.sX[lane] = v4f{(float)xi[0], (float)xi[1], (float)xi[2], (float)w};
                const int pn = base + 64 + lane;
                en_cur = pn < npts ? a.entries[eoff + pn] : 0u;
                __syncthreads();
            }
        }
        // ---- phase 1: constrained basis at the chunk's points (lane = (p, s))
        {
            const int p = lane >> 3, s = lane & 7;
            float b[4] = {0.f, 0.f, 0.f, 0.f}, w = 0.f;
            if (p < np) {
                float xt[3];
                if constexpr (SUB) {
                    const v4f X = *(const v4f *)sm.sX[(base & 63) + p];
                    for (int k = 0; k < 3; ++k) xt[k] = X[k];
                    w = X[3];
                } else {
                    double xi[3], wd;
                    point_xw<false>(a, 0u, p, hd, xi, wd);
                    for (int k = 0; k < 3; ++k) xt[k] = (float)xi[k];
                    w = (float)wd;
                }
                const float hg = 0.5f * (float)two_over_h;
                if (!hang) {
                    // slot s is corner s
                    float f[3], g[3];
                    for (int k = 0; k < 3; ++k) {
                        const bool up = (s >> k) & 1;
                        f[k] = 0.5f * (up ? 1.f + xt[k] : 1.f - xt[k]);
                        g[k] = up ? hg : -hg;
                    }
                    b[0] = f[0] * f[1] * f[2];
                    b[1] = g[0] * f[1] * f[2];
                    b[2] = f[0] * g[1] * f[2];
                    b[3] = f[0] * f[1] * g[2];
                } else {
                    // every corner v with C[v][s] != 0
#pragma unroll 1
                    for (int v = 0; v < 8; ++v) {
                        const float c = sm.sC[v * 8 + s];
                        if (c == 0.f) continue;
                        float f[3], g[3];
                        for (int k = 0; k < 3; ++k) {
                            const bool up = (v >> k) & 1;
                            f[k] = 0.5f * (up ? 1.f + xt[k] : 1.f - xt[k]);
                            g[k] = up ? hg : -hg;
                        }
                        b[0] += c * (f[0] * f[1] * f[2]);
                        b[1] += c * (g[0] * f[1] * f[2]);
                        b[2] += c * (f[0] * g[1] * f[2]);
                        b[3] += c * (f[0] * f[1] * g[2]);
                    }
                }
            }
            *(v4f *)(sm.sB + p * FB + 4 * s) = v4f{b[0], b[1], b[2], b[3]};
            if (s == 0) {
                sm.sQ[p * FQ_N + FQ_UT + 3] = w;
                if (MODE == 2) sm.sSc[p] = 0.f;
            }
        }
        __syncthreads();
        // ---- phase 2: interpolation of the nodal fields (lane = (p, field))
        {
            const int p = lane >> 3, f = lane & 7;
            if (f < 7) {
                const v4f ua = *(const v4f *)(sm.sU + 8 * f), ub = *(const v4f *)(sm.sU + 8 * f + 4);
                v4f v = {0.f, 0.f, 0.f, 0.f};
                for (int s = 0; s < 8; ++s) {
                    const float u = s < 4 ? ua[s & 3] : ub[s & 3];
                    const v4f b = *(const v4f *)(sm.sB + p * FB + 4 * s);
                    for (int k = 0; k < 4; ++k) v[k] += b[k] * u;
                }
                *(v4f *)(sm.sI + p * 28 + 4 * f) = v;
            }
        }
        __syncthreads();
        // ---- phase 3: point quantities, lane = (p, r). (a) Lanes r = 0..3 of
        // point p evaluate the point state; lane r < 3 writes row / component
        // c = r of it and momentum row c of the residual coefficients r^i[k]
        // (times W), lane r = 3 the scalars and the continuity row.
        {
            const int p = lane >> 3, r = lane & 7;
            if (p < np && r < 4) {
                const float *Ip = sm.sI + p * 28;
                v4f I[7];
                for (int f = 0; f < 7; ++f) I[f] = *(const v4f *)(Ip + 4 * f);
                float ut[3], gu[3][3], up[3];
                for (int c = 0; c < 3; ++c) {
                    ut[c] = th * I[c][0] + (1.f - th) * I[4 + c][0];
                    for (int m = 0; m < 3; ++m) gu[c][m] = th * I[c][1 + m] + (1.f - th) * I[4 + c][1 + m];
                }
                float rM[3];
                for (int c = 0; c < 3; ++c) {
                    const float atc = (I[c][0] - I[4 + c][0]) * idt;
                    const float conv = ut[0] * gu[c][0] + ut[1] * gu[c][1] + ut[2] * gu[c][2];
                    rM[c] = rho * (atc + conv) + I[3][1 + c];
                }
                const float div = gu[0][0] + gu[1][1] + gu[2][2];
                const float s0 = tau0 + gG * (ut[0] * ut[0] + ut[1] * ut[1] + ut[2] * ut[2]);
                const float tauM = rsq<float>(s0);
                const float tauC = h2_12 * s0 * tauM;  // (h^2/12) / tau_M
                for (int c = 0; c < 3; ++c) up[c] = -tauM * rM[c];
                const float pp = -rho * tauC * div;
                const float upg = gG * (up[0] * up[0] + up[1] * up[1] + up[2] * up[2]);
                const float tb = upg > 0.f ? rsq<float>(upg) : 0.f;
                float *q = sm.sQ + p * FQ_N;
                const float W = q[FQ_UT + 3];
                if (r < 3) {
                    const int c = r;
                    const v4f Ic = *(const v4f *)(Ip + 4 * c), Jc = *(const v4f *)(Ip + 16 + 4 * c);
                    float guc[3], gcol[3];
                    for (int m = 0; m < 3; ++m) {
                        guc[m] = th * Ic[1 + m] + (1.f - th) * Jc[1 + m];
                        gcol[m] = th * Ip[4 * m + 1 + c] + (1.f - th) * Ip[16 + 4 * m + 1 + c];
                    }
                    const float utc = th * Ic[0] + (1.f - th) * Jc[0];
                    const float atc = (Ic[0] - Jc[0]) * idt;
                    const float convc = ut[0] * guc[0] + ut[1] * guc[1] + ut[2] * guc[2];
                    const float upc = -tauM * (rho * (atc + convc) + Ip[13 + c]);
                    const float svc = up[0] * guc[0] + up[1] * guc[1] + up[2] * guc[2];
                    const float pr = I[3][0];
                    q[FQ_UT + c] = utc;
                    q[FQ_UP + c] = upc;
                    q[FQ_SV + c] = svc;
                    *(v4f *)(q + FQ_G + 4 * c) = v4f{guc[0], guc[1], guc[2], 0.f};
                    float rc[3];
                    for (int k = 0; k < 3; ++k)
                        rc[k] = W * (mu * (guc[k] + gcol[k]) - (k == c ? pr + pp : 0.f) - ut[k] * upc -
                                     up[k] * upc * irho + tb * up[k] * svc);
                    *(v4f *)(q + FQ_RC + 4 * c) = v4f{W * (rho * atc + rho * convc + svc), rc[0], rc[1], rc[2]};
                } else {
                    q[FQ_UP + 3] = tauM;
                    q[FQ_X + 3] = tauC;
                    q[FQ_Y + 3] = tb;
                    *(v4f *)(q + FQ_RC + 12) = v4f{W * div, -W * up[0] * irho, -W * up[1] * irho, -W * up[2] * irho};
                }
            }
        }
        // (b) the factors of the D blocks from the stored point state, lane
        // (p, r): r < 3 the matrix rows c = r, 3 <= r < 6 the vector
        // components c = r - 3. The round trip through LDS bounds the registers
        // the point phase holds.
        __syncthreads();
        {
            const int p = lane >> 3, r = lane & 7;
            if (p < np && r < 6) {
                float *q = sm.sQ + p * FQ_N;
                const float tauM = q[FQ_UP + 3], tb = q[FQ_Y + 3];
                const float tr = tauM * rho, tbtr = tb * tauM * rho, tbt = tb * tauM, tir = tauM * irho;
                if (r < 3) {
                    const int c = r;
                    const v4f gc = *(const v4f *)(q + FQ_G + 4 * c), g0 = *(const v4f *)(q + FQ_G),
                              g1 = *(const v4f *)(q + FQ_G + 4), g2 = *(const v4f *)(q + FQ_G + 8);
                    float ga[3];
                    for (int m = 0; m < 3; ++m) {
                        q[FQ_A + 4 * m + c] = (c == m ? idt : 0.f) + th * gc[m];
                        float v = 0.f;
                        for (int k = 0; k < 3; ++k) {
                            const float gk = k == 0 ? g0[m] : (k == 1 ? g1[m] : g2[m]);
                            v += gc[k] * ((k == m ? idt : 0.f) + th * gk);
                        }
                        ga[m] = v;
                    }
                    *(v4f *)(q + FQ_GA + 4 * c) = v4f{ga[0], ga[1], ga[2], 0.f};
                } else {
                    const int c = r - 3;
                    const float utc = q[FQ_UT + c], upc = q[FQ_UP + c], svc = q[FQ_SV + c];
                    q[FQ_Y + c] = tr * utc + tauM * upc;
                    q[FQ_X + c] = -tbtr * upc;
                    q[FQ_CP + c] = tauM * upc - tbtr * svc;
                    q[FQ_YM + c] = tauM * utc + tir * upc;
                    q[FQ_CM + c] = tir * upc - tbt * svc;
                    q[FQ_XM + c] = -tbt * upc;
                }
            }
        }
        __syncthreads();
        // ---- phase 4: the D blocks of test components {0, 1}, then {2, 3}: one
        // block per lane, momentum/velocity blocks first
        auto dtask = [&](int hf, int &p, int &i, int &j) {
            const int n = hf == 0 ? 48 : 24;
            if (lane < n) {
                p = hf == 0 ? lane / 6 : lane / 3;
                i = hf == 0 ? (lane % 6) / 3 : 2;
                j = lane % 3;
            } else if (hf == 0) {
                p = (lane - n) >> 1;
                i = lane & 1;
                j = 3;
            } else {
                const int u = (lane - n) % 5;
                p = (lane - n) / 5;
                i = u == 0 ? 2 : 3;
                j = u == 0 ? 3 : u - 1;
            }
        };
        auto dcompute = [&](int hf, v4f D[4], int &dst) {
            int p, i, j;
            dtask(hf, p, i, j);
            dst = ((p & 1) * 4 + (p >> 1)) * FD + (4 * (i & 1) + j) * 16;
            if (p >= np) {
                for (int k = 0; k < 4; ++k) D[k] = v4f{0.f, 0.f, 0.f, 0.f};
                return;
            }
            dblock_f(sm.sQ + p * FQ_N, i, j, rho, mu, th, irho, D);
            if constexpr (MODE == 2) {
                // bound of the point's stage-1 operands: row k is sum_l D[k][l] B[l][b]
                // with |B| <= 1 for values and <= 2/h for gradients, times 2/h
                // for gradient rows (their basis rows carry h/2)
                float bnd = 0.f;
                for (int k = 0; k < 4; ++k) {
                    float v = fabsf(D[k][0]);
                    for (int l = 1; l < 4; ++l) v += gh * fabsf(D[k][l]);
                    bnd = fmaxf(bnd, k > 0 ? gh * v : v);
                }
                atomicMax((int *)&sm.sSc[p], __float_as_int(bnd));  // non-negative floats
            }
        };
        v4f D[4];
        int dst;
        dcompute(0, D, dst);
        for (int k = 0; k < 4; ++k) *(v4f *)(sm.sD + dst + 4 * k) = D[k];
        if constexpr (MODE == 2) dcompute(1, D, dst);  // the scale needs every block's bound
        __syncthreads();
        // ---- phase 5: stage 1 (VALU) and stage 2 (MFMA); k-step of 32 = 8 points x
        // 4 derivative rows, lane group g holds points 2g, 2g+1
        const int g = lane >> 4, row = lane & 15, ar = row & 7, bb = row >> 2, jc = lane & 3;
        const bool hi_rows = row < 8;
        // fp16: powers of two put the chunk's largest product near 2^12 and
        // balance it between the two operands of each point (A about 2^ea, F
        // about 2^(s16 - ea)): both split terms stay in the normal fp16 range.
        // A later chunk with larger products lowers s16 and rescales the
        // accumulators (exact).
        int ea[2] = {0, 0};
        float fs[2][2] = {{1.f, 1.f}, {1.f, 1.f}};
        if constexpr (MODE == 2) {
            float bm = 0.f;
            for (int q = 0; q < 8; ++q) bm = fmaxf(bm, sm.sSc[q]);
            if (bm > 0.f) {
                const int sc = 12 - ilogbf(bm);
                if (s16 == INT_MAX) {
                    s16 = sc;
                } else if (sc < s16) {
                    const float f = ldexpf(1.0f, sc - s16);
                    for (int t = 0; t < 8; ++t)
                        for (int r = 0; r < 4; ++r) acc[t >> 1][t & 1][r] *= f;
                    s16 = sc;
                }
            }
            const int sv = s16 == INT_MAX ? 0 : s16;
            for (int pp = 0; pp < 2; ++pp) {
                const float bp = sm.sSc[2 * g + pp];
                ea[pp] = bp > 0.f ? ((ilogbf(bp) + sv) >> 1) : 0;
                fs[pp][0] = ldexpf(1.0f, sv - ea[pp]);
                fs[pp][1] = ldexpf(gh, sv - ea[pp]);
            }
        }
        v8bf Ahm, Alo;
        v8h Ah;
        v4f Bc[2][2];  // basis values of the lane's two points at its two columns b
        for (int pp = 0; pp < 2; ++pp) {
            const float *B = sm.sB + (2 * g + pp) * FB;
            const v4f Av = *(const v4f *)(B + 4 * ar);
            for (int k = 0; k < 4; ++k) {
                const int t = 4 * pp + k;
                if constexpr (MODE == 1) {
                    __bf16 x1, x2, x3;
                    split3(Av[k], x1, x2, x3);
                    Ahm[t] = hi_rows ? x1 : x2;
                    Alo[t] = hi_rows ? x3 : (__bf16)0.0f;
                } else {
                    _Float16 x1, x2;
                    split2h(Av[k] * ldexpf(k == 0 ? 1.0f : hhalf, ea[pp]), x1, x2);
                    Ah[t] = hi_rows ? x1 : x2;
                }
            }
            for (int bh = 0; bh < 2; ++bh) Bc[pp][bh] = *(const v4f *)(B + 4 * (4 * bh + bb));
        }
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            if (hf == 1) {
                if constexpr (MODE == 1) dcompute(1, D, dst);
                __syncthreads();
                for (int k = 0; k < 4; ++k) *(v4f *)(sm.sD + dst + 4 * k) = D[k];
                __syncthreads();
            }
#pragma unroll
            for (int i2 = 0; i2 < 2; ++i2) {
                v8bf F1[2], F2[2], F3[2];
                v8h H1[2], H2[2];
                for (int t = 0; t < 8; t += 2) {
                    const int pp = t >> 2, k = t & 3;
                    const float *dp = sm.sD + (4 * pp + g) * FD + (4 * i2 + jc) * 16 + 4 * k;
                    const v4f d[2] = {*(const v4f *)dp, *(const v4f *)(dp + 4)};
                    for (int bh = 0; bh < 2; ++bh) {
                        v2f F;
                        for (int u = 0; u < 2; ++u) {
                            F[u] = d[u][0] * Bc[pp][bh][0] + d[u][1] * Bc[pp][bh][1] + d[u][2] * Bc[pp][bh][2] +
                                   d[u][3] * Bc[pp][bh][3];
                            // undo the basis scaling and the balance on this operand
                            if (MODE == 2) F[u] *= fs[pp][k + u > 0];
                        }
                        if constexpr (MODE == 1) {
                            v2bf x1, x2, x3;
                            split3x2(F, x1, x2, x3);
                            F1[bh][t] = x1[0]; F1[bh][t + 1] = x1[1];
                            F2[bh][t] = x2[0]; F2[bh][t + 1] = x2[1];
                            F3[bh][t] = x3[0]; F3[bh][t + 1] = x3[1];
                        } else {
                            v2h x1, x2;
                            split2hx2(F, x1, x2);
                            H1[bh][t] = x1[0]; H1[bh][t + 1] = x1[1];
                            H2[bh][t] = x2[0]; H2[bh][t + 1] = x2[1];
                        }
                    }
                }
                for (int bh = 0; bh < 2; ++bh) {
                    v4f c = acc[2 * hf + i2][bh];
                    if constexpr (MODE == 1) {
                        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ahm, F1[bh], c, 0, 0, 0);
                        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ahm, F2[bh], c, 0, 0, 0);
                        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ahm, F3[bh], c, 0, 0, 0);
                        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Alo, F1[bh], c, 0, 0, 0);
                    } else {
                        c = __builtin_amdgcn_mfma_f32_16x16x32_f16(Ah, H1[bh], c, 0, 0, 0);
                        c = __builtin_amdgcn_mfma_f32_16x16x32_f16(Ah, H2[bh], c, 0, 0, 0);
                    }
                    acc[2 * hf + i2][bh] = c;
                }
            }
        }
        // residual: lanes < 32, (a = lane & 7, i = lane >> 3)
        if (lane < 32) {
            for (int p = 0; p < np; ++p) {
                const v4f b = *(const v4f *)(sm.sB + p * FB + 4 * (lane & 7)),
                          r = *(const v4f *)(sm.sQ + p * FQ_N + FQ_RC + 4 * (lane >> 3));
                R += b[0] * r[0] + b[1] * r[1] + b[2] * r[2] + b[3] * r[3];
            }
        }
        __syncthreads();
    }

    // rows 8..15 carry the second split term: fold them onto rows 0..7. The
    // halves of the wave trade their halves of two tiles, so that every lane ends
    // with (rows 4 ((lane / 16) % 2) + r, b = 4 (lane / 32) + bb, j) of each i
    const int bb = (lane >> 2) & 3, jc = lane & 3;
    const float unscale = (MODE == 2 && s16 != INT_MAX) ? ldexpf(1.0f, -s16) : 1.0f;
    const int a0 = 4 * ((lane >> 4) & 1), b = 4 * (lane >> 5) + bb;
    v4f K[4];
    for (int i = 0; i < 4; ++i)
        for (int r = 0; r < 4; ++r) {
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[i][0][r]), __float_as_uint(acc[i][1][r]),
                                                             false, false);
            K[i][r] = (__uint_as_float(sw[0]) + __uint_as_float(sw[1])) * unscale;
        }
    if (a.vals) {
        // atomic scatter: no record; each entry is added into its CSR place
        // (the summation order is the hardware's)
        float *vals = (float *)a.vals;
        const int32_t *mst = a.masters + 8 * (int64_t)e;
        const uint16_t *kk = a.el_kk + 64 * (int64_t)e;
        if (mst[b] >= 0)
            for (int r = 0; r < 4; ++r) {
                const int ma = mst[a0 + r];
                if (ma < 0) continue;
                const int64_t r0 = a.nrow_ptr[ma], deg = a.nrow_ptr[ma + 1] - r0;
                float *dst = vals + 16 * r0 + 4 * (int64_t)kk[8 * (a0 + r) + b] + jc;
                for (int i = 0; i < 4; ++i) atomicAdd(dst + 4 * i * deg, K[i][r]);
            }
    } else {
        // record of the work item, block-major (block (a, b) of master slots,
        // entry 4 i + j)
        for (int r = 0; r < 4; ++r)
            for (int i = 0; i < 4; ++i) sm.sOut[((a0 + r) * 8 + b) * 16 + 4 * i + jc] = K[i][r];
        __syncthreads();
        v4f *dst = (v4f *)((float *)a.em + (a.slot0 + item) * 1024);
        for (int t = 0; t < 4; ++t) dst[64 * t + lane] = ((const v4f *)sm.sOut)[64 * t + lane];
    }
    // residual record of the work item (entry 4 a + i)
    if (lane < 32 && a.rrec) a.rrec[(a.slot0 + item) * 32 + 4 * (lane & 7) + (lane >> 3)] = (double)R;
}

// Waves per SIMD the register allocation aims for. The FP64 matrix kernels fit
// three (OUT elements: 160 VGPRs; at four they spill, 3.00 -> 3.60 ms per step
// on the 194k-octant sphere). The FP64 sub-cell items stay at two: they run
// beside the HBM-bound gather, which needs the other registers for its own
// waves (two-box step of 1.6M octants 12.30 ms at three, 11.75 ms at two; the
// sphere, where the items outlast the gather, 3.01 against 3.03 ms). The mixed
// kernels have the LDS and the registers for four (FP16x2 sphere step 2.14 ms
// at three, 2.07 at four).
#define VMS_ASM_BOUNDS(MODE, SUB) \
    __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu((MODE) == 0 ? ((SUB) ? 2 : 3) : 4, 8)))

// OUT elements (SUB = false) two per workgroup: the second element's data
// and fields load while the first is assembled
template <typename T, int MODE, bool SUB>
__global__ VMS_ASM_BOUNDS(MODE, SUB) void k_asm2(AsmArgs a) {
    __shared__ std::conditional_t<MODE == 0, std::conditional_t<SUB, Smem64Sub<16>, Smem64>,
                                  std::conditional_t<SUB, SmemFSub, SmemF>> sm;
    auto item = [&](int64_t i, const ItemPre *pre) {
        if constexpr (MODE == 0) asm_item64<SUB>(a, i, sm, pre);
        else asm_item32<MODE, SUB>(a, i, sm, pre);
    };
    if constexpr (SUB) {
        item(blockIdx.x, nullptr);
    } else {
        const int64_t i0 = (int64_t)blockIdx.x << a.pair, i1 = i0 + 1;
        const bool has1 = a.pair && i1 < a.n_items;
        ItemPre P0, P1;
        load_pre2(a, i0, i1, has1, P0, P1);
        item(i0, &P0);
        if (has1) item(i1, &P1);
    }
}

// Persistent form over many contexts: every workgroup takes units of work
// from a device counter until none is left, in the order of the unit list
// (heaviest first); a unit is a run of OUT elements or of sub-cell work items
// of one tree. One launch for all units.
template <int MODE, int WPS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WPS, WPS))) void k_asm_batch(
    const AsmArgs *std_args, const AsmArgs *sub_args, const BatchUnit *units, int64_t n_units,
    unsigned long long *counter) {
    __shared__ std::conditional_t<MODE == 0, Smem64Sub<8>, SmemFSub> sm;
    __shared__ int64_t su;
    __shared__ AsmArgs sa;  // the unit's tree, read from LDS where used
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) su = (int64_t)atomicAdd(counter, 1ull);
        __syncthreads();
        const int64_t u = su;
        if (u >= n_units) break;
        const BatchUnit U = units[u];
        if (threadIdx.x == 0) sa = U.sub ? sub_args[U.tree] : std_args[U.tree];
        __syncthreads();
        if constexpr (MODE == 0) {
            if (U.sub) {
                for (int k = 0; k < U.count; ++k) asm_item64<true>(sa, U.first + k, sm, nullptr);
            } else {
                for (int k = 0; k < U.count; ++k) asm_item64<false>(sa, U.first + k, sm, nullptr);
            }
        } else if (U.sub) {
            for (int k = 0; k < U.count; ++k) asm_item32<MODE, true, (WPS > 2)>(sa, U.first + k, sm, nullptr);
        } else {
            for (int k = 0; k < U.count; ++k) asm_item32<MODE, false, (WPS > 2)>(sa, U.first + k, sm, nullptr);
        }
    }
}

__global__ void k_reset_counter(unsigned long long *c) {
    if (threadIdx.x < 2 && blockIdx.x == 0) c[threadIdx.x] = 0ull;
}

void launch_assemble_batch(hipStream_t s, int precision, const AsmArgs *std_args,
                           const AsmArgs *sub_args, const BatchUnit *units, int64_t n_units,
                           unsigned long long *counter, int n_groups, int n_cu) {
    hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(64), 0, s, counter);
    if (n_units <= 0) return;
    dim3 grid((unsigned)n_groups), block(64);
    // mixed forms: up to two workgroups per SIMD have 256 registers each and
    // keep the lane's addresses; more of them run the 128-register build (8
    // trees of 30k octants, BF16x3: 2.98 against 3.23 ms at 8 workgroups per CU,
    // 3.35 against 2.55 ms at 16)
    const bool many = n_groups > 8 * n_cu;
#define VMS_B(MODE, WPS) \
    hipLaunchKernelGGL((k_asm_batch<MODE, WPS>), grid, block, 0, s, std_args, sub_args, units, n_units, counter)
    if (precision == 0) VMS_B(0, 2);
    else if (precision == 1 && many) VMS_B(1, 4);
    else if (precision == 1) VMS_B(1, 2);
    else if (many) VMS_B(2, 4);
    else VMS_B(2, 2);
#undef VMS_B
}

// CSR values from the element-matrix records. A thread takes V consecutive
// entries of one row of a CSR block B (entries e0 .. e0+V-1, e = 4 i + j) and
// sums them over B's contributions in list order (ascending record), fetching
// the record entries V at a time and four contributions at a time; the CSR
// place of entry (i, j) is vbase[B] + i |vstride[B]| + j. A negative stride
// marks the diagonal block of an inactive node: it has no records and becomes
// an identity block. A positive stride may carry the VS_LATE flag (the block
// has records of sub-cell or surface items); SKIP_LATE leaves such blocks out.
template <typename T, int V, bool SKIP_LATE = false>
__device__ inline void gather_block(const T *em, const int64_t *cb_off, const int32_t *contrib,
                                    const int64_t *vbase, const int32_t *vstride, int64_t B, int e0,
                                    T *vals) {
    typedef T vec __attribute__((ext_vector_type(V)));
    const int st = vstride[B];
    if (SKIP_LATE && st > 0 && (st & VS_LATE)) return;
    const int64_t c0 = cb_off[B], c1 = cb_off[B + 1];
    const int64_t base = vbase[B];
    const int stride = st < 0 ? -st : (st & (VS_LATE - 1));
    double s[V];
    for (int q = 0; q < V; ++q) s[q] = (st < 0 && ((e0 + q) >> 2) == ((e0 + q) & 3)) ? 1.0 : 0.0;
    for (int64_t c = c0; c < c1; c += 4) {
        int32_t r[4];
        for (int u = 0; u < 4; ++u) r[u] = c + u < c1 ? contrib[c + u] : -1;
        vec v[4];
        for (int u = 0; u < 4; ++u)
            if (r[u] >= 0) {
                const vec *src = (const vec *)(em + (int64_t)r[u] * 16 + e0);
                v[u] = sizeof(T) == 8 ? __builtin_nontemporal_load(src) : *src;
            }
        for (int u = 0; u < 4; ++u)
            if (r[u] >= 0)
                for (int q = 0; q < V; ++q) s[q] += (double)v[u][q];
    }
    // the CSR values are written once and not read again by this step:
    // streaming (non-temporal) stores keep them from displacing the records
    // in the caches (FP64 gather of the 10^7-octant workload 23.2 -> 20.8 ms)
    T *dst = vals + base + (int64_t)(e0 >> 2) * stride + (e0 & 3);
    vec o;
    for (int q = 0; q < V; ++q) o[q] = (T)s[q];
    __builtin_nontemporal_store(o, (vec *)dst);
}

// residual of node n from the residual records (one thread per node, its entries
// in ascending record order, four in flight)
__device__ inline void res_node(const double *rrec, const int64_t *roff, const int32_t *rlist, int64_t n,
                                double *out) {
    const int64_t c0 = roff[n], c1 = roff[n + 1];
    v4d s = {0.0, 0.0, 0.0, 0.0};
    for (int64_t c = c0; c < c1; c += 4) {
        int32_t q[4];
        for (int u = 0; u < 4; ++u) q[u] = c + u < c1 ? rlist[c + u] : -1;
        v4d v[4];
        for (int u = 0; u < 4; ++u)
            if (q[u] >= 0) v[u] = *(const v4d *)(rrec + 4 * (int64_t)q[u]);
        for (int u = 0; u < 4; ++u)
            if (q[u] >= 0)
                for (int e = 0; e < 4; ++e) s[e] += v[u][e];
    }
    for (int e = 0; e < 4; ++e) out[4 * n + e] = s[e];
}

// The residual's summation rides in the launch of the CSR blocks' (the first nr
// workgroups): on small meshes a launch of its own costs as much as the
// summation (504 octants, FP64: 13.9 us a step, 18.1 us with a second launch).
__device__ inline bool res_part(const ResSum &r, unsigned nr) {
    if (blockIdx.x >= nr) return false;
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n < r.n_nodes) res_node(r.rrec, r.roff, r.rlist, n, r.out);
    return true;
}
static unsigned res_groups(const ResSum &r) { return r.out ? (unsigned)((r.n_nodes + 255) / 256) : 0u; }

// Bound by HBM: records and values alone are 15.8 GB in 3.6 ms for two boxes in
// 1.64 M octants in FP64; with lists and lines read again the counters see 5.4 TB/s
// on 10.2 M octants (a large copy reaches 4.9 TB/s on this GPU, reads alone 6.1).
// Workgroups go round the 8 XCDs in turn; the
// FP64 gather gives each XCD one contiguous range of blocks instead (its grid is a
// multiple of 8), so that workgroups which share lines of the block headers and
// of the CSR rows share an L2, and its records, read once, pass the caches by:
// 16^3 triquadratic elements 482 -> 456 us, the two-box step 11.22 -> 11.07 ms. FP32
// records are more often still in the caches, where going round finds them
// sooner (166k hanging-node octants: 686 us so, 706 us by ranges).
template <typename T, int V, bool SKIP_LATE>
__global__ void k_gather(const T *em, const int64_t *cb_off, const int32_t *contrib,
                         const int64_t *vbase, const int32_t *vstride, int64_t nb, T *vals, ResSum r, unsigned nr) {
    constexpr int TPB = 16 / V;  // threads per block
    if constexpr (!SKIP_LATE)
        if (res_part(r, nr)) return;
    const unsigned b = blockIdx.x - nr;
    const int64_t wg = sizeof(T) == 8 ? (int64_t)(b & 7) * ((gridDim.x - nr) >> 3) + (b >> 3) : b;
    const int64_t g = wg * blockDim.x + threadIdx.x;
    const int64_t B = g / TPB;
    if (B >= nb) return;
    gather_block<T, V, SKIP_LATE>(em, cb_off, contrib, vbase, vstride, B, (int)(g % TPB) * V, vals);
}

// the listed blocks only (the late blocks, after the sub-cell and surface records)
template <typename T, int V>
__global__ void k_gather_list(const T *em, const int64_t *cb_off, const int32_t *contrib,
                              const int64_t *vbase, const int32_t *vstride, const int64_t *list, int64_t n,
                              T *vals, ResSum r, unsigned nr) {
    constexpr int TPB = 16 / V;
    if (res_part(r, nr)) return;
    const int64_t g = (int64_t)(blockIdx.x - nr) * blockDim.x + threadIdx.x;
    const int64_t k = g / TPB;
    if (k >= n) return;
    gather_block<T, V>(em, cb_off, contrib, vbase, vstride, list[k], (int)(g % TPB) * V, vals);
}

// The same summations for every tree of a batch in one launch: the blocks of
// all trees one after the other (prefix[t] = first block of tree t), then the
// nodes of all trees for the residual (node_prefix).
__device__ inline int tree_of(const int64_t *prefix, int n, int64_t g) {
    int lo = 0, hi = n;  // prefix[lo] <= g < prefix[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (prefix[mid] <= g) lo = mid;
        else hi = mid;
    }
    return lo;
}

template <typename T, int V>
__global__ void k_gather_batch(const GatherTab *tabs, const int64_t *prefix, const int64_t *node_prefix, int n_trees,
                               unsigned nr) {
    constexpr int TPB = 16 / V;
    if (blockIdx.x < nr) {
        const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
        if (g >= node_prefix[n_trees]) return;
        const int t = tree_of(node_prefix, n_trees, g);
        const GatherTab &G = tabs[t];
        if (G.resid) res_node(G.rrec, G.roff, G.rlist, g - node_prefix[t], G.resid);
        return;
    }
    const int64_t g = (int64_t)(blockIdx.x - nr) * blockDim.x + threadIdx.x;
    const int64_t Bg = g / TPB;
    if (Bg >= prefix[n_trees]) return;
    const int t = tree_of(prefix, n_trees, Bg);
    const GatherTab &G = tabs[t];
    gather_block<T, V>((const T *)G.em, G.cb_off, G.contrib, G.vbase, G.vstride, Bg - prefix[t],
                       (int)(g % TPB) * V, (T *)G.vals);
}

__global__ void k_res_gather(const double *rrec, const int64_t *roff, const int32_t *rlist, int64_t n_nodes,
                             double *out) {
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= n_nodes) return;
    res_node(rrec, roff, rlist, n, out);
}

void launch_gather_batch(hipStream_t s, int precision, const GatherTab *tabs, const int64_t *blk_prefix,
                         int64_t n_blocks, const int64_t *node_prefix, int64_t n_nodes, int n_trees) {
    const unsigned nr = (unsigned)((n_nodes + 255) / 256);
    const int64_t threads = (precision == 0 ? 8 : 4) * n_blocks;
    const dim3 grid(nr + (unsigned)((threads + 255) / 256));
    if (grid.x == 0) return;
    if (precision == 0)
        hipLaunchKernelGGL((k_gather_batch<double, 2>), grid, dim3(256), 0, s, tabs, blk_prefix, node_prefix, n_trees,
                           nr);
    else
        hipLaunchKernelGGL((k_gather_batch<float, 4>), grid, dim3(256), 0, s, tabs, blk_prefix, node_prefix, n_trees,
                           nr);
}

void launch_res_gather(hipStream_t s, const double *rrec, const int64_t *roff, const int32_t *rlist,
                       int64_t n_nodes, double *out) {
    if (n_nodes <= 0) return;
    hipLaunchKernelGGL(k_res_gather, dim3((unsigned)((n_nodes + 255) / 256)), dim3(256), 0, s, rrec, roff,
                       rlist, n_nodes, out);
}

void launch_gather_f64(hipStream_t s, const double *em, const int64_t *cb_off, const int32_t *contrib,
                       const int64_t *vbase, const int32_t *vstride, int64_t nb, double *vals,
                       bool skip_late, const ResSum &r) {
    const unsigned nr = skip_late ? 0u : res_groups(r);
    const dim3 grid(nr + (unsigned)((8 * nb + 2047) / 2048 * 8));
    if (grid.x == 0) return;
    if (skip_late)
        hipLaunchKernelGGL((k_gather<double, 2, true>), grid, dim3(256), 0, s, em, cb_off, contrib, vbase,
                           vstride, nb, vals, r, nr);
    else
        hipLaunchKernelGGL((k_gather<double, 2, false>), grid, dim3(256), 0, s, em, cb_off, contrib, vbase,
                           vstride, nb, vals, r, nr);
}
void launch_gather_f32(hipStream_t s, const float *em, const int64_t *cb_off, const int32_t *contrib,
                       const int64_t *vbase, const int32_t *vstride, int64_t nb, float *vals,
                       bool skip_late, const ResSum &r) {
    const unsigned nr = skip_late ? 0u : res_groups(r);
    const dim3 grid(nr + (unsigned)((4 * nb + 255) / 256));
    if (grid.x == 0) return;
    if (skip_late)
        hipLaunchKernelGGL((k_gather<float, 4, true>), grid, dim3(256), 0, s, em, cb_off, contrib, vbase,
                           vstride, nb, vals, r, nr);
    else
        hipLaunchKernelGGL((k_gather<float, 4, false>), grid, dim3(256), 0, s, em, cb_off, contrib, vbase,
                           vstride, nb, vals, r, nr);
}
void launch_gather_list(hipStream_t s, bool fp64, const void *em, const int64_t *cb_off, const int32_t *contrib,
                        const int64_t *vbase, const int32_t *vstride, const int64_t *list, int64_t n,
                        void *vals, const ResSum &r) {
    const unsigned nr = res_groups(r);
    const dim3 grid(nr + (unsigned)(((fp64 ? 8 : 4) * n + 255) / 256));
    if (grid.x == 0) return;
    if (fp64)
        hipLaunchKernelGGL((k_gather_list<double, 2>), grid, dim3(256), 0, s, (const double *)em, cb_off, contrib,
                           vbase, vstride, list, n, (double *)vals, r, nr);
    else
        hipLaunchKernelGGL((k_gather_list<float, 4>), grid, dim3(256), 0, s, (const float *)em, cb_off, contrib,
                           vbase, vstride, list, n, (float *)vals, r, nr);
}

// dynamic LDS that holds a kernel to at most wg_per_cu resident workgroups per
// CU (160 KB of LDS each; 512 bytes of slack so that the rounding of the
// allocation cannot cut one more)
size_t lds_for_cap(const void *kernel, int wg_per_cu) {
    if (wg_per_cu <= 0) return 0;
    hipFuncAttributes at{};
    if (hipFuncGetAttributes(&at, kernel) != hipSuccess) return 0;
    const size_t want = (size_t)163840 / (size_t)wg_per_cu - 512;
    return want > at.sharedSizeBytes ? want - at.sharedSizeBytes : 0;
}

int sub_items_per_cu(int precision) {
    const void *k = precision == 0 ? (const void *)&k_asm2<double, 0, true>
                    : precision == 1 ? (const void *)&k_asm2<float, 1, true>
                                     : (const void *)&k_asm2<float, 2, true>;
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, 64, 0) != hipSuccess) return 0;
    return n;
}

int64_t out_items_resident(int precision) {
    const void *k = precision == 0 ? (const void *)&k_asm2<double, 0, false>
                    : precision == 1 ? (const void *)&k_asm2<float, 1, false>
                                     : (const void *)&k_asm2<float, 2, false>;
    int n = 0, dev = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, 64, 0) != hipSuccess || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    return (int64_t)n * cus;
}

// OUT elements go two per workgroup (the second one's loads in flight while the
// first is assembled) only where the GPU goes through many rounds of workgroups: over
// four times the number it holds at once. Below that the workgroups of the next
// round load while others compute, and two in a row only lengthen the last round. The
// FP64 form, with its longer elements, also takes two where one each would leave a
// second round nearly empty. Measured, one / two per workgroup, us:
//   elements    3072         3584         4096         8000         13,824       32,768       262,144
//   FP64        26.6 / 26.8  28.6 / 27.0  29.7 / 31.3  37.5 / 37.9  60.5 / 59.3  120 / 117    916 / 872
//   BF16x3      19.7 / 22.9  22.2 / 24.0  23.5 / 25.2  32.0 / 32.6  47.3 / 48.0  90.1 / 87.9  611 / 594
//   FP16x2      19.1 / 21.8  21.5 / 23.0  22.5 / 24.4  30.8 / 31.5  44.8 / 45.4  87.1 / 85.2  590 / 562
static dim3 item_grid(AsmArgs &a, bool sub, bool fp64, int64_t resident) {
    const int64_t n = a.n_items;
    a.pair = !sub && (n > 4 * resident || (fp64 && n > resident && n < resident + resident / 5));
    return dim3((unsigned)(a.pair ? (n + 1) / 2 : n));
}

void launch_assemble_f64(hipStream_t s, AsmArgs a, bool sub, int wg_per_cu, int64_t resident) {
    if (a.n_items <= 0) return;
    const dim3 grid = item_grid(a, sub, true, resident), block(64);
    if (sub)
        hipLaunchKernelGGL((k_asm2<double, 0, true>), grid, block,
                           lds_for_cap((const void *)&k_asm2<double, 0, true>, wg_per_cu), s, a);
    else
        hipLaunchKernelGGL((k_asm2<double, 0, false>), grid, block, 0, s, a);
}

void launch_assemble_mixed(hipStream_t s, AsmArgs a, bool sub, int fp16, int wg_per_cu, int64_t resident) {
    if (a.n_items <= 0) return;
    const dim3 grid = item_grid(a, sub, false, resident), block(64);
#define VMS_L(MODE)                                                                             \
    do {                                                                                        \
        if (sub)                                                                                \
            hipLaunchKernelGGL((k_asm2<float, MODE, true>), grid, block,                        \
                               lds_for_cap((const void *)&k_asm2<float, MODE, true>, wg_per_cu), s, a); \
        else                                                                                    \
            hipLaunchKernelGGL((k_asm2<float, MODE, false>), grid, block, 0, s, a);             \
    } while (0)
    if (fp16) VMS_L(2);
    else VMS_L(1);
#undef VMS_L
}

}  // namespace vmsk
