// Triquadratic (Q2, 27-node) VMS element assembly of libvms (gfx950), FP64.
//
// The paper compares linear and quadratic bases in its matrix-assembly table
// (uniform 16^3 mesh) and tabulates the basis at the (bf+1)^d Gauss points
// (App. A): here 27 nodes, 3 x 3 x 3 Gauss points, element matrices of 108 x
// 108. The integrand is the trilinear kernel's (eq. (vms), (uprime), (pprime),
// taus frozen), with the same per-point factors and D blocks (vms_point.h).
//
// Workgroups of four waves, two per CU, take elements in turn; the basis at the
// 27 points (24 KB) is tabulated in LDS once per workgroup. Evaluating it in the
// loops instead (189 basis values per lane for the contraction, 81 for the
// interpolation, and one thread per point for the state) cost as much as the
// matrix instructions: 0.90 -> 0.30 ms on 16^3 elements, 1,512 v_mfma_f64_4x4x4
// per wave being 0.18 ms of it.
//   phase 0  node ids and the 27 x 7 nodal fields to LDS;
//   phase 1  fields and gradients at the 27 points;
//   phase 2  per-point state (taus, u', p', residual coefficients, D factors);
//   phase 3  for each third of the points: the 16 D blocks of each point, then
//            wave i (test component i) contracts on v_mfma_f64_4x4x4 (four 4x4
//            blocks per instruction, block = trial component j):
//              stage 1  F^{ij}[k][b] = sum_l D^{ij}[k][l] B[l][b], per 4-column
//                       tile of b, lands in stage 2's second-operand layout;
//              stage 2  K^{ij}[a][b] += sum_k B[k][a] F^{ij}[k][b] over the
//                       7 x 7 tiles (rows and columns padded from 27 to 28);
//   phase 4  residual R[(a,i)] = sum_q sum_k B[k][a] r^i[k] on the VALU;
//   phase 5  the element matrix record, block-major (node pair, then i, j).
#include "kernels.h"
#include "vms_point.h"

namespace vmsk {

namespace {

constexpr double Q2_G = 0x1.8c97ef43f7248p-1;  // sqrt(3/5), correctly rounded
constexpr double Q2_W0 = 5.0 / 9.0, Q2_W1 = 8.0 / 9.0;
constexpr int NQP = NQ2 + 1;  // padded row of the per-point factors

// 1D quadratic Lagrange basis of the nodes -1, 0, 1 at Gauss point g (0..2):
// value of function i, and its xi-derivative
__device__ inline double q2f(int g, int i) {
    const double x = g == 0 ? -Q2_G : (g == 1 ? 0.0 : Q2_G);
    return i == 0 ? 0.5 * x * (x - 1.0) : (i == 1 ? 1.0 - x * x : 0.5 * x * (x + 1.0));
}
__device__ inline double q2g(int g, int i) {
    const double x = g == 0 ? -Q2_G : (g == 1 ? 0.0 : Q2_G);
    return i == 0 ? x - 0.5 : (i == 1 ? -2.0 * x : x + 0.5);
}

// B_q[d][a]: basis function a (d = 0) or its x/y/z derivative (d = 1..3, times
// s = 2/h) at Gauss point q; zero for the padding row a = 27
__device__ inline double q2basis(int q, int a, int d, double s) {
    if (a >= 27) return 0.0;
    const int qx = q % 3, qy = (q / 3) % 3, qz = q / 9;
    const int ax = a % 3, ay = (a / 3) % 3, az = a / 9;
    const double fx = d == 1 ? s * q2g(qx, ax) : q2f(qx, ax);
    const double fy = d == 2 ? s * q2g(qy, ay) : q2f(qy, ay);
    const double fz = d == 3 ? s * q2g(qz, az) : q2f(qz, az);
    return fx * fy * fz;
}

__device__ inline double q2w(int g) { return g == 1 ? Q2_W1 : Q2_W0; }

}  // namespace

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_q2(Q2Args A) {
    __shared__ double sB[27 * 4 * 28];  // B_q[d][a] at (4 q + d) 28 + a; a = 27 is the zero padding
    __shared__ int32_t sN[27];
    __shared__ double sU[27][8];
    __shared__ double sQ[27][NQP];
    __shared__ union {
        double sI[27][29];      // field f, entry d (value, gradient): 4 f + d
        double sD[9][16][17];   // D blocks of a third of the points: [p][4 i + j][4 k + l]
    } u;
    const double h = A.h, s = 2.0 / h;
    for (int k = threadIdx.x; k < 27 * 4 * 28; k += 256) sB[k] = q2basis(k / 112, k % 28, (k / 28) & 3, s);

    for (int64_t e = blockIdx.x; e < A.n_el; e += gridDim.x) {
        // formed anew for every element: the addresses of all phases, kept over
        // the loop, would spill
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        const int lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
        // ---- phase 0
        if (t < 27) sN[t] = A.el_node[27 * e + t];
        __syncthreads();  // also: the table is complete, the previous element is done with the LDS
        if (t < 189) sU[t / 7][t % 7] = A.f[t % 7][sN[t / 7]];
        __syncthreads();

        // ---- phase 1: 27 points x 7 fields x (value, gradient)
        for (int task = t; task < 27 * 28; task += 256) {
            const int q = task / 28, r = task % 28, f = r >> 2;
            const double *B = sB + (4 * q + (r & 3)) * 28;
            double v = 0.0;
            for (int a = 0; a < 27; ++a) v += B[a] * sU[a][f];
            u.sI[q][r] = v;
        }
        __syncthreads();

        // ---- phase 2: per-point state, four threads per point: thread r < 3 takes row /
        // component r with every component index rotated by r (own = index 0),
        // thread 3 the scalars and the continuity row
        if (t < 108) {
            const int q = t >> 2, r = t & 3;
            const int o[3] = {r < 3 ? r : 0, r < 3 ? (r + 1 < 3 ? r + 1 : 0) : 1, r < 3 ? (r + 2 < 3 ? r + 2 : r - 1) : 2};
            const double rho = A.rho, mu = A.mu, th = A.theta, idt = A.idt, irho = A.irho;
            const double g = s * s;  // G = g I
            const double W = q2w(q % 3) * q2w((q / 3) % 3) * q2w(q / 9) * (0.5 * h) * (0.5 * h) * (0.5 * h);
            const double *I = u.sI[q];
            double *Q = sQ[q];
            double ut[3], gu[3][3], up[3], acc[3];
            for (int c = 0; c < 3; ++c) {
                ut[c] = th * I[4 * o[c]] + (1.0 - th) * I[4 * (4 + o[c])];
                for (int m = 0; m < 3; ++m)
                    gu[c][m] = th * I[4 * o[c] + 1 + o[m]] + (1.0 - th) * I[4 * (4 + o[c]) + 1 + o[m]];
            }
            const double s0 = A.tau_a + A.tau_b * g * g + g * (ut[0] * ut[0] + ut[1] * ut[1] + ut[2] * ut[2]);
            const double tauM = rsq<double>(s0);
            const double tauC = (1.0 / (3.0 * g)) * s0 * tauM;  // 1 / (tau_M tr G)
            for (int c = 0; c < 3; ++c) {
                acc[c] = (I[4 * o[c]] - I[4 * (4 + o[c])]) * idt + ut[0] * gu[c][0] + ut[1] * gu[c][1] + ut[2] * gu[c][2];
                up[c] = -tauM * (rho * acc[c] + I[4 * 3 + 1 + o[c]]);
            }
            const double div = gu[0][0] + gu[1][1] + gu[2][2];
            const double pp = -rho * tauC * div;
            const double upg = g * (up[0] * up[0] + up[1] * up[1] + up[2] * up[2]);
            const double tb = upg > 0.0 ? rsq<double>(upg) : 0.0;
            if (r < 3) {
                const int c = r;
                const double svc = up[0] * gu[0][0] + up[1] * gu[0][1] + up[2] * gu[0][2];
                Q[QUT + c] = ut[0];
                Q[QUP + c] = up[0];
                Q[QSV + c] = svc;
                for (int m = 0; m < 3; ++m) {
                    Q[QG + 3 * c + o[m]] = gu[0][m];
                    Q[QA + 3 * c + o[m]] = (m == 0 ? idt : 0.0) + th * gu[0][m];
                    double v = 0.0;
                    for (int k = 0; k < 3; ++k) v += gu[0][k] * ((k == m ? idt : 0.0) + th * gu[k][m]);
                    Q[QGA + 3 * c + o[m]] = v;
                    Q[QRC + 4 * c + 1 + o[m]] = W * (mu * (gu[0][m] + gu[m][0]) - (m == 0 ? I[4 * 3] + pp : 0.0) -
                                                     ut[m] * up[0] - up[m] * up[0] * irho + tb * up[m] * svc);
                }
                Q[QRC + 4 * c] = W * (rho * acc[0] + svc);
                const double tr = tauM * rho, tbtr = tb * tauM * rho, tbt = tb * tauM, tir = tauM * irho;
                Q[QY + c] = tr * ut[0] + tauM * up[0];
                Q[QX + c] = -tbtr * up[0];
                Q[QCP + c] = tauM * up[0] - tbtr * svc;
                Q[QYM + c] = tauM * ut[0] + tir * up[0];
                Q[QCM + c] = tir * up[0] - tbt * svc;
                Q[QXM + c] = -tbt * up[0];
            } else {
                Q[QW] = W;
                Q[QTM] = tauM;
                Q[QTC] = tauC;
                Q[QTB] = tb;
                Q[QRC + 12] = W * div;
                for (int k = 0; k < 3; ++k) Q[QRC + 13 + k] = -W * up[k] * irho;
            }
        }
        __syncthreads();

        // ---- phase 3: D blocks and the two contraction stages, a third of the points at a time
        // lane l: contraction index k = l / 16, block (trial component) j = (l / 4) % 4,
        // row / column n = l % 4; wave wv = test component i
        const int kk = lane >> 4, j4 = (lane >> 2) & 3, n4 = lane & 3, i = wv;
        double acc[7][7];
        for (int at = 0; at < 7; ++at)
            for (int bt = 0; bt < 7; ++bt) acc[at][bt] = 0.0;
        for (int c = 0; c < 3; ++c) {
            if (c > 0) __syncthreads();  // the previous third is done with sD
            if (t < 144) {
                // momentum/velocity blocks first: a wave holds one kind, but for one
                int p, bi, bj;
                if (t < 81) {
                    p = t / 9;
                    bi = (t % 9) / 3;
                    bj = t % 3;
                } else {
                    const int v = t - 81, r = v % 7;
                    p = v / 7;
                    bi = r < 3 ? r : 3;
                    bj = r < 3 ? 3 : (r < 6 ? r - 3 : 3);
                }
                double D[4][4];
                if (bi < 3 && bj < 3) dblock_mv<double>(sQ[9 * c + p], bi, bj, A.rho, A.mu, A.theta, D);
                else dblock_simple<double>(sQ[9 * c + p], bi, bj, A.irho, A.theta, D);
                for (int k = 0; k < 4; ++k)
                    for (int l = 0; l < 4; ++l) u.sD[p][4 * bi + bj][4 * k + l] = D[k][l];
            }
            __syncthreads();
#pragma unroll 1
            for (int p = 0; p < 9; ++p) {
                const double *B = sB + (4 * (9 * c + p) + kk) * 28 + n4;
                double Bt[7];  // B_q[k][4 t + n] (stage 1's second and stage 2's first operand)
                for (int tt = 0; tt < 7; ++tt) Bt[tt] = B[4 * tt];
                const double Dt = u.sD[p][4 * i + j4][4 * n4 + kk];  // D^{ij}[n][k]
                double E[7];
                for (int bt = 0; bt < 7; ++bt) E[bt] = __builtin_amdgcn_mfma_f64_4x4x4f64(Dt, Bt[bt], 0.0, 0, 0, 0);
                for (int at = 0; at < 7; ++at)
                    for (int bt = 0; bt < 7; ++bt)
                        acc[at][bt] = __builtin_amdgcn_mfma_f64_4x4x4f64(Bt[at], E[bt], acc[at][bt], 0, 0, 0);
            }
        }

        // ---- phase 4: residual
        if (t < 108) {
            const int a = t >> 2, ic = t & 3;
            double r = 0.0;
            for (int q = 0; q < 27; ++q)
                for (int k = 0; k < 4; ++k) r += sB[(4 * q + k) * 28 + a] * sQ[q][QRC + 4 * ic + k];
            A.rrec[108 * e + t] = r;
        }

        // ---- phase 5: record, entry ((27 a + b) 16 + 4 i + j)
        double *rec = A.em + (int64_t)e * (729 * 16);
        for (int at = 0; at < 7; ++at)
            for (int bt = 0; bt < 7; ++bt) {
                const int a = 4 * at + kk, b = 4 * bt + n4;
                if (a < 27 && b < 27) rec[(27 * a + b) * 16 + 4 * i + j4] = acc[at][bt];
            }
    }
}

void launch_q2(hipStream_t s, const Q2Args &a) {
    if (a.n_el <= 0) return;
    const int64_t n = a.n_el < 512 ? a.n_el : 512;  // two workgroups per CU
    hipLaunchKernelGGL(k_q2, dim3((unsigned)n), dim3(256), 0, s, a);
}

}  // namespace vmsk
